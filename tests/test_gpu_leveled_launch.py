"""Samples read back in chunks are the samples that were written."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [256, 512, 1024, 2048])
def test_reading_more_samples_than_a_chunk(N):
    import paper_1906_00148_amd as pkg
    rng = np.random.default_rng(N)
    raw = rng.integers(0, 1 << 32, (9, 2, N), dtype=np.uint64).astype(np.uint32)
    with pkg.Context(pkg.Params(n=16, N=N), 77, 4) as ctx:
        ctx.leveled_init(1, 12)
        ctx.trlwe_write(raw, np.arange(9) + 3)
        ids = rng.integers(0, 9, 1025)
        assert np.array_equal(ctx.trlwe_read(ids + 3), raw[ids])
