"""Reading TRLWE samples: lists in the kernel's arguments (up to 256), beyond them, and in chunks of 1024 whose rest is short
again, in any order and with repetitions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [256, 1024, 2048])
def test_samples_are_read_back_as_written(N):
    import paper_1906_00148_amd as pkg
    rng = np.random.default_rng(N)
    slots = 300
    with pkg.Context(pkg.Params(n=4, N=N, l=3, bg_bit=7, ks_t=8, ks_basebit=2), 3, 4) as ctx:
        ctx.leveled_init(1, slots)
        table = rng.integers(0, 2 ** 32, (slots, 2, N), dtype=np.uint32)
        ctx.trlwe_write(table, np.arange(slots))
        for count in (1, 2, 255, 256, 257, 1024, 1025, 1280):
            ids = rng.integers(0, slots, count).astype(np.uint32)
            assert np.array_equal(ctx.trlwe_read(ids), table[ids]), count
