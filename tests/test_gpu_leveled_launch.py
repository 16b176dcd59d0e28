"""Every way a level of CMuxes can be launched gives the same words: four wavefronts per CMux (at most two CMuxes per
compute unit) against one (test_gpu_leveled.py pins that one to the oracle); samples read back in chunks are the samples
that were written."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,l,bg_bit", [(1024, 3, 7), (1024, 2, 8), (1024, 1, 10), (1024, 5, 6), (1024, 8, 3),
                                         (2048, 3, 7), (2048, 2, 8), (2048, 4, 7), (2048, 8, 3)])
@pytest.mark.parametrize("tracking", [False, True])
def test_small_levels_of_cmuxes_give_the_same_words(N, l, bg_bit, tracking):
    import paper_1906_00148_amd as pkg
    per_launch = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    count, data, selectors = per_launch + 5, 60, 7
    rng = np.random.default_rng(N + l)
    with pkg.Context(pkg.Params(n=16, N=N, l=l, bg_bit=bg_bit), 77, 4) as ctx:
        ctx.leveled_init(selectors, data + 2 * count)
        ctx.trgsw_encrypt_bits(rng.integers(0, 2, selectors), 5, np.arange(selectors))
        ctx.trlwe_write(rng.integers(0, 1 << 32, (data, 2, N), dtype=np.uint64).astype(np.uint32), np.arange(data))
        s, i1, i0 = rng.integers(0, selectors, count), rng.integers(0, data, count), rng.integers(0, data, count)
        out = data + np.arange(count)
        ctx.set_round_tracking(tracking)
        ctx.eval_cmux(s, i1, i0, out)                                       # one wavefront per CMux
        want = ctx.trlwe_read(out)
        first = 0
        for size in (1, 4, per_launch):                                     # four
            part = slice(first, first + size)
            ctx.eval_cmux(s[part], i1[part], i0[part], out[part] + count)
            first += size
        assert first == count
        assert np.array_equal(ctx.trlwe_read(out + count), want)
        if tracking:
            assert ctx.get_round_error() < 0.25


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
