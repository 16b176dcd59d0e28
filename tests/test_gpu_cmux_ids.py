"""CMux levels whose ids travel in the kernel's arguments (at most 192 entries) and levels just beyond give the words of
the same entries in one large level, round tracking on and off."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tracking", [False, True])
@pytest.mark.parametrize("N", [1024, 2048])
def test_levels_around_the_argument_limit(N, tracking):
    import paper_1906_00148_amd as pkg
    P = pkg.REAL if N == 1024 else pkg.SECTION4_LEVELED
    selectors, inputs, widest = 7, 64, 700
    rng = np.random.default_rng(N)
    sel, a, b = rng.integers(0, selectors, widest), rng.integers(0, inputs, widest), rng.integers(0, inputs, widest)
    out = np.arange(inputs, inputs + widest)
    with pkg.Context(P, 11, 4) as ctx:
        ctx.leveled_init(selectors, inputs + widest)
        ctx.trgsw_encrypt_bits(rng.integers(0, 2, selectors).astype(np.uint8), 3, np.arange(selectors))
        ctx.trlwe_write(rng.integers(0, 1 << 32, (inputs, 2, N), dtype=np.uint32), np.arange(inputs))
        ctx.set_round_tracking(tracking)
        ctx.eval_cmux(sel, a, b, out)
        want = ctx.trlwe_read(out)
        for count in (1, 2, 191, 192, 193):
            last = slice(widest - count, widest)
            ctx.trlwe_write(np.zeros((count, 2, N), np.uint32), out[last])
            ctx.eval_cmux(sel[last], a[last], b[last], out[last])
            assert np.array_equal(ctx.trlwe_read(out[last]), want[last]), count
