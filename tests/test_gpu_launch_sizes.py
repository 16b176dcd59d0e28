"""Every way a level can be launched gives the same ciphertext words: the launch shapes that depend on the level's size
against one wavefront per rotation (SHE_OPT_SPLIT_BELOW = 0), which test_gpu_parity.py pins to the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

WIDEST = 2600


@pytest.fixture(scope="module")
def level():
    import paper_1906_00148_amd as pkg
    rng = np.random.default_rng(77)
    inputs = 512
    with pkg.Context(pkg.REAL, 190600148, inputs + WIDEST) as ctx:
        ctx.encrypt_bits(rng.integers(0, 2, inputs), 5, np.arange(inputs))
        codes = rng.integers(0, 10, WIDEST).astype(np.uint8)
        a, b = (rng.integers(0, inputs, WIDEST).astype(np.uint32) for _ in range(2))
        out = np.arange(inputs, inputs + WIDEST, dtype=np.uint32)

        def run(count, split_below, tracking=False):
            rows = ctx._pool_tensor.view(ctx.capacity, -1)[inputs:inputs + count]
            rows.zero_()
            ctx.set_option(pkg.OPT_SPLIT_BELOW, split_below)
            ctx.set_round_tracking(tracking)
            ctx.eval_gates(codes[:count], a[:count], b[:count], out[:count])
            ctx.set_round_tracking(False)
            return rows.cpu().numpy().copy()

        default = ctx.get_option(pkg.OPT_SPLIT_BELOW)
        yield run, default, run(WIDEST, 0)


# one gate; around one, two and three gates per compute unit (256 of them)
@pytest.mark.parametrize("tracking", [False, True])
@pytest.mark.parametrize("count", [1, 2, 255, 257, 511, 512, 513, 769])
def test_level_sizes_give_the_same_words(level, count, tracking):
    run, default, want = level
    assert np.array_equal(run(count, default, tracking), want[:count])


# full rounds of four gates per compute unit on a wavefront each, the rest (1 .. 2 per compute unit) on four
@pytest.mark.parametrize("tracking", [False, True])
@pytest.mark.parametrize("count", [1025, 1536, 1537, 2049, 2560])
def test_a_rest_beyond_full_rounds_gives_the_same_words(level, count, tracking):
    run, default, want = level
    assert np.array_equal(run(count, default, tracking), want[:count])
