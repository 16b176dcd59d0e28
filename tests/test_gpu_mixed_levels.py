"""Levels that k_blind_rotate_mixed runs in pairs (two wavefronts per rotation, two rotations per workgroup), alone and beside
the other forms, give the same ciphertext words as one wavefront per rotation (SHE_OPT_SPLIT_BELOW = 0), whose words are the
oracle's (test_gpu_launch_sizes.py): the first and last size of each division on 256 compute units, with a last pair of one.
(That these launches have pairs at all: test_host_mixed.py.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

WIDEST, WIDEST_MUX = 2816, 768


@pytest.fixture(scope="module")
def levels():
    import paper_1906_00148_amd as pkg
    rng = np.random.default_rng(99)
    inputs = 512
    with pkg.Context(pkg.REAL, 190600148, inputs + WIDEST) as ctx:
        ctx.encrypt_bits(rng.integers(0, 2, inputs), 5, np.arange(inputs))
        codes = rng.integers(0, 10, WIDEST).astype(np.uint8)
        a, b, sel = (rng.integers(0, inputs, WIDEST).astype(np.uint32) for _ in range(3))
        out = np.arange(inputs, inputs + WIDEST, dtype=np.uint32)

        def run(count, split_below, tracking=False, mux=False):
            rows = ctx._pool_tensor.view(ctx.capacity, -1)[inputs:inputs + count]
            rows.zero_()
            ctx.set_option(pkg.OPT_SPLIT_BELOW, split_below)
            ctx.set_round_tracking(tracking)
            if mux:
                ctx.eval_mux(sel[:count], a[:count], b[:count], out[:count])
            else:
                ctx.eval_gates(codes[:count], a[:count], b[:count], out[:count])
            ctx.set_round_tracking(False)
            return rows.cpu().numpy().view(np.uint32).copy()

        default = ctx.get_option(pkg.OPT_SPLIT_BELOW)
        yield run, default, run(WIDEST, 0), run(WIDEST_MUX, 0, mux=True)


# a pair and a quad per compute unit (513 to 768); a round and pairs (1281 to 1536); two rounds and pairs (2305 to 2560), and
# a pair and a quad (2561 to 2816)
@pytest.mark.parametrize("tracking", [False, True])
@pytest.mark.parametrize("count", [513, 514, 767, 768, 1281, 1282, 1535, 2305, 2560, 2561, 2562, 2816])
def test_pairs_give_the_same_words(levels, count, tracking):
    run, default, want, _ = levels
    assert np.array_equal(run(count, default, tracking), want[:count])


# the rotations of MUXes leave the samples unswitched: 514, 766, 768, 1282 and 1536 of them
@pytest.mark.parametrize("tracking", [False, True])
@pytest.mark.parametrize("count", [257, 383, 384, 641, 768])
def test_pairs_of_mux_rotations_give_the_same_words(levels, count, tracking):
    run, default, _, want = levels
    assert np.array_equal(run(count, default, tracking, mux=True), want[:count])
