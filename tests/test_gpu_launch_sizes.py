"""Every way a level can be launched gives the same ciphertext words: the launch shapes that depend on the level's size
against one wavefront per rotation (SHE_OPT_SPLIT_BELOW = 0), whose words are the oracle's.  At N = 1024 and l = 3 on 256
compute units that is twelve wavefronts per rotation up to 256 rotations, four up to 512, two up to 1024, and full rounds of
1024 with the rest (at most 512) on four each."""
import numpy as np
import pytest

from oracle import tfhe as O

pytestmark = pytest.mark.gpu

WIDEST, WIDEST_MUX = 2600, 1100


@pytest.fixture(scope="module")
def levels():
    import paper_1906_00148_amd as pkg
    rng = np.random.default_rng(77)
    inputs = 512
    with pkg.Context(pkg.REAL, 190600148, inputs + WIDEST) as ctx:
        ctx.encrypt_bits(rng.integers(0, 2, inputs), 5, np.arange(inputs))
        codes = rng.integers(0, 10, WIDEST).astype(np.uint8)
        a, b = (rng.integers(0, inputs, WIDEST).astype(np.uint32) for _ in range(2))
        out = np.arange(inputs, inputs + WIDEST, dtype=np.uint32)

        sel = rng.integers(0, inputs, WIDEST).astype(np.uint32)

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
        yield {"gates": (run, default, run(WIDEST, 0)), "mux": (run, default, run(WIDEST_MUX, 0, mux=True)),
               "inputs": ctx.read_cts(np.arange(inputs)), "codes": codes, "ids": (a, b, sel)}


@pytest.fixture(scope="module")
def level(levels):
    return levels["gates"]


# one wavefront per rotation, against the oracle: what the other launches are compared with
def test_the_reference_levels_are_the_oracles(levels, real_keys):
    words, codes, (a, b, sel) = levels["inputs"], levels["codes"], levels["ids"]
    n = words.shape[1] - 1
    sample = np.linspace(0, WIDEST - 1, 24).astype(int)
    pool = np.concatenate([words, np.zeros((sample.size, n + 1), np.uint32)])
    O.eval_gates(real_keys, pool, codes[sample], a[sample], b[sample], words.shape[0] + np.arange(sample.size), threads=16)
    assert np.array_equal(levels["gates"][2][sample, :n + 1], pool[words.shape[0]:])
    for m in (0, 511, WIDEST_MUX - 1):
        assert np.array_equal(levels["mux"][2][m, :n + 1], O.mux(real_keys, words[sel[m]], words[a[m]], words[b[m]])), m


# one gate; around one, two and three gates per compute unit (256 of them): twelve wavefronts per gate (1, 2, 255), four (257,
# 511, 512), two (513, 769)
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


# MUX levels leave the samples unswitched: twice as many rotations as entries, on twelve wavefronts (2, 200), on four (512), on
# two (514, 900, 1024) and mixed (1026, 1400, 1536, 2200)
@pytest.mark.parametrize("tracking", [False, True])
@pytest.mark.parametrize("count", [1, 100, 256, 257, 450, 512, 513, 700, 768, 1100])
def test_mux_levels_give_the_same_words(levels, count, tracking):
    run, default, want = levels["mux"]
    assert np.array_equal(run(count, default, tracking, mux=True), want[:count])


# other gadgets (Bg at its largest, and l = 2, which has two wavefronts or one) and a key switch of another base, before which no
# output slot is written: twelve wavefronts (2 rotations), four (300), two (514, 1000), mixed (1026, 1100), MUX included
@pytest.mark.parametrize("l,bg_bit,ks_t,ks_basebit", [(3, 7, 5, 3), (3, 8, 8, 2), (3, 5, 16, 1), (2, 8, 8, 2)])
def test_other_parameters_give_the_same_words(l, bg_bit, ks_t, ks_basebit):
    import paper_1906_00148_amd as pkg
    P = dict(n=24, N=1024, l=l, bg_bit=bg_bit, ks_t=ks_t, ks_basebit=ks_basebit)
    inputs, widest = 64, 1100
    rng = np.random.default_rng(bg_bit)
    bits = rng.integers(0, 2, inputs).astype(np.uint8)
    codes = rng.integers(0, 10, widest).astype(np.uint8)
    a, b, sel = (rng.integers(0, inputs, widest).astype(np.uint32) for _ in range(3))
    out = np.arange(inputs, inputs + widest, dtype=np.uint32)
    with pkg.Context(pkg.Params(**P), 31, inputs + widest) as ctx:
        ctx.encrypt_bits(bits, 5, np.arange(inputs))
        rows = ctx._pool_tensor.view(ctx.capacity, -1)[inputs:]
        default = ctx.get_option(pkg.OPT_SPLIT_BELOW)

        def run(count, mux, split_below):
            ctx.set_option(pkg.OPT_SPLIT_BELOW, split_below)
            words = []
            for tracking in (False, True):
                rows.zero_()
                ctx.set_round_tracking(tracking)
                ctx.get_round_error(reset=True)
                if mux:
                    ctx.eval_mux(sel[:count], a[:count], b[:count], out[:count])
                else:
                    ctx.eval_gates(codes[:count], a[:count], b[:count], out[:count])
                words.append(rows[:count].cpu().numpy().copy())
            assert 0 < ctx.get_round_error() < 0.25
            assert np.array_equal(words[0], words[1])
            return words[0]

        for mux in (False, True):
            want = run(widest, mux, 0)
            for rotations in (2, 300, 514, 1000, 1026, 1100):
                count = rotations // 2 if mux else rotations
                assert np.array_equal(run(count, mux, default), want[:count]), (mux, rotations)
    K = O.keygen(O.Params(**P), 31)
    fresh = O.encrypt_bits(K, bits, 5)
    pool = np.concatenate([fresh, np.zeros((8, P["n"] + 1), np.uint32)])
    with pkg.Context(pkg.Params(**P), 31, inputs + 8) as ctx:
        ctx.encrypt_bits(bits, 5, np.arange(inputs))
        ctx.eval_gates(codes[:8], a[:8], b[:8], out[:8])
        O.eval_gates(K, pool, codes[:8], a[:8], b[:8], out[:8], threads=8)
        assert np.array_equal(ctx.read_cts(out[:8]), pool[inputs:])
