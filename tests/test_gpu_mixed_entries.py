"""A level of gates and native MUXes runs all its rotations in one launch: the same ciphertext words as the gates and the MUXes
by themselves.  Sizes on both sides of a group of 32 entries and in every form of the blind rotation on 256 compute units."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

INPUTS, WIDEST = 128, 1200


def check(pkg, ctx, gates, muxes, seed):
    rng = np.random.default_rng(seed)
    entries = gates + muxes
    codes = rng.integers(0, 10, gates).astype(np.uint8)
    a, b, c = (rng.integers(0, INPUTS, entries).astype(np.uint32) for _ in range(3))
    apart = np.arange(INPUTS, INPUTS + entries, dtype=np.uint32)
    together = apart + WIDEST
    ctx.eval_gates(codes, a[:gates], b[:gates], apart[:gates])
    ctx.eval_mux(a[gates:], b[gates:], c[gates:], apart[gates:])
    # the entries of the circuit in a shuffled order: the library sorts a level's gates before its MUXes
    order = rng.permutation(entries)
    types = np.concatenate([codes, np.full(muxes, pkg.CIRCUIT_MUX, np.uint8)])[order]
    done = ctx.eval_circuit(types, a[order], b[order], c[order], order.argsort().astype(np.uint32) | pkg.WIRE_GATE, together)
    assert done == entries
    sizes = ctx.last_level_sizes()
    assert [int(v[0]) for v in sizes] == [gates, muxes] and ctx.last_timing()["levels"] == 1
    rows = ctx._pool_tensor.view(ctx.capacity, -1)[:, :ctx.params.n + 1].cpu().numpy()
    wrong = np.argwhere(rows[together] != rows[apart])
    assert not wrong.size, (gates, muxes, wrong[:4], wrong.shape)


@pytest.fixture(scope="module")
def real():
    import paper_1906_00148_amd as pkg
    from paper_1906_00148_amd import binding
    with pkg.Context(pkg.REAL, 190600148, INPUTS + 2 * WIDEST) as ctx:
        ctx.encrypt_bits(np.random.default_rng(3).integers(0, 2, INPUTS), 5, np.arange(INPUTS))
        ctx.set_option(binding.OPT_NATIVE_MUX, 1)
        yield binding, ctx


@pytest.mark.parametrize("gates,muxes", [(1, 1), (31, 1), (32, 33), (200, 28), (1, 128), (300, 7), (3, 255), (700, 100), (1000, 40), (1100, 99)])
def test_a_level_of_gates_and_muxes_gives_the_same_words(real, gates, muxes):
    check(*real, gates, muxes, gates)


# no key switch on the matrix units (no output slot is written before it), two gadget levels, a smaller ring
@pytest.mark.parametrize("N,l,ks_t,ks_basebit", [(1024, 3, 5, 3), (1024, 2, 8, 2), (512, 3, 8, 2), (256, 3, 8, 2)])
def test_a_level_of_gates_and_muxes_at_other_parameters(N, l, ks_t, ks_basebit):
    import paper_1906_00148_amd as pkg
    from paper_1906_00148_amd import binding
    with pkg.Context(pkg.Params(n=20, N=N, l=l, bg_bit=7, ks_t=ks_t, ks_basebit=ks_basebit), 31, INPUTS + 2 * WIDEST) as ctx:
        ctx.encrypt_bits(np.random.default_rng(3).integers(0, 2, INPUTS), 5, np.arange(INPUTS))
        ctx.set_option(binding.OPT_NATIVE_MUX, 1)
        for gates, muxes in ((1, 1), (33, 40), (700, 100), (1100, 99)):
            check(binding, ctx, gates, muxes, gates)
