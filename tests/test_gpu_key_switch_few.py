"""The key switch of a few gates, word for word against the CPU oracle: groups of 32 and wavefronts of 64 gates that are full,
nearly empty or missing, the last size that it takes and the first that it does not, coefficient ranges of 8 to 32 per workgroup
and column tiles with one column."""
import numpy as np
import pytest

from oracle import tfhe as O

pytestmark = pytest.mark.gpu

COUNTS = (1, 31, 33, 64, 65, 129, 191, 192, 193, 256)


@pytest.mark.parametrize("N", [256, 512, 1024])
@pytest.mark.parametrize("n", [1, 31, 40])
def test_a_few_gates_match_the_oracle(n, N):
    import paper_1906_00148_amd as pkg
    P = dict(n=n, N=N, l=3, bg_bit=7, ks_t=8, ks_basebit=2)
    inputs, widest = 32, max(COUNTS)
    rng = np.random.default_rng(N + n)
    bits = rng.integers(0, 2, inputs).astype(np.uint8)
    codes = rng.integers(0, 10, widest).astype(np.uint8)
    a, b = (rng.integers(0, inputs, widest).astype(np.uint32) for _ in range(2))
    out = np.arange(inputs, inputs + widest, dtype=np.uint32)
    K = O.keygen(O.Params(**P), 31)
    pool = np.concatenate([O.encrypt_bits(K, bits, 5), np.zeros((widest, n + 1), np.uint32)])
    O.eval_gates(K, pool, codes, a, b, out, threads=16)
    with pkg.Context(pkg.Params(**P), 31, inputs + widest) as ctx:
        ctx.encrypt_bits(bits, 5, np.arange(inputs))
        rows = ctx._pool_tensor.view(ctx.capacity, -1)[inputs:]
        for count in COUNTS:
            rows.zero_()
            ctx.eval_gates(codes[:count], a[:count], b[:count], out[:count])
            got = rows[:, :n + 1].cpu().numpy().view(np.uint32)
            assert np.array_equal(got[:count], pool[inputs:inputs + count]), count
            assert not got[count:].any(), count
