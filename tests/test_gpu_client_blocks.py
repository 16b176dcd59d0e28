"""Client calls at the edges of their kernels: seven samples a workgroup and a lane for each one's error, ten words of a sample
a lane and more at once, word for word and bit for bit against the CPU oracle.  With a deviation of 2^6 torus turns some of the
errors are the host's."""
import numpy as np
import pytest

from oracle import tfhe as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lwe_std", [2.0 ** -15, 64.0])
@pytest.mark.parametrize("n,count", [(2, 6), (630, 7), (639, 8), (640, 13), (641, 14), (704, 15), (1281, 700)])
def test_client_calls_match_the_oracle(n, count, lwe_std):
    import paper_1906_00148_amd as pkg
    K = O.keygen(O.Params(n=n, N=256, lwe_std=lwe_std), 41)
    rng = np.random.default_rng(n)
    bits = rng.integers(0, 2, count).astype(np.uint8)
    ids = rng.permutation(count + 3)[:count].astype(np.uint32)
    with pkg.Context(pkg.Params(n=n, N=256, lwe_std=lwe_std), 41, count + 3) as ctx:
        ctx.encrypt_bits(bits, 1000 + count, ids)
        want = O.encrypt_bits(K, bits, 1000 + count)
        assert np.array_equal(ctx.read_cts(ids), want)
        phase = want[:, n] - (want[:, :n] * K.lwe_key[None, :]).sum(axis=1, dtype=np.uint32)
        assert np.array_equal(ctx.decrypt(ids), (phase.astype(np.int32) > 0).astype(np.uint8))
