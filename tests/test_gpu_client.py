"""Fresh encryptions and decryptions made on the device, word for word and bit for bit against the CPU oracle."""
import numpy as np
import pytest

from oracle import tfhe as O

pytestmark = pytest.mark.gpu


# n around multiples of the 64 lanes that share a sample, counts around the 4 samples of a workgroup.  With a deviation of
# 2^6 torus turns an error is about 2^38, so that 3 % of the samples lie within the device's margin of a rounding boundary
# (2^-44 of the error's size) and the host finishes them.
@pytest.mark.parametrize("lwe_std", [2.0 ** -15, 0.0, 64.0])
@pytest.mark.parametrize("n,count", [(1, 1), (63, 3), (64, 4), (65, 5), (630, 1001)])
def test_fresh_samples_and_decryptions_match_the_oracle(n, count, lwe_std):
    import paper_1906_00148_amd as pkg
    K = O.keygen(O.Params(n=n, N=256, lwe_std=lwe_std), 99)
    rng = np.random.default_rng(count)
    bits = rng.integers(0, 2, count).astype(np.uint8)
    ids = rng.permutation(count + 3)[:count].astype(np.uint32)
    with pkg.Context(pkg.Params(n=n, N=256, lwe_std=lwe_std), 99, count + 3) as ctx:
        ctx.encrypt_bits(bits, 2 ** 63 + count, ids)
        want = O.encrypt_bits(K, bits, 2 ** 63 + count)
        assert np.array_equal(ctx.read_cts(ids), want)
        phase = want[:, n] - (want[:, :n] * K.lwe_key[None, :]).sum(axis=1, dtype=np.uint32)
        assert np.array_equal(ctx.decrypt(ids), (phase.astype(np.int32) > 0).astype(np.uint8))
