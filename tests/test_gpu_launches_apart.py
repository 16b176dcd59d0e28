"""A level whose gates and native MUXes run in two launches gives the same ciphertext words as the gates and the MUXes by
themselves (which levels those are: test_host_launches.py)."""
import numpy as np
import pytest

from test_gpu_mixed_entries import INPUTS, WIDEST, check

pytestmark = pytest.mark.gpu


# both parts in every form: quads, a round beside quads, pairs of one component each, full rounds
@pytest.mark.parametrize("N,l,ks_t,ks_basebit,sizes", [
    (1024, 3, 8, 2, [(500, 525), (430, 560)]), (1024, 3, 5, 3, [(501, 525)]), (1024, 2, 8, 2, [(289, 911)]),
    (512, 3, 8, 2, [(288, 912)]), (256, 3, 8, 2, [(801, 370), (300, 900)])])
def test_two_launches_give_the_same_words(N, l, ks_t, ks_basebit, sizes):
    import paper_1906_00148_amd as pkg
    from paper_1906_00148_amd import binding
    with pkg.Context(pkg.Params(n=20, N=N, l=l, bg_bit=7, ks_t=ks_t, ks_basebit=ks_basebit), 31, INPUTS + 2 * WIDEST) as ctx:
        ctx.encrypt_bits(np.random.default_rng(3).integers(0, 2, INPUTS), 5, np.arange(INPUTS))
        ctx.set_option(binding.OPT_NATIVE_MUX, 1)
        for tracking in (False, True):
            ctx.set_round_tracking(tracking)
            for gates, muxes in sizes:
                check(binding, ctx, gates, muxes, gates)
