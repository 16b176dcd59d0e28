"""Levels of at most one gate per compute unit (N = 1024, l = 3) give the words of one wavefront per gate
(SHE_OPT_SPLIT_BELOW = 0): the smallest key lengths, one gate, and one gate on every compute unit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tracking", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 40])
def test_key_lengths_and_counts(n, tracking):
    import torch
    import paper_1906_00148_amd as pkg
    inputs, widest = 64, torch.cuda.get_device_properties(0).multi_processor_count + 1
    rng = np.random.default_rng(n)
    codes = rng.integers(0, 10, widest).astype(np.uint8)
    a, b = (rng.integers(0, inputs, widest).astype(np.uint32) for _ in range(2))
    out = np.arange(inputs, inputs + widest, dtype=np.uint32)
    with pkg.Context(pkg.Params(n=n, N=1024, l=3, bg_bit=7, ks_t=8, ks_basebit=2), 31, inputs + widest) as ctx:
        ctx.encrypt_bits(rng.integers(0, 2, inputs).astype(np.uint8), 5, np.arange(inputs))
        rows = ctx._pool_tensor.view(ctx.capacity, -1)[inputs:]
        ctx.set_round_tracking(tracking)

        def run(count):
            rows.zero_()
            ctx.eval_gates(codes[:count], a[:count], b[:count], out[:count])
            return rows[:count].cpu().numpy().copy()

        default = ctx.get_option(pkg.OPT_SPLIT_BELOW)
        ctx.set_option(pkg.OPT_SPLIT_BELOW, 0)
        want = run(widest)
        ctx.set_option(pkg.OPT_SPLIT_BELOW, default)
        for count in (1, 2, widest - 1, widest):
            assert np.array_equal(run(count), want[:count]), count
