"""The fp32 contractions on the bf16 matrix cores, layer by layer against 64 bits on the kernels' own operands."""
import numpy as np
import pytest

from paper_2406_05546_amd import synth

pytestmark = pytest.mark.gpu
DROP_SEED, P_DROP = 0xBEEF, 0.25
OFF_W2, OFF_B2 = 160, 4768


@pytest.fixture(scope="module")
def ps():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2406_05546_amd import binding
    return binding


def _d2(ps, ctx, i):
    """Gradient at conv2's outputs [B, 32, 196] in 64 bits, as worker i's own buffers give it."""
    import torch
    act, dbg = ps.ps_debug_last_activations(ctx, i), ps.ps_debug_last_batch(ctx, i)
    code = torch.from_numpy(dbg["pool2"]).cuda().long().view(-1, 32, 49)
    g = torch.from_numpy(act["dpool2"]).cuda().double().view(-1, 32, 49) * ((code & 4) > 0)
    win = torch.zeros(*code.shape, 4, device="cuda", dtype=torch.float64).scatter_(-1, (code & 3).unsqueeze(-1), g.unsqueeze(-1))
    d2 = win.view(-1, 32, 7, 7, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(-1, 32, 196)
    p1 = torch.from_numpy(act["pool1_val"]).cuda().double().view(-1, 16, 14, 14)
    return d2, torch.nn.functional.unfold(p1, 3, padding=1)


# error of the fp32 matrix instructions, a rounding at every step, on these inputs
@pytest.mark.parametrize("n,B,share,fp32", [(8, 200, 1.0, 1.110e-7), (8, 200, 0.2, 1.442e-7), (2, 256, 0.2, 1.506e-7), (2, 32, 1.0, 1.096e-7)])
def test_conv2_weight_gradient_error(ps, n, B, share, fp32):
    """No further from 64 bits than fp32 sums, and on either side of them: the weight gradients of a drain are added
    up, and an error that has a sign is not averaged out.  `share` of the pixels are not zero."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    if share < 1:
        x = torch.where(torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g) < share, x, torch.zeros_like(x))
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
        q = ps.worker_grads_batched(ctx, range(n), [0] * n, [synth.minibatch_id(w, 0) for w in range(n)], x, y)
        ps.ps_sync(ctx)
        want, err = [], []
        for i in range(n):
            d2, u = _d2(ps, ctx, i)
            want.append(torch.matmul(d2, u.transpose(1, 2)).sum(0).flatten())
            err.append(torch.from_numpy(ps.ps_get_grad(ctx, q[i])[OFF_W2:OFF_B2]).cuda().double() - want[-1])
        want, err = torch.cat(want), torch.cat(err)
        assert float(err.norm() / want.norm()) <= fp32
        # independent roundings: the mean of N errors is below 4 / sqrt(N) of one (6e-5 of the cases are above)
        assert abs(float(err.mean())) <= 4 * float(err.std()) / err.numel() ** 0.5
    finally:
        ps.ps_destroy(ctx)


@pytest.mark.parametrize("n,B", [(2, 32), (4, 130), (40, 64)])
@pytest.mark.parametrize("what", ["nan", "infinite conv2 weight", "infinite fc1 weight"])
def test_a_diverged_network_is_not_slow(ps, n, B, what):
    """Sums that the split loses are formed again at the rate of fp32 matrix instructions, 2.7 times slower, from
    operands that come straight from memory; where every sum is NaN not even that."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    theta = synth.he_uniform_theta(1)
    broken = theta.copy()
    if what == "nan":
        broken[:] = np.nan
    else:
        broken[OFF_W2 if "conv2" in what else 4800 + 77 * 1568 + 3] = np.inf
    ctx = ps.ps_init(ps.make_config(n, B, 2, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, theta)
        ps.ps_load_snapshot(ctx, 1, broken, 0)
        ids = [synth.minibatch_id(w, 0) for w in range(n)]
        times = ([], [])
        for i in range(14):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            q = ps.worker_grads_batched(ctx, range(n), [i % 2] * n, ids, x, y)
            b.record()
            ps.ps_apply_sync(ctx, q, 0.0)
            b.synchronize()
            times[i % 2].append(a.elapsed_time(b))
        assert min(times[1]) <= 8 * min(times[0])
    finally:
        ps.ps_destroy(ctx)
