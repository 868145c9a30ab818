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


# wavefronts of one image, of pairs, and of pairs and one, and with fewer images than the others; few blocks for a tap row each, and many for all
@pytest.mark.parametrize("n,B", [(1, 1), (2, 3), (3, 64), (1, 65), (2, 129), (3, 131), (3, 192), (4, 192), (2, 257), (30, 7), (40, 66), (40, 130)])
def test_conv2_weight_gradient_forms(ps, n, B):
    """d W2 within the error of fp32 matrix instructions (1.5e-7, above), d b2 within four roundings of 2^-24: a lane
    adds a value for a row of windows, seven of an image."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(11 * n + B)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
        q = ps.worker_grads_batched(ctx, range(n), [0] * n, [synth.minibatch_id(w, 0) for w in range(n)], x, y)
        ps.ps_sync(ctx)
        for i in {0, n // 2, n - 1}:
            d2, u = _d2(ps, ctx, i)
            got = torch.from_numpy(ps.ps_get_grad(ctx, q[i])).cuda().double()
            want, want_b = torch.matmul(d2, u.transpose(1, 2)).sum(0).flatten(), d2.sum((0, 2))
            assert float((got[OFF_W2:OFF_B2] - want).norm() / want.norm()) <= 1.5e-7
            assert float((got[OFF_B2:OFF_B2 + 32] - want_b).norm() / want_b.norm()) <= 4 * 2.0 ** -24
    finally:
        ps.ps_destroy(ctx)


# the forms above, with a worker behind every worker
@pytest.mark.parametrize("n,B", [(2, 1), (2, 3), (4, 64), (2, 65), (2, 129), (30, 7), (40, 66)])
def test_rows_below_a_map_are_zero(ps, n, B):
    """Rows 14 to 16 of a worker's last map are the first of the next worker's: whether those are infinite must not show."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(23 * n + B)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    theta = synth.he_uniform_theta(5)
    broken = theta.copy()
    broken[144:160] = np.inf  # conv1's bias
    ctx = ps.ps_init(ps.make_config(n, B, 2, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, theta)
        ps.ps_load_snapshot(ctx, 1, broken, 0)
        seen = []
        for other in (0, 1):
            q = ps.worker_grads_batched(ctx, range(n), [0, other] * (n // 2), [synth.minibatch_id(w, 0) for w in range(n)], x, y)
            ps.ps_sync(ctx)
            assert np.isinf(ps.ps_debug_last_activations(ctx, 1)["pool1_val"]).all() == (other == 1)
            seen.append([ps.ps_get_grad(ctx, q[i]) for i in (0, n - 2)])
            for e in q:
                ps.ps_apply_async(ctx, e, 0.0)
        for one, among in zip(*seen):
            assert np.isfinite(one).all()
            np.testing.assert_array_equal(one, among)
    finally:
        ps.ps_destroy(ctx)


@pytest.mark.parametrize("n,B", [(1, 1), (2, 3), (3, 64), (1, 65), (2, 129), (30, 7), (40, 66)])
def test_infinite_activations_that_no_gradient_meets(ps, n, B):
    """A gradient of zero takes nothing out of an infinite pool1 value, wherever the winner of its window is.  (Channel 13
    has two infinite values in an image; they make the outputs that see them minus infinity, which win nothing.)"""
    import torch
    theta = synth.he_uniform_theta(5)
    theta[13 * 9:14 * 9] = 0
    theta[13 * 9 + 4] = 5e37
    theta[160:4768].reshape(32, 16, 9)[:, 13] = -1.2e-38
    theta[4768:4800] = 1.0
    g = torch.Generator(device="cuda")
    g.manual_seed(29 * n + B)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    x.scatter_(-1, torch.randint(0, ps.IMAGE_PIXELS, (n, B, 2), device="cuda", generator=g), 8.0)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, theta)
        q = ps.worker_grads_batched(ctx, range(n), [0] * n, [synth.minibatch_id(w, 0) for w in range(n)], x, y)
        ps.ps_sync(ctx)
        for i in {0, n - 1}:
            d2, u = _d2(ps, ctx, i)
            inf, finite = torch.isinf(u).double(), torch.where(torch.isinf(u), 0.0, u)
            assert inf.any() and torch.isfinite(d2).all() and d2.any()
            assert not torch.matmul((d2 != 0).double(), inf.transpose(1, 2)).any()
            want, size = (torch.matmul(f(d2), f(finite).transpose(1, 2)).sum(0).flatten() for f in (lambda t: t, torch.abs))
            got = torch.from_numpy(ps.ps_get_grad(ctx, q[i])[OFF_W2:OFF_B2]).cuda().double()
            assert bool(((got - want).abs() <= 2.5 * 2.0 ** -24 * 1568 ** 0.5 * size + 1568 * 2.0 ** -150).all())
    finally:
        ps.ps_destroy(ctx)


# several pairs of images for a wavefront, in shares, with fc1's blocks of either width next to them and without
@pytest.mark.parametrize("n,B", [(1, 256), (10, 166), (22, 166), (19, 176), (50, 166)])
def test_gradients_repeat_bit_for_bit(ps, n, B):
    """The next images must not take the place of those that a wavefront still reads.  (Without the wait for those reads they
    did now and then, at 22 workers of 166 and 19 of 176; not in every run, so that this can miss it.)"""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(19 * n + B)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
        rows = ctx.workspace[:(2 + n) * ps.ROW_FLOATS * 4].view(torch.float32).view(-1, ps.ROW_FLOATS)[2:]
        first = None
        for _ in range(200):
            q = ps.worker_grads_batched(ctx, range(n), [0] * n, [synth.minibatch_id(w, 0) for w in range(n)], x, y)
            got = rows[:, :ps.P].clone()
            first = got if first is None else first
            assert bool((got == first).all())
            ps.ps_apply_sync(ctx, q, 0.0)
    finally:
        ps.ps_destroy(ctx)


# both sides of the lines at which eight, four and two wavefronts share an image: 128, 256 and 512 images
@pytest.mark.parametrize("n,B", [(1, 1), (2, 64), (1, 129), (2, 128), (1, 257), (4, 128), (1, 513), (2, 256), (1, 1025)])
def test_images_that_wavefronts_share(ps, n, B):
    """The maps and winners of conv1 and conv2 have the same bytes in a launch of n workers and among so many that no image is shared."""
    import torch
    many = n + 1024 // B + 1
    g = torch.Generator(device="cuda")
    g.manual_seed(17 * n + B)
    x = torch.rand(many, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (many, B), device="cuda", generator=g, dtype=torch.int32)
    seen = []
    ctx = ps.ps_init(ps.make_config(many, B, 1, many, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
        for k in (many, n):
            q = ps.worker_grads_batched(ctx, range(k), [0] * k, [synth.minibatch_id(w, 0) for w in range(k)], x[:k], y[:k])
            ps.ps_sync(ctx)
            seen.append([])
            for i in (0, n - 1):
                act, dbg = ps.ps_debug_last_activations(ctx, i), ps.ps_debug_last_batch(ctx, i)
                seen[-1] += [act["pool1_val"].copy(), act["pool2_val"].copy(), dbg["pool1"].copy(), dbg["pool2"].copy()]
            for e in q:
                ps.ps_apply_async(ctx, e, 0.0)
        for one, other in zip(*seen):
            np.testing.assert_array_equal(one, other)
    finally:
        ps.ps_destroy(ctx)


# one, two, four and eight images of a worker to a wavefront of conv2's forward pass, the last with fewer, and one or two of conv1's
@pytest.mark.parametrize("n,B", [(100, 30), (99, 50), (39, 129), (109, 101), (113, 200), (128, 121)])
def test_images_of_a_wavefront(ps, n, B):
    """The maps and winners of conv1 and conv2 have the same bytes in a launch of n workers and in one of a worker alone."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(31 * n + B)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n + 3, DROP_SEED, P_DROP))

    def maps(i):
        ps.ps_sync(ctx)
        act, dbg = ps.ps_debug_last_activations(ctx, i), ps.ps_debug_last_batch(ctx, i)
        return [act["pool1_val"].copy(), act["pool2_val"].copy(), dbg["pool1"].copy(), dbg["pool2"].copy()]

    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
        mbs = [synth.minibatch_id(w, 0) for w in range(n)]
        ps.worker_grads_batched(ctx, range(n), [0] * n, mbs, x, y)
        workers = (0, n // 2, n - 1)
        among = [maps(i) for i in workers]
        for i, want in zip(workers, among):
            ps.worker_grads_batched(ctx, [i], [0], [mbs[i]], x[i:i + 1], y[i:i + 1])
            for one, other in zip(want, maps(0)):
                np.testing.assert_array_equal(one, other)
    finally:
        ps.ps_destroy(ctx)


# fc1's forward pass and input gradient on both sides of the lines between their forms.  Batches up to 64: 32 x 32, 32 x 64 and
# 128 x 64 tiles; beyond: 32 x 32 tiles, 64 x 64 (up to 512, or up to 1,024 instead of more than 256 wide ones), and 128 x 128 with either half of the forward sums side by side or one after the
# other, and 64 x 64 ones of the input gradient with wavefronts that only multiply.  Whole tiles and remainders down to a column.
@pytest.mark.parametrize("n,B", [(1, 1), (6, 64), (7, 33), (9, 64), (17, 64), (64, 32), (64, 33), (63, 64), (107, 40),
                                 (1, 65), (1, 512), (1, 640), (1, 641), (2, 130), (5, 128), (5, 129), (3, 193), (32, 100), (33, 97), (64, 128), (65, 90), (40, 257),
                                 (21, 129), (22, 130), (33, 176), (43, 129)])
def test_fc1_forms(ps, n, B):
    """Activations and gradients of every image within what an fp32 sum may be off, and with the same bytes when their worker is
    alone.  The partial sums of K terms of size 1 are sqrt(k) large, each rounded by 2^-24 / sqrt(3) of that, and the result is
    sqrt(K) large: 2^-24 sqrt(K / 6) of it, here for halves of K = 1568 and for K = 512.  (A term of the split left out gives
    1e-6 and more.)"""
    import torch
    theta = synth.he_uniform_theta(5)
    g = torch.Generator(device="cuda")
    g.manual_seed(41 * n + B)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n + 2, DROP_SEED, P_DROP))

    def layer(i):
        ps.ps_sync(ctx)
        dbg, act = ps.ps_debug_last_batch(ctx, i), ps.ps_debug_last_activations(ctx, i)
        return {k: v.copy() for k, v in (*dbg.items(), *act.items()) if k in ("keep", "hdrop", "pool2_val", "d3", "dpool2")}

    def off(got, want):
        return float((torch.from_numpy(got).cuda().double() - want).norm(dim=1).div(want.norm(dim=1)).nan_to_num(0.0).max())

    try:
        ps.ps_set_weights(ctx, theta)
        w3, b3 = (torch.from_numpy(theta[a:b]).cuda().double() for a, b in ((4800, 807616), (807616, 808128)))
        w3 = w3.view(512, 1568)
        mbs = [synth.minibatch_id(w, 0) for w in range(n)]
        ps.worker_grads_batched(ctx, range(n), [0] * n, mbs, x, y)
        among = {i: layer(i) for i in {0, n - 1}}
        for i, seen in among.items():
            p2, keep, d3 = (torch.from_numpy(seen[k]).cuda().double() for k in ("pool2_val", "keep", "d3"))
            assert off(seen["hdrop"], (p2 @ w3.t() + b3).clamp_min(0) * keep / (1 - P_DROP)) <= 2.0 ** -24 * (784 / 6) ** 0.5
            assert off(seen["dpool2"], (d3 @ w3) * (p2 > 0)) <= 2.0 ** -24 * (512 / 6) ** 0.5
            ps.worker_grads_batched(ctx, [i], [0], [mbs[i]], x[i:i + 1], y[i:i + 1])
            alone = layer(0)
            for k in ("hdrop", "d3", "dpool2"):
                np.testing.assert_array_equal(alone[k], seen[k])
    finally:
        ps.ps_destroy(ctx)


def test_fc1_forward_of_a_ragged_batch(ps):
    """Batches a little beyond 128 do not pay for an empty half of their tiles: 21 of 129, 504 tiles of 64 x 64, take no longer than
    32 of 128, 512 (measured 48 and 50 us; in 128 x 128 tiles 60)."""
    import torch
    us = []
    for n, B in ((21, 129), (32, 128)):
        x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda")
        y = torch.zeros(n, B, device="cuda", dtype=torch.int32)
        ctx = ps.ps_init(ps.make_config(n, B, 1, n, DROP_SEED, P_DROP))
        try:
            ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
            best = np.inf
            for _ in range(6):
                ps.ps_profile_enable(ctx, True)
                for _ in range(10):
                    ps.worker_grads_batched(ctx, range(n), [0] * n, [synth.minibatch_id(w, 0) for w in range(n)], x, y)
                    ps.ps_drain_buffered(ctx, ps.DRAIN_SUM, 0.0)
                ps.ps_sync(ctx)
                ms, launches = ps.ps_profile_read(ctx)["gemm_split<Fc1FwdEpi>"]
                best = min(best, 1e3 * ms / launches)
            us.append(best)
        finally:
            ps.ps_destroy(ctx)
    print(us)
    assert us[0] <= 1.1 * us[1]


# both sides of the lines between 128 x 64 and 128 x 128 tiles next to conv2's gradients, and between those and a launch of
# their own; whole stages and a remainder
@pytest.mark.parametrize("n", [10, 11, 42, 43])
@pytest.mark.parametrize("B", [5, 16, 48, 51])
def test_fc1_weight_gradient_tiles(ps, n, B):
    """Every row of d fc1.W against 64 bits: within the error of fp32 matrix instructions (1.5e-7, above)."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(13 * n + B)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
        q = ps.worker_grads_batched(ctx, range(n), [0] * n, [synth.minibatch_id(w, 0) for w in range(n)], x, y)
        ps.ps_sync(ctx)
        for i in (0, n - 1):
            act = ps.ps_debug_last_activations(ctx, i)
            d3, p2 = (torch.from_numpy(act[k]).cuda().double().view(B, -1) for k in ("d3", "pool2_val"))
            want = d3.t() @ p2
            got = torch.from_numpy(ps.ps_get_grad(ctx, q[i])[4800:807616]).cuda().double().view(512, 1568)
            some = want.norm(dim=1) > 0
            assert float(((got - want).norm(dim=1)[some] / want.norm(dim=1)[some]).max()) <= 1.5e-7
            assert not bool(got[~some].any())
    finally:
        ps.ps_destroy(ctx)


# both sides of the lines between 64 x 128 and 128 x 128 tiles in a launch of their own; whole stages and a remainder
@pytest.mark.parametrize("n,B", [(43, 1), (43, 17), (170, 96), (170, 97), (160, 97), (160, 128), (161, 128), (43, 128), (43, 129),
                                 (175, 128), (176, 128), (234, 96), (235, 96)])
def test_fc1_weight_gradient_alone(ps, n, B):
    """A sum's order depends on the batch alone: the same bytes as next to conv2's gradients, in 128 x 64 tiles, which are held
    to 64 bits above."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(13 * n + B)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n + 2, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
        mbs = [synth.minibatch_id(w, 0) for w in range(n)]
        q = ps.worker_grads_batched(ctx, range(n), [0] * n, mbs, x, y)
        for i in (0, n - 1):
            q += ps.worker_grads_batched(ctx, [i], [0], [mbs[i]], x[i:i + 1], y[i:i + 1])
        ps.ps_sync(ctx)
        for i, alone in ((0, q[n]), (n - 1, q[n + 1])):
            among = ps.ps_get_grad(ctx, q[i])[4800:807616]
            assert among.any()
            np.testing.assert_array_equal(among, ps.ps_get_grad(ctx, alone)[4800:807616])
    finally:
        ps.ps_destroy(ctx)


# the error of sums that are kept in registers over eight images
@pytest.mark.parametrize("n,B,registers", [(8, 200, 7.92e-8), (8, 1024, 6.45e-8), (4, 4096, 7.16e-8)])
def test_conv1_weight_gradient_error(ps, n, B, registers):
    """conv1 has a partial sum per image; adding up those of a large batch must not lose what the sums had."""
    import torch
    theta = synth.he_uniform_theta(5)
    W2 = torch.from_numpy(theta[OFF_W2:OFF_B2]).cuda().double().view(32, 144)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    ctx = ps.ps_init(ps.make_config(n, B, 1, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, theta)
        q = ps.worker_grads_batched(ctx, range(n), [0] * n, [synth.minibatch_id(w, 0) for w in range(n)], x, y)
        ps.ps_sync(ctx)
        want, err = [], []
        for i in range(n):
            d2, _ = _d2(ps, ctx, i)
            code = torch.from_numpy(ps.ps_debug_last_batch(ctx, i)["pool1"]).cuda().long().view(B, 16, 196)
            dp1 = torch.nn.functional.fold(torch.matmul(W2.t(), d2), (14, 14), 3, padding=1).view(B, 16, 196) * ((code & 4) > 0)
            win = torch.zeros(B, 16, 196, 4, device="cuda", dtype=torch.float64).scatter_(-1, (code & 3).unsqueeze(-1), dp1.unsqueeze(-1))
            d1 = win.view(B, 16, 14, 14, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(B, 16, 784)
            pix = torch.nn.functional.unfold(x[i].double().view(B, 1, 28, 28), 3, padding=1)
            want.append(torch.matmul(d1, pix.transpose(1, 2)).sum(0).flatten())
            err.append(torch.from_numpy(ps.ps_get_grad(ctx, q[i])[:144]).cuda().double() - want[-1])
        assert float(torch.cat(err).norm() / torch.cat(want).norm()) <= registers
    finally:
        ps.ps_destroy(ctx)


@pytest.mark.parametrize("n,B", [(2, 32), (4, 130), (40, 64)])
@pytest.mark.parametrize("what", ["nan", "infinite conv2 weight", "infinite fc1 weight", "half saturated", "saturated"])
def test_a_diverged_network_is_not_slow(ps, n, B, what):
    """Sums that the split loses are formed again at the rate of fp32 matrix instructions, 2.7 times slower, from
    operands that come straight from memory; where every sum is NaN not even that, and images whose gradients are
    tiny cost nothing among others."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    theta = synth.he_uniform_theta(1)
    broken = theta.copy()
    if what == "nan":
        broken[:] = np.nan
    elif "saturated" in what:
        broken[808128:813248] *= 0.1
        broken[813248 + 3] = 70.0
        y[:, :B // 2 if what == "half saturated" else B] = 3
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
        assert min(times[1]) <= (1.3 if what == "half saturated" else 8) * min(times[0])
    finally:
        ps.ps_destroy(ctx)


# ------------------------------------------------------- every contraction against 64 bits on its own operands

OFF_W3, OFF_B3 = 4800, 807616
LAYERS = ("conv2 forward", "fc1 forward", "fc1 input gradient", "fc1 weight gradient", "conv2 input gradient", "conv2 weight gradient",
          "conv2 bias gradient")


def _results(ps, ctx, i, q, theta, x):
    """{layer: (what the kernels made, the same in 64 bits from what they were given, the same of all magnitudes)} of
    worker i, entry q.  No dropout."""
    import torch
    act, dbg = ps.ps_debug_last_activations(ctx, i), ps.ps_debug_last_batch(ctx, i)
    B = dbg["pred"].size
    grad, th = ps.ps_get_grad(ctx, q), torch.from_numpy(theta).cuda().double()
    code2, code1 = (torch.from_numpy(dbg[k]).cuda().long().view(B, c, -1) for k, c in (("pool2", 32), ("pool1", 16)))
    d2, u = _d2(ps, ctx, i)
    pix = torch.nn.functional.unfold(x.double().view(B, 1, 28, 28), 3, padding=1)

    def layers(f):
        W2, b2, W3, b3 = f(th[160:4768]).view(32, 144), f(th[4768:4800]), f(th[4800:807616]).view(512, 1568), f(th[807616:808128])
        p2, d3 = (f(torch.from_numpy(act[k]).cuda().double()) for k in ("pool2_val", "d3"))
        z = torch.matmul(W2, f(u)).view(B, 32, 7, 2, 7, 2).permute(0, 1, 2, 4, 3, 5).reshape(B, 32, 49, 4)
        z = (z.gather(-1, (code2 & 3).unsqueeze(-1))[..., 0] + b2.view(1, 32, 1)).clamp_min(0)
        dp1 = torch.nn.functional.fold(torch.matmul(W2.t(), f(d2)), (14, 14), 3, padding=1).view(B, 16, 196) * ((code1 & 4) > 0)
        w1 = torch.zeros(B, 16, 196, 4, device="cuda", dtype=torch.float64).scatter_(-1, (code1 & 3).unsqueeze(-1), dp1.unsqueeze(-1))
        d1 = w1.view(B, 16, 14, 14, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(B, 16, 784)
        out = (z, (p2 @ W3.t() + b3).clamp_min(0), d3 @ W3 * ((code2 & 4) > 0).view(B, 1568), d3.t() @ p2,
               torch.matmul(d1, f(pix).transpose(1, 2)).sum(0), torch.matmul(f(d2), f(u).transpose(1, 2)).sum(0), f(d2).sum((0, 2)))
        return [t.flatten().cpu().numpy() for t in out]

    got = (act["pool2_val"], dbg["hdrop"], act["dpool2"], grad[OFF_W3:OFF_B3], grad[:144], grad[OFF_W2:OFF_B2], grad[OFF_B2:OFF_W3])
    return {k: (g.astype(np.float64).ravel(), w, m) for k, g, w, m in zip(LAYERS, got, layers(lambda t: t), layers(torch.abs))}


# 2.5 u sqrt(K) of what is summed, as in the parity tests, at K = 1568, and half a unit of the smallest number at each step
def _compare(res, layers=LAYERS, floor=0.0):
    for k in layers:
        got, want, size = res[k]
        assert np.isfinite(got).all() and np.isfinite(want).all(), k
        over = np.abs(got - want) / (2.5 * 2.0 ** -24 * 1568 ** 0.5 * size + 1568 * 2.0 ** -150 + floor * size.max())
        assert over.max() <= 1, (k, over.max(), np.abs(want).max())


def _run(ps, theta, n, B, seed=17, labels=None, seen=None):
    """The last of n workers on `theta`, the others on ordinary weights; no dropout, which would scale values up."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, B), device="cuda", generator=g, dtype=torch.int32)
    if labels is not None:
        y[:] = labels
    ctx = ps.ps_init(ps.make_config(n, B, 2, n, DROP_SEED, 0.0))
    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))
        ps.ps_load_snapshot(ctx, 1, theta, 0)
        q = ps.worker_grads_batched(ctx, range(n), [0] * (n - 1) + [1], [synth.minibatch_id(w, 0) for w in range(n)], x, y)
        ps.ps_sync(ctx)
        if seen is not None:
            seen.update(ps.ps_debug_last_activations(ctx, n - 1))
        return _results(ps, ctx, n - 1, q[-1], theta, x[-1]), _results(ps, ctx, 0, q[0], synth.he_uniform_theta(5) if n > 1 else theta, x[0])
    finally:
        ps.ps_destroy(ctx)


HUGE = np.float32(3.3999e38)  # finite, and infinite when rounded to 16 bits

# launches of every form: images shared or not, fc1 in chunks on tiles of three shapes, its forward sums in halves and its input
# gradient in one chain on tiles of every shape, its weight gradient with conv2's (ragged or not) or by itself, in wide tiles or
# not, conv2's weight gradient in shares or not
FORMS = [(2, 16), (3, 33), (20, 40), (80, 40), (2, 130), (10, 130), (70, 130), (12, 65), (1, 100), (12, 40), (107, 40), (5, 129), (40, 100),
         (33, 176)]


@pytest.mark.parametrize("n,B", FORMS)
@pytest.mark.parametrize("where", ["pool1", "conv2 weight", "fc1 weight", "pool2"])
def test_values_that_cannot_be_split(ps, n, B, where):
    """Finite operands of 3.4e38 in each contraction, next to other operands so small that every sum is finite."""
    theta = synth.he_uniform_theta(5)
    W2, W3 = theta[160:4768].reshape(32, 16, 9), theta[4800:807616].reshape(512, 1568)
    if where == "pool1":            # operand of conv2's forward and weight gradient: channel 13
        theta[144 + 13] = HUGE
        W2[:, 13] *= 1e-5
        W3 *= 1e-3
    elif where == "conv2 weight":   # of conv2's forward and input gradient
        theta[:144] *= 1e-3
        W2[21, 7, 2] = HUGE         # a corner of the window: what lies outside the map must not count
        W3[:, 21 * 49:22 * 49] *= 1e-3
    elif where == "fc1 weight":     # of fc1's forward and input gradient: a feature of the edge tiles
        W2[31] *= 1e-6
        W3[300, 1560] = HUGE
    else:                           # of fc1's forward and weight gradient, features on both sides of the edge
        theta[4768 + 31] = HUGE
        W3[:, 31 * 49:] *= 1e-6
    broken, good = _run(ps, theta, n, B)
    _compare(broken)
    _compare(good)


@pytest.mark.parametrize("n,B", FORMS)
def test_products_just_below_overflow(ps, n, B):
    """A product within 2^-9 of the largest float, whose factors both round up in 16 bits: the leading product of the
    split is infinite, the sum is not."""
    import torch
    theta = synth.he_uniform_theta(5)
    W3 = theta[4800:807616].reshape(512, 1568)
    top = float(np.finfo(np.float32).max)
    with_pool2 = {}
    _run(ps, theta, n, B, seen=with_pool2)
    p2 = torch.from_numpy(with_pool2["pool2_val"])
    bf16 = lambda v: float(torch.tensor(v, dtype=torch.float32).bfloat16())  # noqa: E731
    for feat in range(1567, -1, -1):                            # its largest value is to meet a weight as large as can be
        value = float(p2[:, feat].max())
        w = np.float32(top * (1 - 2.0 ** -12) / max(value, 1.1))
        if value > 1.1 and bf16(w) * bf16(value) > top * (1 + 2.0 ** -20):
            break
    assert feat and top * (1 - 2.0 ** -9) < float(w) * value < top
    W3[300] = 0
    W3[300, feat] = w
    broken, _ = _run(ps, theta, n, B)
    got, want, _ = (a.reshape(B, 512)[:, 300] for a in broken["fc1 forward"])
    assert np.isfinite(want).all() and want.max() > top * (1 - 2.0 ** -9)
    np.testing.assert_allclose(got, want, rtol=2.0 ** -22)     # one product and 1567 zeros, however they are added


@pytest.mark.parametrize("n,B", FORMS)
@pytest.mark.parametrize("what", ["margin 76", "margin 80", "pixels", "conv2 weights", "fc1 weights"])
def test_tiny_operands_keep_their_bits(ps, n, B, what):
    """Parts below 2^-133 do not exist, so operands below 2^-110 have fewer than 24 bits in the split: gradients of a
    minibatch whose every image is classified with a margin of 76 or 80 in the logits, activations and weights of 1e-36."""
    theta = synth.he_uniform_theta(5)
    labels = None
    if what.startswith("margin"):
        labels = 3
        theta[808128:813248] *= 0.01
        theta[813248 + 3] = float(what.split()[1])
    elif what == "pixels":          # pool1 values, by way of conv1's weights
        theta[:144] *= 1e-36
    elif what == "conv2 weights":   # and pool2 values
        theta[160:4768] *= 1e-36
    else:
        theta[4800:807616] *= 1e-36
    broken, good = _run(ps, theta, n, B, labels=labels)
    assert 0 < max(np.abs(want).max() for _, want, _ in broken.values())
    _compare(broken)
    _compare(good)


@pytest.mark.parametrize("n,B", FORMS)
def test_tiny_gradients_among_others(ps, n, B):
    """Every third image is classified with a margin of 76: the gradients are those of the minibatch.  (What comes of such
    an image alone may have fewer bits; that is below 2^-100 of a tensor's largest.)"""
    import torch
    theta = synth.he_uniform_theta(5)
    theta[808128:813248] *= 0.01
    theta[813248 + 3] = 76.0
    labels = torch.full((n, B), 5, device="cuda", dtype=torch.int32)
    labels[:, ::3] = 3
    labels[:, 1] = 3
    broken, _ = _run(ps, theta, n, B, labels=labels)
    _compare(broken, ("conv2 forward", "fc1 forward", "fc1 weight gradient", "conv2 input gradient", "conv2 weight gradient", "conv2 bias gradient"), 2.0 ** -100)


@pytest.mark.parametrize("n,B", [(20, 40), (80, 40), (70, 130), (4, 256), (12, 40), (107, 40), (5, 129), (40, 100), (33, 176)])
@pytest.mark.parametrize("what", ["huge", "tiny", "some tiny"])
def test_sums_formed_again_do_not_depend_on_the_launch(ps, n, B, what):
    """Which sums are lost, and what they are then, is decided by tiles that all forms of a launch share: conv1's, conv2's
    and fc1's weight gradients, fc1's activations and input gradient of a worker have the same bytes alone and among n."""
    import torch

    def layer(i):
        return [v.copy().view(np.int32) for v in (ps.ps_debug_last_batch(ctx, i)["hdrop"], ps.ps_debug_last_activations(ctx, i)["dpool2"])]

    theta = synth.he_uniform_theta(5)
    g = torch.Generator(device="cuda")
    g.manual_seed(19)
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda", generator=g)
    y = torch.full((n, B), 3, device="cuda", dtype=torch.int32)
    if what == "huge":
        theta[144 + 13] = HUGE
        theta[160:4768].reshape(32, 16, 9)[:, 13] *= 1e-5
        theta[4800:807616] *= 1e-3
    else:
        theta[808128:813248] *= 0.01
        theta[813248 + 3] = 80.0
        if what == "some tiny":
            y[:, ::3] = 5
    ctx = ps.ps_init(ps.make_config(n, B, 1, n + 1, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, theta)
        mbs = [synth.minibatch_id(w, 7) for w in range(n)]
        entries = ps.worker_grads_batched(ctx, range(n), [0] * n, mbs, x, y)
        ps.ps_sync(ctx)
        layers = {i: layer(i) for i in (0, n - 1)}
        for i in (0, n - 1):
            (q,) = ps.worker_grads_batched(ctx, [i], [0], [mbs[i]], x[i:i + 1], y[i:i + 1])
            ps.ps_sync(ctx)
            for a, b in zip(layers[i], layer(0)):
                assert a.any() and np.array_equal(a, b)
            among, alone = ps.ps_get_grad(ctx, entries[i]), ps.ps_get_grad(ctx, q)
            assert among[:OFF_B3].any() and np.array_equal(among[:OFF_B3].view(np.int32), alone[:OFF_B3].view(np.int32))
            ps.ps_apply_async(ctx, q, 0.0)
    finally:
        ps.ps_destroy(ctx)
