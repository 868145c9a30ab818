"""Kernels whose launches take different forms, at the sizes where these change."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2406_05546_amd import synth

pytestmark = pytest.mark.gpu
DROP_SEED, P_DROP = 0xBEEF, 0.25


@pytest.fixture(scope="module")
def ps():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_2406_05546_amd import binding
    return binding


@pytest.mark.parametrize("n", [1, 256, 257])
def test_elastic_slots_with_the_launch_and_uploaded(ps, n):
    """Slots in any order, in the kernel's arguments (up to 256) and from an uploaded list."""
    import torch
    alpha = 1 / 512
    ctx = ps.ps_init(ps.make_config(1, 1, n + 2, 1, DROP_SEED, P_DROP))
    try:
        g = torch.Generator(device="cuda")
        g.manual_seed(n)
        rows = ctx.workspace[:(3 + n) * ps.ROW_FLOATS * 4].view(torch.float32).view(-1, ps.ROW_FLOATS)  # server, ring
        rows[:, :ps.P] = torch.rand(3 + n, ps.P, device="cuda", generator=g) - 0.5
        slots = (torch.randperm(n + 2, generator=torch.Generator().manual_seed(n))[:n]).tolist()
        before = rows.clone()
        ps.ps_elastic_average(ctx, slots, alpha)
        ps.ps_sync(ctx)
        at = torch.tensor(slots, device="cuda") + 1
        d = before[at].double() - before[0].double()
        want = before.double()
        want[0] += alpha * d.sum(0)
        want[at] -= alpha * d
        # a difference, a product and n sums, each rounded to 2^-24 of values below 1 and of alpha times their sum
        assert float((rows.double() - want).abs().max()) <= 2.0 ** -24 * (2 + 2 * alpha * n ** 0.5 * n)
        untouched = [s + 1 for s in range(n + 2) if s not in slots]
        assert bool((rows[untouched] == before[untouched]).all())
    finally:
        ps.ps_destroy(ctx)


@pytest.mark.parametrize("n,B", [(1, 1), (3, 15), (2, 17), (5, 40)])
def test_evaluation_of_odd_numbers_of_images(ps, n, B):
    """Groups of 16 images and what is left of them."""
    import torch
    theta = synth.he_uniform_theta(9)
    x, y = synth.minibatches(9, [synth.minibatch_id(w, 0) for w in range(n)], B)
    ctx = ps.ps_init(ps.make_config(n, B, 1, 1, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, theta)
        x, y = x.reshape(n * B, -1), y.reshape(-1)
        loss, accuracy, pred = ps.ps_evaluate(ctx, -1, torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
        want, want_accuracy, want_pred, z = orc.evaluate(orc.Dims(), theta.astype(np.float64), x, y)
        assert abs(loss - want) <= 1e-6 * want  # 2^-24 sqrt(1568 / 6) of a logit, and the others' sums
        top = np.sort(np.asarray(z), axis=1)
        clear = top[:, -1] - top[:, -2] > 1e-5 * np.abs(z).max()
        np.testing.assert_array_equal(np.asarray(pred)[clear], np.asarray(want_pred)[clear])
        assert abs(accuracy - want_accuracy) <= (~clear).mean()
    finally:
        ps.ps_destroy(ctx)


def test_logits_of_an_evaluation(ps):
    """A logit is 512 products, summed in eights and those in a tree: its error over a thousand draws is that of the same sums
    formed here in 32 bits.  (Both are known to 1 part in 45; a chain of 128 to each wavefront has 2.4 times the error.)"""
    import torch
    N = 1000
    rng = np.random.default_rng(3)
    h = np.abs(rng.standard_normal((N, 512))).astype(np.float32)
    w = (1000 * rng.uniform(-1, 1, (N, 512)) * (6 / 512) ** 0.5).astype(np.float32)
    products = h.astype(np.float64) * w
    w *= np.where(products.sum(1) < 0, -1, 1).astype(np.float32)[:, None]
    exact, size = np.abs(products.sum(1)), np.sqrt((products ** 2).sum(1))
    part = np.zeros((N, 64), np.float32)
    for j in range(8):
        part = (h[:, 64 * j:64 * j + 64].astype(np.float64) * w[:, 64 * j:64 * j + 64] + part).astype(np.float32)
    while part.shape[1] > 1:
        part = part[:, :part.shape[1] // 2] + part[:, part.shape[1] // 2:]
    ctx = ps.ps_init(ps.make_config(1, 1, 1, 1, DROP_SEED, P_DROP))
    try:
        # fc1 without weights gives its biases, and the loss of class 1, whose logit is 0, is the logit of class 0
        ps.ps_set_weights(ctx, np.zeros(ps.P, np.float32))
        theta = ctx.workspace.view(torch.float32)[:ps.P]
        x, y = torch.zeros(1, ps.IMAGE_PIXELS, device="cuda"), torch.ones(1, device="cuda", dtype=torch.int32)
        hd, wd, got = torch.from_numpy(h).cuda(), torch.from_numpy(w).cuda(), np.empty(N)
        for i in range(N):
            theta[807616:808128] = hd[i]
            theta[808128:808640] = wd[i]
            got[i] = ps.ps_evaluate(ctx, -1, x, y)[0]
    finally:
        ps.ps_destroy(ctx)
    sure = exact > 30  # or the other classes' exp does not vanish
    assert sure.mean() > 0.95
    off, bound = (float(np.sqrt((((v - exact) / size)[sure] ** 2).mean())) for v in (got, part[:, 0].astype(np.float64)))
    print(f"error {off:.2e}, in 32 bits here {bound:.2e}")
    assert off <= 1.1 * bound


def test_evaluation_of_nan(ps):
    """Weights that are all NaN predict class 0, with a loss that is not a number."""
    import torch
    ctx = ps.ps_init(ps.make_config(1, 20, 1, 1, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, np.full(ps.P, np.nan, np.float32))
        x, y = synth.minibatches(9, [synth.minibatch_id(0, 0)], 20)
        loss, accuracy, pred = ps.ps_evaluate(ctx, -1, torch.from_numpy(x[0]).cuda(), torch.from_numpy(y[0]).cuda())
        assert np.isnan(loss) and not np.asarray(pred).any()
        assert abs(accuracy - float((y[0] == 0).mean())) < 1e-9
    finally:
        ps.ps_destroy(ctx)


def _clipped(theta, rows, mode, lr, clip):
    """In 64 bits: what a clipped drain of `rows` [K, P] makes of theta, on the GPU."""
    import torch
    rows = rows.double()
    c = torch.clamp(clip / rows.norm(dim=1), max=1.0)
    return theta.double() - lr * (c[:, None] * rows).sum(0)


# whole eights of rows, what is left of them, and less
@pytest.mark.parametrize("K", [1, 17, 18, 19, 29, 30, 35, 36, 112, 113])
@pytest.mark.parametrize("mode", [0, 1])
def test_clipped_drain(ps, K, mode):
    """Rows on both sides of the clipping limit, consecutive ones and, in a context, in another order; a second drain over
    other rows, which must not see anything of the first."""
    import torch
    lr, clip = 0.01, 4.0
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    rows = torch.zeros(2 * K, ps.ROW_FLOATS, device="cuda")
    size = torch.tensor([1e-2, 5e-3, 2e-2], device="cuda")[torch.arange(2 * K, device="cuda") % 3]
    rows[:, :ps.P] = (torch.rand(2 * K, ps.P, device="cuda", generator=g) * 2 - 1) * size[:, None]
    theta = torch.zeros(ps.ROW_FLOATS, device="cuda")
    theta[:ps.P] = torch.rand(ps.P, device="cuda", generator=g) - 0.5
    want = theta
    for part in (rows[:K], rows[K:]):
        want = _clipped(want, part, mode, lr, clip)
        ps.ps_drain_rows_mitigated(theta, part, mode, lr, 0.0, clip)
        # K roundings of weights below 1, and of a sum of K gradients below lr * 0.02 each
        assert float((theta.double() - want).abs().max()) <= 2.0 ** -24 * (2 + K)
        want = theta.double()
    ctx = ps.ps_init(ps.make_config(1, 1, 1, K + 2, DROP_SEED, P_DROP))
    try:
        start = np.linspace(-0.5, 0.5, ps.P, dtype=np.float32)
        ps.ps_set_weights(ctx, start)
        host = rows[:K + 1, :ps.P].cpu().numpy()
        first = ps.ps_queue_push_host(ctx, host[K], 0, 0, 0)
        for k in range(K - 1):
            ps.ps_queue_push_host(ctx, host[k], 0, 0, k)
        ps.ps_apply_async(ctx, first, 0.0)  # its place, in front of the others, is the next one handed out
        ps.ps_queue_push_host(ctx, host[K - 1], 0, 0, K)
        ps.ps_drain_buffered_mitigated(ctx, mode, lr, 0.0, clip)
        want = _clipped(torch.from_numpy(start).cuda(), rows[:K, :ps.P], mode, lr, clip)
        assert float((torch.from_numpy(ps.ps_get_weights(ctx)).cuda().double() - want).abs().max()) <= 2.0 ** -24 * (2 + K)
    finally:
        ps.ps_destroy(ctx)


@pytest.mark.parametrize("K", [5, 40])
def test_clipped_drain_beside_other_work(ps, K):
    """Next to matrix products on another stream: the bytes are the same."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    rows = torch.zeros(K, ps.ROW_FLOATS, device="cuda")
    rows[:, :ps.P] = (torch.rand(K, ps.P, device="cuda", generator=g) * 2 - 1) * 1e-2
    a = torch.rand(4096, 4096, device="cuda", generator=g)
    side, first = torch.cuda.Stream(), None
    torch.cuda.synchronize()
    for busy in [False] + [True] * 12:
        if busy:
            with torch.cuda.stream(side):
                for _ in range(3):
                    b = a @ a
        theta = torch.full((ps.ROW_FLOATS,), 0.25, device="cuda")
        for mode in (0, 1):
            ps.ps_drain_rows_mitigated(theta, rows, mode, 0.01, 0.0, 4.0)
        torch.cuda.synchronize()
        first = theta if first is None else first
        assert bool((theta == first).all())
    del b


@pytest.mark.parametrize("pieces", [(100, 100), (112, 113), (1, 8, 29, 30, 64, 120)])
def test_clipped_drain_in_pieces(ps, pieces):
    """A gradient's clip factor is its own: in order, a drain at once and in pieces of few and many rows give the same bytes."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(len(pieces))
    rows = torch.zeros(sum(pieces), ps.ROW_FLOATS, device="cuda")
    rows[:, :ps.P] = (torch.rand(len(rows), ps.P, device="cuda", generator=g) * 2 - 1) * 2e-2  # norms of about 10
    whole, cut = (torch.zeros(ps.ROW_FLOATS, device="cuda") for _ in range(2))
    ps.ps_drain_rows_mitigated(whole, rows, ps.DRAIN_SEQ, 0.5, 0.0, 4.0)
    for piece in rows.split(list(pieces)):
        ps.ps_drain_rows_mitigated(cut, piece, ps.DRAIN_SEQ, 0.5, 0.0, 4.0)
    assert whole.any() and torch.equal(whole, cut)


def test_clipped_drain_shares_the_chip(ps):
    """Next to worker kernels of up to a millisecond a small clipped drain, three launches, finds room between their blocks as a
    plain one of twice the rows does, one launch: measured 47 and 56 us, allowed four times as much.  (Blocks that need a compute
    unit for themselves wait until a worker kernel is through: 486 us.)"""
    import torch
    n = B = 256
    x = torch.rand(n, B, ps.IMAGE_PIXELS, device="cuda")
    y = torch.zeros(n, B, device="cuda", dtype=torch.int32)
    rows = torch.rand(16, ps.ROW_FLOATS, device="cuda")
    theta = torch.zeros(ps.ROW_FLOATS, device="cuda")
    mbs = [synth.minibatch_id(w, 0) for w in range(n)]
    ctx = ps.ps_init(ps.make_config(n, B, 1, n, DROP_SEED, P_DROP))
    try:
        ps.ps_set_weights(ctx, synth.he_uniform_theta(5))

        def next_to_workers(side, K, clip):
            """Median time of a drain, and whether all were through before the workers."""
            at = [torch.cuda.Event(enable_timing=True) for _ in range(26)]
            torch.cuda.synchronize()
            for _ in range(5):
                ps.worker_grads_batched(ctx, range(n), [0] * n, mbs, x, y)
                ps.ps_drain_buffered(ctx, ps.DRAIN_SUM, 0.0)
            workers = torch.cuda.current_stream().record_event()
            with torch.cuda.stream(side):
                at[0].record()
                for e in at[1:]:
                    ps.ps_drain_rows_mitigated(theta, rows[:K], ps.DRAIN_SEQ, 0.0, 0.0, clip)
                    e.record()
            at[-1].synchronize()
            beside = not workers.query()
            torch.cuda.synchronize()
            return float(np.median([a.elapsed_time(b) for a, b in zip(at, at[1:])])), beside

        # streams of a process share a few hardware queues: one that does not share the workers'
        side = next(s for s in (torch.cuda.Stream() for _ in range(8)) if next_to_workers(s, 16, 0.0)[1])
        plain, clipped = (np.median([next_to_workers(side, *how)[0] for _ in range(5)]) for how in ((16, 0.0), (8, 4.0)))
        print(f"plain {1e3 * plain:.0f} us, clipped {1e3 * clipped:.0f} us")
        assert clipped <= 4 * plain
    finally:
        ps.ps_destroy(ctx)


def test_store_runs_ahead_of_the_gpu(ps):
    """Forty appends into a store of two appends' size without a look at the GPU in between: each waits for no more than the
    oldest server step, and the updates are those of the ordered queue."""
    import torch
    n, B, lr = 3, 20, 0.01
    theta = synth.he_uniform_theta(4)
    mbs = [[synth.minibatch_id(w, r) for w in range(n)] for r in range(40)]
    x, y = (torch.from_numpy(a).cuda() for a in synth.minibatches(4, mbs[0], B))
    seen = []
    for lock_free in (True, False):
        ctx = ps.ps_init(ps.make_config(n, B, 2, 2 * n, DROP_SEED, P_DROP))
        try:
            ps.ps_set_weights(ctx, theta)
            for r in range(40):
                if lock_free:
                    ps.worker_grads_append(ctx, range(n), [0] * n, mbs[r], x, y)
                    ps.ps_store_consume(ctx, ps.DRAIN_SEQ, lr)
                    ps.ps_store_publish(ctx, 1)
                else:
                    ps.worker_grads_batched(ctx, range(n), [0] * n, mbs[r], x, y)
                    ps.ps_drain_buffered(ctx, ps.DRAIN_SEQ, lr)
                    ps.ps_snapshot_weights(ctx, 1)
            if lock_free:
                state = ps.ps_store_state(ctx)
                assert (state["claimed"], state["consumed"], state["version"]) == (40 * n, 40 * n, 40 * n)
            seen.append([ps.ps_get_weights(ctx), ps.ps_get_weights(ctx, 1)])
        finally:
            ps.ps_destroy(ctx)
    for one, other in zip(*seen):
        np.testing.assert_array_equal(one, other)
    np.testing.assert_array_equal(seen[0][0], seen[0][1])
