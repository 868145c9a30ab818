"""Work that a user of this library has it do, as cases that can be timed and compared.

Every case is one pass through the calls of include/ps_hotpath.h (by way of
paper_2406_05546_amd.binding), with everything it reads already on the GPU:

  step     a round (or several) of worker gradients followed by what the server does with them: one
           synchronous update, one update and pull per arrival, a buffered drain (summed or in order), or
           the lock-free store's append / consume / publish.  Workers compute on the snapshot they last
           pulled, and the weights the server publishes go into ring slots of their own, as while a
           server restarts: the gradients of a pass are then the same however many passes have gone
           before it, and only the server's weights move.
  drain    the update from buffered gradient rows that the caller owns (no context).
  evaluate inference over a held-out batch, answered on the host.
  elastic  one elastic-averaging step between the server's weights and worker-local copies.

Sizes are those of synth.paper_configs(), of bench.py and of the tests, plus odd ones in between.
"""
import torch

from paper_2406_05546_amd import binding as ps

P, ROW, PIX = ps.P, ps.ROW_FLOATS, ps.IMAGE_PIXELS
P_DROP = 0.25
DROP_SEED = (0x5EED << 32) | 0x2406
OFF_W1, OFF_B1, OFF_W2, OFF_B2, OFF_W3, OFF_B3, OFF_W4, OFF_B4 = 0, 144, 160, 4768, 4800, 807616, 808128, 813248
FLOP_PER_IMAGE = 10718208  # multiply-adds of the layers' forward and backward passes, times two
FLOP_FORWARD = 225792 + 1806336 + 1605632 + 10240


def listed():
    return [
        # the smallest training step: two workers, one synchronous update, weights published
        dict(name="sync_w2_b32", kind="step", rule="sync", n=2, batch=32, slots=1, rounds=1),
        # a ragged one, each worker on a snapshot of its own
        dict(name="sync_w5_b37", kind="step", rule="sync", n=5, batch=37, slots=5, rounds=1),
        # asynchronous server: four arrivals, an update and a pull for each
        dict(name="async_w4_b64", kind="step", rule="async", n=4, batch=64, slots=4, rounds=1),
        # one worker with a large minibatch
        dict(name="async_w1_b256", kind="step", rule="async", n=1, batch=256, slots=1, rounds=1),
        # stateless server down for 50 rounds of eight workers, then 400 gradients applied in order
        dict(name="outage_w8_b64", kind="step", rule="seq", n=8, batch=64, slots=1, rounds=50),
        # workers and server on two streams through the lock-free store
        dict(name="store_w16_b64", kind="step", rule="store", n=16, batch=64, slots=2, rounds=1),
        # 64 workers on eight resident versions, 64 asynchronous updates
        dict(name="versions_w64_b128", kind="step", rule="async", n=64, batch=128, slots=8, rounds=1),
        # the largest round: 65,536 images, the 256 gradients drained as one summed update
        dict(name="outage_w256_b256", kind="step", rule="sum", n=256, batch=256, slots=1, rounds=1),
        # recovery from a small backlog, in order, gradients clipped and the rate turned down
        dict(name="drain_64_seq_clip", kind="drain", rows=64, mode=1, clip=4.0, ref=16.0),
        # recovery from the large backlog (3.3 GB) as one summed update
        dict(name="drain_1024_sum", kind="drain", rows=1024, mode=0, clip=0.0, ref=0.0),
        # periodic evaluation of the server's weights
        dict(name="evaluate_w64_b128", kind="evaluate", n=64, batch=128),
        # one elastic step over 64 worker-local copies
        dict(name="elastic_64", kind="elastic", copies=64),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "drain", "evaluate", "elastic"])
    if kind == "drain":
        return dict(kind=kind, rows=_log(rng, 1, 1000), mode=rng.randrange(2), clip=rng.choice([0.0, 4.0]), ref=rng.choice([0.0, 16.0]))
    if kind == "elastic":
        return dict(kind=kind, copies=_log(rng, 1, 96))
    n, batch = _log(rng, 1, 250), _log(rng, 3, 250)
    if kind == "evaluate":
        return dict(kind=kind, n=n, batch=batch)
    rule = rng.choice(["sync", "async", "sum", "seq", "store"])
    rounds = rng.randint(1, 4) if rule in ("sum", "seq") and n * batch <= 4096 else 1
    return dict(kind=kind, rule=rule, n=n, batch=batch, slots=rng.randint(1, min(n, 8)), rounds=rounds)


# ---------------------------------------------------------------------------------------- inputs

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 16 + stream)
    return g


def _weights(seed, count):
    """`count` snapshots [count, P]: He-uniform weights, small biases, snapshots a few updates apart."""
    g = _gen(seed, 1)
    base = torch.zeros(P, device="cuda")
    for off, n, fan in ((OFF_W1, 144, 9), (OFF_W2, 4608, 144), (OFF_W3, 802816, 1568), (OFF_W4, 5120, 512)):
        base[off:off + n] = (torch.rand(n, device="cuda", generator=g) * 2 - 1) * (6.0 / fan) ** 0.5
    for off, n in ((OFF_B1, 16), (OFF_B2, 32), (OFF_B3, 512), (OFF_B4, 10)):
        base[off:off + n] = (torch.rand(n, device="cuda", generator=g) * 2 - 1) * 0.02
    step = (torch.rand(count, P, device="cuda", generator=g) * 2 - 1) * 1e-3
    return base + step


def _pick(theta, off, *shape):
    n = 1
    for s in shape:
        n *= s
    return theta[off:off + n].view(*shape)


def _unfold(x, h):
    """[N, C, h, h] -> [N, C*9, h*h], 3x3 neighbourhoods with a zero border."""
    return torch.nn.functional.unfold(x.view(x.shape[0], -1, h, h), 3, padding=1)


def _pool(v, h):
    """2x2 windows of [N, C, h*h]: values [N, C, h/2*h/2, 4] in scan order."""
    n, c = v.shape[:2]
    return v.view(n, c, h // 2, 2, h // 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(n, c, h * h // 4, 4)


def _forward(theta, x):
    """The net in 64 bits up to fc1's pre-activations: what a backward pass needs."""
    x = x.double()
    u1 = _unfold(x, 28)
    w1 = _pool(torch.matmul(_pick(theta, OFF_W1, 16, 9), u1) + _pick(theta, OFF_B1, 16, 1), 28)
    p1 = w1.amax(-1).clamp_min(0)
    u2 = _unfold(p1, 14)
    w2 = _pool(torch.matmul(_pick(theta, OFF_W2, 32, 144), u2) + _pick(theta, OFF_B2, 32, 1), 14)
    p2 = w2.amax(-1).clamp_min(0).reshape(-1, 1568)
    h = p2 @ _pick(theta, OFF_W3, 512, 1568).t() + _pick(theta, OFF_B3, 512)
    return u1, w1, p1, u2, w2, p2, h


CHUNK = 4096  # images per 64-bit pass


def _tied(theta, x):
    """Images in which a maximum or a ReLU is so near a tie that 32-bit sums may take it either way.  The
    bounds are 2.5 units of roundoff times the root of the sum's length, of a layer's largest value."""
    bad = []
    for part in x.split(CHUNK):
        _, w1, _, _, w2, _, h = _forward(theta, part)
        b = torch.zeros(part.shape[0], dtype=torch.bool, device=x.device)
        for w, k in ((w1, 9), (w2, 144)):
            reach = 2.5 * 2.0 ** -24 * k ** 0.5 * float(w.abs().amax())
            a, c = torch.maximum(w[..., 0], w[..., 1]), torch.maximum(w[..., 2], w[..., 3])
            top = torch.maximum(a, c)
            lesser = torch.where(a >= c, torch.minimum(w[..., 0], w[..., 1]), torch.minimum(w[..., 2], w[..., 3]))
            second = torch.maximum(torch.minimum(a, c), lesser)
            b |= ((top - second <= 2 * reach) | (top.abs() <= reach)).flatten(1).any(1)
        b |= (h.abs() <= 2.5 * 2.0 ** -24 * 1568 ** 0.5 * float(h.abs().amax())).any(1)
        bad.append(b)
    return torch.cat(bad)


def _images(seed, thetas, slot_of, n, batch):
    """Pixels in [0, 1) and labels for n minibatches.  An image with a decision at a tie, where both outcomes
    are right and lead to different gradients, is drawn again."""
    g = _gen(seed, 2)
    x = torch.rand(n, batch, PIX, device="cuda", generator=g)
    y = torch.randint(0, 10, (n, batch), device="cuda", generator=g, dtype=torch.int32)
    if thetas is not None:
        slot_of = torch.tensor(slot_of, device="cuda")
        for s in range(thetas.shape[0]):
            mine = (slot_of == s).nonzero().flatten()
            if not mine.numel():
                continue
            theta = thetas[s].double()
            part = x[mine].view(-1, PIX)
            todo = torch.arange(part.shape[0], device="cuda")
            while todo.numel():
                todo = todo[_tied(theta, part[todo])]
                part[todo] = torch.rand(todo.numel(), PIX, device="cuda", generator=g)
            x[mine] = part.view(mine.numel(), batch, PIX)
    return x, y


def _ids(case):
    """Per round: worker numbers, the slot each reads, logical minibatch ids."""
    n = case["n"]
    return list(range(n)), [w % case["slots"] for w in range(n)], [[(w << 32) | r for w in range(n)] for r in range(case["rounds"])]


def _rows(ctx, first, count):
    """Rows of the caller's workspace: the server's weights, then the ring slots, then the queue entries."""
    return ctx.workspace[:(first + count) * ROW * 4].view(torch.float32).view(-1, ROW)[first:first + count]


class _Context:
    """A context that goes away with the state that holds it."""

    def __init__(self, *cfg):
        self.ctx = ps.ps_init(ps.make_config(*cfg, seed=DROP_SEED, dropout_p=P_DROP))

    def __del__(self):
        torch.cuda.synchronize()
        ps.ps_destroy(self.ctx)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "drain":
        grads = torch.zeros(case["rows"], ROW, device="cuda")
        g = _gen(seed, 3)
        for k in range(case["rows"]):  # norms on both sides of the clipping limit
            grads[k, :P] = (torch.rand(P, device="cuda", generator=g) * 2 - 1) * (1e-2, 5e-3, 2e-2)[k % 3]
        theta = torch.zeros(ROW, device="cuda")
        theta[:P] = _weights(seed, 1)[0]
        return dict(case=case, theta=theta, grads=grads)
    if kind == "elastic":
        n = case["copies"]
        held = _Context(1, 1, n, 1)
        thetas = _weights(seed, n + 1)
        ps.ps_set_weights(held.ctx, thetas[n].cpu().numpy())
        for s in range(n):
            ps.ps_load_snapshot(held.ctx, s, thetas[s].cpu().numpy(), 0)
        return dict(case=case, held=held, slots=list(range(n)))
    n, batch = case["n"], case["batch"]
    if kind == "evaluate":
        held = _Context(n, batch, 1, 1)
        ps.ps_set_weights(held.ctx, _weights(seed, 1)[0].cpu().numpy())
        x, y = _images(seed, None, None, n, batch)
        return dict(case=case, held=held, x=x.view(-1, PIX), y=y.view(-1))
    workers, slot_of, ids = _ids(case)
    slots, rounds = case["slots"], case["rounds"]
    thetas = _weights(seed, slots)
    x, y = _images(seed, thetas, slot_of * rounds, n * rounds, batch)
    # ring: the snapshots that the workers read, then the slots that the server publishes into
    published = n if case["rule"] == "async" and n <= 8 else 1
    capacity = 2 * n if case["rule"] == "store" else n * rounds
    held = _Context(n, batch, slots + published, capacity)
    ps.ps_set_weights(held.ctx, thetas[0].cpu().numpy())
    for s in range(1, slots):
        ps.ps_load_snapshot(held.ctx, s, thetas[s].cpu().numpy(), 0)
    return dict(case=case, held=held, workers=workers, slot_of=slot_of, ids=ids, published=published, capacity=capacity,
                x=x.view(rounds, n, batch, PIX), y=y.view(rounds, n, batch), loss=torch.zeros(rounds, n, device="cuda"))


# ---------------------------------------------------------------------------------------- one pass

LR = 0.005
ALPHA = 1.0 / 512


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "drain":
        ps.ps_drain_rows_mitigated(state["theta"], state["grads"], case["mode"], LR, case["ref"], case["clip"])
        return state["theta"]
    ctx = state["held"].ctx
    if kind == "evaluate":
        loss, accuracy, pred = ps.ps_evaluate(ctx, -1, state["x"], state["y"])
        return dict(loss=loss, accuracy=accuracy, pred=pred)
    if kind == "elastic":
        ps.ps_elastic_average(ctx, state["slots"], ALPHA)
        return _rows(ctx, 0, 1 + case["copies"])
    rule, slots = case["rule"], case["slots"]
    for r in range(case["rounds"]):
        args = (ctx, state["workers"], state["slot_of"], state["ids"][r], state["x"][r], state["y"][r], state["loss"][r])
        if rule == "store":
            ps.worker_grads_append(*args)
        else:
            entries = ps.worker_grads_batched(*args)
    if rule == "sync":
        ps.ps_apply_sync(ctx, entries, LR)
    elif rule == "async":
        for i, q in enumerate(entries):
            ps.ps_apply_async(ctx, q, LR)
            if state["published"] > 1:  # the worker whose gradient it was pulls
                ps.ps_snapshot_weights(ctx, slots + i)
    elif rule == "store":
        ps.ps_store_consume(ctx, ps.DRAIN_SUM, LR)
        ps.ps_store_publish(ctx, slots)
    else:
        ps.ps_drain_buffered(ctx, ps.DRAIN_SUM if rule == "sum" else ps.DRAIN_SEQ, LR)
    if rule != "store" and state["published"] == 1:
        ps.ps_snapshot_weights(ctx, slots)
    ring = slots + state["published"]
    return dict(weights=_rows(ctx, 0, 1), published=_rows(ctx, 1 + slots, state["published"]),
                grads=_rows(ctx, 1 + ring, state["capacity"]), loss=state["loss"])


def work(case):
    row = P * 4
    kind = case["kind"]
    if kind == "drain":
        return dict(bytes=(case["rows"] + 2) * row, flops=2 * case["rows"] * P)
    if kind == "elastic":
        return dict(bytes=2 * (case["copies"] + 1) * row, flops=4 * case["copies"] * P)
    images = case["n"] * case["batch"]
    if kind == "evaluate":
        return dict(bytes=images * (PIX * 4 + 8) + row, flops=images * FLOP_FORWARD)
    k, images = case["n"] * case["rounds"], images * case["rounds"]
    # pixels, labels and snapshots in; a gradient row written by each worker and read by the server; the
    # server's weights read, written and published
    published = case["n"] if case["rule"] == "async" and case["n"] <= 8 else 1
    return dict(bytes=images * (PIX * 4 + 4) + (case["slots"] + 2 * k + 2 + 2 * published) * row, flops=images * FLOP_PER_IMAGE)


def tolerance(case):
    # Sums in 32 bits: gradient rows are 2 to 5e-7 off 64 bits at every size, weights up to 3e-7 after 400
    # updates, losses up to 1.5e-7; two implementations differ by about 1.4 times that.
    if case["kind"] == "evaluate":
        return dict(rel=2e-6, max=1e-4, differ=1e-3)  # a predicted class may change where two logits tie
    return dict(rel=3e-6, max=1e-4)


# ---------------------------------------------------------------------------------------- in 64 bits

def _mul(a, b):
    """High and low word of a 32 x 32 bit product, on 64-bit integers."""
    p, q = (a & 0xFFFF) * b, (a >> 16) * b
    low = p + ((q & 0xFFFF) << 16)
    return (q >> 16) + (low >> 32), low & 0xFFFFFFFF


def _keep(mb, batch):
    """Keep mask [batch, 512]: word u % 4 of Philox4x32-10 at (id, sample, u / 4) against p * 2^32."""
    dev = "cuda"
    c = [torch.full((batch, 128), mb & 0xFFFFFFFF, device=dev, dtype=torch.int64),
         torch.full((batch, 128), mb >> 32, device=dev, dtype=torch.int64),
         torch.arange(batch, device=dev)[:, None].expand(batch, 128), torch.arange(128, device=dev)[None].expand(batch, 128)]
    k = [DROP_SEED & 0xFFFFFFFF, DROP_SEED >> 32]
    for _ in range(10):
        h0, l0 = _mul(0xD2511F53, c[0])
        h1, l1 = _mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k[0], l1, h0 ^ c[3] ^ k[1], l0]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    return torch.stack(c, -1).reshape(batch, 512) >= int(P_DROP * 2 ** 32)


def _unpool(g, w, h):
    """Gradient at pooled outputs [N, C, h/2*h/2] -> at the window's first maximum, where that is > 0."""
    n, c = w.shape[:2]
    win = torch.zeros_like(w)
    win.scatter_(-1, w.argmax(-1, keepdim=True), (g * (w.amax(-1) > 0)).unsqueeze(-1))
    return win.view(n, c, h // 2, h // 2, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(n, c, h * h)


def _gradients(theta, x, y, mbs):
    """Gradients [m, P] and losses [m] of m minibatches x [m, batch, 784] at `theta`."""
    m, batch = y.shape
    u1, w1, p1, u2, w2, p2, h = _forward(theta, x.reshape(-1, PIX))
    keep = torch.cat([_keep(mb, batch) for mb in mbs]) / (1 - P_DROP)
    a = h.clamp_min(0) * keep
    z = a @ _pick(theta, OFF_W4, 10, 512).t() + _pick(theta, OFF_B4, 10)
    label = y.reshape(-1, 1).long()
    loss = (z.logsumexp(1) - z.gather(1, label)[:, 0]).view(m, batch).mean(1)
    d4 = (torch.softmax(z, 1) - torch.zeros_like(z).scatter_(1, label, 1.0)) / batch
    d3 = (d4 @ _pick(theta, OFF_W4, 10, 512)) * keep * (h > 0)
    dp2 = (d3 @ _pick(theta, OFF_W3, 512, 1568)).view(-1, 32, 49)
    d2 = _unpool(dp2, w2, 14)
    du2 = torch.matmul(_pick(theta, OFF_W2, 32, 144).t(), d2)
    dp1 = torch.nn.functional.fold(du2, (14, 14), 3, padding=1).view(-1, 16, 196)
    d1 = _unpool(dp1, w1, 28)
    per = lambda t: t.reshape(m, batch, *t.shape[1:])  # noqa: E731
    out = torch.empty(m, P, device=x.device, dtype=torch.float64)
    put = lambda off, v: out[:, off:off + v[0].numel()].copy_(v.reshape(m, -1))  # noqa: E731
    for i in range(m):
        out[i, OFF_W1:OFF_B1] = torch.matmul(per(d1)[i], per(u1)[i].transpose(1, 2)).sum(0).flatten()
        out[i, OFF_W2:OFF_B2] = torch.matmul(per(d2)[i], per(u2)[i].transpose(1, 2)).sum(0).flatten()
        out[i, OFF_W3:OFF_B3] = (per(d3)[i].t() @ per(p2)[i]).flatten()
        out[i, OFF_W4:OFF_B4] = (per(d4)[i].t() @ per(a)[i]).flatten()
    put(OFF_B1, per(d1).sum((1, 3)))
    put(OFF_B2, per(d2).sum((1, 3)))
    put(OFF_B3, per(d3).sum(1))
    put(OFF_B4, per(d4).sum(1))
    return out, loss


def exact(case, seed):
    kind = case["kind"]
    if kind == "drain":
        s = prepare(case, seed)
        theta, k = s["theta"].double(), case["rows"]
        lr = LR * min(1.0, case["ref"] / k) if case["ref"] > 0 else LR
        for row in s["grads"]:
            g = row.double()
            norm = float(g.norm())
            theta -= lr * (min(1.0, case["clip"] / norm) if case["clip"] > 0 else 1.0) * g
        return theta
    if kind == "elastic":
        n = case["copies"]
        thetas = _weights(seed, n + 1).double()
        d = thetas[:n] - thetas[n]
        out = torch.zeros(n + 1, ROW, device="cuda", dtype=torch.float64)
        out[0, :P] = thetas[n] + ALPHA * d.sum(0)
        out[1:, :P] = thetas[:n] - ALPHA * d
        return out
    n, batch = case["n"], case["batch"]
    if kind == "evaluate":
        theta = _weights(seed, 1)[0].double()
        x, y = _images(seed, None, None, n, batch)
        loss = 0.0
        for xs, ys in zip(x.view(-1, PIX).split(CHUNK), y.view(-1).split(CHUNK)):
            h = _forward(theta, xs)[-1].clamp_min(0)
            z = h @ _pick(theta, OFF_W4, 10, 512).t() + _pick(theta, OFF_B4, 10)
            loss += float((z.logsumexp(1) - z.gather(1, ys[:, None].long())[:, 0]).sum())
        return dict(loss=loss / (n * batch), accuracy=None, pred=None)
    workers, slot_of, ids = _ids(case)
    slots, rounds, rule = case["slots"], case["rounds"], case["rule"]
    thetas = _weights(seed, slots)
    x, y = _images(seed, thetas, slot_of * rounds, n * rounds, batch)
    published = n if rule == "async" and n <= 8 else 1
    grads = torch.zeros(2 * n if rule == "store" else n * rounds, ROW, device="cuda", dtype=torch.float64)
    loss = torch.empty(n * rounds, device="cuda", dtype=torch.float64)
    mbs, slot_of = [i for r in ids for i in r], slot_of * rounds
    per = max(1, CHUNK // batch)
    for s in range(slots):
        mine = [i for i in range(n * rounds) if slot_of[i] == s]
        for at in range(0, len(mine), per):
            part = mine[at:at + per]
            grads[part, :P], loss[part] = _gradients(thetas[s].double(), x[part], y[part], [mbs[i] for i in part])
    weights = torch.zeros(1, ROW, device="cuda", dtype=torch.float64)
    weights[0, :P] = thetas[0].double()
    out = torch.zeros(published, ROW, device="cuda", dtype=torch.float64)
    for i in range(n * rounds):
        weights[0] -= LR * grads[i]
        out[i if published > 1 else 0] = weights[0]
    return dict(weights=weights, published=out, grads=grads, loss=loss.view(rounds, n))
