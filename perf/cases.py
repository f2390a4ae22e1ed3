"""Workloads of the library as its users run them, for timing and for comparing two builds.

Five kinds of work, all through the public binding:
  loop    the whole expanded-group sampling loop (pg_sample_group and the pg_check the header asks for)
  ratio   the importance-ratio / clipped-surrogate forward pass on a finished loop (pg_policy_ratio)
  own     the loop around a network of the caller's own (PG_NET_NONE): init, previews, prunes, updates, advantages
  select  Optimal Variance Filtering over a batch of groups of rewards (pg_ovf_select / pg_ovf_select_large)
  update  one fused sampler update with its log-prob (pg_sde_step_logprob / pg_sde_step_logprob_bf16)

Everything random is drawn on the GPU from the seed.  The reward probe of a loop is not a random direction: it is the
smallest vector that gives the INITIAL latents of a group evenly spaced scores in random order.  Later steps blur the
order by their noise, but the gaps between scores stay far above what the rounding of a bf16 network moves a score by,
so two correct builds keep the same survivors and the outputs of a pruned loop can be compared value by value.
"""
import math

import torch

from paper_2512_15347_amd import binding as pg

DEV = "cuda:0"


def listed():
    return [
        # ---- whole sampling loops, smallest to largest ----
        # a tiny group: every launch is short, so launches and latency are what counts
        dict(name="tiny_flow_loop", work="loop", kind="adaln", sampler="flow", P=1, N=8, C=4, H=16, W=16, T=10, D=128,
             blocks=2, heads=4, Lc=0, schedule="4:4"),
        # three small groups with funnels of their own (one unpruned), ragged token tiles (64 image + 26 context tokens)
        dict(name="ragged_flow_loop", work="loop", kind="joint", sampler="flow", P=3, N=12, C=4, H=16, W=16, T=6, D=128,
             blocks=2, heads=2, Lc=26, schedule="1:8 3:4|1:7 3:5|"),
        # one diffusion-shaped group: DDIM, cross-attention over 77 context tokens, width 768
        dict(name="diffusion_loop", work="loop", kind="cross", sampler="ddim", P=1, N=24, C=4, H=64, W=64, T=20, D=768,
             blocks=12, heads=12, Lc=77, schedule="5:12"),
        # one flow-shaped group: joint attention over 1024 image + 154 context tokens, width 1536, two prunes
        dict(name="flow_loop", work="loop", kind="joint", sampler="flow", P=1, N=48, C=16, H=64, W=64, T=10, D=1536,
             blocks=24, heads=24, Lc=154, schedule="2:32 4:16"),
        # a batch of such groups packed into one ragged batch, one of them pinned to no pruning
        dict(name="batched_flow_loop", work="loop", kind="joint", sampler="flow", P=2, N=48, C=16, H=64, W=64, T=10,
             D=1536, blocks=24, heads=24, Lc=154, schedule="2:32 4:16|"),
        # the dual-stream network (separate image and context weights, normalised queries / keys), 24 -> 16 -> 12
        dict(name="dual_stream_loop", work="loop", kind="mmdit", sampler="flow", P=1, N=24, C=16, H=64, W=64, T=10,
             D=1536, blocks=24, heads=24, Lc=154, schedule="5:16 7:12"),
        # ---- the policy update's forward pass on the survivors of a 24 -> 16 -> 12 loop, before the first weight step ----
        dict(name="policy_ratio", work="ratio", kind="joint", sampler="flow", P=1, N=24, C=16, H=64, W=64, T=10, D=1536,
             blocks=24, heads=24, Lc=154, schedule="5:16 7:12"),
        # ---- the loop around somebody else's network: eight groups of 48 trajectories, ragged after the prunes ----
        dict(name="own_network_loop", work="own", sampler="flow", P=8, N=48, C=16, H=64, W=64, T=10,
             schedule="2:32 4:16|2:32 4:16|2:32 4:16|2:32 4:16|2:32 4:16|2:32 4:16|2:32 4:16|"),
        # ---- selection on rewards that are already there ----
        dict(name="select_4096", work="select", groups=4096, n=64, k=16, ragged=False),
        dict(name="select_million", work="select", groups=1 << 20, n=64, k=16, ragged=False),
        # ---- one update of a large batch of large latents, fp32 and bf16 storage ----
        dict(name="update_fp32", work="update", dtype="fp32", rows=1024, kept=1024, d=16 * 128 * 128),
        dict(name="update_bf16", work="update", dtype="bf16", rows=1024, kept=1024, d=16 * 128 * 128),
    ]


# ---------------------------------------------------------------- more cases of the same ranges

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_schedule(rng, P, N, T):
    groups = []
    for _ in range(P):
        n, entries, s = N, [], 0
        for _ in range(rng.randint(0, 2)):
            s = rng.randint(s + 1, T) if s + 1 < T else T
            k = rng.randint(max(1, n // 3), n)
            if s >= T or k >= n:
                break
            entries.append("%d:%d" % (s, k))
            n = k
        groups.append(" ".join(entries))
    return "|".join(groups)


def _draw_loop(rng, what):
    kind = rng.choice(["adaln", "joint", "cross", "mmdit"])
    P, N, T = rng.randint(1, 3), _log_int(rng, 4, 64), rng.randint(4, 12)
    D = 64 * _log_int(rng, 2, 24)
    hd = 32 if D <= 256 and rng.random() < 0.5 else 64
    H, W = 2 * _log_int(rng, 4, 32), 2 * _log_int(rng, 4, 32)
    return dict(work=what, kind=kind, sampler=rng.choice(["flow", "ddim"]) if what == "loop" else "flow", P=P, N=N,
                C=rng.choice([4, 16]), H=H, W=W, T=T, D=D, blocks=_log_int(rng, 2, 24), heads=D // hd,
                Lc=0 if kind == "adaln" else rng.randint(5, 160), schedule=_draw_schedule(rng, P, N, T))


def draw(rng):
    largest = max(work(c)["flops"] for c in listed())
    while True:
        what = rng.choice(["loop", "loop", "loop", "ratio", "own", "select", "select", "update", "update"])
        if what in ("loop", "ratio"):
            case = _draw_loop(rng, what)
            if work(case)["flops"] > 0.5 * largest:
                continue
            return case
        if what == "own":
            P, N, T = rng.randint(1, 8), _log_int(rng, 4, 64), rng.randint(4, 12)
            return dict(work="own", sampler=rng.choice(["flow", "ddim"]), P=P, N=N, C=rng.choice([4, 16]),
                        H=2 * _log_int(rng, 8, 64), W=2 * _log_int(rng, 8, 32), T=T, schedule=_draw_schedule(rng, P, N, T))
        if what == "select":
            n = _log_int(rng, 8, 1024) if rng.random() < 0.3 else rng.randint(8, 64)
            groups = _log_int(rng, 64, (1 << 20) if n <= 64 else (1 << 22) // n)
            return dict(work="select", groups=groups, n=n, k=rng.randint(1, max(1, n // 2)), ragged=rng.random() < 0.5)
        rows = _log_int(rng, 8, 1024)
        return dict(work="update", dtype=rng.choice(["fp32", "bf16"]), rows=rows,
                    kept=rows if rng.random() < 0.5 else rng.randint(max(1, rows // 3), rows), d=8 * _log_int(rng, 128, 32768))


# ---------------------------------------------------------------- what a case cannot do without

def _schedule(case):
    groups = [[tuple(int(v) for v in e.split(":")) for e in g.split()] for g in case["schedule"].split("|")]
    assert len(groups) == case["P"]
    return groups


def _active(case):
    """Trajectories that each step evaluates, and those it updates."""
    sched = _schedule(case)
    n = [case["N"]] * case["P"]
    evaluated, updated = [], []
    for s in range(case["T"]):
        evaluated.append(sum(n))
        for g in range(case["P"]):
            n[g] = dict(sched[g]).get(s, n[g])
        updated.append(sum(n))
    return evaluated, updated


def _net_work(case):
    """(flops of one trajectory through the network, step-independent flops per pass, bytes of the weights)"""
    D, blocks, Lc, C = case["D"], case["blocks"], case["Lc"], case["C"]
    Li = case["H"] * case["W"] // 4
    joint = case["kind"] in ("joint", "mmdit")
    L = Li + (Lc if joint else 0)
    block = 24.0 * L * D * D + 4.0 * L * L * D
    params = 18.0 * D * D
    once = 0.0
    if case["kind"] == "cross":
        block += 4.0 * L * D * D + 4.0 * L * Lc * D
        params += 4.0 * D * D
        once = blocks * case["P"] * Lc * 4.0 * D * D
    if joint:
        once = case["P"] * Lc * 2.0 * D * D
    if case["kind"] == "mmdit":
        params *= 2
    return blocks * block + 16.0 * Li * C * D, once, 2.0 * (blocks * params + 4.0 * D * D)


def work(case):
    if case["work"] in ("loop", "ratio"):
        d = case["C"] * case["H"] * case["W"]
        per, once, weights = _net_work(case)
        evaluated, updated = _active(case)
        if case["work"] == "ratio":
            # every stored transition of the final survivors: the states are read, the results are a few numbers
            return dict(flops=case["T"] * updated[-1] * per + once, bytes=weights + 4.0 * (case["T"] + 1) * updated[-1] * d)
        return dict(flops=sum(evaluated) * per + once, bytes=weights + 4.0 * updated[-1] * d)
    if case["work"] == "own":
        d = case["C"] * case["H"] * case["W"]
        evaluated, updated = _active(case)
        total = 4.0 * case["P"] * case["N"] * d                       # initial latents written
        for before, after in zip(evaluated, updated):
            total += 12.0 * after * d + (8.0 * before * d if after < before else 0.0)
        total += 4.0 * updated[-1] * d                                # final rewards
        return dict(flops=0.0, bytes=total)
    if case["work"] == "select":
        kept = case["groups"] * case["k"]
        members = case["groups"] * case["n"] * (0.75 if case["ragged"] else 1.0)
        words = (case["n"] + 63) // 64
        return dict(flops=0.0, bytes=4.0 * members + case["groups"] * (8.0 * words + 12.0) + 4.0 * kept)
    size = 4 if case["dtype"] == "fp32" else 2
    return dict(flops=0.0, bytes=3.0 * size * case["kept"] * case["d"])


def tolerance(case):
    if case["work"] in ("loop", "ratio"):
        return dict(rel=5e-3, max=0.05)     # the products' K order reversed moves the outputs by up to rel 1.3e-3, max 7e-3
    if case["work"] == "own":
        return dict(rel=1e-5)
    if case["work"] == "select":
        return "exact"
    return dict(rel=1e-5) if case["dtype"] == "fp32" else dict(rel=1e-4, max=1e-2)


# ---------------------------------------------------------------- what the caller holds before the call

class State:
    """One context with its buffers (released with the state)."""
    ctx = None

    def __del__(self):
        if self.ctx is not None:
            pg.pg_destroy(self.ctx)


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _config(case):
    sampler = (dict(kind="flow", a=0.7) if case["sampler"] == "flow"
               else dict(kind="ddim", eta=1.0, beta0=1e-4, beta1=0.02, T_train=1000))
    net = {k: case[k] for k in ("kind", "D", "blocks", "heads", "Lc")} if "kind" in case else {}
    return dict(P=case["P"], N=case["N"], C=case["C"], H=case["H"], W=case["W"], T=case["T"], sampler=sampler,
                schedule=_schedule(case), d=case["C"] * case["H"] * case["W"], Dc=case["D"] if case.get("Lc") else 0, **net)


def _weights(ctx, blocks, g):
    """The flat bf16 weight buffer: N(0, 0.02^2) everywhere, norm scales around 1, row padding zero."""
    flat = torch.empty(pg.pg_weights_numel(ctx), dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
    for wid, name in enumerate(pg.WEIGHT_IDS):
        for b in range(1 if wid < pg.FIRST_BLOCK_ID else blocks):
            try:
                off, rows, cols, ld = pg.pg_weight_slot(ctx, wid, b)
            except pg.PgError:                                        # not a tensor of this kind of network
                break
            if name.endswith("_g"):
                flat[off:off + cols] += 1.0
            if ld > cols:
                flat[off:off + rows * ld].view(rows, ld)[:, cols:] = 0.0
    return flat.view(torch.int16)


def _probe(P, N, d, seed, g):
    """Smallest w with <w, x_0> = evenly spaced scores, in random order within each group."""
    x0 = torch.empty(P * N, d, device=DEV)
    pg.pg_init_latents(x0, torch.arange(P * N, dtype=torch.int32, device=DEV), seed)
    scores = torch.cat([torch.randperm(N, device=DEV, generator=g) for _ in range(P)]).double() - (N - 1) / 2
    gram = (x0 @ x0.T).double()
    gram += 1e-6 * gram.diagonal().mean() * torch.eye(P * N, dtype=torch.float64, device=DEV)
    return (torch.linalg.solve(gram, scores).float() @ x0).contiguous()


def _context(case, seed, keep_history=False):
    g = _generator(seed)
    cfg = _config(case)
    s = State()
    s.work, s.P, s.T, s.seed = case["work"], case["P"], case["T"], 1000003 * seed + 17
    config, _ = pg.make_config(cfg, probe_bias=0.1, net="kind" in case)
    s.ctx = pg.pg_create(config)
    b = s.buf = pg.Buffers(s.ctx, cfg, keep_history=keep_history)
    b.probe_w.copy_(_probe(case["P"], case["N"], cfg["d"], s.seed, g))
    if "kind" in case:
        b.weights = _weights(s.ctx, case["blocks"], g)
        b.y = torch.randn(case["P"], case["D"], device=DEV, generator=g)
        b.c.weights, b.c.y = b.weights.data_ptr(), b.y.data_ptr()
        if case["Lc"]:
            b.ctx_tok = torch.randn(case["P"], case["Lc"], cfg["Dc"], device=DEV, generator=g).to(torch.bfloat16)
            b.c.ctx = b.ctx_tok.data_ptr()
    else:
        b.u.normal_(generator=g)
    pg.pg_bind(s.ctx, b)
    return s


def prepare(case, seed):
    if case["work"] in ("loop", "own"):
        s = _context(case, seed)
        s.checkpoints = sorted({e[0] for group in _schedule(case) for e in group})
        return s
    if case["work"] == "ratio":
        s = _context(case, seed, keep_history=True)
        pg.pg_sample_group(s.ctx, s.seed)
        pg.pg_check(s.ctx)
        M0 = case["P"] * case["N"]
        s.new_weights = s.buf.weights.clone()
        s.buf.adv += 1.0              # a shaped reward: centred advantages at ratio 1 would cancel in J to rounding noise
        s.logp, s.ratio = torch.zeros(case["T"], M0, device=DEV), torch.zeros(case["T"], M0, device=DEV)
        s.J = torch.zeros(case["P"], device=DEV)
        return s
    g = _generator(seed)
    s = State()
    s.work, s.case, s.seed = case["work"], case, seed
    if case["work"] == "select":
        G, n, k = case["groups"], case["n"], case["k"]
        sizes = torch.full((G,), n, dtype=torch.int64, device=DEV)
        s.k = torch.full((G,), k, dtype=torch.int32, device=DEV)
        if case["ragged"]:
            sizes = torch.randint((n + 1) // 2, n + 1, (G,), device=DEV, generator=g)
            s.k = torch.randint(1, k + 1, (G,), device=DEV, generator=g).clamp(max=(n + 1) // 2).to(torch.int32)
        s.offsets = torch.zeros(G + 1, dtype=torch.int32, device=DEV)
        s.offsets[1:] = sizes.cumsum(0)
        members = int(sizes.sum())
        # most rewards cluster at the group mean, a fifth spread out
        clustered = torch.rand(members, device=DEV, generator=g) < 0.8
        s.rewards = torch.where(clustered, torch.randn(members, device=DEV, generator=g) * 0.05,
                                torch.rand(members, device=DEV, generator=g) * 2 - 1)
        s.words = (n + 63) // 64
        s.masks = torch.zeros(G * s.words, dtype=torch.int64, device=DEV)
        s.sel = torch.zeros(int(s.k.sum()), dtype=torch.int32, device=DEV)
        s.new_offsets = torch.zeros(G + 1, dtype=torch.int32, device=DEV)
        s.status = torch.zeros(4, dtype=torch.int32, device=DEV)
        s.scratch = torch.zeros(pg.pg_ovf_scratch_ints(G), dtype=torch.int32, device=DEV)
        return s
    rows, kept, d = case["rows"], case["kept"], case["d"]
    dtype = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16
    s.x = torch.empty(rows, d, dtype=dtype, device=DEV).normal_(generator=g)
    s.u = torch.empty(rows, d, dtype=dtype, device=DEV).normal_(generator=g)
    s.out = torch.zeros(kept, d, dtype=dtype, device=DEV)
    if dtype == torch.bfloat16:
        s.x, s.u, s.out = s.x.view(torch.int16), s.u.view(torch.int16), s.out.view(torch.int16)
    s.src = None if kept == rows else torch.randperm(rows, device=DEV, generator=g)[:kept].sort().values.to(torch.int32)
    s.ids = torch.arange(kept, dtype=torch.int32, device=DEV) if s.src is None else s.src
    s.logp, s.hist = torch.zeros(kept, device=DEV), torch.zeros(rows, device=DEV)
    s.partials = torch.zeros(pg.pg_step_scratch_floats(kept, d), device=DEV)
    return s


# ---------------------------------------------------------------- one pass

def _loop_outputs(s):
    b, st = s.buf, pg.pg_state(s.ctx, s.P)
    M = st["M"]
    return dict(x=b.x[st["cur_x"]][:M], survivors=b.orig_id[st["cur_id"]][:M], rewards=b.rewards[:M], adv=b.adv[:M],
                logp=b.logp_hist, logp_sum=b.logp_sum, offsets=b.group_offsets)


def run(s):
    if s.work == "loop":
        pg.pg_sample_group(s.ctx, s.seed)
        pg.pg_check(s.ctx)
        return _loop_outputs(s)
    if s.work == "ratio":
        pg.pg_policy_ratio(s.ctx, s.new_weights, 0.2, s.logp, s.ratio, s.J)
        return dict(logp=s.logp, ratio=s.ratio, J=s.J)
    if s.work == "own":
        # the caller's network would write buf.u before each prune and step; here its last output stays in place
        pg.pg_init_group(s.ctx, s.seed)
        for step in range(s.T):
            pg.pg_net_forward(s.ctx, step)
            if step in s.checkpoints:
                pg.pg_prune(s.ctx, step)
            pg.pg_step(s.ctx, step)
        pg.pg_advantages(s.ctx)
        return _loop_outputs(s)
    if s.work == "select":
        G = s.case["groups"]
        if s.words == 1:
            pg.pg_ovf_select(s.rewards, s.offsets, s.k, G, s.masks, s.sel, s.new_offsets, s.status, s.scratch)
        else:
            pg.pg_ovf_select_large(s.rewards, s.offsets, s.k, G, s.words, s.masks, s.sel, s.new_offsets, s.status, s.scratch)
        return dict(masks=s.masks, selected=s.sel, offsets=s.new_offsets, status=s.status)
    update = pg.pg_sde_step_logprob if s.case["dtype"] == "fp32" else pg.pg_sde_step_logprob_bf16
    update(s.x, s.u, s.out, s.logp, s.hist, None, s.src, s.ids, s.case["kept"], s.case["d"], 0.875, -0.15, 0.35, s.seed, 3, s.partials)
    return dict(x=s.out if s.case["dtype"] == "fp32" else s.out.view(torch.bfloat16), logp=s.logp, hist=s.hist)


# ---------------------------------------------------------------- the same values in 64 bits

_MASK = 0xFFFFFFFF


def _normals(ids, d, step, stream, seed):
    """Noise of rows `ids`: Philox-4x32-10 on (element / 4, step, id, stream) under `seed`, Box-Muller, all in 64 bits."""
    blocks = torch.arange(d // 4, dtype=torch.int64, device=DEV)[None, :]
    c = [blocks.expand(len(ids), -1), torch.full_like(blocks, step), ids.to(torch.int64)[:, None], torch.full_like(blocks, stream)]
    k0, k1 = seed & _MASK, seed >> 32 & _MASK
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]                 # modulo 2^64: only the bit pattern is used
        c = [(p1 >> 32 & _MASK) ^ c[1] ^ k0, p1 & _MASK, (p0 >> 32 & _MASK) ^ c[3] ^ k1, p0 & _MASK]
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    u = [(w.double() + 0.5) / 2.0 ** 32 for w in c]
    r = [(-2.0 * u[0].log()).sqrt(), (-2.0 * u[2].log()).sqrt()]
    a = [2.0 * math.pi * u[1], 2.0 * math.pi * u[3]]
    return torch.stack([r[0] * a[0].cos(), r[0] * a[0].sin(), r[1] * a[1].cos(), r[1] * a[1].sin()], -1).reshape(len(ids), d)


def _coefficients(case):
    """Per step (A, B, C, P, Q): x' = A x + B u + C xi, preview = P x + Q u."""
    T, out = case["T"], []
    if case["sampler"] == "flow":
        for s in range(T):
            tau, delta = 1.0 - s / T, -1.0 / T
            var = 0.7 ** 2 * tau / max(1.0 - tau, 1.0 / T)
            out.append((1.0 + var * delta / (2.0 * tau), delta * (1.0 + var * (1.0 - tau) / (2.0 * tau)),
                        math.sqrt(var * -delta), 1.0, -tau))
        return out
    alphas, prod = [], 1.0
    for i in range(1000):
        prod *= 1.0 - (1e-4 + (0.02 - 1e-4) * i / 999)
        alphas.append(prod)
    steps = [((T - i) * 999 + T // 2) // T for i in range(T + 1)]
    for s in range(T):
        at, ap = alphas[steps[s]], alphas[steps[s + 1]]
        var = (1.0 - ap) / (1.0 - at) * (1.0 - at / ap)
        out.append((math.sqrt(ap / at), math.sqrt(1.0 - ap - var) - math.sqrt(ap * (1.0 - at) / at), math.sqrt(var),
                    1.0 / math.sqrt(at), -math.sqrt((1.0 - at) / at)))
    return out


def _logp(z, C):
    return -0.5 * (z * z).sum(1) - z.shape[1] * (math.log(C) + 0.5 * math.log(2.0 * math.pi))


def _highest_variance(r, k):
    """Slots of the k members with the largest variance: the j lowest and the k - j highest, best j."""
    order = r.argsort(stable=True)
    picks = [torch.cat([order[:j], order[len(r) - (k - j):]]) for j in range(k + 1)]
    return max(picks, key=lambda p: float(r[p].var(unbiased=False))).sort().values


def exact(case, seed):
    if case["work"] == "update":
        s = prepare(case, seed)
        d, out = case["d"], []
        as_is = (lambda t: t) if case["dtype"] == "fp32" else (lambda t: t.view(torch.bfloat16))
        x, u = as_is(s.x), as_is(s.u)
        logp = torch.zeros(case["kept"], dtype=torch.float64, device=DEV)
        rows = max(1, (1 << 24) // d)
        for r in range(0, case["kept"], rows):
            ids = s.ids[r:r + rows].long()
            z = _normals(ids, d, 3, 1, s.seed)
            out.append(0.875 * x[ids].double() - 0.15 * u[ids].double() + 0.35 * z)
            logp[r:r + rows] = _logp(z, 0.35)
        hist = torch.zeros(case["rows"], dtype=torch.float64, device=DEV)
        hist[s.ids.long()] = logp
        return dict(x=torch.cat(out), logp=logp, hist=hist)
    if case["work"] != "own":
        return None          # selections are whole numbers; a bf16 network followed in 64 bits takes far too long
    s = prepare(case, seed)
    P, N, T, d = case["P"], case["N"], case["T"], case["C"] * case["H"] * case["W"]
    u, w, sched = s.buf.u.view(P * N, d).double(), s.buf.probe_w.view(-1).double(), _schedule(case)
    ids, sizes = torch.arange(P * N, device=DEV), [N] * P
    x = _normals(ids, d, 0, 0, s.seed)
    logp = torch.full((T, P * N), math.nan, dtype=torch.float64, device=DEV)
    for step, (A, B, C, pc, qc) in enumerate(_coefficients(case)):
        src = torch.arange(len(ids), device=DEV)
        if step in s.checkpoints:
            reward = 0.1 + (pc * x + qc * u[:len(ids)]) @ w
            kept, first = [], 0
            for g in range(P):
                slots = torch.arange(first, first + sizes[g], device=DEV)
                first += sizes[g]
                if step in dict(sched[g]):
                    sizes[g] = dict(sched[g])[step]
                    slots = slots[_highest_variance(reward[slots], sizes[g])]
                kept.append(slots)
            src = torch.cat(kept)
        ids = ids[src]
        z = _normals(ids, d, step, 1, s.seed)
        logp[step, ids] = _logp(z, C)
        x = A * x[src] + B * u[src] + C * z
    rewards = 0.1 + x @ w
    adv = torch.cat([(r - r.mean()) / (r.std(unbiased=False) + 1e-6) for r in rewards.split(sizes)])
    offsets = torch.tensor([sum(sizes[:g]) for g in range(P + 1)], device=DEV)
    return dict(x=x, survivors=ids, rewards=rewards, adv=adv, logp=logp, logp_sum=logp.nansum(0), offsets=offsets)
