"""GPU parity of the sampling loop (init group, prune, step, advantages) through the C ABI.

The first block drives the loop with the network output taken from the oracle run (written into
the library's `u` buffer before each prune / step), which isolates every non-network stage at the
loop level; the second block runs the library's own network."""
import numpy as np
import pytest
import torch

from oracle import loop, sampler, ovf
from paper_2512_15347_amd import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)


def _config(name):
    """The named configuration; `<name>_layers` has its network of width 128 widened to 256, which takes a launch for the layers between two
    attentions where workgroups that hold a trajectory or 16 rows of it evaluate the narrow one."""
    if not name.endswith("_layers"):
        return workloads.get_config(name)
    cfg = workloads.get_config(name[:-len("_layers")])
    cfg.update(D=256, heads=2 * cfg["heads"], Dc=256 if cfg["Lc"] else 0)
    return cfg


def _oracle(name, seed, **kw):
    cfg = _config(name)
    w = workloads.make_weights(cfg)
    inp = workloads.make_inputs(cfg, w)
    s = cfg["sampler"]
    tables = (sampler.flow_sde_tables(cfg["T"], s["a"]) if s["kind"] == "flow"
              else sampler.ddim_sde_tables(cfg["T"], s["eta"], s["beta0"], s["beta1"], s["T_train"]))
    rec = loop.run(cfg, tables, inp, seed, wts=w, keep_u_steps=range(cfg["T"]), **kw)
    return cfg, w, inp, tables, rec


def _compare_final(lib, ctx, buf, cfg, rec, x_tol, lp_rtol=1e-3):
    st = lib.pg_state(ctx, cfg["P"])
    M = st["M"]
    assert st["offsets"] == rec["offsets"].tolist()
    assert st["evals"] == rec["evals"] and st["updates"] == rec["updates"]
    ids = buf.orig_id[st["cur_id"]].cpu().numpy()[:M]
    np.testing.assert_array_equal(ids, rec["orig_id"])
    np.testing.assert_array_equal(buf.group_offsets.cpu().numpy(), rec["offsets"])
    gof = buf.group_of.cpu().numpy()[:M]
    for g in range(cfg["P"]):
        assert np.all(gof[rec["offsets"][g]:rec["offsets"][g + 1]] == g)
    x = buf.x[st["cur_x"]].cpu().numpy()[:M].astype(np.float64)
    for r in range(M):                                   # max error relative to the trajectory's largest entry
        assert np.max(np.abs(x[r] - rec["x"][r])) <= x_tol * np.max(np.abs(rec["x"][r])), r
    hist = buf.logp_hist.cpu().numpy().astype(np.float64)
    want = rec["logp_hist"]
    assert np.array_equal(np.isnan(hist), np.isnan(want))
    ok = ~np.isnan(want)
    np.testing.assert_allclose(hist[ok], want[ok], rtol=lp_rtol)
    lsum = buf.logp_sum.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(lsum, rec["logp_sum"], rtol=lp_rtol, atol=lp_rtol * np.max(np.abs(want[ok])))
    rew = buf.rewards.cpu().numpy()[:M].astype(np.float64)
    for g in range(cfg["P"]):
        b, e = rec["offsets"][g], rec["offsets"][g + 1]
        scale = max(np.max(np.abs(rec["rewards"][b:e])), np.std(rec["rewards"][b:e]))
        assert np.max(np.abs(rew[b:e] - rec["rewards"][b:e])) <= 1e-3 * scale
    return x, rew


@pytest.mark.parametrize("name", ["cfg1", "cfg4_small", "cfg2_small"])
def test_loop_with_injected_network_output(lib, name):
    say(f"loop (oracle u injected) {name}")
    seed = workloads.MASTER_SEED
    cfg, w, inp, tables, rec = _oracle(name, seed)
    c, keep = lib.make_config(cfg, probe_bias=inp["probe_b"], net=False)
    ctx = lib.pg_create(c)
    buf = lib.Buffers(ctx, cfg, inputs=inp)
    lib.pg_bind(ctx, buf)
    lib.pg_init_group(ctx, seed)
    assert np.max(np.abs(buf.x[0].cpu().numpy().astype(np.float64) - rec["x_init"])) < 2e-5
    for s in range(cfg["T"]):
        ids_s, u_s = rec["u"][s]
        M = lib.pg_state(ctx, cfg["P"])["M"]
        assert M == len(ids_s)
        buf.u[:M].copy_(torch.from_numpy(u_s.astype(np.float32)))
        lib.pg_net_forward(ctx, s)                       # network kind NONE: marks u as supplied
        if s in rec["ovf_masks"]:
            lib.pg_prune(ctx, s)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(buf.masks.cpu().numpy().view(np.uint64), rec["ovf_masks"][s])
            pr = buf.rewards.cpu().numpy()[:M].astype(np.float64)
            assert np.max(np.abs(pr - rec["proxy"][s][1])) <= 1e-3 * max(1.0, np.std(rec["proxy"][s][1]))
        lib.pg_step(ctx, s)
        ids_a, x_a = rec["x_after"][s]
        st = lib.pg_state(ctx, cfg["P"])
        got = buf.x[st["cur_x"]].cpu().numpy()[:st["M"]].astype(np.float64)
        assert np.max(np.abs(got - x_a)) <= 2e-5 * np.max(np.abs(x_a)), s
    lib.pg_advantages(ctx)
    lib.pg_check(ctx)
    _compare_final(lib, ctx, buf, cfg, rec, x_tol=2e-5, lp_rtol=2e-5)
    M = lib.pg_state(ctx, cfg["P"])["M"]
    adv = buf.adv.cpu().numpy()[:M].astype(np.float64)
    np.testing.assert_allclose(adv, rec["adv"], rtol=2e-3, atol=2e-3)
    lib.pg_destroy(ctx)


def test_loop_call_order_is_enforced(lib):
    cfg = workloads.get_config("cfg1")
    c, keep = lib.make_config(cfg, net=False)
    ctx = lib.pg_create(c)
    buf = lib.Buffers(ctx, cfg)
    with pytest.raises(lib.PgError):
        lib.pg_init_group(ctx, 1)                        # not bound yet
    lib.pg_bind(ctx, buf)
    with pytest.raises(lib.PgError):
        lib.pg_step(ctx, 0)                              # not initialised
    lib.pg_init_group(ctx, 1)
    with pytest.raises(lib.PgError) as e:
        lib.pg_step(ctx, 0)                              # no network evaluation yet
    assert e.value.status == lib.PG_ESCHED
    with pytest.raises(lib.PgError) as e:
        lib.pg_net_forward(ctx, 1)                       # the network is evaluated at the step that comes next
    assert e.value.status == lib.PG_ESCHED
    lib.pg_net_forward(ctx, 0)
    with pytest.raises(lib.PgError):
        lib.pg_prune(ctx, 0)                             # step 0 is not a checkpoint
    lib.pg_step(ctx, 0)
    with pytest.raises(lib.PgError) as e:
        lib.pg_advantages(ctx)                           # Eq. 18 is on the final latents: 1 of 10 steps taken
    assert e.value.status == lib.PG_ESCHED
    for s in range(1, 5):
        lib.pg_net_forward(ctx, s)
        if s == 3:
            with pytest.raises(lib.PgError) as e:
                lib.pg_prune(ctx, 4)                     # a prune belongs to the step whose evaluation it uses
            assert e.value.status == lib.PG_ESCHED
        if s == 4:
            with pytest.raises(lib.PgError) as e:
                lib.pg_step(ctx, 4)                      # the schedule prunes here: the funnel must be followed
            assert e.value.status == lib.PG_ESCHED
            lib.pg_prune(ctx, 4)
            with pytest.raises(lib.PgError):
                lib.pg_net_forward(ctx, 5)               # the prune must be consumed by its step first
            with pytest.raises(lib.PgError):
                lib.pg_advantages(ctx)
        lib.pg_step(ctx, s)
    assert lib.pg_state(ctx, 1)["M"] == 4
    with pytest.raises(lib.PgError):
        lib.pg_prune_forced(ctx, 5, [0b10000])           # u is stale
    lib.pg_net_forward(ctx, 5)
    with pytest.raises(lib.PgError):
        lib.pg_prune_forced(ctx, 5, [0b10000])           # names a slot beyond the 4 members
    with pytest.raises(lib.PgError):
        lib.pg_prune_forced(ctx, 5, [0])                 # empty
    lib.pg_check(ctx)
    small = lib.Buffers(ctx, cfg)
    small.c.workspace_bytes = 16
    with pytest.raises(lib.PgError) as e:
        lib.pg_bind(ctx, small)
    assert e.value.status == lib.PG_EWORKSPACE
    lib.pg_destroy(ctx)


def test_nan_reward_is_reported(lib):
    cfg = workloads.get_config("cfg1")
    c, keep = lib.make_config(cfg, net=False)
    ctx = lib.pg_create(c)
    inp = dict(probe_w=np.ones(cfg["d"], np.float32))
    buf = lib.Buffers(ctx, cfg, inputs=inp)
    lib.pg_bind(ctx, buf)
    lib.pg_init_group(ctx, 3)
    for s in range(5):
        buf.u.zero_()
        if s == 4:
            buf.u[2, 7] = float("nan")
        lib.pg_net_forward(ctx, s)
        if s == 4:
            lib.pg_prune(ctx, s)
        lib.pg_step(ctx, s)
    with pytest.raises(lib.PgError) as e:
        lib.pg_check(ctx)
    assert e.value.status == lib.PG_ENAN
    assert lib.pg_state(ctx, 1)["M"] == 4                # the loop itself stayed in bounds
    lib.pg_destroy(ctx)


# ------------------------------------------------------------------ the library's own network
def _gpu_ctx(lib, cfg, w, inp):
    c, keep = lib.make_config(cfg, probe_bias=inp["probe_b"])
    ctx = lib.pg_create(c)
    buf = lib.Buffers(ctx, cfg, inputs=inp, weights_flat=lib.pack_weights(ctx, cfg, w))
    lib.pg_bind(ctx, buf)
    return ctx, buf


@pytest.mark.parametrize("name", ["cfg1", "cfg2_small", "cfg3_small", "cfg4_small", "cfg3_mmdit_small"])
def test_network_output_at_step_0(lib, name):
    say(f"network forward {name}")
    seed = workloads.MASTER_SEED
    cfg, w, inp, tables, rec = _oracle(name, seed)
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    lib.pg_init_group(ctx, seed)
    lib.pg_net_forward(ctx, 0)
    torch.cuda.synchronize()
    u = buf.u.cpu().numpy().astype(np.float64)
    want = rec["u"][0][1]
    err = np.max(np.abs(u - want)) / np.max(np.abs(want))
    rms = np.sqrt(np.mean((u - want) ** 2)) / np.sqrt(np.mean(want ** 2))
    say(f"  u: max err / max|u| = {err:.2e}, rms rel = {rms:.2e}")
    assert err < 2e-2 and rms < 1e-2
    lib.pg_destroy(ctx)


@pytest.mark.parametrize("P,N,tile_rows", [(5, 51, 192), (5, 42, 160), (6, 49, 224)])
def test_network_output_with_every_tile_height_of_the_projection(lib, P, N, tile_rows):
    """The fused query / key / value projection stages its value channels through LDS in groups of four, two and one 16-row
    tiles of a wave; tiles of 192, 160 and 224 rows leave 6 = 4 + 2, 5 = 4 + 1 and 7 = 4 + 2 + 1.  Row counts P * N * 64 chosen
    so that the launcher picks that height for the 768-column projection (255, 252 and 252 tiles for 256 compute units);
    sampled trajectories (first, last, and two whose rows straddle tile boundaries) against the oracle."""
    from oracle import dit, philox
    say(f"network forward with {P * N * 64} rows ({tile_rows}-row tiles in the projection)")
    seed = workloads.MASTER_SEED
    cfg = workloads.get_config("cfg1")
    cfg.update(P=P, N=N, D=256, heads=4, T=2, schedule=[[] for _ in range(P)])
    w = workloads.make_weights(cfg)
    inp = workloads.make_inputs(cfg, w)
    tables = sampler.flow_sde_tables(cfg["T"], cfg["sampler"]["a"])
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    lib.pg_init_group(ctx, seed)
    lib.pg_net_forward(ctx, 0)
    torch.cuda.synchronize()
    u_gpu = buf.u.cpu().numpy().astype(np.float64)
    M = P * N
    for i in sorted({0, 2, tile_rows // 64, M // 2, M - 1}):  # trajectory tile_rows // 64 holds the first tile boundary
        x0 = philox.normals(seed, philox.STREAM_INIT, i, 0, cfg["d"])[None]
        u = dit.forward(w, cfg, x0, tables["t_in"][0], inp["y"][i // N], None)
        err = np.max(np.abs(u_gpu[i].reshape(-1) - u[0].reshape(-1))) / np.max(np.abs(u[0]))
        say(f"  trajectory {i}: max err / max|u| = {err:.2e}")
        assert err < 2e-2
    lib.pg_destroy(ctx)


@pytest.mark.parametrize("P,D,blocks", [(203, 128, 1), (70, 64, 2)])
def test_network_output_of_many_groups(lib, P, D, blocks):
    """Conditioning and modulation vectors of more groups than one workgroup takes, the last workgroup part empty."""
    from oracle import dit
    say(f"network forward, {P} groups of width {D}")
    cfg = workloads.get_config("cfg1")
    cfg.update(P=P, N=2, H=8, W=8, D=D, heads=2, blocks=blocks, T=1, schedule=[[] for _ in range(P)], Li=16, d=4 * 64)
    w = workloads.make_weights(cfg)
    inp = workloads.make_inputs(cfg, w)
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    lib.pg_init_group(ctx, 5)
    lib.pg_net_forward(ctx, 0)
    u, x = buf.u.cpu().numpy().astype(np.float64), buf.x[0].cpu().numpy().astype(np.float64)
    t_in = sampler.flow_sde_tables(1, cfg["sampler"]["a"])["t_in"][0]
    for g in (*range(0, P, 7), P - 2, P - 1):
        want = dit.forward(w, cfg, x[2 * g:2 * g + 2], t_in, inp["y"][g], None)
        assert np.max(np.abs(u[2 * g:2 * g + 2] - want)) < 2e-2 * np.max(np.abs(want)), g
    lib.pg_destroy(ctx)


def test_network_time_does_not_depend_on_the_grouping(lib):
    """4096 trajectories in 1024 groups and in 64 of a one-block network: the same work but for the modulation vectors (1.1
    times; 2.9 times when few workgroups walked all groups)."""
    say("network forward, time with many groups")
    def micros(P, N):
        cfg = workloads.get_config("cfg1")
        cfg.update(P=P, N=N, D=64, heads=2, blocks=1, T=1, schedule=[[] for _ in range(P)])
        w = workloads.make_weights(cfg)
        ctx, buf = _gpu_ctx(lib, cfg, w, workloads.make_inputs(cfg, w))
        lib.pg_init_group(ctx, 5)
        a, b, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), 1e9
        for _ in range(6):
            a.record()
            for _ in range(5):
                lib.pg_net_forward(ctx, 0)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 200)
        lib.pg_destroy(ctx)
        return best
    many, few = micros(1024, 4), micros(64, 64)
    say(f"  1024 groups {many:.0f} us, 64 groups {few:.0f} us")
    assert many < 1.6 * few


def test_projection_time_does_not_depend_on_the_sequence_length(lib):
    """4096 token rows of a 512-wide network as 256 trajectories of 16 tokens and as 16 of 256: the same products (1.05 times; 1.17
    when the values of groups of rows that span several trajectories were stored token by token)."""
    say("network forward, time of the products with short sequences")
    def milliseconds(P, N, H, W):
        cfg = workloads.get_config("cfg1")
        cfg.update(P=P, N=N, H=H, W=W, D=512, heads=8, blocks=8, T=1, schedule=[[] for _ in range(P)], Li=H * W // 4, d=4 * H * W)
        w = workloads.make_weights(cfg)
        ctx, buf = _gpu_ctx(lib, cfg, w, workloads.make_inputs(cfg, w))
        lib.pg_init_group(ctx, 5)
        best = 1e9
        for _ in range(8):
            lib.pg_profile_begin(1000)
            lib.pg_net_forward(ctx, 0)
            best = min(best, lib.pg_profile_read(0)["ms"])
            lib.pg_profile_end()
        lib.pg_destroy(ctx)
        return best
    short, long = milliseconds(8, 32, 8, 8), milliseconds(1, 16, 32, 32)
    say(f"  16 tokens {1e3 * short:.0f} us, 256 tokens {1e3 * long:.0f} us")
    assert short < 1.12 * long                                     # between the two


def _sharpen_attention(w, kind, gain):
    """Makes the attention decide the network output: with weights of 0.02 the softmax is nearly flat and its branch small, and a
    wrong value order or a missing key tile moves u by less than its tolerance.  With sharp scores and values and outputs four
    times as large the oracle's u moves by 0.35 of its maximum or more when the scores are ignored or the values stored in another order,
    by 0.18 when the last 16 keys are left out and, with less than 100 tokens, by 0.04 when one value is wrong (rounding of the
    attention's operands to bf16: 0.01)."""
    def scale(a, factor):
        a[:] = workloads.bf16_round(a * np.float32(factor))
    for blk in w["blocks"]:
        D = len(blk["o_w"])
        for pre in ("", "c_") if kind == "mmdit" else ("",):
            if kind == "mmdit":
                scale(blk[pre + "qn_g"], 1.5)
                scale(blk[pre + "kn_g"], 1.5)
            else:
                scale(blk["qkv_w"][:2 * D], gain)
            scale(blk[pre + "qkv_w"][2 * D:], 4)
            scale(blk[pre + "o_w"], 4)
        if kind == "cross":
            scale(blk["cq_w"], gain)
            scale(blk["ckv_w"][:D], gain)
            scale(blk["ckv_w"][D:], 4)
            scale(blk["co_w"], 4)


def _check_sharp_network(lib, cfg, kind, gain, trajectories):
    from oracle import dit
    w = workloads.make_weights(cfg)
    _sharpen_attention(w, kind, gain)
    inp = workloads.make_inputs(cfg, w)
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    lib.pg_init_group(ctx, 77)
    lib.pg_net_forward(ctx, 0)
    got = buf.u.cpu().numpy().astype(np.float64)
    x = buf.x[0].cpu().numpy().astype(np.float64)
    t_in = sampler.flow_sde_tables(1, 0.7)["t_in"][0]
    for i in trajectories:
        g = i // cfg["N"]
        want = dit.forward(w, cfg, x[i][None], t_in, inp["y"][g], inp["ctx"][g] if cfg["Lc"] else None)[0]
        err = np.max(np.abs(got[i] - want)) / np.max(np.abs(want))
        say(f"  trajectory {i}: max err / max|u| = {err:.2e}")
        assert err < 2e-2, i
    lib.pg_destroy(ctx)


# the rows of the cross and dual-stream networks take a launch between two attentions, with token counts that store the transposed values in
# units of four (64 and 32 tokens; context rows of 16 after 64) and one by one (35 and 30; context rows of 13, 18, 21 and 77); those of the
# other two kinds workgroups of the narrow networks evaluate
@pytest.mark.parametrize("kind,H,W,Lc,heads,gain", [
    ("adaln", 16, 16, 0, 4, 7), ("adaln", 10, 14, 0, 4, 10), ("cross", 10, 14, 13, 2, 7), ("cross", 16, 16, 77, 2, 7),
    ("joint", 10, 14, 26, 2, 7), ("joint", 16, 16, 27, 2, 7), ("mmdit", 10, 14, 18, 2, 1), ("mmdit", 10, 12, 21, 2, 1),
    ("mmdit", 16, 16, 26, 2, 1)])
def test_network_output_with_sharp_attention(lib, kind, H, W, Lc, heads, gain):
    say(f"sharp attention {kind} {H}x{W} Lc={Lc}")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind=kind, P=2, N=5, H=H, W=W, D=128, heads=heads, Lc=Lc, Dc=128 if Lc else 0, blocks=1, T=1, schedule=[[], []],
               Li=H * W // 4, d=4 * H * W)
    _check_sharp_network(lib, cfg, kind, gain, (0, 4, 5, 9))


# a launch between two attentions for the other two kinds, too, at both head widths: units of four (64 tokens, 30 before 26 that make 56 of them),
# and one by one (35; 91)
@pytest.mark.parametrize("kind,H,W,Lc,heads,gain", [
    ("adaln", 16, 16, 0, 6, 7), ("adaln", 10, 14, 0, 3, 10), ("joint", 10, 12, 26, 3, 7), ("joint", 16, 16, 27, 3, 7),
    ("joint", 10, 14, 26, 6, 7), ("cross", 10, 14, 13, 6, 7), ("mmdit", 8, 16, 16, 6, 1)])
def test_network_output_with_sharp_attention_in_layers(lib, kind, H, W, Lc, heads, gain):
    say(f"sharp attention, width 192, {kind} {H}x{W} Lc={Lc}")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind=kind, P=2, N=5, H=H, W=W, D=192, heads=heads, Lc=Lc, Dc=128 if Lc else 0, blocks=1, T=1, schedule=[[], []],
               Li=H * W // 4, d=4 * H * W)
    _check_sharp_network(lib, cfg, kind, gain, (0, 4, 5, 9))


# networks that one workgroup evaluates whole (width 64 up to 192 tokens, 128 up to 96), at the sequence lengths where the kernel
# changes: one token, a whole number of 16-row tiles and one more token, the longest sequence and the first that takes a launch per
# layer; image tokens that end inside a tile before the context's (21 of 25 + ..), 3 and 16 channels, both head widths
@pytest.mark.parametrize("kind,D,heads,C,H,W,Lc", [
    ("adaln", 64, 2, 4, 2, 2, 0), ("adaln", 64, 1, 16, 8, 16, 0), ("joint", 64, 2, 4, 8, 16, 1), ("joint", 64, 2, 3, 10, 10, 39),
    ("joint", 64, 1, 4, 16, 16, 1), ("adaln", 64, 2, 4, 16, 32, 0), ("joint", 64, 1, 4, 16, 32, 1), ("joint", 64, 2, 4, 16, 46, 8),
    ("joint", 64, 2, 4, 16, 46, 9), ("adaln", 128, 4, 16, 8, 16, 0), ("joint", 128, 2, 4, 8, 16, 1), ("adaln", 128, 2, 3, 16, 16, 0),
    ("joint", 128, 4, 4, 16, 16, 1), ("joint", 128, 2, 4, 14, 12, 54), ("joint", 128, 4, 16, 14, 12, 55)])
def test_network_output_of_narrow_networks(lib, kind, D, heads, C, H, W, Lc):
    L = H * W // 4 + Lc
    say(f"narrow network {kind} width {D}, {L} tokens, {C} channels")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind=kind, P=2, N=3, C=C, H=H, W=W, D=D, heads=heads, Lc=Lc, Dc=D if Lc else 0, blocks=2, T=1, schedule=[[], []],
               Li=H * W // 4, d=C * H * W)
    _check_sharp_network(lib, cfg, kind, 7 if L > 1 else 1, (0, 2, 3, 5))


# the layers between two attentions in one launch (widths 128, 192, 256), with 16 rows to a workgroup (few trajectories) and 32 (many):
# one token, whole tiles of either height and one token more, both head widths, one to three blocks, and of the dual-stream network
# context tokens that follow a whole number of fours (32, 16; 34) and that do not (35, 21); a trajectory's output is the same bits either way
@pytest.mark.parametrize("kind,D,heads,H,W,Lc,blocks", [
    ("adaln", 192, 3, 2, 2, 0, 2), ("adaln", 256, 4, 8, 8, 0, 3), ("adaln", 192, 6, 8, 16, 0, 1), ("joint", 256, 8, 8, 16, 1, 2),
    ("joint", 128, 2, 14, 14, 48, 2), ("joint", 192, 3, 10, 6, 2, 2), ("cross", 128, 4, 2, 2, 1, 3), ("cross", 192, 6, 6, 22, 13, 2),
    ("cross", 256, 4, 10, 14, 77, 1), ("cross", 128, 2, 16, 16, 5, 2), ("mmdit", 192, 6, 8, 16, 16, 2), ("mmdit", 128, 2, 10, 14, 18, 3),
    ("mmdit", 256, 4, 8, 8, 1, 2), ("mmdit", 256, 8, 14, 6, 33, 2), ("mmdit", 192, 3, 4, 34, 31, 2), ("mmdit", 128, 4, 2, 2, 2, 1)])
def test_network_output_of_rows_between_attentions(lib, kind, D, heads, H, W, Lc, blocks):
    L = H * W // 4 + (Lc if kind in ("joint", "mmdit") else 0)
    say(f"rows between attentions, {kind} width {D}, {L} tokens, {blocks} blocks")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind=kind, P=2, N=3, H=H, W=W, D=D, heads=heads, Lc=Lc, Dc=128 if Lc else 0, blocks=blocks, T=1, schedule=[[], []],
               Li=H * W // 4, d=4 * H * W)
    # scores grow as gain^2 D, and with them what rounding does to them: as sharp as 7 makes width 128 (7 at width 256, two blocks,
    # is off by 2.1e-2 with a launch per layer, too)
    gain = 7 * (128 / D) ** 0.5 if L > 1 else 1
    _check_sharp_network(lib, cfg, kind, gain, (0, 5))
    N = min(64, 256 // (2 * ((L + 15) // 16)) + 1)
    P = 256 // (N * ((L + 15) // 16)) + 1
    many = dict(cfg, P=P, N=N, schedule=[[]] * P)
    w = workloads.make_weights(cfg)
    _sharpen_attention(w, kind, gain)
    inp = workloads.make_inputs(many, w)
    outs = []
    for c in (dict(cfg, P=1), many):
        part = {k: v[:c["P"]] if k in ("y", "ctx") and v is not None else v for k, v in inp.items()}
        ctx, buf = _gpu_ctx(lib, c, w, part)
        buf.workspace.fill_(255)
        lib.pg_bind(ctx, buf)
        lib.pg_init_group(ctx, 77)
        lib.pg_net_forward(ctx, 0)
        outs.append(buf.u[:3].clone().view(torch.int32))
        lib.pg_destroy(ctx)
    assert torch.equal(outs[0], outs[1])


# what lies between two attentions in one launch or in a launch per layer, on either side of where one gives way to the other; token counts
# that store the transposed values in units of four and one by one
@pytest.mark.parametrize("kind,D,heads,H,W,Lc,P,N,rows", [
    ("adaln", 256, 4, 10, 14, 0, 6, 44, True), ("adaln", 256, 4, 10, 14, 0, 5, 53, False), ("cross", 128, 4, 6, 6, 5, 33, 53, True),
    ("cross", 128, 4, 6, 6, 5, 35, 50, False), ("mmdit", 192, 3, 4, 4, 3, 6, 51, True), ("mmdit", 192, 3, 4, 4, 3, 7, 44, False),
    ("adaln", 192, 6, 8, 10, 0, 20, 59, True), ("adaln", 192, 6, 8, 10, 0, 197, 6, False), ("mmdit", 256, 4, 10, 14, 18, 6, 55, True),
    ("mmdit", 256, 4, 10, 14, 18, 9, 37, False)])
def test_network_output_by_rows_and_by_layers(lib, kind, D, heads, H, W, Lc, P, N, rows):
    say(f"by rows or by layers, {kind} width {D}, {P * N} trajectories")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind=kind, P=P, N=N, H=H, W=W, D=D, heads=heads, Lc=Lc, Dc=128 if Lc else 0, blocks=2, T=1, schedule=[[]] * P,
               Li=H * W // 4, d=4 * H * W)
    lib.pg_profile_begin(1000)
    _check_sharp_network(lib, cfg, kind, 7 * (128 / D) ** 0.5 if H * W > 16 else 1, (0, N, P * N - 1))
    launches = lib.pg_profile_read(0)["launches"]
    lib.pg_profile_end()
    before = 1 + (cfg["blocks"] - 1 if kind == "cross" else 0) if Lc else 0      # the context's projections
    assert (launches - before <= 2 * 2 + 3) == rows, launches


@pytest.mark.parametrize("kind,D,P,N,H,W,Lc", [("adaln", 128, 1, 8, 16, 16, 0), ("joint", 64, 2, 3, 10, 10, 39), ("joint", 192, 1, 3, 10, 10, 6),
                                                ("adaln", 128, 20, 60, 2, 2, 0)])
def test_profile_counts_the_work_of_a_network(lib, kind, D, P, N, H, W, Lc):
    """Networks in one launch and with a launch per layer: the brackets of kinds 0 and 1 together hold all the flops of an evaluation."""
    say(f"profile of a network {kind} width {D}, {P * N} trajectories")
    cfg = workloads.get_config("cfg3_small")
    Li = H * W // 4
    cfg.update(kind=kind, P=P, N=N, C=4, H=H, W=W, D=D, heads=2 if D < 192 else 3, Lc=Lc, Dc=64 if Lc else 0, blocks=2, T=1,
               schedule=[[] for _ in range(P)], Li=Li, d=4 * H * W)
    w = workloads.make_weights(cfg)
    ctx, buf = _gpu_ctx(lib, cfg, w, workloads.make_inputs(cfg, w))
    lib.pg_init_group(ctx, 5)
    lib.pg_profile_begin(1000)
    lib.pg_net_forward(ctx, 0)
    products, attention = lib.pg_profile_read(0), lib.pg_profile_read(1)
    lib.pg_profile_end()
    lib.pg_destroy(ctx)
    L, M = Li + Lc, P * N
    want = M * (2 * (24 * L * D * D + 4 * L * L * D) + 2 * 2 * Li * D * 16)      # the context's projection belongs to pg_init_group
    assert products["work"] + attention["work"] == want
    assert products["launches"] >= 1 and products["ms"] > 0


# a workgroup per 16 rows and the update inside the network's launches (few trajectories) against a workgroup per trajectory and an
# update of its own (many): one row tile, odd and even numbers of them, tiles of context rows alone, both head widths, odd patch rows,
# one and three blocks, modulation vectors of a few steps at a time (many groups)
@pytest.mark.parametrize("kind,D,heads,C,H,W,Lc,blocks,P", [
    ("adaln", 128, 4, 4, 16, 16, 0, 2, 1), ("joint", 128, 2, 4, 10, 10, 40, 1, 2), ("joint", 128, 4, 16, 14, 12, 54, 3, 1),
    ("adaln", 128, 2, 3, 8, 8, 0, 2, 3), ("joint", 128, 2, 4, 6, 6, 24, 2, 33), ("joint", 64, 2, 4, 10, 10, 39, 2, 1),
    ("joint", 64, 1, 16, 16, 46, 8, 1, 1), ("adaln", 64, 2, 4, 4, 18, 0, 3, 2), ("adaln", 64, 1, 4, 16, 28, 0, 2, 9)])
def test_narrow_loops_by_rows_and_by_trajectories_agree(lib, kind, D, heads, C, H, W, Lc, blocks, P):
    L = H * W // 4 + Lc
    say(f"narrow loop {kind} width {D}, {L} tokens, {P} groups")
    cfg = workloads.get_config("cfg3_small")
    first = [(1, 3), (4, 2)]
    cfg.update(kind=kind, P=P, N=4, C=C, H=H, W=W, D=D, heads=heads, Lc=Lc, Dc=D if Lc else 0, blocks=blocks, T=6,
               schedule=[first] + [[]] * (P - 1), Li=H * W // 4, d=C * H * W)
    many = dict(cfg, P=300, schedule=[first] + [[]] * 299)
    w = workloads.make_weights(cfg)
    inp = workloads.make_inputs(many, w)
    seed, ctx, runs = 31, {}, []
    for name, c in (("few", cfg), ("many", many)):
        part = {k: v[:c["P"]] if k in ("y", "ctx") and v is not None else v for k, v in inp.items()}
        cc, keep = lib.make_config(c, probe_bias=part["probe_b"])
        ctx[name] = lib.pg_create(cc)
        buf = lib.Buffers(ctx[name], c, inputs=part, weights_flat=lib.pack_weights(ctx[name], c, w), keep_history=name == "few")
        buf.workspace.fill_(255)
        lib.pg_bind(ctx[name], buf)
        for whole in (True, False) if name == "few" else (True,):
            if whole:
                lib.pg_sample_group(ctx[name], seed)
            else:
                lib.pg_init_group(ctx[name], seed)
                for s in range(6):
                    lib.pg_net_forward(ctx[name], s)
                    if s in (1, 4):
                        lib.pg_prune(ctx[name], s)
                    lib.pg_step(ctx[name], s)
                lib.pg_advantages(ctx[name])
            lib.pg_check(ctx[name])
            st = lib.pg_state(ctx[name], c["P"])
            M = 2 + 4 * (P - 1)                          # survivors of the groups that both contexts have
            runs.append(dict(x=buf.x[st["cur_x"]][:M].clone(), u=buf.u[:M].clone(), ids=buf.orig_id[st["cur_id"]][:M].clone(),
                             hist=buf.logp_hist[:, :4 * P].clone().view(torch.int32), sum=buf.logp_sum[:4 * P].clone(),
                             rewards=buf.rewards[:M].clone()))
            if name == "few":
                runs[-1]["record"] = buf.x_hist.clone()
        lib.pg_destroy(ctx[name])
    for k in runs[1]:
        assert torch.equal(runs[0][k].view(torch.int32), runs[1][k].view(torch.int32)), f"one call and step by step: {k}"
    for k in runs[2]:
        assert torch.equal(runs[0][k], runs[2][k]), f"by rows and by trajectories: {k}"


# on either side of where a loop, and where an evaluation alone, of narrow networks takes a workgroup per 16 rows: 2, 4 and 6 row tiles of
# width 128, 4, 8 and 12 of width 64
@pytest.mark.parametrize("D,H,W,P", [(128, 8, 12, 32), (128, 8, 12, 33), (128, 16, 16, 16), (128, 16, 16, 17), (128, 16, 16, 32), (128, 16, 24, 21),
                                     (128, 16, 24, 22), (64, 16, 16, 8), (64, 16, 16, 9), (64, 16, 16, 16), (64, 16, 16, 17), (64, 16, 32, 16),
                                     (64, 16, 32, 17), (64, 16, 46, 16), (64, 16, 46, 17)])
def test_narrow_loops_on_either_side_of_the_rows_limits(lib, D, H, W, P):
    test_narrow_loops_by_rows_and_by_trajectories_agree(lib, "adaln", D, 2, 4, H, W, 0, 2, P)


# The loop's launches (a prune's and the advantages' rewards by group, a step's log-probs by the last workgroup to arrive) against the
# entry points of the single kernels: latents of one chunk with little and with more to read for a group, of 2 with many trajectories,
# of 5, 16 and 17 chunks, and too large for the sums by arrival
@pytest.mark.parametrize("P,N,C,H,W", [(3, 4, 4, 32, 32), (3, 5, 4, 32, 32), (2, 64, 4, 2, 2), (9, 64, 4, 32, 34), (2, 6, 4, 64, 72),
                                       (2, 4, 16, 64, 64), (1, 3, 16, 66, 64), (1, 3, 16, 214, 214)])
def test_loop_launches_against_the_single_kernels(lib, P, N, C, H, W):
    d, T, seed, M0 = C * H * W, 3, 77, P * N
    say(f"loop launches {P} x {N} latents of {d}")
    cfg = workloads.get_config("cfg1")
    cfg.update(P=P, N=N, C=C, H=H, W=W, T=T, schedule=[[(0, N - 1), (1, 1)]] + [[(1, max(1, N // 2))]] * (P - 1), Li=H * W // 4, d=d)
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    c, keep = lib.make_config(cfg, probe_bias=0.25, net=False)
    ctx = lib.pg_create(c)
    buf = lib.Buffers(ctx, cfg)
    buf.workspace.fill_(255)
    buf.u.normal_(generator=g)
    buf.probe_w.normal_(generator=g)
    lib.pg_bind(ctx, buf)
    lib.pg_init_group(ctx, seed)
    for s in range(T):
        lib.pg_net_forward(ctx, s)
        if s < 2:
            lib.pg_prune(ctx, s)
        lib.pg_step(ctx, s)
    lib.pg_advantages(ctx)
    lib.pg_check(ctx)
    tab = lib.pg_get_tables(ctx, T)
    ints = lambda v: torch.tensor(v, dtype=torch.int32, device=DEV)
    ids, sizes = torch.arange(M0, dtype=torch.int32, device=DEV), [N] * P
    x, other = torch.empty(M0, d, device=DEV), torch.empty(M0, d, device=DEV)
    lib.pg_init_latents(x, ids, seed)
    partials = torch.empty(lib.pg_step_scratch_floats(M0, d), device=DEV)
    rewards, logp = torch.zeros(M0, device=DEV), torch.zeros(M0, device=DEV)
    hist, total = torch.full((T, M0), float("nan"), device=DEV), torch.zeros(M0, device=DEV)
    status, scratch = torch.zeros(4, dtype=torch.int32, device=DEV), torch.zeros(lib.pg_ovf_scratch_ints(P), dtype=torch.int32, device=DEV)
    offsets, masks = ints([N * i for i in range(P + 1)]), torch.zeros(P, dtype=torch.int64, device=DEV)
    for s in range(T):
        sel, M = None, sum(sizes)
        if s < 2:
            lib.pg_preview_reward(x, buf.u, buf.probe_w, rewards, M, d, tab["P"][s], tab["Q"][s], 0.25, partials)
            sizes = [dict(cfg["schedule"][i]).get(s, n) for i, n in enumerate(sizes)]
            M = sum(sizes)
            sel, new = torch.zeros(M, dtype=torch.int32, device=DEV), torch.zeros(P + 1, dtype=torch.int32, device=DEV)
            lib.pg_ovf_select(rewards, offsets, ints(sizes), P, masks, sel, new, status, scratch)
            ids, offsets = ids[sel.long()].contiguous(), new
        lib.pg_sde_step_logprob(x, buf.u, other, logp, hist[s], total, sel, ids, M, d, tab["A"][s], tab["B"][s], tab["C"][s], seed, s, partials)
        x, other = other, x
    adv = torch.zeros(M0, device=DEV)
    lib.pg_preview_reward(x, None, buf.probe_w, rewards, M, d, 1.0, 0.0, 0.25, partials)
    lib.pg_group_advantages(rewards, offsets, P, 1e-6, adv)
    torch.cuda.synchronize()
    st = lib.pg_state(ctx, P)
    assert st["M"] == M and st["offsets"] == offsets.tolist()
    groups = torch.cat([torch.full((n,), i, dtype=torch.int32) for i, n in enumerate(sizes)])
    for name, got, want in (("x", buf.x[st["cur_x"]][:M], x[:M]), ("ids", buf.orig_id[st["cur_id"]][:M], ids), ("masks", buf.masks, masks),
                            ("offsets", buf.group_offsets, offsets), ("groups", buf.group_of[:M], groups.to(DEV)),
                            ("rewards", buf.rewards[:M], rewards[:M]), ("adv", buf.adv[:M], adv[:M]), ("sum", buf.logp_sum, total),
                            ("hist", buf.logp_hist, hist)):
        if name == "adv":                                # a group of one has no spread: 0 / (0 + eps)
            assert torch.isfinite(got).all()
        assert torch.equal(got.contiguous().view(torch.int32), want.contiguous().view(torch.int32)), name
    lib.pg_destroy(ctx)


@pytest.mark.parametrize("C,H,W", [(4, 16, 16), (16, 16, 20)])
def test_init_group_draws_the_initial_latents_alone(lib, C, H, W):
    """A narrow network's run, whose loop in one call wants sums of the noise of all steps: they are not made for a caller who goes step by
    step.  Of the scratch memory nothing but a word per trajectory is written."""
    P, N, T = 1, 8, 40
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind="adaln", P=P, N=N, C=C, H=H, W=W, D=64, heads=2, Lc=0, Dc=0, blocks=1, T=T, schedule=[[]], Li=H * W // 4, d=C * H * W)
    w = workloads.make_weights(cfg)
    ctx, buf = _gpu_ctx(lib, cfg, w, workloads.make_inputs(cfg, w))
    words = buf.workspace[:buf.workspace.numel() // 8 * 8].view(torch.int64)
    before = words.clone()
    lib.pg_init_group(ctx, 5)
    torch.cuda.synchronize()
    written = int((words != before).sum())
    lib.pg_destroy(ctx)
    assert written <= N + 1, f"{written} words written"


@pytest.mark.parametrize("M0,T,C,H,W", [(1, 65600, 16, 16, 18), (128, 65536, 4, 2, 2), (256, 65536, 4, 2, 2)])
def test_narrow_loop_of_very_many_steps(lib, M0, T, C, H, W):
    """As many steps times trajectories as one launch makes the sums of the noise for, and more: log-probs of the first steps, the last ones
    and those around 32768 and 65536 as one update gives them."""
    d = C * H * W
    say(f"{T} steps of {M0} trajectories of {d}")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind="adaln", P=1 if M0 < 64 else M0 // 64, N=min(M0, 64), C=C, H=H, W=W, D=64, heads=2, Lc=0, Dc=0, blocks=1, T=T, Li=H * W // 4, d=d,
               schedule=[[]] * (1 if M0 < 64 else M0 // 64))
    w = workloads.make_weights(cfg)
    ctx, buf = _gpu_ctx(lib, cfg, w, workloads.make_inputs(cfg, w))
    lib.pg_sample_group(ctx, 5)
    lib.pg_check(ctx)
    C_s = lib.pg_get_tables(ctx, T)["C"]
    lib.pg_destroy(ctx)
    x, ids = torch.zeros(M0, d, device=DEV), torch.arange(M0, dtype=torch.int32, device=DEV)
    out, logp, part = torch.zeros(M0, d, device=DEV), torch.zeros(M0, device=DEV), torch.zeros(lib.pg_step_scratch_floats(M0, d), device=DEV)
    for s in (0, 1, 32767, 32768, 65535, 65536, T - 1):
        if s < T:
            lib.pg_sde_step_logprob(x, x, out, logp, None, None, None, ids, M0, d, 1.0, 0.0, float(C_s[s]), 5, s, part)
            assert torch.equal(buf.logp_hist[s], logp), s


# log-probs by the last workgroup to arrive and by a second launch, on either side of where one gives way to the other: 5120 chunks in
# a launch (1024 x 5, the last of them of four elements; the launches after the prunes have fewer) and 32 of a trajectory
@pytest.mark.parametrize("P,N,C,H,W", [(16, 64, 1, 2, 8194), (41, 25, 1, 2, 8194), (2, 4, 16, 64, 128), (2, 4, 16, 64, 130)])
def test_loop_sums_by_arrival_and_by_a_launch(lib, P, N, C, H, W):
    test_loop_launches_against_the_single_kernels(lib, P, N, C, H, W)


def test_start_of_very_many_trajectories(lib):
    """16,777,152 trajectories: their latents take a launch's last lanes, and the state of the run has to find others."""
    P, N, d = 262143, 64, 4
    say(f"start of {P} x {N} trajectories")
    cfg = workloads.get_config("cfg1")
    cfg.update(P=P, N=N, C=1, H=2, W=2, T=1, schedule=[[]] * P, Li=1, d=d)
    c, keep = lib.make_config(cfg, net=False)
    ctx = lib.pg_create(c)
    buf = lib.Buffers(ctx, cfg)
    for t in (buf.x[0], buf.orig_id[0], buf.group_of, buf.group_offsets, buf.logp_hist, buf.logp_sum, buf.status):
        t.fill_(9)
    lib.pg_bind(ctx, buf)
    lib.pg_init_group(ctx, 3)
    torch.cuda.synchronize()
    ids = torch.arange(P * N, dtype=torch.int32, device=DEV)
    x = torch.empty(P * N, d, device=DEV)
    lib.pg_init_latents(x, ids, 3)
    assert torch.equal(buf.x[0], x) and torch.equal(buf.orig_id[0], ids) and torch.equal(buf.group_of, ids // N)
    assert torch.equal(buf.group_offsets, torch.arange(P + 1, dtype=torch.int32, device=DEV) * N)
    assert buf.logp_hist.isnan().all() and not buf.logp_sum.any() and not buf.status.any()
    lib.pg_destroy(ctx)


def test_prune_and_advantages_of_very_many_groups(lib):
    """2^22 groups of three: more than a launch has lanes for with a large workgroup for each.  Of three members the lowest and the
    highest stay."""
    P, N, d = 1 << 22, 3, 4
    say(f"prune and advantages of {P} x {N}")
    cfg = workloads.get_config("cfg1")
    cfg.update(P=P, N=N, C=1, H=2, W=2, T=1, schedule=[[(0, 2)]] * P, Li=1, d=d)
    g = torch.Generator(device=DEV)
    g.manual_seed(8)
    c, keep = lib.make_config(cfg, net=False)
    ctx = lib.pg_create(c)
    buf = lib.Buffers(ctx, cfg)
    buf.u.normal_(generator=g)
    buf.probe_w.normal_(generator=g)
    lib.pg_bind(ctx, buf)
    lib.pg_init_group(ctx, 3)
    lib.pg_net_forward(ctx, 0)
    lib.pg_prune(ctx, 0)
    torch.cuda.synchronize()
    r = buf.rewards.view(P, N)
    # groups whose order of two rewards is not strict are not looked at
    strict = (r.sort(1).values.diff(dim=1) > 0).all(1)
    kept = (1 << r.argmin(1)) | (1 << r.argmax(1))
    assert strict.float().mean() > 0.99 and torch.equal(buf.masks[strict], kept[strict])
    assert torch.equal(buf.group_offsets, 2 * torch.arange(P + 1, dtype=torch.int32, device=DEV))
    assert torch.equal(buf.group_of[:2 * P], torch.arange(2 * P, dtype=torch.int32, device=DEV) // 2)
    del r, strict, kept
    lib.pg_step(ctx, 0)
    lib.pg_advantages(ctx)
    lib.pg_check(ctx)
    r = buf.rewards[:2 * P].view(P, 2).double()
    half = (r[:, :1] - r[:, 1:]).abs() / 2
    want = ((r - r.mean(1, keepdim=True)) / (half + 1e-6)).float()
    # fp32 results of fp64 arithmetic on the same rewards: half a unit of numbers up to 1, and of the comparison's
    assert (buf.adv[:2 * P].view(P, 2) - want).abs().max() < 2.0 ** -23
    lib.pg_destroy(ctx)


# few tokens: the number of trajectories up to which one workgroup each evaluates them, and one group more
@pytest.mark.parametrize("kind,D,P,N,H,W,Lc", [
    ("adaln", 128, 15, 60, 2, 2, 0), ("adaln", 128, 16, 60, 2, 2, 0), ("joint", 64, 40, 43, 2, 6, 1), ("joint", 64, 41, 43, 2, 6, 1),
    ("adaln", 128, 46, 64, 8, 8, 0), ("adaln", 128, 47, 64, 8, 8, 0)])
def test_network_output_of_many_short_sequences(lib, kind, D, P, N, H, W, Lc):
    say(f"narrow network {kind} width {D}, {P} x {N} trajectories of {H * W // 4 + Lc} tokens")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind=kind, P=P, N=N, C=4, H=H, W=W, D=D, heads=2, Lc=Lc, Dc=D if Lc else 0, blocks=2, T=1, schedule=[[] for _ in range(P)],
               Li=H * W // 4, d=4 * H * W)
    _check_sharp_network(lib, cfg, kind, 7 if H * W > 4 else 1, (0, 1, N, P * N // 2, P * N - 1))


@pytest.mark.parametrize("D", [64, 128])
def test_time_of_narrow_networks_goes_with_their_tokens(lib, D):
    """4096 trajectories of 4 tokens against 4096 of 32 (0.68 and 0.55 times; 1.0 when one workgroup evaluated either)."""
    say(f"narrow network of width {D}, time with few tokens")
    def micros(H, W):
        cfg = workloads.get_config("cfg1")
        cfg.update(P=64, N=64, H=H, W=W, D=D, heads=2, blocks=2, T=1, schedule=[[] for _ in range(64)], Li=H * W // 4, d=4 * H * W)
        w = workloads.make_weights(cfg)
        ctx, buf = _gpu_ctx(lib, cfg, w, workloads.make_inputs(cfg, w))
        lib.pg_init_group(ctx, 5)
        a, b, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), 1e9
        for _ in range(6):
            a.record()
            for _ in range(5):
                lib.pg_net_forward(ctx, 0)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 200)
        lib.pg_destroy(ctx)
        return best
    few, many = micros(4, 4), micros(8, 16)
    say(f"  4 tokens {few:.0f} us, 32 tokens {many:.0f} us")
    assert few < 0.85 * many


# enough trajectories and tokens for the 64-queries-per-wave attention (four query tiles of 128 against two of 256, 1.67 rounds
# against one): whole key tiles (484 + 28 tokens), a last tile that ends in its second (484 + 26) or first (462 + 18) half,
# separate streams (462 + 26)
@pytest.mark.parametrize("kind,W,Lc,gain", [("joint", 44, 28, 4), ("joint", 42, 18, 7), ("joint", 44, 26, 4), ("mmdit", 42, 26, 1)])
def test_network_output_with_wide_attention(lib, kind, W, Lc, gain):
    say(f"wide attention {kind} W={W} Lc={Lc} gain={gain}")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind=kind, N=64, H=44, W=W, D=256, heads=4, Lc=Lc, Dc=256, blocks=1, T=1, schedule=[[]], Li=11 * W, d=4 * 44 * W)
    L = cfg["Li"] + Lc
    assert lib.pg_attention_kernel(64, L, L, 4, 64) == 2
    _check_sharp_network(lib, cfg, kind, gain, (0, 63))


@pytest.mark.parametrize("kind", ["joint", "mmdit"])
def test_network_output_of_a_trajectory_does_not_depend_on_the_batch(lib, kind):
    """64 trajectories of 480 tokens take the attention with 64 queries per wave, 48 and 5 the one with 32: the same bits,
    also where scores pass the reference that a query's first key tile set (query and key scales of 8)."""
    say(f"batch independence {kind}")
    cfg = workloads.get_config("cfg3_small")
    cfg.update(kind=kind, H=44, W=42, D=256, heads=4, Lc=18, Dc=256, blocks=2, T=1, schedule=[[]], Li=22 * 21, d=4 * 44 * 42)
    w = workloads.make_weights(cfg)
    for blk in w["blocks"]:
        if kind == "joint":
            blk["qkv_w"][:512] *= 8
        else:
            for name in ("qn_g", "kn_g", "c_qn_g", "c_kn_g"):
                blk[name] *= 8
    inp = workloads.make_inputs(cfg, w)
    u = {}
    for N, kernel in ((64, 2), (48, 1), (5, 1)):
        assert lib.pg_attention_kernel(N, 480, 480, 4, 64) == kernel
        cfg["N"] = N
        ctx, buf = _gpu_ctx(lib, cfg, w, inp)
        lib.pg_init_group(ctx, 9)
        lib.pg_net_forward(ctx, 0)
        u[N] = buf.u.cpu().numpy()
        lib.pg_destroy(ctx)
    assert np.isfinite(u[64]).all()
    np.testing.assert_array_equal(u[64][:48], u[48])
    np.testing.assert_array_equal(u[64][:5], u[5])


@pytest.mark.parametrize("name", ["cfg1", "cfg2_small", "cfg3_small", "cfg4_small", "cfg3_mmdit_small", "cfg1_layers", "cfg4_small_layers"])
def test_full_loop_with_own_network(lib, name):
    """Free-running library loop against the free-running oracle: the survivor sets must be the
    oracle's (the seeds used here leave no near-tie), floats within the stated tolerances."""
    say(f"full loop {name}")
    seed = workloads.MASTER_SEED
    cfg, w, inp, tables, rec = _oracle(name, seed)
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    lib.pg_sample_group(ctx, seed)
    lib.pg_check(ctx)
    x, rew = _compare_final(lib, ctx, buf, cfg, rec, x_tol=2e-2)
    M = lib.pg_state(ctx, cfg["P"])["M"]
    adv = buf.adv.cpu().numpy()[:M].astype(np.float64)
    np.testing.assert_allclose(adv, ovf.group_advantages(rew, rec["offsets"], 1e-6), rtol=1e-4, atol=1e-5)
    for g in range(cfg["P"]):
        a = adv[rec["offsets"][g]:rec["offsets"][g + 1]]
        assert abs(a.mean()) < 1e-5 and abs(a.std() - 1) < 1e-3
    lib.pg_destroy(ctx)


def test_forced_masks_follow_the_oracle(lib):
    """Survivors imposed from the oracle run (test hook): the library still reports its own OVF
    decision for the proxy rewards it computed, and that decision is the oracle's."""
    name, seed = "cfg3_small", 99
    say(f"forced loop {name}")
    cfg, w, inp, tables, rec = _oracle(name, seed)
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    shadow = torch.zeros(cfg["P"], dtype=torch.int64, device=DEV)
    lib.pg_init_group(ctx, seed)
    for s in range(cfg["T"]):
        lib.pg_net_forward(ctx, s)
        if s in rec["used_masks"]:
            lib.pg_prune_forced(ctx, s, rec["used_masks"][s], shadow)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(shadow.cpu().numpy().view(np.uint64), rec["ovf_masks"][s])
            np.testing.assert_array_equal(buf.masks.cpu().numpy().view(np.uint64), rec["used_masks"][s])
        lib.pg_step(ctx, s)
    lib.pg_advantages(ctx)
    lib.pg_check(ctx)
    _compare_final(lib, ctx, buf, cfg, rec, x_tol=2e-2)
    lib.pg_destroy(ctx)


PAPER_SCHEDULES = {
    "paper_std_small": [48] * 6 + [24] * 2 + [12] * 2,
    "paper_flash_small": [24] * 6 + [16] * 2 + [12] * 2,
    "paper_diffusion_small": [48] * 31 + [32] * 10 + [8] * 9,
    "paper_ablation32_small": [32] * 6 + [16] * 2 + [8] * 2,
    "paper_ablation48_small": [48] * 6 + [24] * 2 + [8] * 2,
    "paper_ablation64_small": [64] * 6 + [32] * 2 + [8] * 2,
}


@pytest.mark.parametrize("name", sorted(PAPER_SCHEDULES))
def test_paper_schedules(lib, name):
    """The paper's own schedules (Sec. 6.1: 48 -> 24 -> 12 at steps 5 and 7 of T = 10, the 24 -> 16 -> 12
    efficiency variant, 48 -> 32 -> 8 at steps 30 and 40 of T = 50 for the diffusion model; Sec. 6.3: 32, 48
    and 64 pruned to 8) on small networks: free-running library against the free-running oracle."""
    seed = 2512
    say(f"full loop {name}")
    cfg, w, inp, tables, rec = _oracle(name, seed)
    assert rec["active"] == PAPER_SCHEDULES[name]
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    lib.pg_sample_group(ctx, seed)
    lib.pg_check(ctx)
    _compare_final(lib, ctx, buf, cfg, rec, x_tol=2e-2)
    lib.pg_destroy(ctx)


def test_full_width_group_of_64_and_explicit_tables(lib):
    """Largest group the selection takes (64, the paper's largest G_max), caller-supplied step tables,
    a latent whose size is not a multiple of the streaming chunk."""
    cfg = workloads.get_config("cfg1")
    cfg.update(N=64, C=5, H=18, W=14, T=4, schedule=[[(1, 33), (2, 7)]])
    cfg["d"] = 5 * 18 * 14
    cfg["Li"] = 9 * 7
    say("loop N=64 with explicit tables")
    seed = 77
    w = workloads.make_weights(cfg); inp = workloads.make_inputs(cfg, w)
    tables = sampler.flow_sde_tables(4, 0.35)
    rec = loop.run(cfg, tables, inp, seed, wts=w)
    c, keep = lib.make_config(cfg, probe_bias=inp["probe_b"], tables=tables)
    ctx = lib.pg_create(c)
    buf = lib.Buffers(ctx, cfg, inputs=inp, weights_flat=lib.pack_weights(ctx, cfg, w))
    lib.pg_bind(ctx, buf)
    lib.pg_sample_group(ctx, seed)
    lib.pg_check(ctx)
    _compare_final(lib, ctx, buf, cfg, rec, x_tol=2e-2)
    assert lib.pg_state(ctx, 1)["M"] == 7
    lib.pg_destroy(ctx)


def test_sample_group_is_repeatable_and_seed_dependent(lib):
    cfg = workloads.get_config("cfg3_small")
    w = workloads.make_weights(cfg); inp = workloads.make_inputs(cfg, w)
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    outs = []
    for seed in (5, 5, 6):
        lib.pg_sample_group(ctx, seed)
        lib.pg_check(ctx)
        st = lib.pg_state(ctx, 1)
        outs.append((buf.x[st["cur_x"]][:st["M"]].clone(), buf.logp_sum.clone(), buf.masks.clone()))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    assert not torch.equal(outs[0][0], outs[2][0])
    lib.pg_destroy(ctx)


@pytest.mark.parametrize("name", ["cfg1", "cfg4_small_layers"])
def test_whole_loop_replays_from_a_hip_graph(lib, name):
    """The one-call loop copies nothing from the host and never waits for the device, so it can be recorded into a
    HIP graph (a caller that must not pay 2 400 launches per tiny group does that).  Every replay, with eager work
    of the library and synchronisations in between, must give the eager loop's result bit for bit."""
    seed = 4242
    say(f"graph capture {name}")
    cfg = _config(name)
    w = workloads.make_weights(cfg); inp = workloads.make_inputs(cfg, w)
    ctx, buf = _gpu_ctx(lib, cfg, w, inp)
    P = cfg["P"]
    lib.pg_sample_group(ctx, seed)                       # eager: also warms every one-time set-up of the launches
    lib.pg_check(ctx)
    st = lib.pg_state(ctx, P)
    M = st["M"]
    want = dict(x=buf.x[st["cur_x"]][:M].clone(), adv=buf.adv[:M].clone(), hist=buf.logp_hist.clone(),
                ids=buf.orig_id[st["cur_id"]][:M].clone(), masks=buf.masks.clone())
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        graph.capture_begin()
        lib.pg_sample_group(ctx, seed)                   # launches go to the capturing stream
        graph.capture_end()
    torch.cuda.synchronize()
    for rep in range(3):
        # eager work of the library between the replays, with another seed, so that a replay cannot pass on leftovers
        lib.pg_sample_group(ctx, seed + 1 + rep)
        lib.pg_check(ctx)
        assert not torch.equal(buf.x[lib.pg_state(ctx, P)["cur_x"]][:M], want["x"])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(buf.x[st["cur_x"]][:M], want["x"]), rep
        assert torch.equal(buf.adv[:M], want["adv"]) and torch.equal(buf.masks, want["masks"])
        assert torch.equal(buf.orig_id[st["cur_id"]][:M], want["ids"])
        assert torch.equal(buf.logp_hist.view(torch.int32), want["hist"].view(torch.int32))
        assert int(buf.status[0]) == 0
    lib.pg_destroy(ctx)


@pytest.mark.parametrize("name", ["cfg1", "cfg2_small", "cfg3_small", "cfg3_mmdit_small", "cfg1_layers", "cfg3_small_layers"])
def test_first_run_recorded_but_not_yet_replayed(lib, name):
    """A context whose first run is recorded into a HIP graph: an eager run before any replay gives what a context that was never
    captured gives, and so does the replay.  (The workspace starts as NaN patterns, so nothing can pass on its old contents.)"""
    seed = 91
    say(f"capture first {name}")
    cfg = _config(name)
    w = workloads.make_weights(cfg); inp = workloads.make_inputs(cfg, w)
    c, keep = lib.make_config(cfg, probe_bias=inp["probe_b"])
    runs = []
    for captured in (False, True):
        ctx = lib.pg_create(c)
        buf = lib.Buffers(ctx, cfg, inputs=inp, weights_flat=lib.pack_weights(ctx, cfg, w))
        buf.workspace.fill_(255)
        lib.pg_bind(ctx, buf)
        if captured:
            side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
            with torch.cuda.stream(side):
                graph.capture_begin()
                lib.pg_sample_group(ctx, seed)
                graph.capture_end()
            torch.cuda.synchronize()
        lib.pg_sample_group(ctx, seed + 1)
        lib.pg_check(ctx)
        st = lib.pg_state(ctx, cfg["P"])
        runs.append(buf.x[st["cur_x"]][:st["M"]].clone())
        if not captured:
            lib.pg_sample_group(ctx, seed)
            lib.pg_check(ctx)
            want = buf.x[st["cur_x"]][:st["M"]].clone()
        else:
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(buf.x[st["cur_x"]][:st["M"]], want)
        lib.pg_destroy(ctx)
    assert torch.equal(runs[0], runs[1])
