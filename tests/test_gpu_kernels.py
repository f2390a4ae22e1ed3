"""GPU parity of the kernel-level entry points against the oracle (through the C ABI)."""
import math
import numpy as np
import pytest
import torch

from oracle import philox, sampler, ovf
from paper_2512_15347_amd import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t.to(dtype) if dtype else t).to(DEV)


def say(msg):
    print(msg, flush=True)


# ------------------------------------------------------------------ initial latents / Philox
@pytest.mark.parametrize("n,d", [(3, 1024), (2, 4100), (5, 16384)])
def test_init_latents_matches_oracle(lib, n, d):
    say(f"init_latents n={n} d={d}")
    ids = np.array([7, 0, 123456, 5, 9][:n], dtype=np.int32)
    x = torch.zeros(n, d, device=DEV)
    seed = 0x1234567890ABCDEF
    lib.pg_init_latents(x, dev(ids), seed)
    torch.cuda.synchronize()
    want = np.stack([philox.normals(seed, philox.STREAM_INIT, int(i), 0, d) for i in ids])
    got = x.cpu().numpy().astype(np.float64)
    # fp32 hardware log2 / sin / cos / sqrt against the fp64 transform
    assert np.max(np.abs(got - want)) < 2e-5
    assert abs(got.mean()) < 5 / math.sqrt(got.size) and abs(got.var() - 1) < 0.05


def test_init_latents_empty_and_bad_shape(lib):
    x = torch.zeros(0, 64, device=DEV)
    lib.pg_init_latents(x, torch.zeros(0, dtype=torch.int32, device=DEV), 1)
    with pytest.raises(lib.PgError):
        lib.pg_init_latents(torch.zeros(2, 6, device=DEV), torch.zeros(2, dtype=torch.int32, device=DEV), 1)


# ------------------------------------------------------------------ fused update + log-prob
def _step_case(lib, n, d, seed, step, A, B, Cc, src=None, ids=None):
    x, u = workloads.stress_latents(n, d, seed=seed)
    ids = np.arange(n, dtype=np.int32) * 3 + 1 if ids is None else ids
    n_out = n if src is None else len(src)
    ids_out = ids if src is None else ids[src]
    xo = torch.zeros(n_out, d, device=DEV)
    logp = torch.zeros(n_out, device=DEV)
    hist = torch.full((int(ids.max()) + 1,), float("nan"), device=DEV)
    lsum = torch.ones(int(ids.max()) + 1, device=DEV)
    part = torch.zeros(lib.pg_step_scratch_floats(n_out, d), device=DEV)
    lib.pg_sde_step_logprob(dev(x), dev(u), xo, logp, hist, lsum, None if src is None else dev(src.astype(np.int32)),
                            dev(ids_out.astype(np.int32)), n_out, d, A, B, Cc, seed, step, part)
    torch.cuda.synchronize()
    rows = np.arange(n) if src is None else src
    xi = np.stack([philox.normals(seed, philox.STREAM_STEP, int(i), step, d) for i in ids_out])
    want_x, mean = sampler.sde_step(x[rows].astype(np.float64), u[rows].astype(np.float64), A, B, Cc, xi)
    want_lp = sampler.gaussian_logprob(want_x, mean, Cc)
    got_x = xo.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got_x - want_x)) < 1e-5 * max(1.0, np.max(np.abs(want_x)))
    got_lp = logp.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(got_lp, want_lp, rtol=2e-5)          # bar: 1e-3 relative
    h = hist.cpu().numpy()
    np.testing.assert_array_equal(h[ids_out], logp.cpu().numpy())
    assert np.isnan(np.delete(h, ids_out)).all()
    np.testing.assert_allclose(lsum.cpu().numpy()[ids_out], 1.0 + logp.cpu().numpy(), rtol=1e-6)


@pytest.mark.parametrize("n,d", [(4, 1024), (3, 4096 * 2 + 520), (2, 65536)])
def test_sde_step_logprob_matches_oracle(lib, n, d):
    say(f"sde_step n={n} d={d}")
    t = sampler.flow_sde_tables(10, 0.7)
    _step_case(lib, n, d, seed=42, step=3, A=t["A"][3], B=t["B"][3], Cc=t["C"][3])


def test_sde_step_with_gather_on_read(lib):
    say("sde_step gather")
    src = np.array([0, 2, 3, 7, 8, 11])
    _step_case(lib, 12, 4096 + 256, seed=9, step=5, A=0.93, B=-0.21, Cc=0.31, src=src)


@pytest.mark.parametrize("d", [1024, 4096, 4104, 8200, 12288, 16384, 16392])
def test_sums_over_a_trajectory_do_not_depend_on_the_batch(lib, d):
    """Few trajectories of at most four chunks of 4096 elements are summed by one workgroup each, 513 by one per chunk and a second
    launch: the same bits."""
    say(f"update and preview d={d}")
    n = 513
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    x, u = (torch.randn(n, d, device=DEV, generator=g) for _ in range(2))
    w = torch.randn(d, device=DEV, generator=g)
    ids = torch.arange(n, dtype=torch.int32, device=DEV)
    part = torch.zeros(lib.pg_step_scratch_floats(n, d), device=DEV)
    half = lambda t: t.to(torch.bfloat16).view(torch.int16).contiguous()
    results = []
    for m in (n, 512, 5):
        out, lp, hist, lsum, r = torch.zeros(m, d, device=DEV), *(torch.zeros(m, device=DEV) for _ in range(4))
        lib.pg_sde_step_logprob(x[:m], u[:m], out, lp, hist, lsum, None, ids[:m], m, d, 0.9, -0.2, 0.3, 7, 2, part)
        lib.pg_preview_reward(x[:m], u[:m], w, r, m, d, 1.0, -0.4, 0.1, part)
        out2, lp2 = torch.zeros(m, d, dtype=torch.int16, device=DEV), torch.zeros(m, device=DEV)
        lib.pg_sde_step_logprob_bf16(half(x[:m]), half(u[:m]), out2, lp2, None, None, None, ids[:m], m, d, 0.9, -0.2, 0.3, 7, 2, part)
        results.append([t[:5].cpu().numpy() for t in (out, lp, hist, lsum, r, out2, lp2)])
    for other in results[1:]:
        for a, b in zip(results[0], other):
            np.testing.assert_array_equal(a, b)
    assert np.isfinite(results[0][1]).all() and np.abs(results[0][4]).min() > 0


# the update has 256 lanes to a chunk where less than five sixths of 1024 would have work, else 1024: last chunks on either side of that and of
# one access alone; the same bits as a workgroup per trajectory, which takes few of at most four chunks, else against the oracle
@pytest.mark.parametrize("d", [4100, 6824, 6828, 8188, 8196, 10236, 10240, 12292, 13652, 13656, 16380, 16388, 20484])
def test_update_does_not_depend_on_the_lanes_of_a_chunk(lib, d):
    say(f"update of chunks, d={d}")
    if d > 4 * 4096:
        return _step_case(lib, 3, d, seed=5, step=1, A=0.93, B=-0.21, Cc=0.31)
    n = 513
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    x, u = (torch.randn(n, d, device=DEV, generator=g) for _ in range(2))
    ids = torch.arange(n, dtype=torch.int32, device=DEV)
    part = torch.zeros(lib.pg_step_scratch_floats(n, d), device=DEV)
    outs = [(torch.zeros(m, d, device=DEV), torch.zeros(m, device=DEV)) for m in (n, 512)]
    for out, lp in outs:
        lib.pg_sde_step_logprob(x, u, out, lp, None, None, None, ids, len(lp), d, 0.9, -0.2, 0.3, 7, 2, part)
    for many, few in zip(*outs):
        assert torch.equal(many[:512].view(torch.int32), few.view(torch.int32))


@pytest.mark.parametrize("d", [4100, 8192])
def test_sde_step_of_very_many_chunks(lib, d):
    """2^22 chunks of two to a trajectory: more than a launch has lanes for with one for every 16 bytes.  The sources repeat, so that
    the output alone is large (32 and 64 GiB); rows all over it against a call of their own."""
    n, few = 1 << 21, 64
    say(f"update of {n} trajectories of {d}")
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    x, u = (torch.randn(few, d, device=DEV, generator=g) for _ in range(2))
    ids = torch.arange(n, dtype=torch.int32, device=DEV)
    rows = torch.tensor([0, 1, 2, few + 3, n // 2 - 1, n // 2, n - 2, n - 1], device=DEV)
    got = []
    for some in (ids, ids[rows]):
        m = len(some)
        out, lp, part = torch.empty(m, d, device=DEV), torch.zeros(m, device=DEV), torch.zeros(lib.pg_step_scratch_floats(m, d), device=DEV)
        lib.pg_sde_step_logprob(x, u, out, lp, None, None, some % few, some, m, d, 0.9, -0.2, 0.3, 7, 2, part)
        got.append((out, lp) if m < n else (out[rows], lp[rows]))
        del out
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("n,d,gather", [(4, 1024, False), (3, 4096 * 2 + 520, False), (12, 4096 + 256, True)])
def test_sde_step_bf16_storage_matches_oracle(lib, n, d, gather):
    """Storage variant: bf16 latents and network output in, bf16 latents out.  The oracle takes the same
    bf16-representable inputs; the result may differ from the exactly rounded one by the fp32 arithmetic, i.e.
    by at most one bf16 rounding step; the log-prob is that of the fp32 call."""
    say(f"sde_step bf16 n={n} d={d}")
    seed, step, A, B, Cc = 17, 2, 0.93, -0.21, 0.31
    x, u = workloads.stress_latents(n, d, seed=seed)
    x = workloads.bf16_round(x); u = workloads.bf16_round(u)
    src = np.array([0, 2, 3, 7, 8, 11]) if gather else None
    ids = np.arange(n, dtype=np.int32) * 2 + 5
    rows = np.arange(n) if src is None else src
    ids_out = ids[rows]
    n_out = len(rows)
    bits = lambda a: torch.from_numpy(workloads.bf16_bits(a).view(np.int16)).to(DEV)
    xo = torch.zeros(n_out, d, dtype=torch.int16, device=DEV)
    logp = torch.zeros(n_out, device=DEV)
    part = torch.zeros(lib.pg_step_scratch_floats(n_out, d), device=DEV)
    lib.pg_sde_step_logprob_bf16(bits(x), bits(u), xo, logp, None, None, None if src is None else dev(src.astype(np.int32)),
                                 dev(ids_out.astype(np.int32)), n_out, d, A, B, Cc, seed, step, part)
    torch.cuda.synchronize()
    xi = np.stack([philox.normals(seed, philox.STREAM_STEP, int(i), step, d) for i in ids_out])
    want_x, mean = sampler.sde_step(x[rows].astype(np.float64), u[rows].astype(np.float64), A, B, Cc, xi)
    got = (xo.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    # half a bf16 step is 2^-9 of the value's power of two (<= 2^-8 relative); allow the fp32 arithmetic on top
    assert np.all(np.abs(got - want_x) <= 2.0 ** -8 * np.abs(want_x) * 1.02 + 1e-30 + 2e-6)
    exact = workloads.bf16_round(want_x.astype(np.float32)).astype(np.float64)
    assert np.mean(got == exact) > 0.995                             # rounding decisions differ only near ties
    np.testing.assert_allclose(logp.cpu().numpy().astype(np.float64), sampler.gaussian_logprob(want_x, mean, Cc), rtol=2e-5)
    with pytest.raises(lib.PgError):
        lib.pg_sde_step_logprob_bf16(bits(x), bits(u), xo, logp, None, None, None, dev(ids_out.astype(np.int32)), n_out, 1028, A, B,
                                     Cc, seed, step, part)


def test_sde_step_rejects_bad_arguments(lib):
    x = torch.zeros(2, 64, device=DEV); o = torch.zeros(2, 64, device=DEV)
    ids = torch.zeros(2, dtype=torch.int32, device=DEV); part = torch.zeros(2, device=DEV)
    with pytest.raises(lib.PgError):                                  # C = 0: no density
        lib.pg_sde_step_logprob(x, x, o, None, None, None, None, ids, 2, 64, 1.0, 1.0, 0.0, 1, 0, part)
    with pytest.raises(lib.PgError):                                  # in-place gather would race
        lib.pg_sde_step_logprob(x, x, x, None, None, None, None, ids, 2, 64, 1.0, 1.0, 0.5, 1, 0, part)
    lib.pg_sde_step_logprob(x, x, o, None, None, None, None, ids, 0, 64, 1.0, 1.0, 0.5, 1, 0, part)   # empty: no-op


# ------------------------------------------------------------------ preview + reward, gather
@pytest.mark.parametrize("n,d,with_u", [(5, 1024, True), (3, 16384 + 64, True), (4, 4096, False)])
def test_preview_reward_matches_oracle(lib, n, d, with_u):
    say(f"preview_reward n={n} d={d} u={with_u}")
    x, u = workloads.stress_latents(n, d, seed=5)
    w = np.random.default_rng(1).standard_normal(d).astype(np.float32) / math.sqrt(d)
    Pc, Qc, bias = (1.3, -0.6, 0.25) if with_u else (1.0, 0.0, -0.5)
    r = torch.zeros(n, device=DEV)
    part = torch.zeros(lib.pg_step_scratch_floats(n, d), device=DEV)
    lib.pg_preview_reward(dev(x), dev(u) if with_u else None, dev(w), r, n, d, Pc, Qc, bias, part)
    torch.cuda.synchronize()
    want = sampler.linear_reward(sampler.preview(x.astype(np.float64), u.astype(np.float64), Pc, Qc),
                                 w.astype(np.float64), bias)
    np.testing.assert_allclose(r.cpu().numpy(), want, rtol=0, atol=1e-5)      # bar: 1e-3 of sigma_R ~ 1


def test_compact_gather_is_bit_exact(lib):
    say("compact_gather")
    rng = np.random.default_rng(2)
    for n, d in ((16, 1024), (9, 4096 * 3 + 4)):
        x = rng.standard_normal((n, d), dtype=np.float32)
        x.view(np.uint32)[0, :4] = [0x7FC00001, 0x80000000, 0x00000001, 0xFF800000]   # NaN payload, -0, denormal, -inf
        src = np.sort(rng.choice(n, n // 2, replace=False)).astype(np.int32)
        out = torch.zeros(len(src), d, device=DEV)
        lib.pg_compact_gather(dev(x), out, dev(src), len(src), d)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), ovf.compact(x, src).view(np.uint32))
    lib.pg_compact_gather(dev(x), out, dev(src), 0, d)                   # empty


# ------------------------------------------------------------------ OVF
def _run_ovf(lib, rewards, offsets, ks):
    P = len(ks)
    total = int(np.sum(np.maximum(ks, 0)))          # a negative count reserves no slots
    masks = torch.zeros(P, dtype=torch.int64, device=DEV)
    sel = torch.full((max(total, 1),), -1, dtype=torch.int32, device=DEV)
    newoff = torch.zeros(P + 1, dtype=torch.int32, device=DEV)
    status = torch.zeros(4, dtype=torch.int32, device=DEV)
    scratch = torch.zeros(max(lib.pg_ovf_scratch_ints(P), 1), dtype=torch.int32, device=DEV)
    lib.pg_ovf_select(dev(rewards.astype(np.float32)), dev(np.asarray(offsets, np.int32)), dev(np.asarray(ks, np.int32)),
                      P, masks, sel, newoff, status, scratch)
    torch.cuda.synchronize()
    return (masks.cpu().numpy().view(np.uint64), sel.cpu().numpy()[:total], newoff.cpu().numpy(),
            int(status.cpu()[0]))


def test_ovf_stress_config_bit_exact(lib):
    say("ovf 4096 x 64 -> 16")
    for offset in (0.0, 23.0):
        r = workloads.stress_rewards(4096, 64, offset=offset)
        off = np.arange(4097) * 64
        ks = np.full(4096, 16)
        masks, sel, newoff, status = _run_ovf(lib, r.reshape(-1), off, ks)
        w_masks, w_sel, w_off = ovf.ovf_groups(r.reshape(-1), off, ks)
        assert status == 0
        np.testing.assert_array_equal(masks, w_masks)
        np.testing.assert_array_equal(sel, w_sel)
        np.testing.assert_array_equal(newoff, w_off)


@pytest.mark.parametrize("groups", [40, 16400])                     # a wave each; the rest of many groups, k > 32
def test_ovf_values_that_several_members_have(lib, groups):
    """Groups of 1 to 64 members with one value for all, two, pairs of every value, pairs and one more, and one pair among single values."""
    say(f"ovf ties, {groups} groups")
    rng = np.random.default_rng(groups)
    sizes = np.array([64, 64, 64, 63, 64, 33, 2, 40] * (groups // 8))
    ks = np.array([40, 33, 35, 34, 63, 17, 1, 39] * (groups // 8))
    off = np.concatenate([[0], np.cumsum(sizes)])
    r = np.empty(off[-1], np.float32)
    for g, n in enumerate(sizes):
        levels = (1, 2, 32, 32, 63, 16, 1, 12)[g % 8]
        r[off[g]:off[g + 1]] = rng.permutation(np.arange(n) % levels) * 0.37 - 3
    masks, sel, newoff, status = _run_ovf(lib, r, off, ks)
    w_masks, w_sel, w_off = ovf.ovf_groups(r, off, ks)
    assert status == 0
    np.testing.assert_array_equal(masks, w_masks)
    np.testing.assert_array_equal(sel, w_sel)
    np.testing.assert_array_equal(newoff, w_off)


def test_ovf_ragged_groups_ties_and_degenerate_k(lib):
    say("ovf ragged")
    rng = np.random.default_rng(8)
    sizes = [48, 48, 32, 17, 64, 1, 2, 64, 33, 5, 48, 64]
    ks =    [32, 48, 16, 5, 16, 1, 1, 64, 32, 5, 1, 63]
    off = np.concatenate([[0], np.cumsum(sizes)])
    r = rng.standard_normal(off[-1]).astype(np.float32)
    r[off[2]:off[3]] = np.round(r[off[2]:off[3]] * 2) / 2        # many exact ties
    r[off[8]:off[9]] = 0.75                                       # all equal
    r[off[4]] = -0.0; r[off[4] + 1] = 0.0
    masks, sel, newoff, status = _run_ovf(lib, r, off, ks)
    w_masks, w_sel, w_off = ovf.ovf_groups(r, off, ks)
    assert status == 0
    np.testing.assert_array_equal(masks, w_masks)
    np.testing.assert_array_equal(sel, w_sel)
    np.testing.assert_array_equal(newoff, w_off)


def test_ovf_groups_above_64_members(lib):
    """Groups of up to 1024 members (one workgroup per group), ragged, with ties, bit for bit against the
    oracle; groups of at most 64 members must get the 64-slot routine's answer."""
    say("ovf large groups")
    rng = np.random.default_rng(21)
    sizes = [1024, 65, 100, 513, 64, 48, 1, 777, 200, 1000, 129, 2]
    ks =    [512, 7, 50, 40, 16, 24, 1, 776, 200, 1, 64, 1]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    r = (rng.standard_normal(off[-1]) * np.where(rng.random(off[-1]) < 0.8, 0.05, 1.0)).astype(np.float32)
    r[off[2]:off[3]] = np.round(r[off[2]:off[3]] * 4) / 4         # many exact ties
    r[off[10]:off[11]] = -1.5                                      # all equal
    words = 16
    w_masks, w_sel, w_off = ovf.ovf_groups_large(r, off, ks, words)
    P = len(sizes)
    masks = torch.full((P, words), -1, dtype=torch.int64, device=DEV)
    sel = torch.full((int(np.sum(ks)),), -1, dtype=torch.int32, device=DEV)
    noff = torch.zeros(P + 1, dtype=torch.int32, device=DEV)
    status = torch.zeros(4, dtype=torch.int32, device=DEV)
    scratch = torch.zeros(lib.pg_ovf_scratch_ints(P), dtype=torch.int32, device=DEV)
    lib.pg_ovf_select_large(torch.from_numpy(r).to(DEV), torch.from_numpy(off).to(DEV),
                            torch.tensor(ks, dtype=torch.int32, device=DEV), P, words, masks, sel, noff, status, scratch)
    torch.cuda.synchronize()
    assert status[0].item() == 0
    np.testing.assert_array_equal(masks.cpu().numpy().view(np.uint64), w_masks)
    np.testing.assert_array_equal(noff.cpu().numpy(), w_off)
    np.testing.assert_array_equal(sel.cpu().numpy(), w_sel)
    # the small groups agree with the one-wave kernel
    for g in (4, 5, 6, 11):
        m64, _, _ = ovf.ovf_groups(r[off[g]:off[g + 1]], [0, sizes[g]], [ks[g]])
        assert int(w_masks[g, 0]) == int(m64[0])
    # a group that does not fit the mask, a bad k and a non-finite reward are flagged
    off2 = torch.tensor([0, 200, 210, 300], dtype=torch.int32, device=DEV)
    k2 = torch.tensor([5, 11, 3], dtype=torch.int32, device=DEV)
    r2 = torch.from_numpy(r[:300].copy()).to(DEV); r2[250] = float("inf")
    masks2 = torch.full((3, 2), -1, dtype=torch.int64, device=DEV)
    sel2 = torch.full((19,), -1, dtype=torch.int32, device=DEV)
    status.zero_()
    lib.pg_ovf_select_large(r2, off2, k2, 3, 2, masks2, sel2, noff[:4], status, scratch)
    torch.cuda.synchronize()
    assert status[0].item() == 3
    m2 = masks2.cpu().numpy().view(np.uint64)
    assert not m2[0].any() and not m2[1].any() and int(m2[2, 0]) == 0b111
    assert sel2.cpu().numpy()[16:].tolist() == [210, 211, 212]


def test_ovf_many_groups_and_schedule_sizes(lib):
    say("ovf 20000 groups")
    rng = np.random.default_rng(9)
    sizes = rng.choice([24, 32, 48, 64], size=20000)
    ks = np.array([{24: 12, 32: 16, 48: 32, 64: 8}[int(s)] for s in sizes])
    off = np.concatenate([[0], np.cumsum(sizes)])
    r = (rng.standard_normal(off[-1]) * 0.3 + 22.0).astype(np.float32)
    masks, sel, newoff, status = _run_ovf(lib, r, off, ks)
    w_masks, w_sel, w_off = ovf.ovf_groups(r, off, ks)
    assert status == 0
    np.testing.assert_array_equal(masks, w_masks)
    np.testing.assert_array_equal(sel, w_sel)
    np.testing.assert_array_equal(newoff, w_off)


@pytest.mark.parametrize("lo,hi,kmax", [(2, 16, 15), (9, 32, 16), (20, 32, 31), (33, 64, 16), (2, 64, 32), (1, 64, 64)])
def test_ovf_one_lane_per_group(lib, lo, hi, kmax):
    """Enough groups for the one-lane-per-group kernel, last wave and workgroup part empty: every sort width and scan
    length, ties across the thresholds, a wave with an unsuitable group (k = n, k > 32, one member, a NaN)."""
    G = 32768 + 77
    say(f"ovf lanes {lo}..{hi}")
    rng = np.random.default_rng(hi * 100 + kmax)
    sizes = rng.integers(lo, hi + 1, G)
    ks = np.minimum(rng.integers(1, kmax + 1, G), np.maximum(sizes - (kmax < 64), 1))
    off = np.concatenate([[0], np.cumsum(sizes)])
    r = (rng.standard_normal(off[-1]) * np.where(rng.random(off[-1]) < 0.8, 0.05, 1.0)).astype(np.float32)
    r[: off[G // 2]] = np.round(r[: off[G // 2]] * 4) / 4            # exact ties, signed zeros among them
    masks, sel, newoff, status = _run_ovf(lib, r, off, ks)
    w_masks, w_sel, w_off = ovf.ovf_groups(r, off, ks)
    assert status == 0
    np.testing.assert_array_equal(masks, w_masks)
    np.testing.assert_array_equal(sel, w_sel)
    np.testing.assert_array_equal(newoff, w_off)
    r[off[70]] = np.nan                                              # second wave: flagged, the other groups as before
    masks, sel, newoff, status = _run_ovf(lib, r, off, ks)
    assert status == 1 and off[70] <= sel[w_off[70]] < off[71]
    np.testing.assert_array_equal(np.delete(masks, 70), np.delete(w_masks, 70))


@pytest.mark.parametrize("sizes_of", ["proper", "any"])
def test_ovf_one_lane_per_group_against_one_wave_per_group(lib, sizes_of):
    """Groups that need no selection, keep more than 32, hold a reward that is not finite or have a bad count, mixed into one
    call that is large enough for the one-lane-per-group kernel: what the calls below its threshold give, slice by slice.
    `any`: some sizes lie outside 0..64 as well."""
    say(f"ovf lanes against waves, {sizes_of} sizes")
    G, part = 16384 + 333, 8000
    rng = np.random.default_rng(31)
    sizes = rng.integers(1, 65, G)
    sizes[rng.random(G) < 0.05] = 0
    ks = np.minimum(rng.integers(1, 33, G), sizes)
    form = rng.integers(0, 60, G)
    ks = np.where(form < 3, sizes, ks)                               # keeps all
    ks = np.where((form == 3) & (sizes > 34), sizes - 1, ks)         # more than 32
    ks[(form == 4) | (sizes == 0) & (form == 5)] = 3                 # bad where larger than the group
    ks[form == 6] = 0
    ks[form == 7] = -2
    ks[form == 8] += 70
    ks[2048:2048 + 640] = np.maximum(sizes[2048:2048 + 640] - 1, 0)  # whole waves that keep nearly all
    ks[4096:4096 + 640] = sizes[4096:4096 + 640]
    sizes[6400:6464], ks[6400:6464] = 0, 0                           # a wave of empty groups
    if sizes_of == "any":
        odd = rng.choice(G - 1, 40, replace=False) + 1
        sizes[odd] = rng.integers(65, 200, 40)
        sizes[odd - 1] = -5
    off = np.concatenate([[300], 300 + np.cumsum(sizes)])
    r = rng.standard_normal(int(off.max()) + 1).astype(np.float32)
    r[rng.random(len(r)) < 2e-4] = np.nan
    r[rng.random(len(r)) < 1e-4] = -np.inf
    rd, od, kd = dev(r), dev(off.astype(np.int32)), dev(ks.astype(np.int32))

    def select(first, last):
        n = last - first
        masks = torch.full((n,), -1, dtype=torch.int64, device=DEV)
        sel = torch.full((int(np.maximum(ks[first:last], 0).sum()),), -1, dtype=torch.int32, device=DEV)
        noff = torch.full((n + 1,), -1, dtype=torch.int32, device=DEV)
        status = torch.zeros(4, dtype=torch.int32, device=DEV)
        scratch = torch.zeros(lib.pg_ovf_scratch_ints(n), dtype=torch.int32, device=DEV)
        lib.pg_ovf_select(rd, od[first:last + 1], kd[first:last], n, masks, sel, noff, status, scratch)
        return masks.cpu().numpy(), sel.cpu().numpy(), noff.cpu().numpy(), status.cpu().numpy()

    masks, sel, noff, status = select(0, G)
    assert status.tolist() == [3, 0, 0, 0]
    np.testing.assert_array_equal(noff, np.concatenate([[0], np.cumsum(np.maximum(ks, 0))]))
    for first in range(0, G, part):
        last = min(first + part, G)
        w_masks, w_sel, _, _ = select(first, last)
        np.testing.assert_array_equal(masks[first:last], w_masks)
        np.testing.assert_array_equal(sel[noff[first]:noff[last]], w_sel)


@pytest.mark.parametrize("n,k", [(64, 16), (64, 17), (64, 32), (64, 1), (32, 16), (32, 31), (16, 15), (16, 4), (48, 16), (20, 7), (4, 3)])
def test_ovf_lanes_with_groups_of_whole_chunks(lib, n, k):
    """Groups that start and end on 16 bytes are staged by direct loads, others through registers: the oracle's selection with
    the rewards aligned, the same with them one float further on; equal sizes (nothing to pad when they fill the sort), then sizes
    that are multiples of four; ties across the thresholds, a reward that is not finite, groups that keep everything."""
    say(f"ovf lanes, whole chunks, {n} -> {k}")
    G = 16384 + 77
    for mixed in (False, True):
        rng = np.random.default_rng(1000 * n + k + mixed)
        sizes = np.full(G, n) if not mixed else 4 * rng.integers(1, n // 4 + 1, G)
        ks = np.minimum(np.full(G, k), sizes - (sizes > 1))
        ks[rng.random(G) < 0.01] = 1
        ks[40:44] = sizes[40:44]
        off = np.concatenate([[0], np.cumsum(sizes)])
        r = rng.standard_normal(off[-1] + 1).astype(np.float32)
        r[: off[G // 2]] = np.round(r[: off[G // 2]] * 4) / 4
        want = ovf.ovf_groups(r[:-1], off, ks)
        for shift in (0, 1):
            base = dev(np.concatenate([np.zeros(shift, np.float32), r]))[shift:]
            assert base.data_ptr() % 16 == 4 * shift
            for bad in (False, True):
                if bad:
                    base[int(off[200])] = float("inf")
                masks = torch.full((G,), -1, dtype=torch.int64, device=DEV)
                sel = torch.full((int(ks.sum()),), -1, dtype=torch.int32, device=DEV)
                noff, status = torch.zeros(G + 1, dtype=torch.int32, device=DEV), torch.zeros(4, dtype=torch.int32, device=DEV)
                scratch = torch.zeros(lib.pg_ovf_scratch_ints(G), dtype=torch.int32, device=DEV)
                lib.pg_ovf_select(base, dev(off.astype(np.int32)), dev(ks.astype(np.int32)), G, masks, sel, noff, status, scratch)
                got = masks.cpu().numpy().view(np.uint64)
                np.testing.assert_array_equal(noff.cpu().numpy(), want[2])
                assert int(status[0]) == (1 if bad else 0)
                if bad:                                             # the first slots are kept where a reward is not finite
                    assert got[200] == np.uint64((1 << int(ks[200])) - 1)
                    np.testing.assert_array_equal(np.delete(got, 200), np.delete(want[0], 200))
                else:
                    np.testing.assert_array_equal(got, want[0])
                    np.testing.assert_array_equal(sel.cpu().numpy(), want[1])


def test_ovf_unsuited_groups_do_not_hold_up_a_batch(lib):
    """A batch whose groups all keep more than 32, or in which every 64th group keeps everything, takes no longer than a few
    times the batch that suits the one-lane-per-group kernel best (about 1.5 and 1.1 times; 11 times when the wave that met
    such a group did its 64 groups one after another)."""
    say("ovf lanes, time with unsuited groups")
    G = 16384
    off = torch.arange(G + 1, dtype=torch.int32, device=DEV) * 64
    r = torch.randn(G * 64, device=DEV)
    masks, noff = torch.zeros(G, dtype=torch.int64, device=DEV), torch.zeros(G + 1, dtype=torch.int32, device=DEV)
    status, scratch = torch.zeros(4, dtype=torch.int32, device=DEV), torch.zeros(lib.pg_ovf_scratch_ints(G), dtype=torch.int32, device=DEV)

    def micros(k):
        sel = torch.zeros(int(k.sum()), dtype=torch.int32, device=DEV)
        a, b, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), 1e9
        for _ in range(6):
            a.record()
            for _ in range(20):
                lib.pg_ovf_select(r, off, k, G, masks, sel, noff, status, scratch)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    suited = micros(torch.full((G,), 16, dtype=torch.int32, device=DEV))
    many = micros(torch.full((G,), 40, dtype=torch.int32, device=DEV))
    one_in_64 = torch.full((G,), 16, dtype=torch.int32, device=DEV)
    one_in_64[5::64] = 64
    unpruned = micros(one_in_64)
    say(f"  {suited:.1f} us, all keep 40: {many:.1f} us, one in 64 keeps all: {unpruned:.1f} us")
    assert many < 4 * suited and unpruned < 4 * suited


@pytest.mark.parametrize("n,k", [(64, 16), (32, 8), (16, 4)])
def test_ovf_groups_with_nothing_to_sort_cost_what_they_write(lib, n, k):
    """Sizes that fill the sort, one group in 64 unpruned: the other lanes' time does not change, and the unpruned groups write n - k
    more indices each (3 % of the batch's bytes).  One such group in a wave took it to 1.65 (64 -> 16), 1.52 and 1.35 times while its
    lane sent the others through the route of ties."""
    say(f"ovf lanes, time with unpruned groups, {n} -> {k}")
    G = 1 << 18
    off = torch.arange(G + 1, dtype=torch.int32, device=DEV) * n
    r = torch.randn(G * n, device=DEV)
    masks, noff = torch.zeros(G, dtype=torch.int64, device=DEV), torch.zeros(G + 1, dtype=torch.int32, device=DEV)
    status, scratch = torch.zeros(4, dtype=torch.int32, device=DEV), torch.zeros(lib.pg_ovf_scratch_ints(G), dtype=torch.int32, device=DEV)
    micros = []
    for kept in (k, n):
        ks = torch.full((G,), k, dtype=torch.int32, device=DEV)
        ks[5::64] = kept
        sel = torch.zeros(int(ks.sum()), dtype=torch.int32, device=DEV)
        a, b, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), 1e9
        for _ in range(8):
            a.record()
            for _ in range(20):
                lib.pg_ovf_select(r, off, ks, G, masks, sel, noff, status, scratch)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        micros.append(best)
    say(f"  plain {micros[0]:.1f} us, one in 64 unpruned {micros[1]:.1f} us")
    assert micros[1] < 1.2 * micros[0]


@pytest.mark.parametrize("words", [1, 2, 3, 4, 5, 8, 9, 16])
def test_ovf_large_at_every_workgroup_size(lib, words):
    say(f"ovf large, {words} mask words")
    rng = np.random.default_rng(words)
    P, top = 4096 + 5, 64 * words                                    # the count sums of two launches
    sizes = np.where(rng.random(P) < 0.02, rng.integers(1, top + 1, P), rng.integers(1, 9, P))
    sizes[:3] = [top, max(1, top - 1), top // 2 + 1]
    ks = np.array([rng.integers(1, n + 1) for n in sizes])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    r = np.round(rng.standard_normal(off[-1]) * 8).astype(np.float32) / 8
    w_masks, w_sel, w_off = ovf.ovf_groups_large(r, off, ks, words)
    masks = torch.full((P, words), -1, dtype=torch.int64, device=DEV)
    sel = torch.full((int(ks.sum()),), -1, dtype=torch.int32, device=DEV)
    noff = torch.zeros(P + 1, dtype=torch.int32, device=DEV)
    status = torch.zeros(4, dtype=torch.int32, device=DEV)
    scratch = torch.zeros(lib.pg_ovf_scratch_ints(P), dtype=torch.int32, device=DEV)
    lib.pg_ovf_select_large(dev(r), dev(off), dev(ks.astype(np.int32)), P, words, masks, sel, noff, status, scratch)
    assert status[0].item() == 0
    np.testing.assert_array_equal(masks.cpu().numpy().view(np.uint64), np.asarray(w_masks).reshape(P, words))
    np.testing.assert_array_equal(sel.cpu().numpy(), w_sel)
    np.testing.assert_array_equal(noff.cpu().numpy(), w_off)


def test_ovf_flags_non_finite_and_bad_counts(lib):
    say("ovf error flags")
    r = np.array([0.1, np.nan, 0.3, 0.4, 1.0, 2.0, 3.0, 4.0], dtype=np.float32)
    masks, sel, newoff, status = _run_ovf(lib, r, [0, 4, 8], [2, 2])
    assert status & 1
    assert masks[1] == np.uint64(ovf.ovf_select(r[4:], 2)[0])    # the clean group is still selected
    assert set(sel[:2].tolist()) <= {0, 1, 2, 3}                  # indices stay inside the group
    r[1] = np.inf
    assert _run_ovf(lib, r, [0, 4, 8], [2, 2])[3] & 1
    r[1] = 0.2
    masks, sel, newoff, status = _run_ovf(lib, r, [0, 4, 8], [5, 2])   # k > n
    assert status & 2 and masks[0] == 0
    # the five slots reserved for the bad group hold rows of that group, and the clean group behind it is intact
    assert newoff.tolist() == [0, 5, 7] and set(sel[:5].tolist()) <= {0, 1, 2, 3}
    assert sel[5:7].tolist() == [4 + i for i in range(4) if (int(masks[1]) >> i) & 1]
    # a negative count reserves nothing: the groups behind it keep non-negative offsets
    masks, sel, newoff, status = _run_ovf(lib, r, [0, 4, 8], [-3, 2])
    assert status & 2 and masks[0] == 0 and newoff.tolist() == [0, 0, 2]
    assert masks[1] == np.uint64(ovf.ovf_select(r[4:], 2)[0])
    masks, sel, newoff, status = _run_ovf(lib, r, [0, 0, 8], [0, 3])   # an empty group is fine
    assert status == 0 and masks[0] == 0 and newoff.tolist() == [0, 0, 3]


# ------------------------------------------------------------------ advantages
def test_group_advantages_match_oracle(lib):
    say("advantages")
    rng = np.random.default_rng(3)
    sizes = [16, 12, 4, 1, 8, 64, 16]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    r = (rng.standard_normal(off[-1]) * 0.3 + 22.0).astype(np.float32)
    r[off[4]:off[5]] = 1.25
    adv = torch.zeros(int(off[-1]), device=DEV)
    for eps in (1e-6, 1e-2):
        lib.pg_group_advantages(dev(r), dev(off), len(sizes), eps, adv)
        torch.cuda.synchronize()
        want = ovf.group_advantages(r.astype(np.float64), off, eps)
        np.testing.assert_allclose(adv.cpu().numpy(), want, rtol=1e-5, atol=1e-6)
    a = adv.cpu().numpy()
    assert np.all(a[off[3]:off[5]] == 0)
