"""GPU parity of the network kernels (MFMA GEMM, attention, whole forward) against the oracle."""
import math
import numpy as np
import pytest
import torch

from oracle import dit
from paper_2512_15347_amd import workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)


def bf16_dev(a):
    """fp32 host array of bf16-representable values -> int16 device tensor of bit patterns."""
    return torch.from_numpy(workloads.bf16_bits(a).view(np.int16)).to(DEV)


# ragged last tiles in both directions, by the launcher's choice
@pytest.mark.parametrize("M,N,K", [(300, 200, 128), (2356, 384, 512), (256, 256, 64), (1, 16, 64), (777, 4608, 1536),
                                   (12251, 768, 128), (12251, 2304, 64), (12283, 3072, 128), (24571, 1532, 64),
                                   (18848, 1536, 64), (9001, 520, 192)])
def test_gemm_matches_oracle_linear(lib, M, N, K):
    say(f"gemm M={M} N={N} K={K}")
    rng = np.random.default_rng(M + N + K)
    A = workloads.bf16_round(rng.standard_normal((M, K), dtype=np.float32))
    W = workloads.bf16_round(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    b = workloads.bf16_round(rng.standard_normal(N, dtype=np.float32))
    out = torch.full((M, N), float("nan"), device=DEV)
    lib.pg_gemm_bf16(bf16_dev(A), K, bf16_dev(W), K, bf16_dev(b), out, N, M, N, K)
    torch.cuda.synchronize()
    want = dit.linear(A.astype(np.float64), W, b)
    got = out.cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    # fp32 accumulation of exact bf16 products: error ~ sqrt(K) * 2^-24 * |a||w|
    assert np.max(np.abs(got - want)) < 2e-5 * math.sqrt(K) * np.max(np.abs(want)) + 1e-6


# tiles by the launcher's choice, one row and column short of or past a tile
@pytest.mark.parametrize("M,N,K", [(3213, 4484, 256), (14100, 1540, 192), (3697, 6140, 192), (4000, 4100, 128), (5000, 1000, 64),
                                   (4099, 1404, 320), (4097, 1020, 192), (63, 252, 64), (65, 68, 192), (64, 64, 128)])
def test_gemm_tiles_with_short_k(lib, M, N, K):
    test_gemm_matches_oracle_linear(lib, M, N, K)


# tiles by the launcher's choice with fewer K steps than their operands have stages in LDS, as many, and more (test_gemm_tile_by_tile has
# all of them)
@pytest.mark.parametrize("M,N", [(28673, 260), (14337, 516), (16385, 516), (12289, 516), (14337, 260), (5121, 516), (4097, 260), (70, 68)])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 7])
def test_gemm_stages_in_lds(lib, M, N, steps):
    test_gemm_matches_oracle_linear(lib, M, N, 64 * steps)


# every tile with fewer K steps than its operands have stages in LDS, as many, and more: 256 x 256 and 128 x 128 (two stages of either
# operand), 192 and 224 rows (three of A, two of W), 160 rows, 128 x 256 and 128 x 64 (three), 64 x 64 (two; three); stored and added, with
# rows and columns that fill no last tile, and with fewer of them than a tile has
@pytest.mark.parametrize("tile", range(1, 10))
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 7])
def test_gemm_tile_by_tile(lib, tile, steps):
    K = 64 * steps
    say(f"gemm tile {tile}, {steps} K steps")
    for M, N in ((485, 292), (39, 20)):
        rng = np.random.default_rng(M + steps)
        A = workloads.bf16_round(rng.standard_normal((M, K), dtype=np.float32))
        W = workloads.bf16_round(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
        b = workloads.bf16_round(rng.standard_normal(N, dtype=np.float32))
        Ad, Wd, bd = bf16_dev(A), bf16_dev(W), bf16_dev(b)
        out, chosen = (torch.full((M + 1, N), float("nan"), device=DEV) for _ in range(2))
        lib.pg_gemm_bf16_tile(Ad, K, Wd, K, bd, out, N, M, N, K, tile=tile)
        lib.pg_gemm_bf16(Ad, K, Wd, K, bd, chosen, N, M, N, K)
        added = torch.randn(M + 1, N, device=DEV, generator=torch.Generator(device=DEV).manual_seed(tile))
        before = added.clone()
        lib.pg_gemm_bf16_tile(Ad, K, Wd, K, bd, added, N, M, N, K, accumulate=True, tile=tile)
        want = dit.linear(A.astype(np.float64), W, b)
        # fp32 accumulation of exact bf16 products: error ~ sqrt(K) * 2^-24 * |a||w|
        assert np.max(np.abs(out[:M].cpu().numpy() - want)) < 2e-5 * math.sqrt(K) * np.max(np.abs(want)) + 1e-6
        assert torch.equal(out[:M], chosen[:M]) and out[M].isnan().all()
        assert torch.equal(added[:M], before[:M] + out[:M]) and torch.equal(added[M], before[M])


@pytest.mark.parametrize("ld", [1 << 23, (1 << 23) + 64])
def test_gemm_rows_far_apart(lib, ld):
    """Row strides on both sides of what a 32-bit byte offset inside a tile can express."""
    say(f"gemm ld={ld}")
    M, N, K = 9, 12, 128
    rng = np.random.default_rng(5)
    A = workloads.bf16_round(rng.standard_normal((M, K), dtype=np.float32))
    W = workloads.bf16_round(rng.standard_normal((N, K), dtype=np.float32))
    Ad = torch.zeros(M * ld, dtype=torch.int16, device=DEV)
    Ad.view(M, ld)[:, :K] = bf16_dev(A)
    Wd = torch.zeros(N * ld, dtype=torch.int16, device=DEV)
    Wd.view(N, ld)[:, :K] = bf16_dev(W)
    out = torch.full((M, N), float("nan"), device=DEV)
    lib.pg_gemm_bf16(Ad, ld, Wd, ld, None, out, N, M, N, K)
    want = dit.linear(A.astype(np.float64), W, np.zeros(N, np.float32))
    assert np.max(np.abs(out.cpu().numpy() - want)) < 2e-5 * math.sqrt(K) * np.max(np.abs(want))


def test_gemm_rejects_bad_shapes(lib):
    A = torch.zeros(64, 96, dtype=torch.int16, device=DEV)
    out = torch.zeros(64, 64, device=DEV)
    with pytest.raises(lib.PgError):
        lib.pg_gemm_bf16(A, 96, A, 96, None, out, 64, 64, 64, 96)       # K not a multiple of 64
    lib.pg_gemm_bf16(A, 96, A, 96, None, out, 64, 0, 64, 64)           # empty: no-op


@pytest.mark.parametrize("B,Lq,Lk,heads,hd", [(2, 90, 90, 2, 64), (1, 64, 13, 2, 64), (3, 64, 64, 4, 32),
                                              (1, 300, 1178, 3, 64), (2, 130, 77, 2, 32)])
def test_attention_matches_oracle(lib, B, Lq, Lk, heads, hd):
    say(f"attention B={B} Lq={Lq} Lk={Lk} heads={heads} hd={hd}")
    rng = np.random.default_rng(Lq * 7 + Lk)
    D = heads * hd
    q = workloads.bf16_round(rng.standard_normal((B, Lq, D), dtype=np.float32) * 1.5)
    k = workloads.bf16_round(rng.standard_normal((B, Lk, D), dtype=np.float32))
    v = workloads.bf16_round(rng.standard_normal((B, Lk, D), dtype=np.float32))
    Lkpad = (Lk + 63) // 64 * 64
    vt = np.full((B, D, Lkpad), np.nan, dtype=np.float32)          # padding must be ignored, whatever it holds
    vt[:, :, :Lk] = v.transpose(0, 2, 1)
    out = torch.zeros(B, Lq, D, dtype=torch.int16, device=DEV)
    lib.pg_attention_bf16(bf16_dev(q), bf16_dev(k), bf16_dev(vt), out, B, Lq, Lk, heads, hd)
    torch.cuda.synchronize()
    got = out.view(torch.bfloat16).float().cpu().numpy().astype(np.float64)
    want = dit.attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), heads)
    assert np.isfinite(got).all()
    # probabilities and outputs are rounded to bf16 (2^-9 relative)
    assert np.max(np.abs(got - want)) < 1.5e-2 * np.max(np.abs(want))
    assert np.sqrt(np.mean((got - want) ** 2)) < 4e-3 * np.sqrt(np.mean(want ** 2))


@pytest.mark.parametrize("hd,Lk", [(64, 128), (64, 20), (32, 77)])
def test_attention_with_every_score_far_below_zero(lib, hd, Lk):
    """The first key tile sets a query's reference exponent; here it lies at -1000 or below, and 2^1000 has no fp32 value."""
    say(f"attention far below zero hd={hd} Lk={Lk}")
    rng = np.random.default_rng(hd + Lk)
    B, Lq, heads = 1, 40, 2
    D = heads * hd
    q = workloads.bf16_round(8.0 + rng.standard_normal((B, Lq, D), dtype=np.float32) * 0.1)
    k = workloads.bf16_round(-90.0 * (1.0 if hd == 64 else 1.5) / math.sqrt(hd) + rng.standard_normal((B, Lk, D), dtype=np.float32) * 0.05)
    v = workloads.bf16_round(rng.standard_normal((B, Lk, D), dtype=np.float32))
    Lkpad = (Lk + 63) // 64 * 64
    vt = np.zeros((B, D, Lkpad), dtype=np.float32)
    vt[:, :, :Lk] = v.transpose(0, 2, 1)
    out = torch.zeros(B, Lq, D, dtype=torch.int16, device=DEV)
    lib.pg_attention_bf16(bf16_dev(q), bf16_dev(k), bf16_dev(vt), out, B, Lq, Lk, heads, hd)
    got = out.view(torch.bfloat16).float().cpu().numpy().astype(np.float64)
    want = dit.attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), heads)
    assert np.isfinite(got).all()
    # rounding of the scaled queries to bf16 moves the output by 2e-3 of its maximum (the part common to all keys cancels), fp32
    # scores of this size (ulp 1e-4) by less; probabilities and outputs are rounded to bf16
    assert np.max(np.abs(got - want)) < 1.5e-2 * np.max(np.abs(want))


def _network_attention(lib, q, k, v, heads, kernel):
    """Output [B, Lq, D] of the kernel on queries already in the softmax's log2 units; values in the network's key order, NaN in
    the padding."""
    B, Lq, D = q.shape
    Lk, Lkpad = k.shape[1], (k.shape[1] + 63) // 64 * 64
    vt = np.full((B, D, Lkpad), np.nan, dtype=np.float32)
    t = np.arange(Lk)
    vt[:, :, (t & ~12) | ((t & 4) << 1) | ((t & 8) >> 1)] = v.transpose(0, 2, 1)
    out = torch.full((B, Lq, D), -1, dtype=torch.int16, device=DEV)
    lib.pg_attention_network(bf16_dev(q), bf16_dev(k), bf16_dev(vt), out, B, Lq, Lk, Lkpad, heads, D // heads, kernel)
    return out.view(torch.bfloat16).float().cpu().numpy().astype(np.float64)


# whole key tiles, last tiles that end in their first and second half, on and inside a group of 16 and of 4 keys, one key; query
# counts that leave a wave's second 32, whole waves, or nearly a workgroup without work.  gain: scale of the scores; rising: later
# keys score higher, so that tile after tile raises the reference
@pytest.mark.parametrize("B,Lq,Lk,heads,hd,gain,rising", [
    (1, 256, 128, 2, 64, 1.0, False), (2, 90, 90, 2, 64, 1.0, False), (1, 300, 1178, 3, 64, 1.0, False), (3, 33, 211, 1, 64, 1.0, False),
    (1, 130, 77, 2, 64, 1.0, False), (1, 64, 13, 2, 64, 1.0, False), (2, 5, 1, 2, 64, 1.0, False), (1, 260, 506, 2, 64, 12.0, False),
    (1, 257, 484, 2, 64, 1.0, True), (1, 100, 330, 2, 64, 12.0, True), (2, 130, 77, 2, 32, 1.0, False), (3, 64, 64, 4, 32, 1.0, False),
    (1, 140, 186, 3, 32, 12.0, True), (1, 40, 29, 2, 32, 1.0, False)])
def test_network_attention_kernels_match_oracle(lib, B, Lq, Lk, heads, hd, gain, rising):
    say(f"network attention B={B} Lq={Lq} Lk={Lk} heads={heads} hd={hd} gain={gain} rising={rising}")
    rng = np.random.default_rng(Lq * 7 + Lk)
    D = heads * hd
    scale = np.float32(1.4426950408889634 / math.sqrt(hd))
    q = workloads.bf16_round(rng.standard_normal((B, Lq, D), dtype=np.float32) * (1.5 * gain * scale))
    k = rng.standard_normal((B, Lk, D), dtype=np.float32)
    if rising:                                         # one channel of every head: 0 .. 40 in log2 units over the keys
        q[:, :, ::hd] = 1.0
        k[:, :, ::hd] = np.linspace(0, 40, Lk, dtype=np.float32)[None, :, None]
    k = workloads.bf16_round(k)
    v = workloads.bf16_round(rng.standard_normal((B, Lk, D), dtype=np.float32))
    want = dit.attention(q.astype(np.float64) / float(scale), k.astype(np.float64), v.astype(np.float64), heads)
    outs = {kernel: _network_attention(lib, q, k, v, heads, kernel) for kernel in ((1, 2) if hd == 64 else (1,))}
    for got in outs.values():
        assert np.isfinite(got).all()
        # probabilities and outputs are rounded to bf16 (2^-9 relative)
        assert np.max(np.abs(got - want)) < 1.5e-2 * np.max(np.abs(want))
        assert np.sqrt(np.mean((got - want) ** 2)) < 4e-3 * np.sqrt(np.mean(want ** 2))
    if hd == 64:
        np.testing.assert_array_equal(outs[1], outs[2])            # the choice is made by size and may not show


# a constant added to the scores of the queries of one block of 32 (exact in bf16: one channel holds 1 and the constant), inside the
# range in which probabilities are taken as they are and outside it on either side, where that block alone is done again
@pytest.mark.parametrize("offset", [50.0, 90.0, 130.0, 1000.0, -50.0, -70.0, -140.0, -1000.0])
@pytest.mark.parametrize("Lk", [13, 64, 130, 331])
def test_network_attention_outside_the_range_of_plain_probabilities(lib, offset, Lk):
    say(f"network attention, scores moved by {offset}, {Lk} keys")
    rng = np.random.default_rng(Lk)
    B, Lq, heads, hd = 2, 300, 1, 64
    scale = np.float32(1.4426950408889634 / math.sqrt(hd))
    q = workloads.bf16_round(rng.standard_normal((B, Lq, hd), dtype=np.float32) * scale)
    k = workloads.bf16_round(rng.standard_normal((B, Lk, hd), dtype=np.float32))
    v = workloads.bf16_round(rng.standard_normal((B, Lk, hd), dtype=np.float32))
    v *= np.float32(2.0 ** 60)                             # exact; times an unnormalised probability of 2^90 it has no fp32 value
    q[:, :, 5], k[:, :, 5] = 0.0, offset
    plain = {kernel: _network_attention(lib, q, k, v, heads, kernel) for kernel in (1, 2)}
    q[1, 96:128, 5] = 1.0
    want = dit.attention(q.astype(np.float64) / float(scale), k.astype(np.float64), v.astype(np.float64), heads)
    for kernel in (1, 2):
        got = _network_attention(lib, q, k, v, heads, kernel)
        assert np.isfinite(got).all()
        # fp32 scores of size 1000 (ulp 6e-5) do not show beside probabilities and outputs rounded to bf16 (2^-9 relative)
        assert np.max(np.abs(got - want)) < 1.5e-2 * np.max(np.abs(want))
        others = np.ones((B, Lq), bool)
        others[1, 96:128] = False
        np.testing.assert_array_equal(got[others], plain[kernel][others])          # nobody else notices
        np.testing.assert_array_equal(plain[kernel], plain[1])
        if kernel == 1:
            first = got
        np.testing.assert_array_equal(got, first)


# values so large or so small that beside a normaliser inside the range of plain probabilities (2^offset and more) their products
# leave fp32's range: the reference exponent of the online softmax keeps them
@pytest.mark.parametrize("offset,exponent", [(50.0, 80), (30.0, 110), (0.0, 115), (-38.0, -112), (-20.0, -115), (-58.0, -100)])
@pytest.mark.parametrize("Lk", [13, 128, 331])
def test_network_attention_with_values_of_any_size(lib, offset, exponent, Lk):
    say(f"network attention, scores moved by {offset}, values of size 2^{exponent}, {Lk} keys")
    rng = np.random.default_rng(Lk)
    B, Lq, heads, hd = 1, 300, 1, 64
    scale = np.float32(1.4426950408889634 / math.sqrt(hd))
    q = workloads.bf16_round(rng.standard_normal((B, Lq, hd), dtype=np.float32) * scale)
    k = workloads.bf16_round(rng.standard_normal((B, Lk, hd), dtype=np.float32))
    v = workloads.bf16_round(rng.standard_normal((B, Lk, hd), dtype=np.float32)) * np.float32(2.0 ** exponent)     # exact
    q[:, :, 5], k[:, :, 5] = 1.0, offset
    want = dit.attention(q.astype(np.float64) / float(scale), k.astype(np.float64), v.astype(np.float64), heads)
    outs = [_network_attention(lib, q, k, v, heads, kernel) for kernel in (1, 2)]
    np.testing.assert_array_equal(outs[0], outs[1])
    assert np.isfinite(outs[0]).all()
    # probabilities and outputs are rounded to bf16 (2^-9 relative)
    assert np.max(np.abs(outs[0] - want)) < 1.5e-2 * np.max(np.abs(want))


# One key far above the others for one block of 32 queries: inside the range in which probabilities are taken as they are, past it
# in a tile that fp32 still holds (the block goes on with a reference), and in one it does not (the block is done again), in the first
# half of the first tile, later, and in the part-filled last tile
@pytest.mark.parametrize("score", [50.0, 70.0, 100.0, 140.0, 600.0])
@pytest.mark.parametrize("Lk,key", [(64, 40), (331, 3), (331, 63), (331, 130), (331, 255), (331, 328), (90, 77), (192, 64)])
def test_network_attention_with_one_key_far_above_the_others(lib, score, Lk, key):
    say(f"network attention, key {key} of {Lk} at {score}")
    rng = np.random.default_rng(Lk + key)
    B, Lq, heads, hd = 1, 300, 1, 64
    scale = np.float32(1.4426950408889634 / math.sqrt(hd))
    q = workloads.bf16_round(rng.standard_normal((B, Lq, hd), dtype=np.float32) * scale)
    k = workloads.bf16_round(rng.standard_normal((B, Lk, hd), dtype=np.float32))
    v = workloads.bf16_round(rng.standard_normal((B, Lk, hd), dtype=np.float32))
    q[:, :, 5], k[:, :, 5] = 0.0, 0.0
    k[0, key, 5] = score
    plain = _network_attention(lib, q, k, v, heads, 1)
    q[0, 128:160, 5] = np.linspace(0.5, 1.0, 32)                   # not all of the block's queries leave the range
    q = workloads.bf16_round(q)
    want = dit.attention(q.astype(np.float64) / float(scale), k.astype(np.float64), v.astype(np.float64), heads)
    got = _network_attention(lib, q, k, v, heads, 1)
    assert np.isfinite(got).all()
    # fp32 scores of size 600 (ulp 6e-5) do not show beside probabilities and outputs rounded to bf16 (2^-9 relative)
    assert np.max(np.abs(got - want)) < 1.5e-2 * np.max(np.abs(want))
    others = np.ones((B, Lq), bool)
    others[0, 128:160] = False
    np.testing.assert_array_equal(got[others], plain[others])      # nobody else notices
    np.testing.assert_array_equal(_network_attention(lib, q, k, v, heads, 2), got)


@pytest.mark.parametrize("B,Lq,Lk,heads", [(48, 1178, 1178, 24), (24, 1024, 1024, 12), (24, 1024, 77, 12)])
def test_sharp_attention_takes_little_longer_than_flat(lib, B, Lq, Lk, heads):
    """Scores of standard deviation 29 in log2 units (largest of a row 60 to 100), which need a reference exponent, against scores of
    1.4: 1.31, 1.21 and 1.10 times as long (2.2, 2.1 and 1.4 times when every block was done twice)."""
    say(f"sharp attention, time, {B} x {heads} heads x {Lq} on {Lk}")
    D, Lkpad = heads * 64, (Lk + 63) // 64 * 64
    g = torch.Generator(device=DEV)
    g.manual_seed(Lk)
    rand = lambda *s: torch.randn(*s, device=DEV, generator=g)
    bits = lambda t: t.to(torch.bfloat16).view(torch.int16)
    q, k, vt = rand(B, Lq, D) * (1.4426950408889634 / 8), bits(rand(B, Lk, D)), bits(rand(B, D, Lkpad))
    out = torch.zeros(B, Lq, D, dtype=torch.int16, device=DEV)
    micros = []
    for gain in (1.0, 20.0):
        qb = bits(q * gain)
        a, b, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), 1e9
        for _ in range(6):
            a.record()
            for _ in range(10):
                lib.pg_attention_network(qb, k, vt, out, B, Lq, Lk, Lkpad, heads, 64, 0)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 100)
        micros.append(best)
    say(f"  flat {micros[0]:.1f} us, sharp {micros[1]:.1f} us")
    assert micros[1] < (1.6 if Lk > 100 else 1.25) * micros[0]
