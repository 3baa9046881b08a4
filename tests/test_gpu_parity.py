"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Codes and scales must match bit for bit; products must satisfy
max|C - C_ref| <= 4e-3 max|C_ref| (fp16) / 1.6e-2 max|C_ref| (bf16).
"""
import numpy as np
import pytest

import oracle
from paper_2308_09723_amd import workloads

from gpu_util import (TOL, assert_gemm_close, assert_quantizer_parity, from_dev_act, gpu_quantize, round_to_act,
                      to_dev_act, torch_mod)

pytestmark = pytest.mark.gpu


def _fq():
    from paper_2308_09723_amd import fq
    return fq


def _say(msg):
    print(msg, flush=True)


# ------------------------------------------------------------------ quantiser
@pytest.mark.parametrize("bits,g", [(8, 0), (4, 128)])
def test_quantize_config1(bits, g):
    _say(f"quantize config1 bits={bits} g={g}")
    _, W = workloads.config1(0)
    assert_quantizer_parity(W, bits, g)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("K,N,g", [(384, 80, 32), (512, 272, 64), (768, 48, 96), (1024, 16, 0), (256, 1040, 256)])
def test_quantize_ragged_shapes_and_outliers(bits, K, N, g):
    _say(f"quantize ragged bits={bits} K={K} N={N} g={g}")
    W = workloads.weights_gaussian(K, N, seed=K + N + bits, outlier_prob=0.01)
    assert_quantizer_parity(W, bits, g)
    Wh = workloads.weights_heavy_tail(K, N, seed=K + N + bits + 1, col_prob=0.05)
    assert_quantizer_parity(Wh, bits, g)


@pytest.mark.parametrize("bits", [4, 8])
def test_quantize_edge_values(bits):
    _say(f"quantize edge values bits={bits}")
    K, N, g = 256, 32, 64
    W = workloads.weights_gaussian(K, N, seed=99)
    W[:, 0] = 0                                   # all-zero column
    W[:64, 1] = 0                                 # one all-zero group
    W[:, 2] = np.float16(6e-8)                    # smallest subnormal everywhere
    W[64:128, 3] = np.float16(6e-8)
    W[70, 3] = np.float16(-1.2e-7)
    W[0, 4] = np.float16(65504.0)
    W[1, 4] = np.float16(-65504.0)
    W[:, 5] = np.float16(6.1e-5)                  # smallest normal
    # exact ties: with max 7.5 (int4) / 127.5 (int8) the scale is exactly 1
    top = 7.5 if bits == 4 else 127.5
    W[:64, 6] = np.float16(0.5)
    W[0, 6] = np.float16(top)
    W[1, 6] = np.float16(1.5)
    W[2, 6] = np.float16(2.5)
    W[3, 6] = np.float16(-3.5)
    W[4, 6] = np.float16(-top)
    _, _, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
    assert s_ref[0, 6] == np.float16(1.0) and q_ref[1, 6] == 2 and q_ref[2, 6] == 2 and q_ref[3, 6] == -4


def test_quantize_exhaustive_quotient_window():
    """Every (numerator, scale) pair of a dense window goes through the GPU divide/round path."""
    _say("quantize exhaustive window")
    s_vals = np.arange(0x2C00, 0x3000, 8, dtype=np.uint16).view(np.float16)      # 128 scales in [2^-4, 2^-3)
    K = 2048
    N = len(s_vals)
    all16 = np.arange(0x1000, 0x3C00, dtype=np.uint16).view(np.float16)          # positive halves up to 1.0
    W = np.empty((K, N), dtype=np.float16)
    rng = np.random.default_rng(5)
    for j, sj in enumerate(s_vals):
        top = np.float16(float(sj) * 15 / 2.0)
        cand = all16[all16 <= top]
        col = rng.choice(cand, size=K, replace=True)
        col[0] = top
        sign = rng.integers(0, 2, size=K) * 2 - 1
        W[:, j] = (col.astype(np.float32) * sign).astype(np.float16)
    assert_quantizer_parity(W, 4, 0)


@pytest.mark.parametrize("bits", [3, 4, 8])
def test_quantize_quotients_next_to_ties(bits):
    """Numerators chosen next to (k + 1/2) * s for every code k and 256 scales of every mantissa pattern:
    the binary16 values just below and above each tie (two on each side), both signs.  Hundreds of the
    quotients are exact ties (counted below; with binary16 numerators nothing else comes within 2^-13 of
    one), the rest are the closest misses there are: where a product with the reciprocal and the IEEE
    quotient could round differently."""
    _say(f"quantize next to ties int{bits}")
    qmax = (1 << (bits - 1)) - 1
    L = float((1 << bits) - 1)
    tops = np.arange(0x3000, 0x3400, 4, dtype=np.uint16).view(np.float16)         # 256 column maxima in [1/8, 1/4)
    N = len(tops)
    s_col = oracle.scale_from_absmax(tops, bits).astype(np.float64)
    all16 = np.arange(0x0001, 0x3400, dtype=np.uint16).view(np.float16).astype(np.float64)   # ascending
    per_col = 4 * qmax
    K = 128 * (-(-(2 * per_col + 1) // 128))
    W = np.zeros((K, N), dtype=np.float16)
    near = 0
    for n in range(N):
        ties = (np.arange(qmax) + 0.5) * s_col[n]
        at = np.searchsorted(all16, ties)                     # first value >= tie
        idx = np.concatenate([at - 2, at - 1, at, at + 1])
        vals = all16[np.clip(idx, 0, len(all16) - 1)]
        vals = vals[vals <= float(tops[n])]
        quo = (vals.astype(np.float32) / np.float32(s_col[n])).astype(np.float64)
        near += int(np.sum(np.abs(np.abs(quo - np.rint(quo)) - 0.5) < 2.0 ** -13))
        col = np.concatenate([[float(tops[n])], vals, -vals])
        W[: len(col), n] = col.astype(np.float16)
    _say(f"  {near} quotients within 2^-13 of a tie")
    assert near >= 400
    _, _, _, s_ref = assert_quantizer_parity(W, bits, 0)
    assert np.array_equal(s_ref[0].astype(np.float64), s_col)


# ------------------------------------------------------------------ product, oracle-sized cases
def _gemm_case(M, K, N, dtype, bits, g, seed, heavy=False):
    fq = _fq()
    A = workloads.activations(M, K, dtype, seed)
    if heavy:
        W = workloads.weights_heavy_tail(K, N, seed + 1, col_prob=0.02)
    else:
        W = workloads.weights_gaussian(K, N, seed + 1, outlier_prob=1e-3)
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
    C_ref = oracle.gemm_ref(A, q_ref, s_ref)
    Ad = to_dev_act(A, dtype)
    C = from_dev_act(fq.gemm(Ad, codes, scales, bits, g), dtype)
    rel = assert_gemm_close(C, C_ref, dtype, f"M={M} K={K} N={N} {dtype} int{bits} g={g}")
    # determinism: a second call returns the same bits
    C2 = from_dev_act(fq.gemm(Ad, codes, scales, bits, g), dtype)
    assert np.array_equal(C, C2)
    return rel


def test_gemm_config1():
    for bits, g in ((8, 0), (4, 128)):
        _say(f"gemm config1 int{bits} g={g}")
        fq = _fq()
        A, W = workloads.config1(0)
        codes, scales, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
        C = from_dev_act(fq.gemm(to_dev_act(A, "f16"), codes, scales, bits, g), "f16")
        assert_gemm_close(C, oracle.gemm_ref(A, q_ref, s_ref), "f16", "config1")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bits,g", [(4, 32), (4, 64), (4, 128), (4, 256), (4, 0), (8, 32), (8, 64), (8, 128), (8, 0)])
@pytest.mark.parametrize("M", [1, 5, 16])
def test_gemm_small_m(dtype, bits, g, M):
    _say(f"gemm small-M {dtype} int{bits} g={g} M={M}")
    # 9 column tiles (ragged against the 4-tile wave groups), 6 k-blocks of 128
    _gemm_case(M, 768, 144, dtype, bits, g, seed=1000 + M + bits + g)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bits,g", [(4, 32), (4, 64), (4, 128), (4, 0), (8, 64), (8, 0)])
@pytest.mark.parametrize("M", [17, 40, 130])
def test_gemm_tiled(dtype, bits, g, M):
    _say(f"gemm tiled {dtype} int{bits} g={g} M={M}")
    _gemm_case(M, 768, 304, dtype, bits, g, seed=2000 + M + bits + g)


def _sweep_cases():
    """Seeded draw of (M, K, N, dtype, bits, g): M on both sides of every plan boundary, K from one to a
    few k-blocks (so that the pipelined loops run their prologue, their unrolled body and their tail with
    clamped prefetches), N from one column tile to several ragged column blocks."""
    rng = np.random.default_rng(20240611)
    Ms = [1, 2, 7, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 200, 257, 300]
    cases = []
    for i in range(48):
        bits = int(rng.choice([4, 8]))
        kblk = 128 if bits == 4 else 64
        K = kblk * int(rng.choice([1, 2, 3, 4, 5, 7, 12]))
        N = 16 * int(rng.choice([1, 2, 3, 5, 12, 13, 24, 25, 31, 49]))
        gs = [g for g in (32, 64, 96, 128, 256, 0) if g == 0 or (g <= K and K % g == 0)]
        g = int(rng.choice(gs))
        M = int(Ms[i % len(Ms)])
        dtype = "f16" if rng.integers(2) else "bf16"
        cases.append((M, K, N, dtype, bits, g))
    return cases


@pytest.mark.parametrize("M,K,N,dtype,bits,g", _sweep_cases())
def test_gemm_shape_sweep(M, K, N, dtype, bits, g):
    _say(f"gemm sweep M={M} K={K} N={N} {dtype} int{bits} g={g}")
    _gemm_case(M, K, N, dtype, bits, g, seed=7000 + M + K + N + bits + g)


@pytest.mark.parametrize("dtype,bits,g,M", [("f16", 4, 96, 8), ("bf16", 4, 192, 33), ("f16", 8, 96, 3), ("bf16", 8, 160, 70)])
def test_gemm_group_sizes_that_are_not_powers_of_two(dtype, bits, g, M):
    _say(f"gemm odd group {dtype} int{bits} g={g} M={M}")
    K = 960 * 2 if g in (96, 160, 192) else 768           # 1920 = lcm-friendly: divisible by 96, 160, 192 and 128
    _gemm_case(M, K, 64, dtype, bits, g, seed=3000 + g)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bits", [4, 8])
def test_gemm_heavy_tailed_weights(dtype, bits):
    _say(f"gemm heavy tail {dtype} int{bits}")
    for g in (32, 128, 0):
        for M in (1, 16, 48):
            _gemm_case(M, 1024, 224, dtype, bits, g, seed=4000 + M + g, heavy=True)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bits,g", [(4, 32), (4, 128), (8, 0), (8, 32)])
def test_gemm_one_hot_rows_return_the_dequantised_weights_exactly(dtype, bits, g):
    """A = e_k: no accumulation error, so C must equal q*s rounded once to the output type.

    Every k of two k-blocks is visited, which checks the packed layout element by element."""
    _say(f"gemm one-hot {dtype} int{bits} g={g}")
    fq = _fq()
    K, N = 256, 48
    W = workloads.weights_gaussian(K, N, seed=77 + bits, outlier_prob=0.01)
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
    gg = g or K
    for k0 in range(0, K, 16):
        A = np.zeros((16, K), dtype=np.float32)
        for r in range(16):
            A[r, k0 + r] = 1.0
        A_in = A.astype(np.float16) if dtype == "f16" else A
        C = from_dev_act(fq.gemm(to_dev_act(A_in, dtype), codes, scales, bits, g), dtype)
        for r in range(16):
            k = k0 + r
            expect = round_to_act(q_ref[k].astype(np.float64) * s_ref[k // gg].astype(np.float64), dtype)
            assert np.array_equal(C[r], expect), (k, dtype, bits, g)


def test_gemm_rows_beyond_m_are_not_written():
    _say("gemm guard rows")
    fq = _fq()
    torch = torch_mod()
    K, N, M = 512, 128, 5
    A = workloads.activations(M, K, "f16", 1)
    W = workloads.weights_gaussian(K, N, 2)
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, 4, 128)
    for Mcase in (5, 21):
        A = workloads.activations(Mcase, K, "f16", 1)
        out = torch.full((Mcase + 3, N), 7.0, dtype=torch.float16, device="cuda")
        fq.gemm(to_dev_act(A, "f16"), codes, scales, 4, 128, out=out[:Mcase])
        host = out.cpu().numpy()
        assert np.all(host[Mcase:] == 7.0)
        assert_gemm_close(host[:Mcase].astype(np.float64), oracle.gemm_ref(A, q_ref, s_ref), "f16", "guard")


# ------------------------------------------------------------------ heuristic
def test_choose_group_matches_oracle():
    fq = _fq()
    torch = torch_mod()
    cases = []
    W = workloads.weights_gaussian(1024, 256, 11, outlier_prob=1e-3)
    for alpha in (0.0, 0.3, 0.6, 0.75, 0.9, 0.97, 0.995, 1.0):
        cases.append((W, 256, 64, alpha))
        cases.append((W, 0, 32, alpha))
    Wp = np.full((512, 64), 1.0, dtype=np.float16)
    Wp[:64, 3] = 8.0
    cases += [(Wp, 0, 16, 0.5), (Wp, 0, 16, 0.9), (Wp, 64, 16, 0.5)]
    Wq = np.full((64, 32), 1.0, dtype=np.float16)
    Wq[:32, 1] = 4.0
    cases += [(Wq, 0, 32, 0.5), (Wq, 0, 32, 0.75), (Wq, 0, 32, 0.8)]
    Wo = workloads.weights_gaussian(96 * 4, 32, 5)
    cases += [(Wo, 96, 1, 0.0), (Wo, 0, 32, 0.0), (Wo, 0, 32, 0.4)]
    for W_, gs, gm, alpha in cases:
        _say(f"choose_group K={W_.shape[0]} N={W_.shape[1]} g_start={gs} g_min={gm} alpha={alpha}")
        want = oracle.choose_group(W_, gs, gm, alpha)
        got = fq.choose_group(torch.from_numpy(W_).cuda(), gs, gm, alpha)
        assert got == want, (gs, gm, alpha, got, want)


# ------------------------------------------------------------------ round-trip error (section 3.2)
@pytest.mark.parametrize("K,N", [(32 * 512, 80), (32 * 1024, 48), (32 * 2048, 32), (48 * 256, 272)])
def test_choose_group_deep_halving_trees(K, N):
    """Per-column start with 9, 10, 11 and 8 halving levels (the fold over the levels runs in LDS with 32, 16
    or 64 columns per block, or per column in registers beyond 1024 fine blocks).  One column carries 8.0 in
    its first K / 2^(d+1) rows and 1.0 elsewhere: the halving test then fires at levels 0 .. d and nowhere
    else, so the answer is K / 2^(d+1); plus Gaussian weights at several thresholds."""
    fq = _fq()
    torch = torch_mod()
    f = 48 if K % 48 == 0 and (K // 48) & (K // 48 - 1) == 0 else 32
    levels = (K // f).bit_length() - 1
    assert f << levels == K
    for d in sorted({0, 1, levels // 2, levels - 2, levels - 1}):
        W = np.full((K, N), 1.0, dtype=np.float16)
        W[: K >> (d + 1), N - 3] = 8.0
        want = oracle.choose_group(W, 0, f, 0.5)
        assert want == K >> (d + 1)
        _say(f"choose_group deep K={K} N={N} levels={levels} d={d} -> {want}")
        assert fq.choose_group(torch.from_numpy(W).cuda(), 0, f, 0.5) == want
        assert fq.choose_group(torch.from_numpy(W).cuda(), 0, f, 0.8) == want     # 1 < 0.2 * 8 still holds
        assert fq.choose_group(torch.from_numpy(W).cuda(), 0, f, 0.9) == K        # 1 < 0.1 * 8 does not
        assert oracle.choose_group(W, 0, f, 0.8) == want and oracle.choose_group(W, 0, f, 0.9) == K
    Wg = workloads.weights_gaussian(K, N, 77, outlier_prob=1e-4)
    Wd = torch.from_numpy(Wg).cuda()
    for alpha in (0.2, 0.6, 0.9, 0.99):
        want = oracle.choose_group(Wg, 0, f, alpha)
        _say(f"choose_group deep gaussian K={K} alpha={alpha} -> {want}")
        assert fq.choose_group(Wd, 0, f, alpha) == want


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("K,N,g", [(384, 80, 32), (512, 272, 64), (1024, 16, 0), (256, 1040, 256), (768, 304, 128)])
def test_quant_error_matches_oracle(bits, K, N, g):
    _say(f"quant error int{bits} K={K} N={N} g={g}")
    fq = _fq()
    torch = torch_mod()
    W = workloads.weights_gaussian(K, N, 90 + K + N, outlier_prob=2e-3)
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
    sse, mx = fq.quant_error(torch.from_numpy(W).cuda(), codes, scales, bits, g)
    sse_ref, mx_ref = oracle.quant_error(W, q_ref, s_ref)
    assert mx == mx_ref                                   # one exact difference: bit-exact
    # both sides add the same exactly rounded squares, in different orders: K * N <= 3e5 terms of
    # relative rounding 2^-53 each
    assert abs(sse - sse_ref) <= 1e-11 * sse_ref, (sse, sse_ref)
    sse2, mx2 = fq.quant_error(torch.from_numpy(W).cuda(), codes, scales, bits, g)
    assert (sse2, mx2) == (sse, mx)                       # deterministic


def test_quant_error_heavy_tail_and_zero_matrix():
    fq = _fq()
    torch = torch_mod()
    W = workloads.weights_heavy_tail(512, 96, seed=17)
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, 4, 64)
    sse, mx = fq.quant_error(torch.from_numpy(W).cuda(), codes, scales, 4, 64)
    sse_ref, mx_ref = oracle.quant_error(W, q_ref, s_ref)
    assert mx == mx_ref and abs(sse - sse_ref) <= 1e-11 * sse_ref
    Z = np.zeros((256, 32), dtype=np.float16)
    codes, scales, _, _ = assert_quantizer_parity(Z, 8, 128)
    assert fq.quant_error(torch.from_numpy(Z).cuda(), codes, scales, 8, 128) == (0.0, 0.0)


# ------------------------------------------------------------------ grouped (mixture of experts)
@pytest.mark.parametrize("dtype,bits,g", [("f16", 4, 64), ("bf16", 4, 64), ("f16", 8, 0)])
def test_grouped_gemm_small(dtype, bits, g):
    _say(f"grouped small {dtype} int{bits} g={g}")
    fq = _fq()
    torch = torch_mod()
    E, K, N = 6, 256, 96
    rows = [70, 0, 1, 16, 130, 0]
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    A = workloads.activations(int(offsets[-1]), K, dtype, 8)
    qs, ss, codes_l, scales_l = [], [], [], []
    for e in range(E):
        W = workloads.weights_gaussian(K, N, 50 + e, outlier_prob=1e-3)
        c, s, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
        codes_l.append(c)
        scales_l.append(s.reshape(-1))
        qs.append(q_ref)
        ss.append(s_ref)
    codes = torch.cat(codes_l)
    scales = torch.cat(scales_l)
    out = torch.full((int(offsets[-1]), N), 3.0, dtype=torch.float16 if dtype == "f16" else torch.bfloat16, device="cuda")
    fq.gemm_grouped(to_dev_act(A, dtype), offsets.tolist(), codes, scales, bits, g, N, out=out)
    C = from_dev_act(out, dtype)
    C_ref = oracle.gemm_ref_grouped(A, offsets, qs, ss)
    assert_gemm_close(C, C_ref, dtype, "grouped")
    for e in range(E):
        if rows[e]:
            sl = slice(offsets[e], offsets[e + 1])
            assert_gemm_close(C[sl], C_ref[sl], dtype, f"expert {e}")


def _grouped_case(dtype, bits, g, K, N, rows, seed, shared_weights=False):
    """Experts with the given row counts; returns nothing, asserts parity per expert."""
    fq = _fq()
    torch = torch_mod()
    E = len(rows)
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    A = workloads.activations(int(offsets[-1]), K, dtype, seed)
    qs, ss, codes_l, scales_l = [], [], [], []
    for e in range(E):
        if e == 0 or not shared_weights:
            W = workloads.weights_gaussian(K, N, seed + 50 + e, outlier_prob=1e-3)
            c, s, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
        codes_l.append(c)
        scales_l.append(s.reshape(-1))
        qs.append(q_ref)
        ss.append(s_ref)
    codes = torch.cat(codes_l)
    scales = torch.cat(scales_l)
    out = torch.full((int(offsets[-1]), N), 3.0, dtype=torch.float16 if dtype == "f16" else torch.bfloat16, device="cuda")
    fq.gemm_grouped(to_dev_act(A, dtype), offsets.tolist(), codes, scales, bits, g, N, out=out)
    C = from_dev_act(out, dtype)
    C_ref = oracle.gemm_ref_grouped(A, offsets, qs, ss)
    for e in range(E):
        if rows[e]:
            sl = slice(offsets[e], offsets[e + 1])
            assert_gemm_close(C[sl], C_ref[sl], dtype, f"expert {e} ({rows[e]} rows)")


@pytest.mark.parametrize("dtype,bits,g", [("f16", 4, 64), ("bf16", 4, 128), ("bf16", 8, 32), ("f16", 8, 0),
                                          ("f16", 4, 128), ("bf16", 4, 64), ("f16", 4, 0)])
def test_grouped_gemm_tile_boundaries(dtype, bits, g):
    """Row counts on both sides of every row-tile size (32 / 64 / 128) and several column blocks with a
    ragged last one for both the 4-wave (192 columns) and the 8-wave (384 columns) block shapes."""
    _say(f"grouped tile boundaries {dtype} int{bits} g={g}")
    _grouped_case(dtype, bits, g, 256, 400, [32, 33, 64, 65, 128, 129, 0, 193, 40, 161, 1], seed=31)


@pytest.mark.parametrize("dtype,bits,g", [("f16", 4, 64), ("bf16", 4, 128), ("f16", 8, 0), ("bf16", 3, 64)])
def test_grouped_gemm_wide_matrix_uses_eight_wave_blocks_for_every_tile_size(dtype, bits, g):
    """49 column tiles: two full 8-wave column blocks and one with a single tile, for the 32-, 64- and
    128-row tiles alike."""
    _say(f"grouped wide {dtype} int{bits} g={g}")
    _grouped_case(dtype, bits, g, 256, 784, [31, 33, 64, 0, 130, 1, 97], seed=33)


def test_grouped_gemm_more_tiles_than_one_launch_holds():
    """260 row tiles of 128 rows: the by-value tile list holds 256, so a second launch takes the rest."""
    _say("grouped 130 experts x 256 rows")
    _grouped_case("f16", 4, 128, 128, 48, [256] * 130, seed=32, shared_weights=True)


# ------------------------------------------------------------------ bf16 activations on the fp16 matrix path
def _rows_case(M, K, N, bits, g, seed, row_scales):
    """bf16 activations whose rows are scaled by `row_scales` (wide matrix, 128-row blocks: the rows are
    rewritten as binary16 over a power of two per row); parity per row, relative to that row's largest output."""
    fq = _fq()
    W = workloads.weights_gaussian(K, N, seed, outlier_prob=1e-3)
    A = workloads.activations(M, K, "bf16", seed + 1).astype(np.float64)
    A *= np.asarray(row_scales, dtype=np.float64)[:, None]
    A = workloads.round_to_bf16(A.astype(np.float32))
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
    assert fq.gemm_workspace_bytes_for(M, N, K, bits, g, fq.FQ_BF16) > fq.gemm_workspace_bytes_for(M, N, K, bits, g, fq.FQ_F16)
    C = from_dev_act(fq.gemm(to_dev_act(A, "bf16"), codes, scales, bits, g), "bf16")
    C_ref = oracle.gemm_ref(A, q_ref, s_ref)
    assert np.all(np.isfinite(C))
    for r in range(M):
        top = np.max(np.abs(C_ref[r]))
        err = np.max(np.abs(C[r] - C_ref[r]))
        assert err <= TOL["bf16"] * top, f"row {r} (scale {row_scales[r]:.3g}): {err} > {TOL['bf16']} * {top}"


@pytest.mark.parametrize("bits,g", [(4, 128), (4, 64), (8, 0), (3, 32)])
def test_gemm_bf16_rows_rewritten_as_binary16(bits, g):
    _say(f"bf16 via fp16 path int{bits} g={g}")
    M, K, N = 270, 256, 8192            # more than 256 rows: 128-row blocks
    rng = np.random.default_rng(77)
    row_scales = 2.0 ** rng.integers(-60, 60, size=M).astype(np.float64)
    row_scales[0] = 0.0                 # an all-zero row
    row_scales[1] = 2.0 ** -120         # far below the binary16 range
    row_scales[2] = 2.0 ** 110          # far above it
    row_scales[3] = 1.0
    _rows_case(M, K, N, bits, g, 9100 + bits + g, row_scales)


def test_gemm_bf16_rows_with_outliers_inside_a_row():
    """One element 2^20 times larger than the rest of its row: the small elements keep their relative
    precision (they are still normal binary16 numbers after the row's division)."""
    _say("bf16 via fp16 path, outlier inside rows")
    fq = _fq()
    M, K, N = 260, 384, 8192
    W = workloads.weights_gaussian(K, N, 9200, outlier_prob=1e-3)
    A = workloads.activations(M, K, "bf16", 9201).astype(np.float32)
    A[:, 5] *= np.float32(2.0 ** 20)
    A = workloads.round_to_bf16(A)
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, 4, 128)
    assert fq.gemm_workspace_bytes_for(M, N, K, 4, 128, fq.FQ_BF16) > fq.gemm_workspace_bytes_for(M, N, K, 4, 128, fq.FQ_F16)
    C = from_dev_act(fq.gemm(to_dev_act(A, "bf16"), codes, scales, 4, 128), "bf16")
    assert_gemm_close(C, oracle.gemm_ref(A, q_ref, s_ref), "bf16", "outlier column")
    # without the outlier column the same rows: the small elements alone must still be accurate
    A2 = A.copy()
    A2[:, 5] = 0
    C2 = from_dev_act(fq.gemm(to_dev_act(A2, "bf16"), codes, scales, 4, 128), "bf16")
    assert_gemm_close(C2, oracle.gemm_ref(A2, q_ref, s_ref), "bf16", "rows without the outlier")


def test_gemm_bf16_wide_matrix_split_k_and_tail():
    """Wide matrices whose plans split K (uniformly, or for the tail round only) on the fp16 path."""
    _say("bf16 via fp16 path with split K")
    fq = _fq()
    for M, K, N in ((384, 2048, 8192), (300, 1024, 12288)):
        assert fq.gemm_workspace_bytes_for(M, N, K, 4, 128, fq.FQ_BF16) > fq.gemm_workspace_bytes_for(M, N, K, 4, 128, fq.FQ_F16)
        _say("  " + fq.gemm_describe(M, N, K, 4, 128))
        _gemm_case(M, K, N, "bf16", 4, 128, seed=9300 + M)


@pytest.mark.parametrize("M,K,N,dtype,g", [(300, 4224, 6160, "f16", 128), (260, 4224, 6160, "bf16", 0),
                                           (1100, 1152, 6160, "f16", 0), (900, 1152, 12288, "bf16", 128),
                                           (1030, 1280, 9232, "f16", 256), (300, 4224, 6160, "f16", 64),
                                           (600, 128, 12288, "f16", 128)])
def test_gemm_int8_two_layout_blocks_per_k_block(M, K, N, dtype, g):
    """8-bit codes in the 128-row, 8-wave shape: the kernel takes two 64-row k-blocks of the packed layout
    per k-block when K is a multiple of 128 and the group size too (checked through the plan's k-block
    count: K / 128 instead of K / 64 blocks in all); an odd number of them, a ragged split of K, ragged
    last row blocks, the fp16 path for bf16 rows (N >= 8192), a single k-block, and g = 64, which keeps
    the 64-row blocks."""
    import re
    fq = _fq()
    desc = fq.gemm_describe(M, N, K, 8, g)
    _say(f"int8 wide M={M} K={K} N={N} {dtype} g={g}: {desc}")
    m = re.match(r"tiled mt=8 waves=8 splits=(\d+) kb_per_split=(\d+)", desc)
    assert m, desc
    splits, kbs = int(m.group(1)), int(m.group(2))
    unit = 128 if (g or K) % 128 == 0 else 64
    assert kbs * splits >= K // unit > kbs * (splits - 1)
    _gemm_case(M, K, N, dtype, 8, g, seed=9500 + M + g)


@pytest.mark.parametrize("dtype,g,K", [("bf16", 128, 384), ("f16", 0, 640), ("f16", 64, 384)])
def test_grouped_gemm_int8_two_layout_blocks_per_k_block(dtype, g, K):
    """8-bit experts: the 128-row tiles take two 64-row layout k-blocks per k-block when K and the group size
    are multiples of 128 (an odd number of them here), the smaller tiles and g = 64 keep the 64-row blocks."""
    _say(f"grouped int8 wide {dtype} g={g} K={K}")
    _grouped_case(dtype, 8, g, K, 784, [130, 31, 64, 0, 257, 1, 97], seed=35)


@pytest.mark.parametrize("rows", [[16, 1, 0, 15, 4], [1], [17, 16, 1, 2, 3, 16, 4, 5, 16], [32, 16, 3], [130, 16, 0, 33, 9, 20]],
                         ids=["at-most-16", "one-row", "one-of-nine-17", "32-and-16", "every-size"])
@pytest.mark.parametrize("dtype,bits,g,K,N", [("f16", 4, 64, 640, 112), ("bf16", 4, 128, 1664, 1040), ("bf16", 8, 0, 192, 48),
                                              ("f16", 8, 32, 256, 816), ("f16", 3, 96, 384, 16),
                                              ("f16", 4, 128, 128, 33200), ("bf16", 4, 64, 256, 33200)])
def test_grouped_gemm_few_rows_per_expert(dtype, bits, g, K, N, rows):
    """Experts of at most 16 rows take the small-M kernel, those of 17 .. 32 too (as two items) where they are few and
    nobody has more; neighbours with more rows take the tiled kernel, and so does every expert beside such a neighbour
    where all tiles are resident at once (the narrow matrices here, not the wide ones).  Column counts that leave idle column groups, k
    ranges shorter than the k-workers' turn, and every expert's rows next to another expert's."""
    _say(f"grouped few rows {dtype} int{bits} g={g} {rows}")
    fq = _fq()
    torch = torch_mod()
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    A = workloads.activations(int(offsets[-1]), K, dtype, 60 + K)
    qs, ss, codes, scales = [], [], [], []
    for e in range(len(rows)):
        c, s, q_ref, s_ref = assert_quantizer_parity(workloads.weights_gaussian(K, N, 700 + e, outlier_prob=1e-3), bits, g)
        qs.append(q_ref); ss.append(s_ref); codes.append(c); scales.append(s.reshape(-1))
    C = torch.full((int(offsets[-1]) + 2, N), 7.0, dtype=to_dev_act(A[:1], dtype).dtype, device="cuda")
    fq.gemm_grouped(to_dev_act(A, dtype), offsets.tolist(), torch.cat(codes), torch.cat(scales), bits, g, N,
                    out=C[:int(offsets[-1])])
    assert_gemm_close(from_dev_act(C[:int(offsets[-1])], dtype), oracle.gemm_ref_grouped(A, offsets, qs, ss), dtype)
    assert bool((C[int(offsets[-1]):] == 7.0).all())


@pytest.mark.parametrize("M", [17, 31, 32, 33, 48])
@pytest.mark.parametrize("dtype,bits,g,K,N", [("f16", 4, 128, 128, 16), ("bf16", 4, 128, 640, 144), ("f16", 4, 64, 1664, 1040),
                                              ("bf16", 4, 32, 3200, 208), ("bf16", 8, 0, 64, 80), ("f16", 8, 128, 2048, 656),
                                              ("f16", 3, 0, 1152, 336), ("bf16", 3, 96, 768, 96), ("f16", 8, 32, 448, 48)])
def test_gemm_mid_rows(dtype, bits, g, K, N, M):
    """17 .. 48 rows: both row-tile counts at their edges, fewer k-blocks than k-workers, last super-blocks that are not
    full, idle column groups, K split over the grid, and every number of scale rows per k-block."""
    _say(f"gemm mid {dtype} int{bits} g={g} K={K} N={N} M={M}")
    assert "mid-m" in _fq().gemm_describe(M, N, K, bits, g)
    _gemm_case(M, K, N, dtype, bits, g, seed=8000 + M + K + N)


@pytest.mark.parametrize("form", ["M=20", "M=40", "grouped"])
@pytest.mark.parametrize("dtype,bits", [("f16", 4), ("f16", 8), ("f16", 3), ("bf16", 4), ("bf16", 8), ("bf16", 3)])
def test_rows_with_infinities_nans_and_the_largest_magnitudes(dtype, bits, form):
    """The kernels whose operands carry the storage bias remove it with row sums; a row whose sums are not finite must
    still give what the product gives: infinities and NaNs in its own row only, and (bf16) finite results for
    magnitudes at which the biased sums overflow."""
    _say(f"non-finite rows {dtype} int{bits} {form}")
    fq = _fq()
    K, N, g = 768, 112, 128
    rows = [16, 9] if form == "grouped" else [int(form[2:])]
    M = sum(rows)
    A = workloads.activations(M, K, dtype, 5).astype(np.float32)
    A[1, 3] = np.inf
    A[4, 700] = -np.inf
    A[6, 100] = np.nan
    A[M - 1, 0], A[M - 1, 767] = np.inf, -np.inf
    if dtype == "bf16":
        A[2] = workloads.round_to_bf16(A[2] * np.float32(1e36))
    W = workloads.weights_gaussian(K, N, 6, outlier_prob=1e-3)
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
    Ad = to_dev_act(A.astype(np.float16) if dtype == "f16" else A, dtype)
    if form == "grouped":
        torch = torch_mod()
        offsets = [0, rows[0], M]
        C = from_dev_act(fq.gemm_grouped(Ad, offsets, torch.cat([codes] * 2), torch.cat([scales.reshape(-1)] * 2), bits, g, N),
                         dtype)
    else:
        C = from_dev_act(fq.gemm(Ad, codes, scales, bits, g), dtype)
    Wd = q_ref.astype(np.float64) * np.repeat(s_ref.astype(np.float64), g, axis=0)
    with np.errstate(invalid="ignore"):
        ref = A.astype(np.float64) @ Wd
    for r in range(M):
        want = ref[r]
        assert np.array_equal(np.isnan(C[r]), np.isnan(want)), (r, C[r], want)
        assert np.array_equal(C[r][np.isinf(want)], want[np.isinf(want)]), r
        ok = np.isfinite(want)
        if ok.any():
            assert_gemm_close(C[r][ok], want[ok], dtype, f"row {r}")


@pytest.mark.parametrize("M,K,N", [(4, 1024, 1024), (200, 6016, 8208)])
def test_gemm_replaces_a_workspace_that_is_too_small(M, K, N):
    """fq.gemm with no workspace, one of 16 bytes and one that is large enough: the same bits."""
    fq = _fq()
    torch = torch_mod()
    codes, scales, _, _ = assert_quantizer_parity(workloads.weights_gaussian(K, N, 61), 4, 128)
    need = fq.gemm_workspace_bytes(M, N, K, 4, 128)
    assert need > 16
    for dtype in ("f16", "bf16"):
        A = to_dev_act(workloads.activations(M, K, dtype, 62), dtype)
        C = fq.gemm(A, codes, scales, 4, 128)
        for size in (16, need):
            assert torch.equal(C, fq.gemm(A, codes, scales, 4, 128, workspace=torch.empty(size, dtype=torch.uint8, device="cuda")))


@pytest.mark.parametrize("form", ["M=20", "M=40", "grouped"])
@pytest.mark.parametrize("dtype,bits,g", [("f16", 4, 128), ("bf16", 4, 128), ("bf16", 3, 64), ("bf16", 4, 32), ("bf16", 8, 128)])
def test_rows_do_not_depend_on_another_row_that_is_not_finite(dtype, bits, g, form):
    """Infinities and a NaN in three rows: every other row gives the same bits as without them."""
    _say(f"rows beside non-finite ones {dtype} int{bits} g={g} {form}")
    fq = _fq()
    torch = torch_mod()
    K, N = 2048, 1040
    rows = [16, 9] if form == "grouped" else [int(form[2:])]
    M = sum(rows)
    codes, scales, _, _ = assert_quantizer_parity(workloads.weights_gaussian(K, N, 51, outlier_prob=1e-3), bits, g)
    A = to_dev_act(workloads.activations(M, K, dtype, 52), dtype)
    B = A.clone()
    B[1, 3], B[7, 2000], B[M - 1, 77] = float("inf"), float("nan"), float("-inf")

    def product(X):
        if form == "grouped":
            return fq.gemm_grouped(X, [0, rows[0], M], torch.cat([codes] * 2), torch.cat([scales.reshape(-1)] * 2), bits, g, N)
        return fq.gemm(X, codes, scales, bits, g)

    keep = [r for r in range(M) if r not in (1, 7, M - 1)]
    assert torch.equal(product(A)[keep], product(B)[keep])


@pytest.mark.parametrize("form", ["M=20", "M=40", "grouped"])
@pytest.mark.parametrize("dtype,bits,g", [("f16", 3, 128), ("f16", 4, 128), ("f16", 4, 64), ("f16", 4, 32), ("f16", 8, 128),
                                          ("f16", 8, 32), ("bf16", 8, 128), ("bf16", 8, 32), ("bf16", 4, 32), ("bf16", 3, 96)])
def test_outlying_activations_on_zero_weights(dtype, bits, g, form):
    """Every 96th activation is huge (near the top of binary16's range; 10^8 in bfloat16) and its weights are zero.  Such a
    product adds nothing, and what it leaves behind is bounded by the other terms alone: the weights' and the result's
    roundings to 16 bits, 2^-11 (2^-8) relative each, and the sums' to binary32 (operands with a bias leave 2^-24 * bias
    * a * s per sum: 30 to 500 times as much)."""
    _say(f"outliers on zero weights {dtype} int{bits} g={g} {form}")
    fq = _fq()
    torch = torch_mod()
    K, N = 768, 112
    rows = [16, 9] if form == "grouped" else [int(form[2:])]
    W = workloads.weights_gaussian(K, N, 41)
    W[::96] = 0
    A = workloads.activations(sum(rows), K, dtype, 42).astype(np.float32)
    A[:, ::96] = 60000.0 if dtype == "f16" else workloads.round_to_bf16(np.float32([1e8]))[0]
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
    Ad = to_dev_act(A.astype(np.float16) if dtype == "f16" else A, dtype)
    if form == "grouped":
        C = fq.gemm_grouped(Ad, [0, rows[0], sum(rows)], torch.cat([codes] * 2), torch.cat([scales.reshape(-1)] * 2), bits, g, N)
    else:
        C = fq.gemm(Ad, codes, scales, bits, g)
    Wd = q_ref.astype(np.float64) * np.repeat(s_ref.astype(np.float64), g, axis=0)
    terms = np.abs(A.astype(np.float64)) @ np.abs(Wd)
    err = np.abs(from_dev_act(C, dtype) - A.astype(np.float64) @ Wd)
    assert np.max(err / terms) <= 2 * (2.0 ** -11 if dtype == "f16" else 2.0 ** -8) + 2.0 ** -20


@pytest.mark.parametrize("M,K,N,rows,cols", [(257, 640, 8208, 80, 256), (563, 1152, 8208, 96, 256), (578, 640, 10256, 112, 256),
                                             (563, 640, 12304, 128, 256), (386, 640, 16400, 80, 384), (200, 6016, 8208, 112, 256)])
@pytest.mark.parametrize("dtype,bits,g", [("f16", 4, 128), ("bf16", 4, 128), ("bf16", 4, 64), ("f16", 4, 32), ("f16", 3, 128),
                                          ("bf16", 8, 128), ("f16", 8, 64), ("bf16", 8, 32)])
def test_gemm_shapes_between_64_and_128_rows(dtype, bits, g, M, K, N, rows, cols):
    """Every block shape of 80 .. 128 rows beside 128 x 384 (odd numbers of row tiles load padded LDS tiles), ragged in rows
    and columns, odd numbers of k-blocks, every number of scale rows per k-block, and K split over the grid."""
    desc = _fq().gemm_describe(M, N, K, bits, g)
    _say(f"gemm {dtype} int{bits} g={g} M={M} K={K} N={N}: {desc}")
    if (N, bits, g) != (16400, 4, 32):   # (keeps the former shape)
        assert f"rows={rows} cols={cols}" in desc
        assert (K == 6016) == ("splits=1 " not in desc)
    _gemm_case(M, K, N, dtype, bits, g, seed=9700 + M + K + bits)


def _grouped_plan(rows, K, N, bits, g):
    import re
    d = _fq().gemm_grouped_describe(np.concatenate([[0], np.cumsum(rows)]).tolist(), N, K, bits, g)
    return {k: int(v) for k, v in re.findall(r"([\w-]+)=(\d+)", d)}


@pytest.mark.parametrize("rows", [[16, 1, 17, 33, 0, 48, 32, 49, 80, 97, 145, 2], [48, 3], [31], [96] * 135],
                         ids=["every-height", "48-and-3", "31", "more-than-one-launch"])
@pytest.mark.parametrize("dtype,bits,g,K,N", [("f16", 4, 64, 640, 112), ("bf16", 4, 128, 1664, 1040), ("bf16", 8, 0, 192, 48),
                                              ("f16", 8, 32, 256, 816), ("f16", 3, 96, 384, 16), ("bf16", 3, 128, 256, 304),
                                              ("bf16", 4, 32, 256, 64)])
def test_grouped_gemm_tiles_of_the_streaming_kernel(dtype, bits, g, K, N, rows):
    """Row tiles of 16, 32 and 48 rows in one launch: every height on both sides of its limits, experts cut into several
    tiles of nearly equal height, idle column groups, k ranges shorter than the k-workers' turn, more tiles than one
    launch holds."""
    if len(rows) > 100 and K * N > 40000:
        pytest.skip("the number of tiles is what matters: small matrices")
    _say(f"grouped streaming tiles {dtype} int{bits} g={g} {rows[:12]}")
    plan = _grouped_plan(rows, K, N, bits, g)
    assert plan["rows128"] == plan["rows64"] == plan["small-m"] == 0 and plan["streams"] == 1
    assert plan["mid-m"] == sum(-(-r // 48) for r in rows)
    _grouped_case(dtype, bits, g, K, N, rows, seed=91, shared_weights=len(rows) > 100)


@pytest.mark.parametrize("dtype,bits,g", [("f16", 4, 64), ("bf16", 4, 128), ("bf16", 8, 128), ("f16", 8, 64), ("bf16", 3, 32)])
def test_grouped_gemm_tall_experts_beside_the_streaming_kernel(dtype, bits, g):
    """Enough tall experts for tiles of 128 and 64 rows of the tiled kernel (one column tile in the last column block),
    with what is left below 49 rows in the streaming kernel."""
    _say(f"grouped tall {dtype} int{bits} g={g}")
    rows = [256] * 12 + [64, 177, 33, 49, 30, 17, 130, 0]
    plan = _grouped_plan(rows, 1024, 6160, bits, g)
    assert (plan["rows128"], plan["rows64"], plan["mid-m"], plan["small-m"]) == (26, 3, 4, 0)
    _grouped_case(dtype, bits, g, 1024, 6160, rows, seed=93, shared_weights=True)


@pytest.mark.parametrize("bits,g", [(4, 128), (4, 64), (8, 64)])
def test_grouped_gemm_rows_beside_one_that_is_not_finite(bits, g):
    """bf16, one expert per tile height: an infinity in one row leaves the bits of every other row as they are."""
    _say(f"grouped non-finite row int{bits} g={g}")
    fq, torch = _fq(), torch_mod()
    rows, K, N = [9, 30, 47], 512, 208
    offsets = np.concatenate([[0], np.cumsum(rows)]).tolist()
    parts = [assert_quantizer_parity(workloads.weights_gaussian(K, N, 40 + e), bits, g)[:2] for e in range(3)]
    codes, scales = torch.cat([p[0] for p in parts]), torch.cat([p[1].reshape(-1) for p in parts])
    A = to_dev_act(workloads.activations(offsets[-1], K, "bf16", 17), "bf16")
    want = fq.gemm_grouped(A, offsets, codes, scales, bits, g, N).clone()
    B = A.clone()
    hit = [4, 20, 60]
    B[hit, 100] = float("inf")
    got = fq.gemm_grouped(B, offsets, codes, scales, bits, g, N)
    keep = [r for r in range(offsets[-1]) if r not in hit]
    assert torch.equal(got[keep].view(torch.int16), want[keep].view(torch.int16))
    assert not bool(torch.isfinite(got[hit]).all())


@pytest.mark.parametrize("M", [49, 64, 97, 145])
@pytest.mark.parametrize("dtype,bits,g,K,N", [("f16", 4, 128, 2304, 2064), ("bf16", 4, 128, 2304, 2064), ("f16", 4, 64, 1280, 1552),
                                              ("bf16", 4, 64, 1280, 1552), ("bf16", 4, 32, 768, 784), ("bf16", 8, 128, 1024, 1552),
                                              ("f16", 8, 64, 1152, 1552), ("f16", 3, 96, 768, 784), ("bf16", 3, 96, 768, 784)])
def test_gemm_row_blocks_of_the_streaming_kernel(dtype, bits, g, K, N, M):
    """49 rows and more on small matrices: row blocks of 48 and 32 rows and a lower last one, every number of scale rows per
    k-block, last super-blocks that are not full, idle column groups."""
    desc = _fq().gemm_describe(M, N, K, bits, g)
    _say(f"gemm row blocks {dtype} int{bits} g={g} K={K} N={N} M={M}: {desc}")
    assert "mid-m rows=48" in desc
    _gemm_case(M, K, N, dtype, bits, g, seed=8100 + M + K + N)


@pytest.mark.parametrize("form", ["M=97", "M=145", "grouped"])
@pytest.mark.parametrize("dtype,bits,g", [("f16", 4, 128), ("bf16", 4, 128), ("bf16", 4, 64), ("bf16", 3, 64), ("bf16", 8, 128),
                                          ("bf16", 4, 32)])
def test_outlying_activations_on_zero_weights_in_row_blocks(dtype, bits, g, form):
    """As test_outlying_activations_on_zero_weights: row blocks of more than 48 rows, and the tiles of experts of more than 48
    rows, have no bias in their operands whatever the format."""
    _say(f"outliers on zero weights in row blocks {dtype} int{bits} g={g} {form}")
    fq, torch = _fq(), torch_mod()
    K, N = 2304, (112 if form == "grouped" else 2064)
    rows = [50, 97] if form == "grouped" else [int(form[2:])]
    W = workloads.weights_gaussian(K, N, 41)
    W[::96] = 0
    A = workloads.activations(sum(rows), K, dtype, 42).astype(np.float32)
    A[:, ::96] = 60000.0 if dtype == "f16" else workloads.round_to_bf16(np.float32([1e8]))[0]
    codes, scales, q_ref, s_ref = assert_quantizer_parity(W, bits, g)
    Ad = to_dev_act(A.astype(np.float16) if dtype == "f16" else A, dtype)
    if form == "grouped":
        assert _grouped_plan(rows, K, N, bits, g)["mid-m"] == 5
        C = fq.gemm_grouped(Ad, [0, rows[0], sum(rows)], torch.cat([codes] * 2), torch.cat([scales.reshape(-1)] * 2), bits, g, N)
    else:
        assert "mid-m rows=48" in fq.gemm_describe(sum(rows), N, K, bits, g)
        C = fq.gemm(Ad, codes, scales, bits, g)
    Wd = q_ref.astype(np.float64) * np.repeat(s_ref.astype(np.float64), g, axis=0)
    terms = np.abs(A.astype(np.float64)) @ np.abs(Wd)
    err = np.abs(from_dev_act(C, dtype) - A.astype(np.float64) @ Wd)
    assert np.max(err / terms) <= 2 * (2.0 ** -11 if dtype == "f16" else 2.0 ** -8) + 2.0 ** -20


@pytest.mark.parametrize("M,K,N,dtype,bits,g,shape", [(1009, 640, 2064, "f16", 4, 32, " rows=32 cols=384"), (1345, 640, 1584, "bf16", 3, 64, " rows=64 cols=192"),
                                                      (600, 1536, 3968, "f16", 8, 32, " rows=64 cols=192"), (2048, 512, 2064, "bf16", 4, 64, " rows=64 cols=384"),
                                                      (270, 7168, 2112, "f16", 4, 64, " rows=64 cols=192"), (1000, 640, 4400, "f16", 4, 0, " f16: rows=64 cols=384"),
                                                      (1020, 640, 5744, "bf16", 4, 128, " f16: rows=64 cols=384")])
def test_gemm_small_row_blocks_above_256_rows(M, K, N, dtype, bits, g, shape):
    """Narrow matrices: 32- and 64-row blocks of the tiled kernel for 257 .. 2048 rows (last row blocks of 1 .. 40 rows, split K);
    binary16 products alone where these blocks' bfloat16 operands have a bias."""
    desc = _fq().gemm_describe(M, N, K, bits, g)
    _say(f"M={M} K={K} N={N} {dtype} int{bits} g={g}: {desc}")
    assert shape in desc, desc
    _gemm_case(M, K, N, dtype, bits, g, seed=9700 + M)


@pytest.mark.parametrize("M,K,N,dtype,bits,g,shape", [(257, 640, 144, "f16", 4, 32, "gp=1 kw=5"), (625, 1536, 208, "bf16", 3, 64, "gp=1 kw=6"),
                                                      (2332, 2176, 288, "bf16", 8, 64, "gp=2 kw=6"), (2332, 2176, 288, "f16", 4, 128, "gp=2 kw=6"),
                                                      (12241, 640, 144, "f16", 4, 128, "gp=3 kw=4"), (12288, 768, 80, "bf16", 4, 32, "gp=2 kw=6"),
                                                      (12288, 1536, 208, "f16", 8, 64, "gp=5 kw=2")])
def test_gemm_row_blocks_of_the_streaming_kernel_above_256_rows(M, K, N, dtype, bits, g, shape):
    """Row blocks of 48 rows from 257 rows to the most that one launch takes (256 of them, the last of 1 row, lower or full);
    block shapes chosen so that all blocks are resident at once."""
    desc = _fq().gemm_describe(M, N, K, bits, g)
    _say(f"gemm row blocks {dtype} int{bits} g={g} K={K} N={N} M={M}: {desc}")
    assert f"mid-m rows=48 {shape}" in desc and _fq().gemm_workspace_bytes(M, N, K, bits, g) == 0
    assert "mid-m" not in _fq().gemm_describe(12289, N, K, bits, g)
    _gemm_case(M, K, N, dtype, bits, g, seed=8900 + M + K)


@pytest.mark.parametrize("K,N,g", [(2048, 48, 32), (384, 48, 96), (640, 48, 160), (4480, 16, 224), (896, 16, 448), (3200, 272, 800),
                                   (128 * 33, 16, 128 * 33), (31 * 128, 32, 31 * 32), (160 * 256, 144, 160)])
def test_quantizer_group_abs_max_row_remainders(K, N, g):
    """The abs-max of groups whose rows do not fill the last round of loads: 2 to 14 rows per thread and one more or less, few blocks
    (eight rows in flight) and 256 or more (four), groups of whole 128-row blocks; the largest value in a group's last row."""
    W = workloads.weights_gaussian(K, N, seed=g, outlier_prob=2e-3)
    W[g - 1 :: g, 3] = np.float16(-9.0)
    W[g - 1 :: g, 5] = np.float16(7.0)
    assert_quantizer_parity(W, 4, g)


@pytest.mark.parametrize("M,K,N,bits,g,dtype,narrow", [
    (17, 1024, 1040, 4, 128, "f16", True), (32, 1280, 4032, 4, 0, "bf16", True), (33, 1920, 5504, 4, 32, "bf16", True),
    (48, 1408, 2768, 8, 32, "f16", True), (30, 1152, 336, 3, 64, "bf16", True), (20, 128, 16, 4, 128, "bf16", True),
    (24, 640, 8208, 4, 64, "f16", True), (41, 2048, 528, 8, 0, "bf16", True), (18, 1536, 3088, 4, 96, "bf16", True),
    (17, 640, 12304, 4, 64, "bf16", False), (48, 384, 12320, 3, 128, "f16", False), (33, 1536, 8480, 8, 64, "bf16", False),
    (40, 512, 12304, 4, 32, "f16", False), (21, 5120, 4400, 4, 64, "f16", False), (48, 10240, 2064, 8, 128, "bf16", False)])
def test_gemm_mid_rows_16_and_48_columns_per_wave(M, K, N, bits, g, dtype, narrow):
    """17 .. 48 rows: waves of 16 columns on matrices that they spread over more of the chip, of 48 on wide ones and where K is
    split over the grid (the last two), each with a last block that is not full and every number of scale rows per k-block."""
    desc = _fq().gemm_describe(M, N, K, bits, g)
    assert "mid-m" in desc and ("cols=16" in desc) == narrow, desc
    _gemm_case(M, K, N, dtype, bits, g, seed=M + K + N)


@pytest.mark.parametrize("M,K,N,bits,g,dtype,narrow", [
    (49, 1152, 1104, 4, 64, "bf16", True), (96, 1408, 816, 3, 128, "f16", True), (97, 1536, 3952, 4, 32, "f16", True),
    (143, 1664, 976, 8, 128, "bf16", True), (145, 2304, 3280, 4, 128, "f16", True), (197, 3840, 2832, 4, 0, "bf16", True),
    (256, 1152, 1552, 4, 96, "f16", True), (66, 896, 16, 4, 32, "bf16", True),
    (257, 1152, 1552, 4, 96, "bf16", False), (133, 1152, 8192, 4, 64, "f16", False),
    (89, 6912, 288, 8, 64, "f16", False)])
def test_gemm_row_blocks_of_16_columns_per_wave(M, K, N, bits, g, dtype, narrow):
    """49 .. 256 rows on less than 8192 columns: row blocks of 48 and fewer rows with waves of 16 columns, a last row block and a
    last column block that are not full, and the first sizes beyond the range."""
    desc = _fq().gemm_describe(M, N, K, bits, g)
    assert ("cols=16" in desc) == narrow, desc
    _gemm_case(M, K, N, dtype, bits, g, seed=M + K + N)
