"""GPU parity for the bfloat16 scale format (section 4.1, "GPU kernel implementations": scales of the
activation's data type): quantiser bit-exact against the oracle's bf16-format encoder, products of
bf16 activations within 1.6e-2 max|C_ref|, through the *_sf entry points of the C ABI.
"""
import numpy as np
import pytest

import oracle
from paper_2308_09723_amd import workloads

from gpu_util import assert_gemm_close, from_dev_act, to_dev_act, torch_mod

pytestmark = pytest.mark.gpu


def _fq():
    from paper_2308_09723_amd import fq
    return fq


def _say(msg):
    print(msg, flush=True)


def _quantize_parity(W, bits, g):
    fq = _fq()
    torch = torch_mod()
    q_ref, s_ref = oracle.quantize(W, bits, g, "bf16")
    codes, scales = fq.quantize(torch.from_numpy(W).cuda(), bits, g, fq.FQ_SCALE_BF16)
    assert scales.dtype == torch.bfloat16
    s_bits = scales.view(torch.int16).cpu().numpy().view(np.uint16)
    q = fq.unpack(codes, W.shape[0], W.shape[1], bits).cpu().numpy()
    assert np.array_equal(s_bits, oracle.bf16_scale_bits(s_ref)), "scales differ"
    assert np.array_equal(q, q_ref), "codes differ"
    return codes, scales, q_ref, s_ref


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("K,N,g", [(384, 80, 32), (512, 272, 64), (768, 48, 96), (1024, 16, 0), (256, 1040, 256),
                                   (2048, 144, 1024), (768, 304, 128)])
def test_quantize_bf16_scales(bits, K, N, g):
    _say(f"quantize bf16 scales int{bits} K={K} N={N} g={g}")
    W = workloads.weights_gaussian(K, N, 4000 + K + N + bits, outlier_prob=1e-3)
    _quantize_parity(W, bits, g)


@pytest.mark.parametrize("bits", [4, 8])
def test_quantize_bf16_scales_edge_values(bits):
    """Zero groups, the smallest subnormal, the largest binary16 values and heavy tails."""
    _say(f"quantize bf16 scales edge values int{bits}")
    W = workloads.weights_heavy_tail(256, 64, 11)
    W[:32, 0] = np.float16(0.0)
    W[:, 1] = np.float16(0.0)
    W[32:64, 2] = np.float16(6e-8)
    W[64, 3] = np.float16(65504.0)
    W[65, 3] = np.float16(-65504.0)
    _quantize_parity(W, bits, 32)
    _quantize_parity(W, bits, 0)


def test_quantize_every_binary16_absmax():
    """One group per possible abs-max: column n of block b holds the n-th value of a slab of the binary16
    range as its only non-zero element, so every scale of the format is exercised."""
    _say("quantize bf16 scales, all abs-max values")
    vals = np.arange(0, 0x7C00, dtype=np.uint16).view(np.float16)
    N = 1024
    G = (len(vals) + N - 1) // N                 # 31 groups of 32 rows
    assert G == 31
    W = np.zeros((1024, N), dtype=np.float16)    # 32 groups; the last one stays zero
    flat = np.zeros(G * N, dtype=np.float16)
    flat[:len(vals)] = vals
    W[5:G * 32:32, :] = flat.reshape(G, N)
    W[6:G * 32:32, :] = -(flat.reshape(G, N).astype(np.float32) * 0.37).astype(np.float16)
    for bits in (4, 8):
        _quantize_parity(W, bits, 32)


def _gemm_case(M, K, N, bits, g, seed):
    fq = _fq()
    W = workloads.weights_gaussian(K, N, seed, outlier_prob=1e-3)
    A = workloads.activations(M, K, "bf16", seed + 1)
    codes, scales, q_ref, s_ref = _quantize_parity(W, bits, g)
    C_ref = oracle.gemm_ref(A, q_ref, s_ref)
    Ad = to_dev_act(A, "bf16")
    C = from_dev_act(fq.gemm(Ad, codes, scales, bits, g), "bf16")
    assert_gemm_close(C, C_ref, "bf16", f"bf16 scales M={M} K={K} N={N} int{bits} g={g}")
    C2 = from_dev_act(fq.gemm(Ad, codes, scales, bits, g), "bf16")
    assert np.array_equal(C, C2)


@pytest.mark.parametrize("bits,g", [(4, 32), (4, 64), (4, 128), (4, 256), (4, 0), (8, 32), (8, 64), (8, 0)])
@pytest.mark.parametrize("M", [1, 5, 16])
def test_gemm_small_m_bf16_scales(bits, g, M):
    _say(f"gemm bf16 scales small-M int{bits} g={g} M={M}")
    _gemm_case(M, 768, 144, bits, g, seed=5000 + M + bits + g)


@pytest.mark.parametrize("bits,g", [(4, 32), (4, 64), (4, 128), (4, 0), (8, 32), (8, 64), (8, 0)])
@pytest.mark.parametrize("M", [17, 40, 130, 300])
def test_gemm_tiled_bf16_scales(bits, g, M):
    _say(f"gemm bf16 scales tiled int{bits} g={g} M={M}")
    _gemm_case(M, 768, 304, bits, g, seed=6000 + M + bits + g)


@pytest.mark.parametrize("bits,g,M", [(4, 128, 300), (4, 64, 130), (4, 32, 260), (8, 0, 300), (8, 64, 140), (3, 128, 300)])
def test_gemm_wide_matrix_bf16_scales_on_the_fp16_matrix_path(bits, g, M):
    """Wide matrices (N >= 8192): at 260 and 300 rows bfloat16 scales are brought to binary16 through a common power of
    two and the product runs on the fp16 matrix path; at 130 and 140 rows it keeps 32-row blocks and bfloat16 operands
    (the plan's description names the block shape)."""
    fq = _fq()
    K, N = 512, 8192
    desc = fq.gemm_describe(M, N, K, bits, g)
    _say(f"gemm bf16 scales wide int{bits} g={g} M={M}: {desc}")
    _gemm_case(M, K, N, bits, g, seed=6200 + M + bits + g)


@pytest.mark.parametrize("M,K,N", [(257, 640, 8208), (563, 640, 12304), (386, 640, 16400)])
@pytest.mark.parametrize("bits,g", [(4, 128), (4, 64), (4, 32), (8, 128), (3, 128)])
def test_gemm_shapes_between_64_and_128_rows_bf16_scales(bits, g, M, K, N):
    """80 x 256, 128 x 256 and 80 x 384 blocks: post-scaled with one scale row per k-block, where the scales are widened as
    they are, times the matrix's common power of two; pre-scaled otherwise."""
    _say(f"gemm bf16 scales M={M} K={K} N={N} int{bits} g={g}")
    _gemm_case(M, K, N, bits, g, seed=6400 + M + bits + g)


def test_gemm_wide_matrix_bf16_scales_spread_over_many_binades():
    """Columns scaled by powers of two from 2^-12 to 2^3 (scales spread over 15 binades inside one matrix), a
    zero column and a matrix that is tiny as a whole (every scale near 2^-22): the common power of two follows
    the largest scale, and what falls more than 2^14 below it is far below the tolerance."""
    fq = _fq()
    torch = torch_mod()
    K, N, M, g = 512, 8192, 300, 128
    W = workloads.weights_gaussian(K, N, 6301, outlier_prob=1e-3).astype(np.float32)
    W *= (2.0 ** ((np.arange(N) % 16) - 12)).astype(np.float32)[None, :]
    W[:, 5] = 0
    W = W.astype(np.float16)
    A = workloads.activations(M, K, "bf16", 6302)
    for Wm in (W, (workloads.weights_gaussian(K, N, 6303).astype(np.float32) * 2.0 ** -14).astype(np.float16)):
        codes, scales, q_ref, s_ref = _quantize_parity(Wm, 4, g)
        C_ref = oracle.gemm_ref(A, q_ref, s_ref)
        C = from_dev_act(fq.gemm(to_dev_act(A, "bf16"), codes, scales, 4, g), "bf16")
        assert np.max(np.abs(C_ref)) > 0
        assert_gemm_close(C, C_ref, "bf16", "bf16 scales over many binades")
        # column by column as well where the column is not negligible: each column's own scale of error
        col_scale = np.max(np.abs(C_ref), axis=0)
        big = col_scale >= 2.0 ** -10 * col_scale.max()
        err = np.max(np.abs(C - C_ref), axis=0)
        assert np.all(err[big] <= 1.6e-2 * col_scale[big])


def _columns_over_binades(K, N, binades, seed):
    """N(0, 0.02) weights, columns times powers of two from 2^14 down over `binades` binades, and a zero column."""
    W = workloads.weights_gaussian(K, N, seed, outlier_prob=1e-3).astype(np.float32)
    W *= (2.0 ** (14.0 - (np.arange(N) * 7) % (binades + 1))).astype(np.float32)[None, :]
    W[:, 5] = 0
    return W.astype(np.float16)


@pytest.mark.parametrize("bits,g,M,K,N", [(4, 64, 250, 2048, 12304), (8, 128, 250, 2048, 12304), (4, 32, 130, 2048, 24592)])
@pytest.mark.parametrize("what", ["scales", "activations"])
def test_gemm_65_to_256_rows_keep_bfloat16_range(bits, g, M, K, N, what):
    """Where binary16 activations take blocks of 80 rows and more in place of 32- and 64-row ones, bfloat16 ones do not: their operands
    stay bfloat16.  Scales over 24 binades, and activations 2^40 times their neighbours on zero weights: every result
    within the roundings of its terms' weights and of itself to bfloat16, 2^-9 each (a column or a neighbour that vanishes
    is off by some 20 times that)."""
    fq = _fq()
    torch = torch_mod()
    desc = fq.gemm_describe(M, N, K, bits, g)
    _say(f"range int{bits} g={g} M={M} {what}: {desc}")
    assert "f16: rows=" in desc and "mt=8" not in desc
    A = workloads.activations(M, K, "bf16", 6602)
    if what == "scales":
        W = _columns_over_binades(K, N, 24, 6601)
        codes, scales, q_ref, s_ref = _quantize_parity(W, bits, g)
    else:
        W = workloads.weights_gaussian(K, N, 6601)
        W[::96] = 0
        A[:, ::96] = 2.0 ** 40
        codes, scales = fq.quantize(torch.from_numpy(W).cuda(), bits, g)
        q_ref, s_ref = oracle.quantize(W, bits, g)
    C_ref = oracle.gemm_ref(A, q_ref, s_ref)
    C = from_dev_act(fq.gemm(to_dev_act(A, "bf16"), codes, scales, bits, g), "bf16")
    terms = np.abs(A.astype(np.float64)) @ np.abs(oracle.dequantize(q_ref, s_ref))
    assert np.all(np.abs(C - C_ref) <= 1.01 * 2.0 ** -9 * (np.abs(C_ref) + terms))


@pytest.mark.parametrize("bits,g,M,K,N,shape", [(4, 64, 300, 512, 8192, "rows=80 cols=256"), (4, 32, 300, 512, 8192, "rows=80 cols=256"),
                                                (8, 64, 300, 512, 8192, "rows=80 cols=256"), (4, 128, 300, 512, 8192, "rows=80 cols=256"),
                                                (4, 64, 578, 640, 10256, "rows=112 cols=256"), (4, 128, 1040, 512, 8208, "mt=8 waves=8"),
                                                (4, 64, 1040, 512, 8208, "mt=8 waves=8"), (8, 128, 1040, 512, 8208, "mt=8 waves=8")])
def test_gemm_bf16_scales_over_many_binades_on_the_fp16_matrix_path(bits, g, M, K, N, shape):
    """Scales over 20 binades on the shapes that bring them to binary16 (and the post-scaled one, which does not): with 2^E
    the largest scale's power of two a scale times its code is off by at most 2^-24 2^E |q| beside the roundings of the
    weight (2^-11) and the result (2^-9)."""
    fq = _fq()
    desc = fq.gemm_describe(M, N, K, bits, g)
    _say(f"binades int{bits} g={g} M={M}: {desc}")
    assert shape in desc and ("rows=" in shape or "rows=" not in desc)
    W = _columns_over_binades(K, N, 20, 6701)
    codes, scales, q_ref, s_ref = _quantize_parity(W, bits, g)
    A = workloads.activations(M, K, "bf16", 6702)
    C = from_dev_act(fq.gemm(to_dev_act(A, "bf16"), codes, scales, bits, g), "bf16")
    C_ref = oracle.gemm_ref(A, q_ref, s_ref)
    top = 2.0 ** np.floor(np.log2(s_ref.astype(np.float64).max()))
    mag = np.abs(A.astype(np.float64))
    terms = mag @ np.abs(oracle.dequantize(q_ref, s_ref))
    lost = 2.0 ** -24 * top * (mag @ np.abs(q_ref.astype(np.float64)))
    assert np.all(np.abs(C - C_ref) <= 2.0 ** -8 * np.abs(C_ref) + 2.0 ** -10 * terms + lost)


def test_gemm_split_k_bf16_scales():
    """A shape whose plan splits K (few column blocks, many k-blocks)."""
    _say("gemm bf16 scales split-K")
    _gemm_case(64, 4096, 48, 4, 128, seed=6100)
    _gemm_case(8, 4096, 48, 4, 64, seed=6101)


@pytest.mark.parametrize("bits,g", [(4, 32), (8, 0)])
def test_one_hot_rows_return_the_dequantised_weights(bits, g):
    """M = 16 one-hot rows: C[i, :] = q[k_i, :] * s[k_i / g, :] rounded once to bf16 (no accumulation error),
    which also proves that the scale bits are widened as bfloat16 and not as binary16."""
    _say(f"one-hot rows, bf16 scales int{bits} g={g}")
    fq = _fq()
    K, N = 512, 96
    W = workloads.weights_gaussian(K, N, 6200 + bits, outlier_prob=1e-3)
    codes, scales, q_ref, s_ref = _quantize_parity(W, bits, g)
    ks = [0, 1, 31, 32, 63, 64, 127, 128, 129, 255, 256, 300, 383, 384, 500, 511]
    A = np.zeros((16, K), dtype=np.float32)
    for i, k in enumerate(ks):
        A[i, k] = 1.0
    C = from_dev_act(fq.gemm(to_dev_act(A, "bf16"), codes, scales, bits, g), "bf16")
    Wd = oracle.dequantize(q_ref, s_ref)
    want = workloads.round_to_bf16(Wd[ks].astype(np.float32)).astype(np.float64)
    assert np.array_equal(C, want)


def test_grouped_bf16_scales():
    _say("grouped bf16 scales")
    fq = _fq()
    torch = torch_mod()
    K, N, bits, g = 256, 400, 4, 64
    rows = [32, 33, 0, 65, 129, 1]
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    A = workloads.activations(int(offsets[-1]), K, "bf16", 6300)
    qs, ss, codes_l, scales_l = [], [], [], []
    for e in range(len(rows)):
        W = workloads.weights_gaussian(K, N, 6310 + e, outlier_prob=1e-3)
        c, s, q_ref, s_ref = _quantize_parity(W, bits, g)
        codes_l.append(c)
        scales_l.append(s.reshape(-1))
        qs.append(q_ref)
        ss.append(s_ref)
    out = torch.full((int(offsets[-1]), N), 3.0, dtype=torch.bfloat16, device="cuda")
    fq.gemm_grouped(to_dev_act(A, "bf16"), offsets.tolist(), torch.cat(codes_l), torch.cat(scales_l), bits, g, N,
                    out=out)
    C = from_dev_act(out, "bf16")
    C_ref = oracle.gemm_ref_grouped(A, offsets, qs, ss)
    for e in range(len(rows)):
        if rows[e]:
            sl = slice(offsets[e], offsets[e + 1])
            assert_gemm_close(C[sl], C_ref[sl], "bf16", f"expert {e}")


def test_quant_error_bf16_scales():
    _say("quant_error bf16 scales")
    fq = _fq()
    torch = torch_mod()
    W = workloads.weights_gaussian(512, 272, 6400, outlier_prob=1e-3)
    for bits, g in ((4, 64), (8, 0)):
        codes, scales, q_ref, s_ref = _quantize_parity(W, bits, g)
        sse, mx = fq.quant_error(torch.from_numpy(W).cuda(), codes, scales, bits, g)
        sse_ref, mx_ref = oracle.quant_error(W, q_ref, s_ref)
        assert mx == mx_ref
        assert abs(sse - sse_ref) <= 1e-11 * sse_ref


@pytest.mark.parametrize("bits", [3, 4, 8])
def test_quant_error_of_the_largest_bf16_scales(bits):
    """A caller's bfloat16 scales next to binary32's largest: the error is that scale times the code, in binary64."""
    fq = _fq()
    torch = torch_mod()
    W = workloads.weights_gaussian(256, 48, 6401)
    codes, scales, q_ref, s_ref = _quantize_parity(W, bits, 64)
    scales[1, 7] = 2.0 ** 127
    s64 = s_ref.astype(np.float64)
    s64[1, 7] = 2.0 ** 127
    err = W.astype(np.float64) - q_ref.astype(np.float64) * np.repeat(s64, 64, axis=0)
    sse, mx = fq.quant_error(torch.from_numpy(W).cuda(), codes, scales, bits, 64)
    assert mx == np.abs(err).max() and abs(sse - np.sum(err * err)) <= 1e-11 * np.sum(err * err)


def test_bf16_scales_need_bf16_activations():
    fq = _fq()
    torch = torch_mod()
    W = workloads.weights_gaussian(256, 32, 6500)
    codes, scales = fq.quantize(torch.from_numpy(W).cuda(), 4, 64, fq.FQ_SCALE_BF16)
    A = torch.zeros((4, 256), dtype=torch.float16, device="cuda")
    with pytest.raises(fq.FqError) as ei:
        fq.gemm(A, codes, scales, 4, 64)
    assert ei.value.status == fq.FQ_ERR_UNSUPPORTED
