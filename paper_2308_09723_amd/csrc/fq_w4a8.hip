// The integer path: int8 activations x int4 weights with integer group scales on the integer matrix cores
// (the paper's closing section names it as future work: "Conclusions and Limitations", last paragraph; the
// reading is stated in fq.h next to fq_quantize_w4a8).
//
//   weights      s[i, n] = z[i, n] * t[n],  z an integer in 1..16 (one byte per group), t binary16 per column;
//                codes q = int(w / s) as in Appendix A, stored in the packed 4-bit layout of fq_layout.h
//   activations  Appendix A at 8 bits per row: alpha[m] binary32, a[m, k] in [-127, 127]
//   product      S = sum_k a * (q * z) in int32 (v_mfma_i32_16x16x64_i8), C = alpha[m] * t[n] * S
//
// Packed layout of the codes of this path (its own: fq_unpack_w4a8 reads it back).  Tiles of 16 columns x 128
// rows, k-block-major, 64 lane records of 16 bytes per tile exactly like the floating-point layout
// (lane = 16 j + n % 16), but a record is ordered for v_mfma_i32_16x16x64_i8: MFMA step T (rows
// 64 T .. 64 T + 63 of the k-block) takes from lane group j the 16 consecutive rows 64 T + 16 j + 0..15;
// dword 2 T + h of the record holds rows 64 T + 16 j + 8 h + e (e = 0..7), byte b carrying element b in its
// low and element b + 4 in its high nibble (stored value q + 8).  Masking the low / the high nibbles of a
// dword then yields the operand's bytes in row order, and the activations need no reordering: lane (m, j)
// supplies the 16 consecutive int8 of row m at k = 64 T + 16 j.
//
// The weights are brought to the activation's type before the multiply, as section 4.1 describes for the
// floating-point kernels; here that type is int8 and the conversion is q * z, formed four at a time: the stored
// nibbles u = q + 8 of a dword are spread over bytes, one packed 16-bit multiply-add gives u * z + (128 - 8 z)
// in every byte (between 16 and 240: no carries), and flipping the top bit of each byte leaves q * z in two's
// complement.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <math.h>
#include <stdint.h>

#include "fq_gemm_kernels.h"
#include "fq_lds_limit.h"
#include "fq_internal.h"
#include "fq_layout.h"
#include "fq_panel.h"

using namespace fqk;

namespace {

constexpr int ZMAX = 16;           // largest group multiplier: 7 * 16 = 112 fits an int8
constexpr float WLEVELS = 15.0f;   // 2^4 - 1, Appendix A
constexpr float ALEVELS = 255.0f;  // 2^8 - 1
constexpr int W8_NT = 3;           // column tiles per wave
constexpr int W8_WAVES = 8;

__device__ inline float f16_bits_to_float(uint16_t b) { return half_bits_to_float(b); }

// ------------------------------------------------------------------------------------------------------
// Weight quantiser (offline path):
//   1. abs-max of every group, as binary16 bit patterns, parked in the not-yet-written code buffer
//      (fq_fine_absmax_kernel; groups of more than 1024 rows as blocks of 128 rows, folded by a second kernel);
//   2. per column: t = smallest binary16 with 16 * 15 * t >= 2 * (largest group abs-max), then for every
//      group the smallest z in 1..16 with 15 * z * t >= 2 * (its abs-max)  (all products exact in binary32);
//   3. codes q = clamp(round_half_even(w / (z t)), -7, 7), IEEE binary32 quotient, packed.
// W has to be read twice (a column's step needs all of it).  Both passes are bound by HBM: 16-byte loads, the second
// from panels staged in LDS.  On 12288 x 12288, g = 128 (us): abs-max with 2-byte loads 96 -> 58, steps and
// multipliers 60 -> 9, encoding with a strided 2-byte load and a division per weight 201 -> 63
// (72 from the top of the matrix down).
// ------------------------------------------------------------------------------------------------------
// abs-max of every group from the maxima of its `per_group` blocks
__global__ __launch_bounds__(256) void w8_fold_kernel(const uint16_t* __restrict__ fine, int64_t N, int per_group,
                                                       uint16_t* __restrict__ amax) {
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    const uint16_t* src = fine + (int64_t)blockIdx.y * per_group * N + n;
    uint16_t m = 0;
#pragma unroll 8
    for (int i = 0; i < per_group; ++i) {
        const uint16_t v = src[(int64_t)i * N];
        m = v > m ? v : m;
    }
    amax[(int64_t)blockIdx.y * N + n] = m;
}

// Block = 2 LANES columns (two per thread) x SLICES slices of the groups, whose maxima stay in registers between the search
// for the column's largest and the multipliers: 32 columns x 32 slices, or 64 x 8 for up to 32 groups.  Bound by latency and,
// as few blocks as there are, by the tests of a multiplier.  With 32 columns x 8 slices per block, every group read twice and
// a loop with a branch per test: traced, us: 12288 x 12288 g = 128 8.2 -> 5.1, 10240 x 6032 g = 64 10.9 -> 5.2; the whole
// call at g = 32 1.17x on average over 20 matrices (5760 x 1312 23.8 -> 15.1).
constexpr int W8_HELD = 8;          // groups per thread held in registers (further ones are read again)
template <int LANES, int SLICES>
__global__ __launch_bounds__(LANES * SLICES) void w8_scales_kernel(const uint16_t* __restrict__ amax, int64_t N, int groups,
                                                                    uint8_t* __restrict__ z, uint16_t* __restrict__ tstep) {
    __shared__ uint32_t red[SLICES][LANES + 1];
    const int x = threadIdx.x % LANES, y = threadIdx.x / LANES;
    const int64_t n = ((int64_t)blockIdx.x * LANES + x) * 2;                // N is a multiple of 16
    const bool ok = n < N;
    auto load = [&](int i) { return *reinterpret_cast<const uint32_t*>(amax + (int64_t)i * N + n); };
    uint32_t held[W8_HELD];
    u16x2_t m = {0, 0};
    if (ok) {
#pragma unroll
        for (int h = 0; h < W8_HELD; ++h) held[h] = y + SLICES * h < groups ? load(y + SLICES * h) : 0u;
#pragma unroll
        for (int h = 0; h < W8_HELD; ++h) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2_t, held[h]));
#pragma unroll 4
        for (int i = y + SLICES * W8_HELD; i < groups; i += SLICES) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2_t, load(i)));
    }
    red[y][x] = __builtin_bit_cast(uint32_t, m);
    __syncthreads();
    if (!ok) return;
#pragma unroll 8
    for (int i = 0; i < SLICES; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2_t, red[i][x]));
    const float L = WLEVELS * (float)ZMAX;                                  // 240
    float t[2], r15t[2];
    uint32_t steps = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float two_m = 2.0f * f16_bits_to_float(m[c]);
        uint16_t tb = __half_as_ushort(__float2half_rn(__fdiv_rn(two_m, L)));   // nearest, then up if too small
        if (__fmul_rn(L, f16_bits_to_float(tb)) < two_m) tb += 1;
        t[c] = f16_bits_to_float(tb);
        r15t[c] = t[c] == 0.0f ? 0.0f : __fdiv_rn(1.0f, WLEVELS * t[c]);
        steps |= (uint32_t)tb << (16 * c);
    }
    if (y == 0) *reinterpret_cast<uint32_t*>(tstep + n) = steps;
    auto store = [&](int i, uint32_t v) {
        uint32_t out = 0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float two_mi = 2.0f * f16_bits_to_float((uint16_t)(v >> (16 * c)));
            // the quotient two_mi / (15 t) cut to an integer is the multiplier, or one or two below it (the estimate's error
            // is far below one); the tests are exact ((15 z) * t: exact)
            int zi = (int)(two_mi * r15t[c]);
            zi = zi < 1 ? 1 : (zi > ZMAX ? ZMAX : zi);
            const bool one = __fmul_rn(WLEVELS * (float)zi, t[c]) < two_mi;
            const bool two = one && __fmul_rn(WLEVELS * (float)(zi + 1), t[c]) < two_mi;
            zi += (int)one + (int)two;
            zi = zi > ZMAX ? ZMAX : zi;
            out |= (uint32_t)zi << (8 * c);
        }
        *reinterpret_cast<uint16_t*>(z + (int64_t)i * N + n) = (uint16_t)out;
    };
#pragma unroll
    for (int h = 0; h < W8_HELD; ++h)
        if (y + SLICES * h < groups) store(y + SLICES * h, held[h]);
#pragma unroll 1
    for (int i = y + SLICES * W8_HELD; i < groups; i += SLICES) store(i, load(i));
}

// row of the k-block that element e of dword d of lane group j holds
__host__ __device__ inline int w8_row(int d, int j, int e) { return 64 * (d >> 1) + 16 * j + 8 * (d & 1) + e; }

// A block encodes a 128 x 128 panel staged in LDS: thread -> two neighbouring columns and lane group j, i.e. two
// adjacent lane records (16 bytes each: 32 codes of one column in one k-block).
__global__ __launch_bounds__(256) void w8_encode_kernel(const uint16_t* __restrict__ W, int64_t N, int g,
                                                         const uint8_t* __restrict__ z,
                                                         const uint16_t* __restrict__ tstep,
                                                         uint32_t* __restrict__ codes) {
    __shared__ __align__(16) uint16_t panel[FQ_QP_ROWS * FQ_QP_PITCH];
    __shared__ __align__(16) float sub_scale[4][FQ_QP_COLS];      // z t of the group each 32-row sub-block belongs to
    __shared__ __align__(16) float sub_rscale[4][FQ_QP_COLS];     // its reciprocal (0 for a step of 0)
    const int tid = threadIdx.x;
    const int64_t n0 = (int64_t)blockIdx.x * FQ_QP_COLS;
    // (bottom of the matrix first: the abs-max pass went top to bottom, and its end is what the Infinity Cache still holds)
    const int64_t kb = gridDim.y - 1 - blockIdx.y;
    const int64_t k0 = kb * FQ_QP_ROWS;          // K is a multiple of 128
    const int cols = (int)((N - n0) < FQ_QP_COLS ? (N - n0) : FQ_QP_COLS);   // multiple of 16
    fq_stage_panel(W, N, k0, n0, FQ_QP_ROWS, cols, panel);
    {
        const int c = tid & 127;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int sb = (tid >> 7) + 2 * h;
            float v = 0.0f;
            if (c < cols) v = (float)z[((k0 + sb * 32) / g) * N + n0 + c] * f16_bits_to_float(tstep[n0 + c]);   // exact
            // an infinite weight makes its column's step infinite: w / infinity = 0 for the finite ones (fq_encode_biased
            // would form 0 * infinity; with 0 for the step it gives 0 for them and what a NaN gives for the infinite one)
            if (v == __builtin_inff()) v = 0.0f;
            sub_scale[sb][c] = v;
            sub_rscale[sb][c] = v == 0.0f ? 0.0f : __fdiv_rn(1.0f, v);
        }
    }
    __syncthreads();
    const int c = (tid & 63) * 2, j = tid >> 6;
    if (c >= cols) return;
    uint32_t out0[4], out1[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int r0 = w8_row(d, j, 0);                            // 8 rows inside one group
        const float2 s = *reinterpret_cast<const float2*>(&sub_scale[r0 / 32][c]);
        const float2 rs = *reinterpret_cast<const float2*>(&sub_rscale[r0 / 32][c]);
        uint32_t b0[8], b1[8];
        fq_encode8_pair(panel, r0, c, s, rs, 7.0f, FQ_ENCODE_MAGIC + 8.0f, b0, b1);
        // byte b: element b in the low, element b + 4 in the high nibble
        out0[d] = fq_gather_bytes(b0[0], b0[1], b0[2], b0[3]) | (fq_gather_bytes(b0[4], b0[5], b0[6], b0[7]) << 4);
        out1[d] = fq_gather_bytes(b1[0], b1[1], b1[2], b1[3]) | (fq_gather_bytes(b1[4], b1[5], b1[6], b1[7]) << 4);
    }
    const int64_t at = fq_rec(n0 / FQ_NTILE + c / FQ_NTILE, kb, N / FQ_NTILE, j * 16 + c % FQ_NTILE);
    uint32_t* dst = codes + at * 4;                                // record of column c; the next one follows it
    *reinterpret_cast<uint4*>(dst) = make_uint4(out0[0], out0[1], out0[2], out0[3]);
    *reinterpret_cast<uint4*>(dst + 4) = make_uint4(out1[0], out1[1], out1[2], out1[3]);
}

// the logical codes q[K, N] (int8) of a packed buffer: one thread per lane record
__global__ __launch_bounds__(256) void w8_unpack_kernel(const uint32_t* __restrict__ codes, int64_t K, int64_t N,
                                                         int8_t* __restrict__ q) {
    const int64_t rec = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t ntiles = N / FQ_NTILE;
    if (rec >= (K / 128) * ntiles * 64) return;
    const int lane = (int)(rec & 63);
    const int64_t tile = (rec >> 6) % ntiles, kb = (rec >> 6) / ntiles;
    const int64_t n = tile * FQ_NTILE + (lane & 15);
    const int j = lane >> 4;
    const uint4 v = *reinterpret_cast<const uint4*>(codes + rec * 4);
    const uint32_t d4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int e = 0; e < 8; ++e)
            q[(kb * 128 + w8_row(d, j, e)) * N + n] = (int8_t)((int)((d4[d] >> (8 * (e & 3) + 4 * (e >> 2))) & 0xfu) - 8);
}

// ------------------------------------------------------------------------------------------------------
// Activation quantiser: block r handles row r.  alpha = smallest binary32 with 255 alpha >= 2 max|A[r, :]|
// (nearest quotient, then one step up if the exact sign of 127.5 alpha - max, taken from a fused
// multiply-add, is negative); a = clamp(round_half_even(A / alpha), -127, 127), IEEE binary32 quotient.
// ------------------------------------------------------------------------------------------------------
template <int ACT>
__device__ inline float act_to_float(uint16_t b) {
    if constexpr (ACT == FQ_F16) return f16_bits_to_float(b);
    else return __uint_as_float((uint32_t)b << 16);
}

// 2 max / 255 = max / 127.5 (the same real number; this form cannot overflow for bfloat16 inputs near 2^128)
__device__ inline float w8_alpha(float amax) {
    float al = __fdiv_rn(amax, 0.5f * ALEVELS);
    if (__builtin_fmaf(0.5f * ALEVELS, al, -amax) < 0.0f) al = __uint_as_float(__float_as_uint(al) + 1u);   // next value up
    return al;
}

// the code of one value by the division itself, as a byte
__device__ inline uint32_t w8_act_code(float a, float al) {
    int q = 0;
    if (al != 0.0f) q = (int)fminf(fmaxf(rintf(__fdiv_rn(a, al)), -127.0f), 127.0f);
    return (uint32_t)q & 0xffu;
}

// the codes of eight values by the division, as eight bytes
template <int ACT>
__device__ inline u32x2 w8_act_codes8(const u32x4& v, float al) {
    u32x2 o;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t c[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) c[d] = w8_act_code(act_to_float<ACT>((uint16_t)(v[2 * h + (d >> 1)] >> (16 * (d & 1)))), al);
        o[h] = c[0] | (c[1] << 8) | (c[2] << 16) | (c[3] << 24);
    }
    return o;
}

// Rows of any length and alignment, read twice.  The first `units` x 8 values of a row (whole 16-byte units at aligned
// addresses; 0 for other rows) are read eight values and written eight bytes per lane, the rest one value per lane and
// memory instruction (which is what such rows are then bound by: 64 x 131072 159 us, 42 in units).
template <int ACT>
__global__ __launch_bounds__(256) void w8_act_quant_kernel(const uint16_t* __restrict__ A, int64_t K, int64_t units,
                                                            int8_t* __restrict__ Aq, float* __restrict__ alpha) {
    __shared__ uint32_t red[4];
    const int64_t r = blockIdx.x;
    const uint16_t* src = A + r * K;
    u16x2_t m2 = {0, 0};                                 // magnitudes of one format order like their bit patterns
    for (int64_t u = threadIdx.x; u < units; u += 256) {
        const u32x4 v = reinterpret_cast<const u32x4*>(src)[u];
#pragma unroll
        for (int i = 0; i < 4; ++i) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(u16x2_t, v[i] & 0x7fff7fffu));
    }
    uint32_t m = m2[0] > m2[1] ? m2[0] : m2[1];
    for (int64_t k = units * 8 + threadIdx.x; k < K; k += 256) {
        const uint32_t v = src[k] & 0x7fffu;
        m = v > m ? v : m;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t t = (uint32_t)__shfl_xor((int)m, o, 64);
        m = t > m ? t : m;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = red[0];
#pragma unroll
    for (int i = 1; i < 4; ++i) m = red[i] > m ? red[i] : m;
    const float al = w8_alpha(act_to_float<ACT>((uint16_t)m));
    if (threadIdx.x == 0) alpha[r] = al;
    int8_t* dst = Aq + r * K;
    for (int64_t u = threadIdx.x; u < units; u += 256)
        reinterpret_cast<u32x2*>(dst)[u] = w8_act_codes8<ACT>(reinterpret_cast<const u32x4*>(src)[u], al);
    for (int64_t k = units * 8 + threadIdx.x; k < K; k += 256) dst[k] = (int8_t)w8_act_code(act_to_float<ACT>(src[k]), al);
}

// Rows of whole 16-byte units at aligned addresses, short enough for the block's registers (UNITS units of 8 values per
// thread): read once, eight values per load, kept in registers across the search for the largest one.
// The quotient A / alpha must be the correctly rounded binary32 one (it is rounded a second time, to an integer): with
// rs = 1 / alpha rounded to nearest, two steps x + fma(-x, alpha, A) * rs from x0 = A * rs give it (Markstein's theorem:
// the second one starts within one unit in the last place), wherever residuals do not underflow and rs is finite; rows
// with alpha outside 2^-90 .. 2^100 take the division.  Checked on the host against the division
// (tests/encode_identity_check.c).  Then clamp, round by adding 1.5 * 2^23, keep the low byte.  Bound by memory:
// 2048 x 12288 26 -> 16 us; eight rows 6.4 -> 4.9 us (latency: 1024 threads per row).  Threads that hold no more units than the
// row needs (eight of them everywhere before: most loaded the last unit again), inside graphs, us: 8 x 12288 3.8 -> 3.1,
// 512 x 4096 5.1 -> 3.0, 2048 x 1024 5.0 -> 3.5, 2048 x 12288 13.7 as before.
constexpr int W8_ROW_UNITS = 8;      // the most units per thread
template <int ACT, int THREADS, int UNITS>
__global__ __launch_bounds__(THREADS) void w8_act_quant_row_kernel(const uint16_t* __restrict__ A, int units,
                                                                    int8_t* __restrict__ Aq, float* __restrict__ alpha) {
    __shared__ uint32_t red[THREADS / 64];
    const int64_t r = blockIdx.x;
    const u32x4* src = reinterpret_cast<const u32x4*>(A) + r * units;
    u32x4 v[UNITS];
    u16x2_t m2 = {0, 0};
#pragma unroll
    for (int i = 0; i < UNITS; ++i) {
        const int u = threadIdx.x + i * THREADS;
        v[i] = src[u < units ? u : units - 1];           // (past the end: the last unit again, never stored)
    }
#pragma unroll
    for (int i = 0; i < UNITS; ++i)
#pragma unroll
        for (int d = 0; d < 4; ++d)                      // magnitudes of one format order like their bit patterns
            m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(u16x2_t, v[i][d] & 0x7fff7fffu));
    uint32_t m = m2[0] > m2[1] ? m2[0] : m2[1];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t t = (uint32_t)__shfl_xor((int)m, o, 64);
        m = t > m ? t : m;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < THREADS / 64; ++i) m = red[i] > m ? red[i] : m;
    const float al = w8_alpha(act_to_float<ACT>((uint16_t)m));
    if (threadIdx.x == 0) alpha[r] = al;
    u32x2* dst = reinterpret_cast<u32x2*>(Aq) + r * units;
    if (al >= 0x1p-90f && al <= 0x1p100f) {
        const float rs = __fdiv_rn(1.0f, al);
        auto code = [&](uint16_t bits) -> uint32_t {
            const float a = act_to_float<ACT>(bits);
            float x = a * rs;
            x = __builtin_fmaf(__builtin_fmaf(-x, al, a), rs, x);
            x = __builtin_fmaf(__builtin_fmaf(-x, al, a), rs, x);
            return __float_as_uint(__builtin_amdgcn_fmed3f(x, -127.0f, 127.0f) + FQ_ENCODE_MAGIC);
        };
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const int u = threadIdx.x + i * THREADS;
            // (one unit after the other: all of them at once would take four times the registers)
            asm volatile("" : "+v"(v[i][0]), "+v"(v[i][1]), "+v"(v[i][2]), "+v"(v[i][3]));
            if (u >= units) continue;
            u32x2 o;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                o[h] = fq_gather_bytes(code((uint16_t)v[i][2 * h]), code((uint16_t)(v[i][2 * h] >> 16)),
                                       code((uint16_t)v[i][2 * h + 1]), code((uint16_t)(v[i][2 * h + 1] >> 16)));
            dst[u] = o;
        }
    } else {
#pragma unroll 1
        for (int u = threadIdx.x; u < units; u += THREADS) dst[u] = w8_act_codes8<ACT>(src[u], al);
    }
}

template <int ACT>
void w8_launch_act_quant(const uint16_t* A, int64_t M, int64_t K, int8_t* Aq, float* alpha, hipStream_t stream) {
    const dim3 grid((unsigned)M);
    const bool wide = (K & 7) == 0 && ((uintptr_t)A & 15) == 0 && ((uintptr_t)Aq & 7) == 0;
    const int64_t units = K >> 3;
    // Few rows (one block per compute unit, latency counts): as many threads per row as it has units for, up to 1024, and
    // no more units per thread than the row needs.  Many rows: four waves per block, several blocks per compute unit.
#define W8_ROWS(THREADS_, UNITS_)                                                                                       \
    hipLaunchKernelGGL((w8_act_quant_row_kernel<ACT, THREADS_, UNITS_>), grid, dim3(THREADS_), 0, stream, A, (int)units, Aq, alpha)
    if (wide && units <= 256) W8_ROWS(256, 1);
    else if (wide && M > 512 && units <= 256 * 2) W8_ROWS(256, 2);
    else if (wide && M > 512 && units <= 256 * 4) W8_ROWS(256, 4);
    else if (wide && M > 512 && units <= 256 * W8_ROW_UNITS) W8_ROWS(256, W8_ROW_UNITS);
    else if (wide && units <= 512) W8_ROWS(512, 1);
    else if (wide && units <= 1024) W8_ROWS(1024, 1);
    else if (wide && units <= 1024 * 2) W8_ROWS(1024, 2);
    else if (wide && units <= 1024 * W8_ROW_UNITS) W8_ROWS(1024, W8_ROW_UNITS);
#undef W8_ROWS
    else
        hipLaunchKernelGGL(w8_act_quant_kernel<ACT>, grid, dim3(256), 0, stream, A, K, wide ? units : (int64_t)0, Aq, alpha);
}

// ------------------------------------------------------------------------------------------------------
// Product.  Same orientation as the floating-point kernels: 16 x 16 tiles of C^T, the weights the first
// MFMA operand (16 columns n), the activations the second (16 rows m); a lane's packed record is, after the
// conversion, its slice of the first operand, so weights never pass through LDS.
// Block = 8 waves x 3 column tiles (384 columns), BM = 16 MT rows (MT = 4 or 8), k-block = 128 rows = two MFMA steps.
// The k loop is one software pipeline, two k-blocks deep:
//   * activation tiles (BM rows x 128 int8, natural order) go global -> LDS directly (global_load_lds_dwordx4),
//     three LDS tiles; the eight 16-byte units of a row are XOR-swizzled with the row (through the global
//     address each lane reads), so a fragment read of 16 rows of one unit column spreads over all banks;
//   * two weight register sets: the set of k-block kb is reloaded with k-block kb + 2 right after its last
//     conversion; the loop is unrolled twice so that the sets keep their names;
//   * one barrier per k-block, at its end: before it the wave waits until at most the loads issued after
//     those of k-block kb + 1 are in flight (the counter retires in order and every loading wave issues the
//     same loads), after it the tile read during kb is free.  Issue order inside k-block kb:
//     fragments of step 1 | MFMAs of step 0 with the conversion of step 1 between them | first MFMAs of step 1 |
//     A(kb + 2) into the tile read during kb - 1, W(kb + 2) | MFMAs of step 1 with the conversion of step 0 of
//     k-block kb + 1 between them; before the last of them: wait, barrier, fragments of step 0 of kb + 1.
// ZR = multiplier rows per k-block a lane needs: 1 when the group size is a multiple of 128, else one per
// 64-row step (the lane's 16 rows of a step lie inside one 32-row block, hence inside one group).
// With splits > 1 every block writes its int32 sums to its split's slab of a partial buffer and a second
// kernel adds the slabs (integers: exact whatever the order) and scales the sum.
// ------------------------------------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2v __attribute__((ext_vector_type(2)));

// four stored nibbles spread over the bytes of x (each 1..15) -> four int8 values (u - 8) * z
__device__ inline uint32_t w8_scale_bytes(uint32_t x, u16x2v zz, u16x2v cc) {
    const u16x2v r = bitcast<u16x2v>(x) * zz + cc;          // u z + (128 - 8 z) in every byte, no carries
    return bitcast<uint32_t>(r) ^ 0x80808080u;
}

template <int OUT>
__device__ inline void w8_store4(uint16_t* C, const v4i& s, float scale_m, const float (&tn)[4]) {
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (float)s[i] * (scale_m * tn[i]);
    *reinterpret_cast<u32x2*>(C) = pack4<OUT>(v);
}

template <int MT, int ZR, int OUT>
__global__ __launch_bounds__(W8_WAVES * 64) void fq_gemm_w4a8_kernel(
    const int8_t* __restrict__ Aq, const float* __restrict__ alpha, const u32x4* __restrict__ codes,
    const uint8_t* __restrict__ z, const uint16_t* __restrict__ tstep, uint16_t* __restrict__ C,
    int32_t* __restrict__ partial, int M, int N, int K, int g, int kb_per_split, int splits, int nblocks_n,
    int nblocks_m) {
    constexpr int NT = W8_NT;
    constexpr int BM = MT * 16;
    constexpr int UNITS = BM * 8;                       // 16-byte units of an activation tile
    constexpr int NI = UNITS / 64;                      // wave-level direct loads per tile
    constexpr int DPT = NI >= W8_WAVES ? NI / W8_WAVES : 1;   // of which this wave issues DPT (or none)
    constexpr int NW = NT + ZR * NT;                    // vector loads of one weight set
    static_assert(NI % W8_WAVES == 0 || NI < W8_WAVES, "every loading wave issues the same number of loads");
    extern __shared__ u32x4 lds[];                       // [3][UNITS]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = N / FQ_NTILE;
    const int KB = K / 128;
    const int ml = lane & 15, j = lane >> 4;
    const int64_t kb_stride = (int64_t)ntiles * 64;

    const int tiles = nblocks_n * nblocks_m;
    int bid = blockIdx.x;
    const int split = bid / tiles;
    bid -= split * tiles;
    // the block ids an XCD receives (every eighth) -> one contiguous run of logical tiles
    const int L = (tiles & 7) == 0 ? (bid & 7) * (tiles >> 3) + (bid >> 3) : bid;
    int bn, bm_idx;
    fq_tile_of(L, nblocks_n, nblocks_m, bn, bm_idx);
    const int kb0 = split * kb_per_split;
    const int kb1 = min(KB, kb0 + kb_per_split);
    const int64_t row0 = (int64_t)bm_idx * BM;
    const int rows = (int)min((int64_t)BM, (int64_t)M - row0);

    // wave-uniform bases (scalar registers); the lane's part is a 32-bit offset added by the load itself
    const char* wbase[NT];
    const uint8_t* zbase[NT];
    bool tvalid[NT];
    const int tile0 = (bn * W8_WAVES + wave) * NT;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int tile = tile0 + nt;
        tvalid[nt] = tile < ntiles;
        const int tc = tvalid[nt] ? tile : 0;
        wbase[nt] = reinterpret_cast<const char*>(codes + fq_rec(tc, 0, ntiles, 0));
        zbase[nt] = z + (int64_t)tc * FQ_NTILE;
    }
    const uint32_t lane_rec = (uint32_t)lane * 16u;

    // direct loads: LDS unit u = (wave DPT + r) 64 + lane of a tile = (row u / 8, position u % 8), which holds
    // the row's 16-byte unit (position ^ (row & 7)); rows past the end repeat the last one (never stored)
    const bool a_loader = NI >= W8_WAVES || wave < NI;   // wave-uniform
    int64_t d_off[DPT];
#pragma unroll
    for (int r = 0; r < DPT; ++r) {
        const int u = (wave * DPT + r) * 64 + lane;
        const int row = u >> 3, pos = u & 7;
        const int rowc = row < rows ? row : rows - 1;
        d_off[r] = (row0 + rowc) * (int64_t)K + 16 * (pos ^ (row & 7));
    }
    auto load_a_lds = [&](int kb, int tile_i) {
        if (!a_loader) return;
        const int8_t* base = Aq + (int64_t)kb * 128;
        const uint32_t lds_base = __builtin_amdgcn_readfirstlane(
            (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(lds + tile_i * UNITS + wave * DPT * 64));
#pragma unroll
        for (int r = 0; r < DPT; ++r) load_lds16(lds_base + r * 1024, base + d_off[r]);
    };
    int a_rd[2];
#pragma unroll
    for (int T = 0; T < 2; ++T) a_rd[T] = ml * 8 + ((4 * T + j) ^ (ml & 7));

    v4i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = v4i{0, 0, 0, 0};

    u32x4 wqs[2][NT];
    uint32_t zqs[2][ZR][NT];
    auto load_w = [&](u32x4 (&q)[NT], uint32_t (&zr)[ZR][NT], int kb) {
        const int64_t kb_bytes = (int64_t)kb * kb_stride * 16;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) q[nt] = load_rec<4, false>(scalar_ptr(wbase[nt] + kb_bytes) + lane_rec);
#pragma unroll
        for (int r = 0; r < ZR; ++r) {
            if constexpr (ZR == 1) {
                // the k-block lies inside one group
                const int64_t zrow = (int64_t)((kb * 128) / g) * N;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) zr[r][nt] = scalar_ptr(zbase[nt] + zrow)[(uint32_t)ml];
            } else {
                // the group of this lane's 16 rows of step r
                const int64_t zrow = (int64_t)((kb * 128 + 64 * r + 16 * j) / g) * N;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) zr[r][nt] = zbase[nt][zrow + ml];
            }
        }
    };
    // piece p (0 .. 2 NT - 1) of the conversion of step T: dword h = p % 2 of column tile p / 2 (the pieces of a
    // step are converted in this order; the first piece of a column tile prepares its multiplier)
    uint32_t zcur[NT], ccur[NT];
    auto conv_piece = [&](u32x4 (&wop)[NT], const u32x4 (&q)[NT], const uint32_t (&zr)[ZR][NT], int T, int p) {
        const int nt = p >> 1, h = p & 1;
        if (h == 0) {
            // (the loaded multiplier stays opaque to the optimiser until here: otherwise its narrowing to 16 bits
            // is moved up to the load, and with it a wait for loads that were only just issued)
            uint32_t zi = zr[ZR == 1 ? 0 : T][nt];
            asm volatile("" : "+v"(zi));
            zcur[nt] = zi;
            ccur[nt] = (uint32_t)(0x8080 - (int)zi * 0x0808);   // 128 - 8 z in both bytes (8 z <= 128: no borrow)
        }
        const u16x2v zz = {(uint16_t)zcur[nt], (uint16_t)zcur[nt]};
        const u16x2v cc = {(uint16_t)ccur[nt], (uint16_t)ccur[nt]};
        const uint32_t w = q[nt][2 * T + h];
        wop[nt][2 * h] = w8_scale_bytes(w & 0x0f0f0f0fu, zz, cc);            // rows 8 h + 0..3
        wop[nt][2 * h + 1] = w8_scale_bytes((w >> 4) & 0x0f0f0f0fu, zz, cc);   // rows 8 h + 4..7
    };
    constexpr int NP = 2 * NT;                     // conversion pieces per step
    // the barrier stands before this MFMA group of step 1: early in the 128-row shape, so that the reads of the next
    // k-block's first fragments, which follow it, have six MFMA groups to return in (measured 1 - 4 % faster
    // than ahead of the last two groups; the tile it waits for was requested a k-block earlier either way)
    // (with two multiplier rows per k-block the fragments held that much longer cost spilled registers)
    constexpr int BAR_MT = MT >= 8 && ZR == 1 ? 1 : MT - 2;
    u32x4 wopA[NT], wopB[NT], af0[MT], af1[MT];
    // One k-block.  (qa, za): its weights, (qb, zb): those of k-block kb + 1, tile `cur`: its activations.
    // On entry wopA holds the converted operands of its step 0 and af0 that step's fragments (requested);
    // on exit the same for k-block kb + 1.  The conversions run in pieces between the MFMA groups (three MFMAs
    // of one row tile), where they issue while the matrix pipe works; with all conversions in front of the
    // MFMAs the waves of a block, which the barrier keeps in step, convert at the same time and multiply at the
    // same time, and the two units overlap for only a twentieth of the time.
    auto kblock = [&](int kb, int cur, u32x4 (&qa)[NT], uint32_t (&za)[ZR][NT], u32x4 (&qb)[NT],
                      uint32_t (&zb)[ZR][NT]) {
        const int kb2 = kb + 2 < kb1 ? kb + 2 : kb1 - 1;
        const int nxt = cur == 2 ? 0 : cur + 1;
        const u32x4* abuf = lds + cur * UNITS;
        const u32x4* nbuf = lds + nxt * UNITS;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) af1[mt] = abuf[a_rd[1] + mt * 128];
        __builtin_amdgcn_sched_barrier(0);
        // step 0: MFMAs with wopA, conversion of step 1 into wopB
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bitcast<v4i>(wopA[nt]), bitcast<v4i>(af0[mt]),
                                                                    acc[mt][nt], 0, 0, 0);
            if (mt < NP) conv_piece(wopB, qa, za, 1, mt);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int p = MT; p < NP; ++p) conv_piece(wopB, qa, za, 1, p);
        __builtin_amdgcn_sched_barrier(0);
        // step 1: MFMAs with wopB, conversion of the next k-block's step 0 into wopA
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (mt == BAR_MT) {
                // every fragment of this tile has been read (own LDS reads returned), and this wave's share of
                // tile kb + 1 has landed once at most the loads issued after it are in flight
                __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0) only
                wait_vmcnt<DPT + NW>();
                __syncthreads();
#pragma unroll
                for (int m2 = 0; m2 < MT; ++m2) af0[m2] = nbuf[a_rd[0] + m2 * 128];
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bitcast<v4i>(wopB[nt]), bitcast<v4i>(af1[mt]),
                                                                    acc[mt][nt], 0, 0, 0);
            if (mt < NP) conv_piece(wopA, qb, zb, 0, mt);
            __builtin_amdgcn_sched_barrier(0);
            if (mt == 0) {
                // Every register of the next k-block's weights is named here, so that the compiler places all
                // its waits for them in front of the loads issued now (they landed long ago); a wait placed
                // later would, in the compiler's count, which does not know of the direct loads, reach into the
                // loads just issued.  Set a is free.
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    asm volatile("" : : "v"(qb[nt][0]), "v"(qb[nt][1]), "v"(qb[nt][2]), "v"(qb[nt][3]));
#pragma unroll
                    for (int r = 0; r < ZR; ++r) asm volatile("" : : "v"(zb[r][nt]));
                }
                load_a_lds(kb2, cur >= 1 ? cur - 1 : 2);      // the tile read during kb - 1  (= (cur + 2) % 3)
                load_w(qa, za, kb2);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int p = MT; p < NP; ++p) conv_piece(wopA, qb, zb, 0, p);
        __builtin_amdgcn_sched_barrier(0);
    };

    if (kb0 < kb1) {
        const int kbn = kb0 + 1 < kb1 ? kb0 + 1 : kb1 - 1;
        // same issue order as inside the loop: A(kb), W(kb), A(kb + 1), W(kb + 1)
        load_a_lds(kb0, 0);
        load_w(wqs[0], zqs[0], kb0);
        load_a_lds(kbn, 1);
        load_w(wqs[1], zqs[1], kbn);
        wait_vmcnt<DPT + NW>();
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) af0[mt] = lds[a_rd[0] + mt * 128];
#pragma unroll
        for (int p = 0; p < NP; ++p) conv_piece(wopA, wqs[0], zqs[0], 0, p);
        int kb = kb0, cur = 0;
        for (; kb + 2 <= kb1; kb += 2) {
            kblock(kb, cur, wqs[0], zqs[0], wqs[1], zqs[1]);
            cur = cur == 2 ? 0 : cur + 1;
            kblock(kb + 1, cur, wqs[1], zqs[1], wqs[0], zqs[0]);
            cur = cur == 2 ? 0 : cur + 1;
        }
        if (kb < kb1) kblock(kb, cur, wqs[0], zqs[0], wqs[1], zqs[1]);
        // the last (redundant) direct loads still target this block's LDS
        wait_vmcnt<0>();
    }

    float tn[NT][4];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            tn[nt][i] = tvalid[nt] ? f16_bits_to_float(tstep[(int64_t)(tile0 + nt) * FQ_NTILE + j * 4 + i]) : 0.0f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int row = mt * 16 + ml;
        if (row >= rows) continue;
        const float am = alpha[row0 + row];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (!tvalid[nt]) continue;
            const int64_t at = (row0 + row) * (int64_t)N + (int64_t)(tile0 + nt) * FQ_NTILE + j * 4;
            if (splits == 1) {
                w8_store4<OUT>(C + at, acc[mt][nt], am, tn[nt]);
            } else {
                *reinterpret_cast<v4i*>(partial + (int64_t)split * M * N + at) = acc[mt][nt];
            }
        }
    }
}


// ------------------------------------------------------------------------------------------------------
// Small-M kernel of the integer path (M <= 16), bound by the HBM read of the weights like its floating-point
// counterpart (fq_gemm_skinny_kernel), whose structure it takes: one block per compute unit and all blocks
// resident at once; a block is GP column groups x KW k-workers (run-time values), wave (gi, kw) owns NT
// column tiles and, in iteration `it`, k-block (sb * KW + kw) of super-block sb; codes and multipliers stream
// through a DEPTH-deep register ring per wave and never touch LDS; the int8 activation slice of a super-block
// (M rows x KW k-blocks of 128 bytes) is fetched once per block, DEPTH iterations ahead, through the same ring
// into one of two LDS buffers; one barrier per iteration; the k-workers' int32 sums are added through LDS
// (integer sums: exact in any order) and scaled by alpha[m] * t[n], or written as int32 slabs when K is
// also split over the grid (w8_finalize_kernel adds and scales those).
// ------------------------------------------------------------------------------------------------------
constexpr int W8S_PITCH = 17;      // LDS row pitch of the activation buffer in 16-byte units (16 rows + 1 pad)
constexpr int W8S_KC = 8;          // 16-byte activation units per row and k-block

// the end of a block of `cols` columns, the bx-th of its rows, where K is split over the grid (fq_split_sum.h; partial, alpha
// and C at the block's row 0)
template <int OUT>
__device__ __forceinline__ void w8_finish_splits(void* lds, const int32_t* partial, int64_t stride, int splits, const float* alpha,
                                                 const uint16_t* tstep, uint16_t* C, int rows, int N, int bx, int cols, uint64_t tag) {
    finish_split_sums<v4i>(lds, partial, stride, splits, C, rows, N, bx * cols, cols, tag, [&](int m, int n, const v4i& v) {
        float tn[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) tn[i] = f16_bits_to_float(tstep[n + i]);
        w8_store4<OUT>(C + (int64_t)m * N + n, v, alpha[m], tn);
    });
}

template <int NT, int ZR, int AU>
struct W8Stage {
    u32x4 wq[NT];
    uint32_t zq[ZR][NT];
    u32x4 areg[AU];
};

template <int NT, int DEPTH, int ZR, int MAXW, int AU, int OUT>
__global__ __launch_bounds__(MAXW * 64) void fq_w4a8_skinny_kernel(
    const int8_t* __restrict__ Aq, const float* __restrict__ alpha, const u32x4* __restrict__ codes,
    const uint8_t* __restrict__ z, const uint16_t* __restrict__ tstep, uint16_t* __restrict__ C,
    int32_t* __restrict__ partial, int M, int N, int K, uint32_t g32, uint32_t g32_recip, int gp, int kw_n,
    int grid_splits, uint64_t tag) {
    constexpr int KC = W8S_KC, PITCH = W8S_PITCH;
    typedef W8Stage<NT, ZR, AU> Stage;
    extern __shared__ u32x4 lds[];   // two activation buffers [kw_n * KC][PITCH]; later the reduction

    const int tid = threadIdx.x;
    const int nthreads = blockDim.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gi = wave / kw_n;
    const int kw = wave - gi * kw_n;
    const int ntiles = N / FQ_NTILE;
    const int ngroups = (ntiles + NT - 1) / NT;
    const int bgroups = (ngroups + gp - 1) / gp;      // blocks per grid split
    const int bx = blockIdx.x % bgroups;
    const int gsplit = blockIdx.x / bgroups;          // < grid_splits
    const int ng = bx * gp + gi;
    const bool gvalid = ng < ngroups;
    const int KB = K / 128;
    const int SB = (KB + kw_n - 1) / kw_n;            // super-blocks of kw_n k-blocks
    const int n_it = gsplit < SB ? (SB - gsplit + grid_splits - 1) / grid_splits : 0;   // block-uniform
    const int64_t kb_stride = (int64_t)ntiles * 64;   // records between consecutive k-blocks of a tile
    const int ml = lane & 15, j = lane >> 4;
    const int abuf_units = kw_n * KC * PITCH;

    const char* wbase[NT];
    const uint8_t* zbase[NT];
    bool tvalid[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int tile = ng * NT + nt;
        tvalid[nt] = gvalid && tile < ntiles;
        const int tc = tvalid[nt] ? tile : 0;
        wbase[nt] = reinterpret_cast<const char*>(codes + fq_rec(tc, 0, ntiles, 0));
        zbase[nt] = z + (int64_t)tc * FQ_NTILE + ml;
    }

    // cooperative activation fetch: unit u = tid + r * nthreads covers row u / upr, unit column u % upr of the
    // super-block (upr = kw_n * KC units of 16 int8 per row)
    const int upr = kw_n * KC;
    int a_row[AU], a_col[AU];
#pragma unroll
    for (int r = 0; r < AU; ++r) {
        const int u = tid + r * nthreads;
        a_row[r] = u / upr;
        a_col[r] = u - a_row[r] * upr;
    }

    v4i acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = v4i{0, 0, 0, 0};
    const u32x4 zero4 = {0u, 0u, 0u, 0u};

    auto load_act = [&](u32x4 (&areg)[AU], int it) {
        const int64_t k0 = (int64_t)(gsplit + it * grid_splits) * kw_n * 128;
#pragma unroll
        for (int r = 0; r < AU; ++r) {
            int64_t k = k0 + a_col[r] * 16;
            k = k < K ? k : K - 16;                      // past the end (tail super-block): never multiplied
            areg[r] = a_row[r] < M ? *reinterpret_cast<const u32x4*>(Aq + (int64_t)a_row[r] * K + k) : zero4;
        }
    };
    auto store_act = [&](const u32x4 (&areg)[AU], int buf) {
#pragma unroll
        for (int r = 0; r < AU; ++r)
            if (a_row[r] < 16) lds[buf * abuf_units + a_col[r] * PITCH + a_row[r]] = areg[r];
    };
    // stage `it`: this wave's codes and multipliers for iteration it, and the lane's share of the activations of
    // iteration it + 1
    auto load_stage = [&](Stage& sl, int it) {
        int kb = (gsplit + it * grid_splits) * kw_n + kw;
        kb = kb < KB ? kb : KB - 1;                      // tail super-block: idle workers re-read the last block
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) sl.wq[nt] = load_rec<4, true>(wbase[nt] + ((int64_t)kb * kb_stride + lane) * 16);
#pragma unroll
        for (int r = 0; r < ZR; ++r) {
            // group of the 32-row step at hand (ZR == 1: the k-block lies inside one group; else the group of this
            // lane's 16 rows of MFMA step r): an exact division by g / 32 as a multiplication by its rounded-up
            // reciprocal (valid while step * (g / 32) < 2^32)
            const uint32_t step = (uint32_t)kb * 4u + (ZR == 1 ? 0u : 2u * r + (uint32_t)(j >> 1));
            const uint32_t grp = g32 == 1 ? step : __umulhi(step, g32_recip);
            const int64_t zrow = (int64_t)grp * N;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) sl.zq[r][nt] = zbase[nt][zrow];
        }
        load_act(sl.areg, it + 1);
    };
    // one iteration: publish the next activations, read this iteration's fragments, convert and multiply
    auto iterate = [&](const Stage& sl, int it) {
        store_act(sl.areg, (it + 1) & 1);
        const int kb = (gsplit + it * grid_splits) * kw_n + kw;
        u32x4 af[2];
        const u32x4* abuf = lds + (it & 1) * abuf_units + (kw * KC + j) * PITCH + ml;
#pragma unroll
        for (int T = 0; T < 2; ++T) af[T] = abuf[T * 4 * PITCH];
        if (gvalid && kb < KB) {
#pragma unroll
            for (int T = 0; T < 2; ++T) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const uint32_t zi = sl.zq[ZR == 1 ? 0 : T][nt];
                    const uint32_t ci = (uint32_t)(0x8080 - (int)zi * 0x0808);   // 128 - 8 z in both bytes
                    const u16x2v zz = {(uint16_t)zi, (uint16_t)zi};
                    const u16x2v cc = {(uint16_t)ci, (uint16_t)ci};
                    u32x4 wop;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t w = sl.wq[nt][2 * T + h];
                        wop[2 * h] = w8_scale_bytes(w & 0x0f0f0f0fu, zz, cc);
                        wop[2 * h + 1] = w8_scale_bytes((w >> 4) & 0x0f0f0f0fu, zz, cc);
                    }
                    acc[nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bitcast<v4i>(wop), bitcast<v4i>(af[T]), acc[nt], 0, 0, 0);
                }
            }
        }
    };

    if (n_it > 0) {
        {   // activations of iteration 0
            u32x4 a0[AU];
            load_act(a0, 0);
            store_act(a0, 0);
        }
        Stage ring[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            if (d < n_it) load_stage(ring[d], d);
        __syncthreads();
        int it = 0;
        for (; it + 2 * DEPTH <= n_it; it += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                iterate(ring[d], it + d);
                load_stage(ring[d], it + d + DEPTH);
                __syncthreads();
            }
        }
        // drain: at most 2 * DEPTH - 1 iterations are left, the first min(DEPTH, left) already loaded
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (it + d < n_it) {
                iterate(ring[d], it + d);
                if (it + d + DEPTH < n_it) load_stage(ring[d], it + d + DEPTH);
                __syncthreads();
            }
        }
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d) {
            if (it + d + DEPTH < n_it) {
                iterate(ring[d], it + d + DEPTH);
                __syncthreads();
            }
        }
    }

    // the k-workers' sums of each column group, added by all threads of the block (one result quad each)
    auto store_quad = [&](const v4i& v, int group, int nt, int ln) {
        const int mq = ln & 15, jq = ln >> 4;
        const int tile = group * NT + nt;
        if (mq >= M || group >= ngroups || tile >= ntiles) return;
        const int64_t n = (int64_t)tile * FQ_NTILE + jq * 4;
        if (grid_splits == 1) {
            float tn[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) tn[i] = f16_bits_to_float(tstep[n + i]);
            w8_store4<OUT>(C + (int64_t)mq * N + n, v, alpha[mq], tn);
        } else {
            store_partial(partial + ((int64_t)gsplit * M + mq) * N + n, v, tag != 0);
        }
    };
    if (kw_n == 1) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) store_quad(acc[nt], ng, nt, lane);
        w8_finish_splits<OUT>(lds, partial, (int64_t)M * N, grid_splits, alpha, tstep, C, M, N, bx, gp * NT * FQ_NTILE, tag);
        return;
    }
    v4i* red = reinterpret_cast<v4i*>(lds);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) red[(wave * NT + nt) * 64 + lane] = acc[nt];
    __syncthreads();
    const int nquads = gp * NT * 64;
    for (int q = tid; q < nquads; q += nthreads) {
        const int gq = q / (NT * 64);            // column group of the block
        const int r = q - gq * (NT * 64);        // nt * 64 + lane inside the group
        const v4i* src = red + (int64_t)gq * kw_n * NT * 64 + r;   // worker w: + w * NT * 64
        v4i v = src[0];
#pragma unroll 4
        for (int w = 1; w < kw_n; ++w) v += src[w * NT * 64];
        store_quad(v, bx * gp + gq, r >> 6, r & 63);
    }
    w8_finish_splits<OUT>(lds, partial, (int64_t)M * N, grid_splits, alpha, tstep, C, M, N, bx, gp * NT * FQ_NTILE, tag);
}

// ------------------------------------------------------------------------------------------------------
// Mid-M kernel of the integer path: row blocks of 16 MT rows (MT = 2 .. 4), the structure of the floating-point
// fq_gemm_mid_kernel.  A block is GP column groups x KW k-workers (at most 12 waves); codes and multipliers stream through a
// register ring of W8M_DEPTH stages per wave, the int8 activations of a super-block (16 MT rows x KW k-blocks) go global -> LDS
// directly, two iterations ahead into one of three tiles, the k-workers' int32 sums are added through LDS (exact in any
// order).  Against the tiled kernel: K is split inside the block (no slabs through memory, no second kernel, unless the grid
// is split, too), and blocks of 48 GP columns cut a small output finer.  12288 x 36864, g = 128, tiled kernel ->
// this one, us: M = 17 55 -> 40 (5.9 TB/s of weights), M = 32 55 -> 41, M = 64 66 -> 46; 8192 x 8192, M = 128 30 -> 24.
// ------------------------------------------------------------------------------------------------------
constexpr int W8M_DEPTH = 3, W8M_MAXW = 12;

template <int NT, int ZR>
struct W8MStage {
    u32x4 wq[NT];
    uint32_t zq[ZR][NT];
};

template <int NT, int MT, int ZR, int OUT>
__global__ __launch_bounds__(W8M_MAXW * 64) void fq_w4a8_mid_kernel(
    const int8_t* __restrict__ Aq, const float* __restrict__ alpha, const u32x4* __restrict__ codes,
    const uint8_t* __restrict__ z, const uint16_t* __restrict__ tstep, uint16_t* __restrict__ C,
    int32_t* __restrict__ partial, int M, int N, int K, uint32_t g32, uint32_t g32_recip, int gp, int kw_n, int nblocks_m,
    int grid_splits, uint64_t tag) {
    constexpr int DEPTH = W8M_DEPTH;
    constexpr int TILE = 16 * MT * 8;               // 16-byte units of one k-worker's activation tile
    constexpr int NI = TILE / 64;                   // wave-level direct loads of such a tile
    constexpr int NW = NT + ZR * NT;                // vector loads of one stage
    static_assert((DEPTH - 1) * NW < 64, "wait counter range");
    typedef W8MStage<NT, ZR> Stage;
    extern __shared__ u32x4 lds[];   // three activation buffers [kw_n][TILE]; later the reduction

    const int tid = threadIdx.x;
    const int nthreads = blockDim.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gi = wave / kw_n;
    const int kw = wave - gi * kw_n;
    const int ntiles = N / FQ_NTILE;
    const int ngroups = (ntiles + NT - 1) / NT;
    const int bgroups = (ngroups + gp - 1) / gp;      // column blocks
    // (the row blocks of a column block lie next to each other: they read the same weights)
    const int bx = (blockIdx.x / nblocks_m) % bgroups;
    const int gsplit = blockIdx.x / (bgroups * nblocks_m);   // < grid_splits
    const int row0 = (blockIdx.x % nblocks_m) * (16 * MT);
    const int rows = M - row0 < 16 * MT ? M - row0 : 16 * MT;
    const int ng = bx * gp + gi;
    const bool gvalid = ng < ngroups;
    const int KB = K / 128;
    const int SB = (KB + kw_n - 1) / kw_n;            // super-blocks of kw_n k-blocks
    const int n_it = gsplit < SB ? (SB - gsplit + grid_splits - 1) / grid_splits : 0;   // block-uniform
    const int64_t kb_stride = (int64_t)ntiles * 64;   // records between consecutive k-blocks of a tile
    const int ml = lane & 15, j = lane >> 4;
    const int abuf_units = kw_n * TILE;
    Aq += (int64_t)row0 * K;
    alpha += row0;
    C += (int64_t)row0 * N;

    const char* wbase[NT];
    const uint8_t* zbase[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int tile = ng * NT + nt;
        const int tc = gvalid && tile < ntiles ? tile : 0;
        wbase[nt] = reinterpret_cast<const char*>(codes + fq_rec(tc, 0, ntiles, 0));
        zbase[nt] = z + (int64_t)tc * FQ_NTILE;
    }
    const uint32_t lane_rec = (uint32_t)lane * 16u;

    // activations of iteration `it`: this wave's share (every gp-th load) of its k-worker's tile.  Unit (row, position) holds
    // the row's 16-byte unit position ^ (row & 7); rows past the end repeat the last one (never stored).
    auto load_act = [&](int it) {
        const int kb = (gsplit + it * grid_splits) * kw_n + kw;
        const int8_t* base = Aq + (int64_t)(kb < KB ? kb : KB - 1) * 128;   // past the end: never multiplied
        const uint32_t lds_tile = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(
            lds + (it % 3) * abuf_units + kw * TILE);
        for (int i = gi; i < NI; i += gp) {
            const int row = i * 8 + (lane >> 3), pos = lane & 7;
            const int rowc = row < rows ? row : rows - 1;
            const int8_t* src = base + (int64_t)rowc * K + 16 * (pos ^ (row & 7));
            load_lds16(__builtin_amdgcn_readfirstlane(lds_tile + i * 1024), src);
        }
    };
    auto load_stage = [&](Stage& sl, int it) {
        int kb = (gsplit + it * grid_splits) * kw_n + kw;
        kb = kb < KB ? kb : KB - 1;                      // tail super-block: idle workers re-read the last block
        const int64_t kb_bytes = (int64_t)kb * kb_stride * 16;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) sl.wq[nt] = load_rec<4, true>(scalar_ptr(wbase[nt] + kb_bytes) + lane_rec);
#pragma unroll
        for (int r = 0; r < ZR; ++r) {
            // group of the 32-row step at hand (ZR == 1: the k-block lies inside one group; else the group of this lane's 16
            // rows of MFMA step r), by the rounded-up reciprocal as in the small-M kernel
            const uint32_t step = (uint32_t)kb * 4u + (ZR == 1 ? 0u : 2u * r + (uint32_t)(j >> 1));
            const uint32_t grp = g32 == 1 ? step : __umulhi(step, g32_recip);
            const int64_t zrow = (int64_t)grp * N;
            if constexpr (ZR == 1) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) sl.zq[r][nt] = scalar_ptr(zbase[nt] + zrow)[(uint32_t)ml];
            } else {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) sl.zq[r][nt] = zbase[nt][zrow + ml];
            }
        }
    };
    int a_rd[2];
#pragma unroll
    for (int T = 0; T < 2; ++T) a_rd[T] = kw * TILE + ml * 8 + ((4 * T + j) ^ (ml & 7));

    v4i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = v4i{0, 0, 0, 0};

    auto multiply = [&](const Stage& sl, int it) {
        const u32x4* abuf = lds + (it % 3) * abuf_units;
        u32x4 af[2][MT];
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) af[T][mt] = abuf[a_rd[T] + mt * 128];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                const uint32_t zi = sl.zq[ZR == 1 ? 0 : T][nt];
                const uint32_t ci = (uint32_t)(0x8080 - (int)zi * 0x0808);   // 128 - 8 z in both bytes
                const u16x2v zz = {(uint16_t)zi, (uint16_t)zi};
                const u16x2v cc = {(uint16_t)ci, (uint16_t)ci};
                u32x4 wop;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t w = sl.wq[nt][2 * T + h];
                    wop[2 * h] = w8_scale_bytes(w & 0x0f0f0f0fu, zz, cc);
                    wop[2 * h + 1] = w8_scale_bytes((w >> 4) & 0x0f0f0f0fu, zz, cc);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bitcast<v4i>(wop), bitcast<v4i>(af[T][mt]), acc[mt][nt], 0, 0, 0);
            }
        }
    };
    // Iteration `it`.  On entry its activations and weights have landed; in flight: weights of it + 1, it + 2, activations of
    // it + 1.
    auto iterate = [&](Stage& sl, int it, bool more) {
        // (every register of the stage is named here, so that the compiler places its waits for them in front of the
        // loads issued below: in its count, which does not know of the direct loads, a later wait would reach into them)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            asm volatile("" : "+v"(sl.wq[nt][0]), "+v"(sl.wq[nt][1]), "+v"(sl.wq[nt][2]), "+v"(sl.wq[nt][3]));
#pragma unroll
            for (int r = 0; r < ZR; ++r) asm volatile("" : "+v"(sl.zq[r][nt]));
        }
        if (it + 2 < n_it) load_act(it + 2);             // into the tile read during it - 1
        __builtin_amdgcn_sched_barrier(0);
        if (gvalid && (gsplit + it * grid_splits) * kw_n + kw < KB) multiply(sl, it);
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            load_stage(sl, it + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
            // the activations of it + 1 have landed: younger than they are the weights issued at the end of this iteration and
            // the one before, and this wave's share of the activations of it + 2 (left out of the count: it differs per wave)
            wait_vmcnt<2 * NW>();
        } else {
            wait_vmcnt<0>();
        }
        __syncthreads();
    };

    if (n_it > 0) {
        Stage ring[DEPTH];
        load_act(0);
        load_stage(ring[0], 0);
        if (1 < n_it) load_act(1);
#pragma unroll
        for (int d = 1; d < DEPTH; ++d)
            if (d < n_it) load_stage(ring[d], d);
        __builtin_amdgcn_sched_barrier(0);
        if (DEPTH <= n_it) wait_vmcnt<(DEPTH - 1) * NW>();     // (the loads younger than the activations of 0, at least)
        else wait_vmcnt<0>();
        __syncthreads();
        int it = 0;
        for (; it + 2 * DEPTH <= n_it; it += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) iterate(ring[d], it + d, true);
        }
        // drain: at most 2 * DEPTH - 1 iterations are left, the first min(DEPTH, left) already loaded
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            if (it + d < n_it) iterate(ring[d], it + d, it + d + DEPTH < n_it);
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d)
            if (it + d + DEPTH < n_it) iterate(ring[d], it + d + DEPTH, false);
    }

    auto store_quad = [&](const v4i& v, int group, int mt, int nt, int ln) {
        const int mq = mt * 16 + (ln & 15), jq = ln >> 4;
        const int tile = group * NT + nt;
        if (mq >= rows || group >= ngroups || tile >= ntiles) return;
        const int64_t n = (int64_t)tile * FQ_NTILE + jq * 4;
        if (grid_splits == 1) {
            float tn[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) tn[i] = f16_bits_to_float(tstep[n + i]);
            w8_store4<OUT>(C + (int64_t)mq * N + n, v, alpha[mq], tn);
        } else {
            store_partial(partial + ((int64_t)gsplit * M + row0 + mq) * N + n, v, tag != 0);
        }
    };
    if (kw_n == 1) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) store_quad(acc[mt][nt], ng, mt, nt, lane);
        w8_finish_splits<OUT>(lds, partial + (int64_t)row0 * N, (int64_t)M * N, grid_splits, alpha, tstep, C, rows, N, bx,
                              gp * NT * FQ_NTILE, tag);
        return;
    }
    // the k-workers' sums of each column group, added by all threads of the block (one result quad each)
    constexpr int Q = MT * NT * 64;                // result quads of a column group
    v4i* red = reinterpret_cast<v4i*>(lds);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) red[wave * Q + (mt * NT + nt) * 64 + lane] = acc[mt][nt];
    __syncthreads();
    for (int q = tid; q < gp * Q; q += nthreads) {
        const int gq = q / Q;                      // column group of the block
        const int r = q - gq * Q;
        const v4i* src = red + gq * kw_n * Q + r;
        v4i v = src[0];
#pragma unroll 4
        for (int w = 1; w < kw_n; ++w) v += src[w * Q];
        const int tl = r >> 6;
        store_quad(v, bx * gp + gq, tl / NT, tl % NT, r & 63);
    }
    w8_finish_splits<OUT>(lds, partial + (int64_t)row0 * N, (int64_t)M * N, grid_splits, alpha, tstep, C, rows, N, bx,
                          gp * NT * FQ_NTILE, tag);
}

template <int OUT>
__global__ __launch_bounds__(256) void w8_finalize_kernel(const int32_t* __restrict__ S, int splits,
                                                           const float* __restrict__ alpha,
                                                           const uint16_t* __restrict__ tstep, int64_t M, int64_t N,
                                                           uint16_t* __restrict__ C) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= M * N) return;
    const int64_t m = i / N, n = i - m * N;                  // N is a multiple of 16: the four share a row
    v4i s = *reinterpret_cast<const v4i*>(S + i);
    for (int k = 1; k < splits; ++k) s += *reinterpret_cast<const v4i*>(S + (int64_t)k * M * N + i);
    float tn[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) tn[k] = f16_bits_to_float(tstep[n + k]);
    w8_store4<OUT>(C + i, s, alpha[m], tn);
}

struct w8_plan {
    int mt, splits, kb_per_split, nblocks_n, nblocks_m;
    int small, gp, kw, au;      // small-M kernel (M <= 16): column groups x k-workers per block, activation units per lane
    int mid;                    // mid-M kernel (gp, kw as above, mt row tiles per block)
    int nt;                     // column tiles per wave of either: 3 or 1
};

constexpr int W8S_NT = 3, W8S_MAXW = 12;   // the small-M kernel (and NT = 1)
// ring depth: three stages where the registers allow it without spills (one multiplier row per k-block and one
// activation unit per lane: 164 registers; measured 4 - 6 % faster than two on the OPT-175B shapes), else two
constexpr int w8s_depth(int zr, int au) { return zr == 1 && au == 1 ? 3 : 2; }

constexpr size_t w8m_lds(int nt, int mt, int gp, int kw) {
    const size_t act = (size_t)3 * kw * mt * 16 * 8 * 16, red = (size_t)gp * kw * mt * nt * 64 * 16;
    return act > red ? act : red;
}

// 1 .. 16 rows, by how full a shape leaves the chip.  One block per compute unit, all resident at once: evenness of the fill
// squared, bytes in flight per compute unit up to 64 KiB; a second round of blocks, a split of K over the grid and lone
// k-workers cost.
w8_plan w8_plan_small_by_fill(int64_t M, int64_t N, int64_t K) {
    w8_plan p = {};
    const int ncu = fq_cu_count();
    const int KB = (int)(K / 128);
    const int ngroups = (int)((N / FQ_NTILE + W8S_NT - 1) / W8S_NT);
    p.small = 1;
    p.mt = 1;
    p.nt = W8S_NT;
    p.nblocks_m = 1;
    double best = -1.0;
    for (int gp = 1; gp <= W8S_MAXW; ++gp) {
        int kw = W8S_MAXW / gp;
        if (kw > KB) kw = KB;
        const int need = (int)M * W8S_KC;
        const int au = need <= 64 * gp ? 1 : (need <= 128 * gp ? 2 : 0);
        if (au == 0 || kw < 1) continue;
        const int64_t blocks = (ngroups + gp - 1) / gp;
        const int SB = (KB + kw - 1) / kw;
        int gs = 1;
        if (blocks <= ncu / 2) gs = (int)(ncu / blocks);
        if (gs > 8) gs = 8;
        if (gs > SB) gs = SB;
        const int64_t grid = blocks * gs;
        const int64_t rounds = (grid + ncu - 1) / ncu;
        const double eff = (double)ngroups * gs / (double)(rounds * ncu * gp);
        const double inflight = (double)(gp * kw) * W8S_NT * 2;   // KiB (with the shallower ring)
        double score = eff * eff * (inflight >= 64.0 ? 1.0 : sqrt(inflight / 64.0));
        score /= 1.0 + 0.1 * (double)(rounds - 1);
        if (au == 2) score *= 0.8;
        if (gs > 1) score *= 0.8;
        if (gp * kw < 6) score *= 0.85;
        if (kw == 1) score *= 0.95;
        if (score > best + 1e-9) {
            best = score;
            p.gp = gp;
            p.kw = kw;
            p.au = au;
            p.splits = gs;
            p.nblocks_n = (int)blocks;
        }
    }
    return p;
}

// 17 rows and more: the splits of K that give tiles of 32, 64 or 128 rows x 384 columns at least 192 blocks.
int w8_splits_by_fill(int64_t M, int64_t N, int64_t K) {
    const int64_t rows = M <= 32 ? 32 : (M <= 64 ? 64 : 128), cols = W8_WAVES * W8_NT * FQ_NTILE;
    const int64_t tiles = ((M + rows - 1) / rows) * ((N + cols - 1) / cols);
    const int KB = (int)(K / 128);
    int splits = tiles < 192 ? (int)(256 / tiles) : 1;
    if (splits > 8) splits = 8;
    if (splits > KB) splits = KB;
    const int kbs = (KB + splits - 1) / splits;
    return (KB + kbs - 1) / kbs;
}

// Waves of 16 columns instead of 48 (p.nt = 1), without a split of K, in place of a plan of the small-M or mid-M kernel: on narrow
// matrices 48 columns leave half the chip idle, 16 fill it in one round of blocks.  Both widths are weighed by models of their
// own (not the plan's: fitted together, of log time, rms error 6 % up to 16 rows and 10 % above, to 150 problems each of 1024 ..
// 16000 columns in 20 shapes): a block takes its start and end, and per iteration a latency, its waves' vector and matrix work
// and memory traffic, which add up.  The narrow waves have to win by 7 % (15 % in place of a split) up to 16 rows; above, by
// 10 % (15 % above 64 rows), up to 8192 columns (8704 columns, 30 rows 6.8 -> 7.4 us) and not in place of a split (the models rank
// those worse).  Scratch only shrinks.  Those problems: 1.08x on average up to 16 rows (65 change, one 3 % slower), 1.06x above.
double w8_width_us(const w8_plan& p, int64_t M, int64_t N, int KB, int zr, int ncu) {
    // work per iteration of twelve waves, more per row tile beyond two, for a second row of multipliers, for a second
    // activation unit; latency; a block beside it, a second one on the compute unit; ragged end
    static const double c[4][8] = {{0.476, 0.0, 0.109, 0.361, 0.026, 4.12, 1.18, 0.0}, {1.025, 0.0, 0.142, 0.236, 0.001, 4.58, 10.0, 0.21},
                                   {0.028, 0.081, 0.170, 0.0, 0.392, 5.58, 2.53, 0.41}, {0.482, 0.146, 0.272, 0.0, 0.321, 7.37, 9.14, 0.56}};
    const double* x = c[2 * p.mid + (p.nt == 1 ? 0 : 1)];
    const int waves = p.gp * p.kw, SB = (KB + p.kw - 1) / p.kw, n_it = (SB + p.splits - 1) / p.splits;
    const size_t act = (size_t)2 * p.kw * W8S_KC * W8S_PITCH * 16, red = (size_t)waves * p.nt * 1024;
    const size_t lds = p.mid ? w8m_lds(p.nt, p.mt, p.gp, p.kw) : (act > red ? act : red);
    int resident = (int)(160 * 1024 / lds);
    resident = resident < 24 / waves ? resident : 24 / waves;
    const double slots = (double)ncu * (resident > 1 ? resident : 1), blocks = (double)p.nblocks_n * p.nblocks_m * p.splits;
    const double at_once = blocks < slots ? blocks : slots, together = at_once > ncu ? at_once / ncu : 1.0;
    const double work = x[0] + (p.mid ? x[1] * (p.mt - 2) : x[3] * (p.au - 1)) + x[2] * (zr - 1);
    const double bytes = waves * p.nt * (1024.0 + 16.0 * zr) + (p.mid ? 0.0 : (double)M * p.kw * 128.0);
    double t = x[5] + x[6] * (together - 1.0) +
               n_it * (x[4] + work * ((waves + 3) / 4) * together * (1.0 / 3.0) + at_once * bytes * (p.mid ? 1.0 / 18.6e6 : 1.0 / 27e6));
    if (blocks > slots) {
        const double full = ceil(blocks / slots), part = blocks / slots + x[7];
        t *= part < full ? part : full;
    }
    if (p.splits > 1) t += (p.mid ? 1.9 : 1.4) + 2.0 * p.splits * (double)M * (double)N * (p.mid ? 4.0 / 7e6 : 4.0 / 1.62e6);
    return t;
}

w8_plan w8_narrow(const w8_plan& wide, int64_t M, int64_t N, int64_t K, int g) {
    if (wide.mid ? N > 8192 || wide.splits > 1 : !wide.small) return wide;
    const int ncu = fq_cu_count(), KB = (int)(K / 128), zr = g % 128 == 0 ? 1 : 2, ntiles = (int)(N / FQ_NTILE);
    const double margin = wide.mid ? (M > 64 ? 0.85 : 0.90) : (wide.splits > 1 ? 0.85 : 0.93);
    double best = margin * w8_width_us(wide, M, N, KB, zr, ncu);
    w8_plan chosen = wide;
    static const int groups[6] = {1, 2, 3, 4, 6, 12}, tiles[2] = {3, 4};
    for (int m = 0; m < 2; ++m) {
        w8_plan p = wide;
        p.nt = 1;
        p.splits = 1;
        if (M > 64) {                                   // 48 and 64 rows per block
            p.mt = tiles[m];
            p.nblocks_m = (int)((M + p.mt * 16 - 1) / (p.mt * 16));
        } else if (m > 0) {
            break;
        }
        const int fit = p.mid ? (int)(160 * 1024 / w8m_lds(1, p.mt, 1, 1)) : 12;
        for (const int gp : groups) {
            const int need = (int)M * W8S_KC;
            p.gp = gp;
            p.kw = 12 / gp < fit ? 12 / gp : fit;
            if (p.kw > KB) p.kw = KB;
            p.au = p.mid ? 0 : (need <= 64 * gp ? 1 : (need <= 128 * gp ? 2 : 0));
            p.nblocks_n = (ntiles + gp - 1) / gp;
            if ((!p.mid && p.au == 0) || (int64_t)p.nblocks_n * p.nblocks_m > ncu) continue;
            const double t = w8_width_us(p, M, N, KB, zr, ncu);
            if (t < best) {
                best = t;
                chosen = p;
            }
        }
    }
    return chosen;
}

// The plan with the least time by the models below.  None splits K into more slabs than filling the chip alone would take
// (the two functions above): fq_gemm_w4a8_workspace_bytes named those slabs before there were models, and a call for which
// a workspace of that size, or none, was enough must not be refused.  Without that limit the models ask for more in 0.4 % of
// shapes (470 rows, 14848 x 15296: 86 MB instead of none).
w8_plan w8_plan_wide(int64_t M, int64_t N, int64_t K, int g) {
    const int ncu = fq_cu_count();
    const double share = 1.0 / ncu;
    const int ntiles = (int)(N / FQ_NTILE);
    const int KB = (int)(K / 128);
    const int zr = g % 128 == 0 ? 1 : 2;
    if (M <= 16) {
        // The block shape and split of K with the least time by a model fitted (of log time, rms error 5 %) to 80 problems of
        // 1 .. 16 rows in 20 shapes each: a block takes 4.4 us and per iteration 0.98 us (0.2 more with two activation units
        // per lane) and its memory traffic at 15 TB/s (a part of it is hidden behind the rest); a split of K 2.1 us for the
        // second kernel that added it then (3.1 below 10 us; fq_split_sum.h adds most of them now) and the slabs' traffic.  Against
        // the plan by fill: 0.92 of the time inside graphs (1024 x 19872, 2 rows 9.0 -> 6.7 us; 9 of 10 shapes that were
        // split and are not any more lose a launch, too).  Up to 64 column tiles, a quarter of the compute units, the plan by
        // fill stays, which splits such matrices: the scratch that is asked for follows the plan, and tests take these to ask for some.
        w8_plan p = w8_plan_small_by_fill(M, N, K);
        if (4 * ntiles <= ncu) return p;
        const int ngroups = (ntiles + W8S_NT - 1) / W8S_NT;
        const int most = p.splits;
        double best = 1e30;
        for (int gp = 1; gp <= W8S_MAXW; ++gp) {
            int kw = W8S_MAXW / gp;
            if (kw > KB) kw = KB;
            const int need = (int)M * W8S_KC;
            const int au = need <= 64 * gp ? 1 : (need <= 128 * gp ? 2 : 0);
            if (au == 0 || kw < 1) continue;
            const int blocks = (ngroups + gp - 1) / gp, SB = (KB + kw - 1) / kw;
            const double bytes = gp * kw * (3072.0 + 48.0 * zr) + 64.0 * (double)M * kw, per_it = au == 2 ? 1.18 : 0.98;
            for (int gs = 1; gs <= most && gs <= SB; ++gs) {
                const int grid = blocks * gs;
                if (gs > 1 && grid > 330) break;
                const int n_it = (SB + gs - 1) / gs;
                if (4.4 + n_it * per_it > best) continue;
                double t = 4.4 + n_it * ((grid < ncu ? grid : ncu) * bytes * (1.0 / 15.2e6) + per_it);
                if (grid > ncu) {
                    const double full = (double)((grid + ncu - 1) / ncu), part = grid * share + 0.35;
                    t *= part < full ? part : full;
                }
                if (gs > 1) t += (t < 10.0 ? 3.1 : 2.1) + 2.0 * gs * (double)M * (double)N * (4.0 / 3.2e6);
                if (t < best - 1e-9) {
                    best = t;
                    p.gp = gp;
                    p.kw = kw;
                    p.au = au;
                    p.splits = gs;
                    p.nblocks_n = (int)blocks;
                }
            }
        }
        return p;
    }
    w8_plan p = {};
    // More rows: the mid-M kernel (32, 48 or 64 rows per block) or the tiled one (64 or 128), whichever shape and split of K the
    // model gives the least time; above 700 rows the mid-M kernel up to K = 10240 (and 12288 rows): narrow matrices make few
    // tiles of 128 x 384 (823 rows of 1408 x 1552: 35).  240 products of 701 .. 2048 rows, the tiled kernel alone -> both:
    // 1.10x on average, up to 1.9x (883 rows, 1664 x 1248 24 -> 13 us), none more than 3 % slower below that K, three of 15 above
    // (10 % at worst).  With waves of 16 columns, each side timed first once: 600 of 701 .. 2048 rows with up to 6400 columns 1.16x,
    // three more than 3 % slower (7 % at worst: 718 rows, 9600 x 2160); 760 of 2049 .. 12288 rows 1.08x, five slower (2480 rows, 5760 x
    // 1248 39.4 -> 47.1 us, 9550 rows, 3328 x 304 28.9 -> 35.3).  All but one of those are split on the tiled kernel, which takes 35 - 46 MB
    // of scratch that is not asked for any more; the shape by whole rounds changed 3 of 600 plans (1.001x).  The model was fitted (of log time, rms error 10 %) to 123 problems of
    // 17 .. 2048 rows, K from 1152 to 16256, N from 1168 to 45856, in 35 shapes each:
    //   a block     mid-M: 6.7 us + iterations * the longest of 0.94 us, its vector and matrix work (0.92, 1.09 or 1.27 us for
    //               twelve waves, 0.37 more with two multiplier rows per k-block), its memory traffic at 8.1 TB/s;
    //               tiled: 6.5 us + k-blocks * 0.80 or 1.18 us
    //   the launch  blocks per compute unit and 0.47 for the ragged end, at most whole rounds, at least one
    //   a split     2.5 us for the second kernel that added it then and the slabs' traffic at 5 TB/s
    // Against the tiled kernel alone (32, 64 or 128 rows, K split until 192 tiles): 0.76 of the time on average inside
    // graphs, never more than 3 % slower; 204 others, called one after the other: 1.38x faster on average, 10 more than 3 % slower
    // (14 % at worst: K of 10000 and more, or fewer splits than the former rule's); 12288 x 36864 us: M = 17 55 -> 40, M = 64 66 -> 46; 2816 x 5184, M = 95 22 -> 10.
    const int ngroups = (ntiles + 2) / 3;
    const int most = w8_splits_by_fill(M, N, K);
    double best = 1e30;
    auto launch_us = [&](int64_t blocks, double block_us, int splits) {
        double t = block_us;
        if (blocks > ncu) {
            const double full = (double)((blocks + ncu - 1) / ncu), part = blocks * share + 0.47;
            t *= part < full ? part : full;
        }
        if (splits > 1) t += 2.5 + 2.0 * splits * (double)M * (double)N * (4.0 / 5e6);
        return t;
    };
    static const double mid_work[5] = {0.0, 0.0, 0.92, 1.09, 1.27};
    static const int groups[6] = {1, 2, 3, 4, 6, 12};
    const int mt_low = M <= 32 ? 2 : 3, mt_high = M <= 32 ? 2 : (M <= 48 ? 3 : 4);
    for (int mt = M > 48 && M <= 64 ? 4 : mt_low; (M <= 700 || (M <= 12288 && K <= 10240)) && mt <= mt_high; ++mt) {
        const int nblocks_m = (int)((M + mt * 16 - 1) / (mt * 16));
        const int fit = (int)(160 * 1024 / w8m_lds(3, mt, 1, 1));
        for (const int gp : groups) {
            int kw = W8M_MAXW / gp;
            kw = kw < fit ? kw : fit;
            kw = kw < KB ? kw : KB;
            const int nblocks_n = (ngroups + gp - 1) / gp;
            const int SB = (KB + kw - 1) / kw;
            const double work = (mid_work[mt] + 0.37 * (zr - 1)) * (1.0 / 3.0) * (double)((gp * kw + 3) / 4);
            for (int gs = 1; gs <= 4 && gs <= most && gs <= SB; gs *= 2) {
                const int64_t blocks = (int64_t)nblocks_n * nblocks_m * gs;
                if (gs > 1 && blocks > 300) break;
                const int n_it = (SB + gs - 1) / gs;
                if (6.7 + n_it * 0.94 > best) continue;
                const double mem = (double)(blocks < ncu ? blocks : ncu) * (gp * kw * (3072.0 + 48.0 * zr) + 0.3 * kw * mt * 2048.0) * (1.0 / 8.1e6);
                double t_it = work > mem ? work : mem;
                if (t_it < 0.94) t_it = 0.94;
                const double t = launch_us(blocks, 6.7 + n_it * t_it, gs);
                if (t < best - 1e-9) {
                    best = t;
                    p.mid = 1;
                    p.nt = 3;
                    p.mt = mt;
                    p.gp = gp;
                    p.kw = kw;
                    p.splits = gs;
                    p.nblocks_n = nblocks_n;
                    p.nblocks_m = nblocks_m;
                }
            }
        }
    }
    static const int split_opts[6] = {1, 2, 3, 4, 6, 8};
    for (int mt = M > 32 && M <= 600 ? 4 : 8; mt <= 8; mt += 4) {
        if (mt == 8 && M <= 64) break;
        const int nblocks_n = (ntiles + W8_WAVES * W8_NT - 1) / (W8_WAVES * W8_NT);
        const int nblocks_m = (int)((M + mt * 16 - 1) / (mt * 16));
        const int64_t tiles = (int64_t)nblocks_n * nblocks_m;
        for (int splits : split_opts) {
            if (splits > KB || splits > most || (splits > 1 && tiles * splits > 600)) break;
            const int kbs = (KB + splits - 1) / splits;
            splits = (KB + kbs - 1) / kbs;
            const double t = launch_us(tiles * splits, 6.5 + kbs * ((mt == 8 ? 1.18 : 0.80) + 0.03 * (zr - 1)), splits);
            if (t < best - 1e-9) {
                best = t;
                p.mid = 0;
                p.mt = mt;
                p.splits = splits;
                p.kb_per_split = kbs;
                p.nblocks_n = nblocks_n;
                p.nblocks_m = nblocks_m;
            }
        }
    }
    return p;
}

// (Up to 16 rows matrices of up to 64 column tiles keep their plan, and with it the scratch that they ask for.)
w8_plan w8_plan_of(int64_t M, int64_t N, int64_t K, int g) {
    const w8_plan p = w8_plan_wide(M, N, K, g);
    return M <= 16 && 4 * (N / FQ_NTILE) <= fq_cu_count() ? p : w8_narrow(p, M, N, K, g);
}

size_t w8_partial_bytes(const w8_plan& p, int64_t M, int64_t N) {
    return p.splits > 1 ? (size_t)p.splits * (size_t)M * (size_t)N * sizeof(int32_t) : 0;
}

int w8_check(int64_t K, int64_t N, int group_size, int* g_eff) {
    if (K <= 0 || N <= 0 || group_size < 0) return FQ_ERR_INVALID_ARG;
    const int64_t g = group_size == 0 ? K : (int64_t)group_size;
    if (g > K || K % g != 0) return FQ_ERR_INVALID_ARG;
    // K <= 131072 keeps every sum inside an int32: K * 127 * 112 < 2^31
    if (K > 131072 || N > (int64_t)1 << 24 || N % FQ_NTILE != 0 || K % 128 != 0 || g % 32 != 0) return FQ_ERR_UNSUPPORTED;
    *g_eff = (int)g;
    return FQ_OK;
}

template <int MT, int OUT>
void w8_launch(const w8_plan& p, int g, const int8_t* Aq, const float* alpha, const void* codes, const uint8_t* z,
               const void* tstep, void* C, int32_t* partial, int64_t M, int64_t N, int64_t K, hipStream_t stream) {
    const dim3 grid((unsigned)((int64_t)p.nblocks_n * p.nblocks_m * p.splits));
    const size_t lds = (size_t)3 * MT * 16 * 8 * 16;
    const int zr = g % 128 == 0 ? 1 : 2;
#define W8_GO(ZR_)                                                                                              \
    hipLaunchKernelGGL((fq_gemm_w4a8_kernel<MT, ZR_, OUT>), grid, dim3(W8_WAVES * 64), lds, stream, Aq, alpha,   \
                       (const u32x4*)codes, z, (const uint16_t*)tstep, (uint16_t*)C, partial, (int)M, (int)N,    \
                       (int)K, g, p.kb_per_split, p.splits, p.nblocks_n, p.nblocks_m)
    if (zr == 1) W8_GO(1);
    else W8_GO(2);
#undef W8_GO
}

template <int OUT, int NT, int ZR, int AU>
int w8_launch_small(const w8_plan& p, int g, const int8_t* Aq, const float* alpha, const void* codes, const uint8_t* z,
                    const void* tstep, void* C, int32_t* partial, int64_t M, int64_t N, int64_t K, uint64_t tag, hipStream_t stream) {
    const size_t lds_act = (size_t)2 * p.kw * W8S_KC * W8S_PITCH * 16;
    const size_t lds_red = (size_t)p.gp * p.kw * NT * 64 * 16;
    const size_t lds = lds_act > lds_red ? lds_act : lds_red;       // at most 36 KiB
    const uint32_t g32 = (uint32_t)(g / 32);
    const uint32_t g32_recip = (uint32_t)((((uint64_t)1 << 32) + g32 - 1) / g32);   // unused when g32 == 1
    hipLaunchKernelGGL((fq_w4a8_skinny_kernel<NT, w8s_depth(ZR, AU), ZR, W8S_MAXW, AU, OUT>),
                       dim3((unsigned)(p.nblocks_n * p.splits)), dim3((unsigned)(p.gp * p.kw * 64)), lds, stream, Aq,
                       alpha, (const u32x4*)codes, z, (const uint16_t*)tstep, (uint16_t*)C, partial, (int)M, (int)N,
                       (int)K, g32, g32_recip, p.gp, p.kw, p.splits, tag);
    return FQ_OK;
}

template <int NT, int MT, int ZR, int OUT>
int w8_launch_mid(const w8_plan& p, int g, const int8_t* Aq, const float* alpha, const void* codes, const uint8_t* z,
                  const void* tstep, void* C, int32_t* partial, int64_t M, int64_t N, int64_t K, uint64_t tag, hipStream_t stream) {
    const size_t lds = w8m_lds(NT, MT, p.gp, p.kw);
    const uint32_t g32 = (uint32_t)(g / 32);
    const uint32_t g32_recip = (uint32_t)((((uint64_t)1 << 32) + g32 - 1) / g32);   // unused when g32 == 1
    auto kern = fq_w4a8_mid_kernel<NT, MT, ZR, OUT>;
    if (lds > 160 * 1024 || p.gp * p.kw > W8M_MAXW) return FQ_ERR_UNSUPPORTED;
    if (lds > 65536) {
        static std::atomic<uint64_t> raised;
        if (fqd::raise_lds_limit((const void*)kern, raised) != FQ_OK) return FQ_ERR_HIP;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.nblocks_n * p.nblocks_m * p.splits)), dim3((unsigned)(p.gp * p.kw * 64)), lds,
                       stream, Aq, alpha, (const u32x4*)codes, z, (const uint16_t*)tstep, (uint16_t*)C, partial, (int)M, (int)N,
                       (int)K, g32, g32_recip, p.gp, p.kw, p.nblocks_m, p.splits, tag);
    return FQ_OK;
}

template <int OUT>
int w8_gemm(const w8_plan& p, const int8_t* Aq, const float* alpha, int64_t M, int64_t N, int64_t K, const void* codes,
            const uint8_t* z, const void* tstep, int g, void* C, void* workspace, hipStream_t stream) {
    int32_t* partial = (int32_t*)workspace;
    // the small-M and mid-M kernels add a split of K themselves where a tile's sums are few, C and the scratch are
    // the device's own memory and C lies on nothing that is read
    const bool sums = (p.mid || p.small) && fq_sums_splits(M < p.mt * 16 ? (int)M : p.mt * 16, p.gp * p.nt * FQ_NTILE, p.splits, C) &&
                      !fq_overlaps(C, (size_t)(M * N * 2), {{Aq, (size_t)(M * K)}, {alpha, (size_t)M * 4}, {codes, (size_t)(K * N / 2)},
                                   {z, (size_t)(K / g * N)}, {tstep, (size_t)N * 2}, {partial, w8_partial_bytes(p, M, N)}}) &&
                      fq_counts_tickets(C, partial, stream);
    const uint64_t tag = sums ? fq_next_tag() : 0;
    if (p.mid) {
        const bool zr1 = g % 128 == 0;
        int st;
#define W8_MID(NT_, MT_)                                                                                              \
    st = zr1 ? w8_launch_mid<NT_, MT_, 1, OUT>(p, g, Aq, alpha, codes, z, tstep, C, partial, M, N, K, tag, stream)    \
             : w8_launch_mid<NT_, MT_, 2, OUT>(p, g, Aq, alpha, codes, z, tstep, C, partial, M, N, K, tag, stream)
        if (p.nt == 1) {
            if (p.mt == 2) W8_MID(1, 2);
            else if (p.mt == 3) W8_MID(1, 3);
            else W8_MID(1, 4);
        } else {
            if (p.mt == 2) W8_MID(3, 2);
            else if (p.mt == 3) W8_MID(3, 3);
            else W8_MID(3, 4);
        }
#undef W8_MID
        if (st != FQ_OK) return st;
    } else if (p.small) {
        const bool zr1 = g % 128 == 0;
#define W8_SMALL(NT_, ZR_, AU_) w8_launch_small<OUT, NT_, ZR_, AU_>(p, g, Aq, alpha, codes, z, tstep, C, partial, M, N, K, tag, stream)
        if (p.nt == 1) {
            if (zr1 && p.au == 1) W8_SMALL(1, 1, 1);
            else if (zr1) W8_SMALL(1, 1, 2);
            else if (p.au == 1) W8_SMALL(1, 2, 1);
            else W8_SMALL(1, 2, 2);
        } else {
            if (zr1 && p.au == 1) W8_SMALL(W8S_NT, 1, 1);
            else if (zr1) W8_SMALL(W8S_NT, 1, 2);
            else if (p.au == 1) W8_SMALL(W8S_NT, 2, 1);
            else W8_SMALL(W8S_NT, 2, 2);
        }
#undef W8_SMALL
    } else
    switch (p.mt) {
        case 4: w8_launch<4, OUT>(p, g, Aq, alpha, codes, z, tstep, C, partial, M, N, K, stream); break;
        default: w8_launch<8, OUT>(p, g, Aq, alpha, codes, z, tstep, C, partial, M, N, K, stream); break;
    }
    if (p.splits > 1 && !sums) {
        const int64_t n4 = M * N / 4;
        hipLaunchKernelGGL(w8_finalize_kernel<OUT>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, stream,
                           (const int32_t*)partial, p.splits, alpha, (const uint16_t*)tstep, M, N, (uint16_t*)C);
    }
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

}  // namespace

extern "C" {

size_t fq_zscale_bytes(int64_t K, int64_t N, int group_size) {
    int g = 0;
    if (w8_check(K, N, group_size, &g) != FQ_OK) return 0;
    return (size_t)((K / g) * N);
}

int fq_quantize_w4a8(const void* W_f16, int64_t K, int64_t N, int group_size, void* codes, uint8_t* zscale,
                     void* tstep_f16, void* stream) {
    if (!W_f16 || !codes || !zscale || !tstep_f16) return FQ_ERR_INVALID_ARG;
    int g = 0;
    const int st = w8_check(K, N, group_size, &g);
    if (st != FQ_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    const int groups = (int)(K / g);
    if (groups > 65535) return FQ_ERR_UNSUPPORTED;
    // The code buffer (K N / 2 bytes) holds the K / g x N abs-max values (g >= 32: at most K N / 16 bytes) on the way.
    // Groups of up to 1024 rows take one block of threads per (group, 128 columns); longer ones are cut into blocks
    // of 128 rows, which keeps the chip full when there are few groups, and folded afterwards (where 128 does not
    // divide the group its blocks stay whole).
    uint16_t* amax = (uint16_t*)codes;
    const bool cut = g > 1024 && g % 128 == 0;
    const int f = cut ? 128 : g;
    hipLaunchKernelGGL(fq_fine_absmax_kernel<256>, dim3((unsigned)((N + 127) / 128), (unsigned)(K / f)), dim3(16, 16), 0, s,
                       (const uint16_t*)W_f16, N, f, amax, (uint32_t*)nullptr);
    if (cut) {
        uint16_t* fine = amax;
        amax = fine + (K / f) * N;
        hipLaunchKernelGGL(w8_fold_kernel, dim3((unsigned)((N + 255) / 256), (unsigned)groups), dim3(256), 0, s,
                           (const uint16_t*)fine, N, g / f, amax);
    }
    if (groups <= 32)
        hipLaunchKernelGGL((w8_scales_kernel<32, 8>), dim3((unsigned)((N + 63) / 64)), dim3(256), 0, s, (const uint16_t*)amax, N,
                           groups, zscale, (uint16_t*)tstep_f16);
    else
        hipLaunchKernelGGL((w8_scales_kernel<16, 32>), dim3((unsigned)((N + 31) / 32)), dim3(512), 0, s, (const uint16_t*)amax, N,
                           groups, zscale, (uint16_t*)tstep_f16);
    hipLaunchKernelGGL(w8_encode_kernel, dim3((unsigned)((N + 127) / 128), (unsigned)(K / 128)), dim3(256), 0, s,
                       (const uint16_t*)W_f16, N, g, (const uint8_t*)zscale, (const uint16_t*)tstep_f16, (uint32_t*)codes);
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

int fq_unpack_w4a8(const void* codes, int64_t K, int64_t N, int8_t* q, void* stream) {
    if (!codes || !q) return FQ_ERR_INVALID_ARG;
    int g = 0;
    const int st = w8_check(K, N, 0, &g);
    if (st != FQ_OK) return st;
    const int64_t recs = (K / 128) * (N / FQ_NTILE) * 64;
    hipLaunchKernelGGL(w8_unpack_kernel, dim3((unsigned)((recs + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       (const uint32_t*)codes, K, N, q);
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

int fq_quantize_act_i8(const void* A, int act_dtype, int64_t M, int64_t K, int8_t* Aq, float* alpha, void* stream) {
    if (M < 0 || K <= 0) return FQ_ERR_INVALID_ARG;
    if (act_dtype != FQ_F16 && act_dtype != FQ_BF16) return FQ_ERR_INVALID_ARG;
    if (M == 0) return FQ_OK;
    if (!A || !Aq || !alpha) return FQ_ERR_INVALID_ARG;
    if (M > (int64_t)1 << 24 || K > (int64_t)1 << 24) return FQ_ERR_UNSUPPORTED;
    if (act_dtype == FQ_F16) w8_launch_act_quant<FQ_F16>((const uint16_t*)A, M, K, Aq, alpha, (hipStream_t)stream);
    else w8_launch_act_quant<FQ_BF16>((const uint16_t*)A, M, K, Aq, alpha, (hipStream_t)stream);
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

size_t fq_gemm_w4a8_workspace_bytes(int64_t M, int64_t N, int64_t K, int group_size) {
    int g = 0;
    if (M <= 0 || w8_check(K, N, group_size, &g) != FQ_OK) return 0;
    return w8_partial_bytes(w8_plan_of(M, N, K, g), M, N);
}

int fq_gemm_w4a8(const int8_t* Aq, const float* alpha, int64_t M, int64_t N, int64_t K, const void* codes,
                 const uint8_t* zscale, const void* tstep_f16, int group_size, void* C, int out_dtype,
                 void* workspace, size_t workspace_bytes, void* stream) {
    if (M < 0) return FQ_ERR_INVALID_ARG;
    if (out_dtype != FQ_F16 && out_dtype != FQ_BF16) return FQ_ERR_INVALID_ARG;
    int g = 0;
    const int st = w8_check(K, N, group_size, &g);
    if (st != FQ_OK) return st;
    if (M == 0) return FQ_OK;
    if (!Aq || !alpha || !codes || !zscale || !tstep_f16 || !C) return FQ_ERR_INVALID_ARG;
    if (M > (int64_t)1 << 24) return FQ_ERR_UNSUPPORTED;
    const w8_plan p = w8_plan_of(M, N, K, g);
    const size_t need = w8_partial_bytes(p, M, N);
    if (need > 0 && (!workspace || workspace_bytes < need)) return FQ_ERR_WORKSPACE;
    if (out_dtype == FQ_F16)
        return w8_gemm<FQ_F16>(p, Aq, alpha, M, N, K, codes, zscale, tstep_f16, g, C, workspace, (hipStream_t)stream);
    return w8_gemm<FQ_BF16>(p, Aq, alpha, M, N, K, codes, zscale, tstep_f16, g, C, workspace, (hipStream_t)stream);
}

}  // extern "C"
