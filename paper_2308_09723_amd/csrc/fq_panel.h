// Device code shared by the weight quantisers (fq_quantize.hip, fq_w4a8.hip): a 128 x 128 panel of binary16
// weights staged in LDS, and the encoding of eight consecutive rows of one column from it.
#ifndef FQ_PANEL_H_
#define FQ_PANEL_H_

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#define FQ_QP_ROWS 128
#define FQ_QP_COLS 128
#define FQ_QP_PITCH (FQ_QP_COLS + 8)   // binary16 elements per LDS row (16-byte units stay aligned)

typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));

__device__ inline float half_bits_to_float(uint16_t b) { return __half2float(__ushort_as_half(b)); }

// abs-max bit patterns of 8 columns (four packed pairs) over rows ty, ty + 16, ... < rows: four rows in flight, or eight where
// there are fewer blocks than the 256 compute units, which are bound by this chain of loads, and what is left in one go (rows past
// the end are the last one again).  Four in flight and the rest one by one -> this, the heuristic's call, us: 16256 x 2176 in
// blocks of 4064 rows 41.4 -> 32.4, 10368 x 1888 in blocks of 162 32.9 -> 27.3.  With eight in flight everywhere 12672 x 9392
// in blocks of 3168 (296 blocks) took 64.4 instead of 62.2.
__device__ inline uint4 absmax8_slice(const uint16_t* __restrict__ base, int64_t N, int rows, int ty) {
    u16x2_t m[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
    auto fold = [&](const uint4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t a = w[i] & 0x7fff7fffu;
            m[i] = __builtin_elementwise_max(m[i], __builtin_bit_cast(u16x2_t, a));
        }
    };
    auto some = [&](int r, auto count) {
        constexpr int COUNT = decltype(count)::value;
        uint4 v[COUNT];
#pragma unroll
        for (int i = 0; i < COUNT; ++i)
            v[i] = *reinterpret_cast<const uint4*>(base + (int64_t)(r + 16 * i < rows ? r + 16 * i : rows - 1) * N);
#pragma unroll
        for (int i = 0; i < COUNT; ++i) fold(v[i]);
    };
    int r = ty;
    if (gridDim.x * gridDim.y < 256)
        for (; r + 64 < rows; r += 128) some(r, std::integral_constant<int, 8>());
    for (; r + 32 < rows; r += 64) some(r, std::integral_constant<int, 4>());
    if (r < rows) some(r, std::integral_constant<int, 2>());
    return make_uint4(__builtin_bit_cast(uint32_t, m[0]), __builtin_bit_cast(uint32_t, m[1]),
                      __builtin_bit_cast(uint32_t, m[2]), __builtin_bit_cast(uint32_t, m[3]));
}
// the sixteen slices of a block combined: valid in the threads with ty == 0
__device__ inline uint4 absmax8_block(uint4 mine, uint4 (&red)[16][16], int tx, int ty) {
    red[ty][tx] = mine;
    __syncthreads();
    if (ty != 0) return mine;
    u16x2_t m[4];
    m[0] = __builtin_bit_cast(u16x2_t, mine.x); m[1] = __builtin_bit_cast(u16x2_t, mine.y);
    m[2] = __builtin_bit_cast(u16x2_t, mine.z); m[3] = __builtin_bit_cast(u16x2_t, mine.w);
    for (int y = 1; y < 16; ++y) {
        const uint4 o = red[y][tx];
        m[0] = __builtin_elementwise_max(m[0], __builtin_bit_cast(u16x2_t, o.x));
        m[1] = __builtin_elementwise_max(m[1], __builtin_bit_cast(u16x2_t, o.y));
        m[2] = __builtin_elementwise_max(m[2], __builtin_bit_cast(u16x2_t, o.z));
        m[3] = __builtin_elementwise_max(m[3], __builtin_bit_cast(u16x2_t, o.w));
    }
    return make_uint4(__builtin_bit_cast(uint32_t, m[0]), __builtin_bit_cast(uint32_t, m[1]),
                      __builtin_bit_cast(uint32_t, m[2]), __builtin_bit_cast(uint32_t, m[3]));
}

// Abs-max of blocks of f rows -> fine[K / f, N] as binary16 bit patterns; block = 16 x 16 threads, thread (tx, ty)
// takes 8 consecutive columns (16-byte loads) of the rows ty, ty + 16, ...; grid (N / 128 rounded up, K / f).
// `clear` (may be null): two words set to zero for the kernels that follow.
template <int THREADS>   // (a template so that every translation unit may hold a copy)
__global__ __launch_bounds__(THREADS) void fq_fine_absmax_kernel(const uint16_t* __restrict__ W, int64_t N, int f,
                                                                 uint16_t* __restrict__ fine,
                                                                 uint32_t* __restrict__ clear) {
    static_assert(THREADS == 256, "16 x 16 threads");
    __shared__ uint4 red[16][16];
    const int tx = threadIdx.x, ty = threadIdx.y;
    const int64_t n = ((int64_t)blockIdx.x * 16 + tx) * 8;      // N is a multiple of 16
    const int64_t blk = blockIdx.y;
    if (clear != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && tx == 0 && ty == 0) clear[0] = clear[1] = 0u;
    uint4 m = make_uint4(0u, 0u, 0u, 0u);
    if (n < N) m = absmax8_slice(W + (blk * f) * N + n, N, f, ty);
    m = absmax8_block(m, red, tx, ty);
    if (ty == 0 && n < N) *reinterpret_cast<uint4*>(fine + blk * N + n) = m;
}

// Stage rows k0 .. k0 + rows - 1, columns n0 .. n0 + cols - 1 of W in LDS (256 threads, coalesced 16-byte loads;
// the rest of the panel is zero).  No barrier.
__device__ inline void fq_stage_panel(const uint16_t* __restrict__ W, int64_t N, int64_t k0, int64_t n0, int rows,
                                      int cols, uint16_t* panel) {
    const int tid = threadIdx.x;
    const int c8 = (tid & 15) * 8;
    uint4 v[FQ_QP_ROWS / 16];
#pragma unroll
    for (int i = 0; i < FQ_QP_ROWS / 16; ++i) {
        const int r = (tid >> 4) + 16 * i;
        v[i] = make_uint4(0u, 0u, 0u, 0u);
        if (r < rows && c8 < cols) v[i] = *reinterpret_cast<const uint4*>(W + (k0 + r) * N + n0 + c8);
    }
#pragma unroll
    for (int i = 0; i < FQ_QP_ROWS / 16; ++i)
        *reinterpret_cast<uint4*>(&panel[((tid >> 4) + 16 * i) * FQ_QP_PITCH + c8]) = v[i];
}

// Encode: divide (IEEE binary32), round half to even, clamp (Appendix A's q = int(w / s)); the low byte of the
// returned word is q + bias.
//
// The quotient is formed without the division instruction sequence: with rs = 1 / s rounded to nearest
// (once per group; 0 for s = 0), x0 = w * rs is within two units in the last place of w / s, its residual
// e = w - x0 * s comes exactly out of one fused multiply-add, and x = x0 + e * rs (fused again) is the
// quotient rounded to nearest wherever that matters here: an exact tie k + 1/2 is representable and is
// returned exactly, and any other quotient of a binary16 weight by a binary16 or bfloat16 scale lies at
// least 2^-12 away from a tie (numerator and denominator are integers of at most 11 bits times powers of
// two; 2^-16 for the integer path's z * t with its 15 bits), far beyond the error of x.  Checked on the host
// (tests/encode_identity_check.c).  What the general division adds (scaling against overflow and subnormal
// quotients, the fix-ups for zero, infinity and NaN operands) cannot occur: |w / s| <= (2^bits - 1) / 2.
// Clamping before the rounding gives the same integer (the bound is an integer).  The rounding itself is the
// addition of 1.5 * 2^23 + bias: at that magnitude binary32 holds integers only, halves go to the even one
// (1.5 * 2^23 and the biases used are even, so it is the even q), and the low byte of the sum's bit pattern is
// q + bias, ready to be packed.  Seven vector instructions with the conversion to binary32; with a rounding,
// two comparisons and a conversion to integer it was ten, and the panel kernels are bound by their instructions
// next to the memory.
__device__ inline uint32_t fq_encode_biased(float w, float s, float rs, float qmax, float magic) {
    const float x0 = w * rs;
    const float e = __builtin_fmaf(-x0, s, w);
    const float x = __builtin_fmaf(e, rs, x0);
    return __float_as_uint(__builtin_amdgcn_fmed3f(x, -qmax, qmax) + magic);
}
#define FQ_ENCODE_MAGIC 12582912.0f   // 1.5 * 2^23

// the low bytes of four words as one word (byte i from b[i])
__device__ inline uint32_t fq_gather_bytes(uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3) {
    const uint32_t lo = __builtin_amdgcn_perm(b1, b0, 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(b3, b2, 0x04000c0cu);
    return lo | hi;
}

// Eight consecutive rows of two neighbouring columns of the staged panel, encoded: b0[e], b1[e] = words whose low
// bytes are q + bias of row r0 + e of columns c and c + 1 (c even: one 4-byte LDS read per row serves both).
__device__ inline void fq_encode8_pair(const uint16_t* panel, int r0, int c, float2 s, float2 rs, float qmax, float magic,
                                       uint32_t (&b0)[8], uint32_t (&b1)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t v = *reinterpret_cast<const uint32_t*>(&panel[(r0 + e) * FQ_QP_PITCH + c]);
        b0[e] = fq_encode_biased(half_bits_to_float((uint16_t)v), s.x, rs.x, qmax, magic);
        b1[e] = fq_encode_biased(half_bits_to_float((uint16_t)(v >> 16)), s.y, rs.y, qmax, magic);
    }
}

#endif  // FQ_PANEL_H_
