// Quantiser, packer, unpacker and group-size heuristic kernels (gfx950).
//
// Appendix A: s = 2 max|w| / (2^b - 1), q = int(w / s); section 4.1: one scale per block
// of g consecutive rows of a column; Appendix B: scales stored in half precision.
// Rounding choices (scale rounded up to binary16, quotient in binary32, ties to even,
// clamp) are stated in fq.h.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <mutex>
#include <stdint.h>
#include <string.h>

#include "fq_internal.h"
#include "fq_layout.h"
#include "fq_panel.h"

namespace {

// stored scale (16 bits, binary16 or bfloat16) -> binary32
__device__ inline float scale_bits_to_float(uint16_t b, int sfmt) {
    return sfmt == FQ_SCALE_BF16 ? __uint_as_float((uint32_t)b << 16) : half_bits_to_float(b);
}

// Appendix A's scale for a group whose abs-max has the binary16 bit pattern m:
// the smallest s of the storage format with L * s >= 2 m (L = 2^bits - 1), as a 16-bit pattern.
// The candidate is the binary32 quotient rounded to nearest (binary16) or cut (bfloat16: at or
// below the quotient); the products L * candidate are exact in binary32 (8 x 11 bits at most),
// so one comparison decides whether the next value up is needed.
__device__ inline uint32_t scale_bits_from_absmax_bits(uint32_t m, float L, int sfmt) {
    const float two_m = 2.0f * half_bits_to_float((uint16_t)m);
    const float t32 = __fdiv_rn(two_m, L);
    uint32_t tb = sfmt == FQ_SCALE_BF16 ? (__float_as_uint(t32) >> 16)
                                        : (uint32_t)__half_as_ushort(__float2half_rn(t32));
    if (__fmul_rn(L, scale_bits_to_float((uint16_t)tb, sfmt)) < two_m) tb += 1;   // next value up
    return tb;
}

// ---------------------------------------------------------------------------------
// Scales: abs-max over each block of g rows, then the smallest storable s with
// L * s >= 2 m.  Block = 16 x 16 threads: thread (tx, ty) takes 8 consecutive columns (one
// 16-byte load per row, so a row of the block is 256 contiguous bytes) of the rows ty, ty + 16,
// ... of the group; the sixteen row slices are combined through LDS.
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fq_scales_kernel(const uint16_t* __restrict__ W, int64_t K,
                                                        int64_t N, int g, float L, int sfmt,
                                                        uint16_t* __restrict__ scales) {
    __shared__ uint4 red[16][16];
    const int tx = threadIdx.x, ty = threadIdx.y;
    const int64_t n = ((int64_t)blockIdx.x * 16 + tx) * 8;      // N is a multiple of 16
    const int64_t grp = blockIdx.y;
    uint4 m = make_uint4(0u, 0u, 0u, 0u);
    if (n < N) m = absmax8_slice(W + (grp * g) * N + n, N, g, ty);
    m = absmax8_block(m, red, tx, ty);
    if (ty == 0 && n < N) {
        const uint32_t w[4] = {m.x, m.y, m.z, m.w};
        uint32_t out[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            out[i] = scale_bits_from_absmax_bits(w[i] & 0xffffu, L, sfmt) |
                     (scale_bits_from_absmax_bits(w[i] >> 16, L, sfmt) << 16);
        *reinterpret_cast<uint4*>(scales + grp * N + n) = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

// Coarse groups (few groups per column): the abs-max of 128-row blocks is taken first by
// fq_fine_absmax_kernel, with one block of threads per (128 rows x 128 columns), and this
// kernel folds the g / 128 block maxima of each group into its scale.  One kernel walking a
// whole 12288-row column per thread slice leaves most of the GPU idle.
__global__ __launch_bounds__(256) void fq_scales_fold_kernel(const uint16_t* __restrict__ fine, int64_t N,
                                                             int per_group, float L, int sfmt,
                                                             uint16_t* __restrict__ scales) {
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    const int64_t grp = blockIdx.y;
    uint32_t m = 0;
    int i = 0;
    for (; i + 8 <= per_group; i += 8) {     // eight loads in flight
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = fine[(grp * per_group + i + u) * N + n];
#pragma unroll
        for (int u = 0; u < 8; ++u) m = v[u] > m ? v[u] : m;
    }
    for (; i < per_group; ++i) {
        const uint32_t v = fine[(grp * per_group + i) * N + n];
        m = v > m ? v : m;
    }
    scales[grp * N + n] = (uint16_t)scale_bits_from_absmax_bits(m, L, sfmt);
}

// ---------------------------------------------------------------------------------
// One-pass quantiser for group sizes that divide 128 (32, 64, 128): a block stages a panel of
// 128 rows x 128 columns of W in LDS with coalesced 16-byte loads, takes the abs-max of every
// 32-row sub-block, derives the scales of the panel's groups, and encodes and packs the panel
// from LDS.  W is read from HBM once.
// A thread works on pairs of neighbouring columns: one 4-byte LDS read per row serves two weights (one 2-byte
// read per weight made the LDS reads a third of the kernel's instructions), and its two lane records are
// adjacent in memory.  Bound by HBM next to its own instructions (about 10 per weight; 20 with per-weight reads
// and roundings): 8192 x 28672 to int4, g = 128: 152 -> 108 us (5.4 TB/s;
// a device copy reaches 4.9).
// ---------------------------------------------------------------------------------
// Packs the eight biased codes of one 32-row step (rows 32 t + 8 j .. + 7) into the record dwords.
template <int BITS>
__device__ inline void pack_step(uint32_t (&rec)[4], int t, const uint32_t (&b)[8]) {
    if constexpr (BITS == 8) {
        rec[2 * t] = fq_gather_bytes(b[0], b[1], b[2], b[3]);
        rec[2 * t + 1] = fq_gather_bytes(b[4], b[5], b[6], b[7]);
    } else {
        // nibble slots 0..7 hold elements 0, 2, 4, 6, 1, 3, 5, 7: low nibbles of the bytes 0, 4, 1, 5, high 2, 6, 3, 7
        const uint32_t v = fq_gather_bytes(b[0], b[4], b[1], b[5]) | (fq_gather_bytes(b[2], b[6], b[3], b[7]) << 4);
        if (BITS == 4 || t < 3) {
            rec[t] |= v;
        } else {
            // 3-bit codes, step 3: bit i of the value goes to the fourth bit of the same nibble of dword i
#pragma unroll
            for (int i = 0; i < 3; ++i) rec[i] |= (v << (3 - i)) & 0x88888888u;
        }
    }
}

// OWN_SCALES = false: the scales were computed before (groups larger than the panel) and are only read.
template <int BITS, bool OWN_SCALES>
__global__ __launch_bounds__(256) void fq_quantize_panel_kernel(const uint16_t* __restrict__ W, int64_t K,
                                                                int64_t N, int g, float L, int sfmt,
                                                                uint16_t* __restrict__ scales,
                                                                uint32_t* __restrict__ codes) {
    constexpr int KBLK = fq_kblk(BITS);
    constexpr int STEPS = KBLK / FQ_KSTEP;
    constexpr int RW = fq_rec_bytes(BITS) / 4;           // dwords per lane record
    constexpr float QMAX = (float)((1 << (BITS - 1)) - 1);
    constexpr float MAGIC = FQ_ENCODE_MAGIC + (float)(1 << (BITS - 1));
    __shared__ __align__(16) uint16_t panel[FQ_QP_ROWS * FQ_QP_PITCH];
    __shared__ __align__(16) uint16_t submax[8][FQ_QP_COLS];      // abs-max bits of 16-row slices
    __shared__ __align__(16) float sub_scale[4][FQ_QP_COLS];      // scale of the group each 32-row sub-block belongs to
    __shared__ __align__(16) float sub_rscale[4][FQ_QP_COLS];     // its reciprocal (0 for an all-zero group)
    const int tid = threadIdx.x;
    const int64_t n0 = (int64_t)blockIdx.x * FQ_QP_COLS;
    // Bottom of the matrix first: whatever read W before (the abs-max pass of coarse groups, the group-size heuristic)
    // went top to bottom, and its end is what a matrix larger than the Infinity Cache has left there (108 -> 100 us
    // after the heuristic; no difference on a matrix nobody read before).
    const int64_t k0 = (int64_t)(gridDim.y - 1 - blockIdx.y) * FQ_QP_ROWS;
    const int cols = (int)((N - n0) < FQ_QP_COLS ? (N - n0) : FQ_QP_COLS);   // multiple of 16
    const int rows = (int)((K - k0) < FQ_QP_ROWS ? (K - k0) : FQ_QP_ROWS);   // 128, or 64 at the end (8-bit)

    fq_stage_panel(W, N, k0, n0, rows, cols, panel);
    __syncthreads();
    if constexpr (OWN_SCALES) {
        // abs-max of 16-row slices: thread -> four columns 4 (tid % 32), slice tid / 32; 8-byte LDS reads and
        // packed 16-bit maxima
        {
            const int c4 = (tid & 31) * 4;
            const int sl = tid >> 5;
            u16x2_t m0 = {0, 0}, m1 = {0, 0};
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint2 v = *reinterpret_cast<const uint2*>(&panel[(sl * 16 + r) * FQ_QP_PITCH + c4]);
                m0 = __builtin_elementwise_max(m0, __builtin_bit_cast(u16x2_t, v.x & 0x7fff7fffu));
                m1 = __builtin_elementwise_max(m1, __builtin_bit_cast(u16x2_t, v.y & 0x7fff7fffu));
            }
            *reinterpret_cast<uint2*>(&submax[sl][c4]) =
                make_uint2(__builtin_bit_cast(uint32_t, m0), __builtin_bit_cast(uint32_t, m1));
        }
        __syncthreads();
        // scales: one per (group, column); a group is g / 16 consecutive slices
        {
            const int per = g / 32;                 // 1, 2 or 4 sub-blocks of 32 rows
            const int c = tid & 127;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int sb = (tid >> 7) + 2 * h;
                const int first = (sb / per) * per;
                uint32_t m = 0;
                for (int i = 0; i < 2 * per; ++i) {
                    const uint32_t a = submax[2 * first + i][c];
                    m = a > m ? a : m;
                }
                const uint32_t sbits = scale_bits_from_absmax_bits(m, L, sfmt);
                const float sv = scale_bits_to_float((uint16_t)sbits, sfmt);
                sub_scale[sb][c] = sv;
                sub_rscale[sb][c] = sv == 0.0f ? 0.0f : __fdiv_rn(1.0f, sv);
                if (sb == first && sb * 32 < rows && c < cols) scales[((k0 + sb * 32) / g) * N + n0 + c] = (uint16_t)sbits;
            }
        }
        __syncthreads();
    } else {
        const int c = tid & 127;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int sb = (tid >> 7) + 2 * h;
            float v = 0.0f;
            if (sb * 32 < rows && c < cols) v = scale_bits_to_float(scales[((k0 + sb * 32) / g) * N + n0 + c], sfmt);
            sub_scale[sb][c] = v;
            sub_rscale[sb][c] = v == 0.0f ? 0.0f : __fdiv_rn(1.0f, v);
        }
        __syncthreads();
    }
    // encode + pack: thread -> columns c, c + 1 and lane group j; its records of every k-block of the panel
    const int c = (tid & 63) * 2, j = tid >> 6;
    if (c >= cols) return;                               // (no barrier below)
    const int64_t ntiles = N / FQ_NTILE;
    for (int kb = 0; kb * KBLK < rows; ++kb) {
        uint32_t rec0[4] = {0u, 0u, 0u, 0u}, rec1[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            const int r0 = kb * KBLK + t * FQ_KSTEP + j * 8;
            const float2 s = *reinterpret_cast<const float2*>(&sub_scale[r0 / 32][c]);
            const float2 rs = *reinterpret_cast<const float2*>(&sub_rscale[r0 / 32][c]);
            uint32_t b0[8], b1[8];
            fq_encode8_pair(panel, r0, c, s, rs, QMAX, MAGIC, b0, b1);
            pack_step<BITS>(rec0, t, b0);
            pack_step<BITS>(rec1, t, b1);
        }
        const int64_t kblock = (k0 / KBLK) + kb;
        const int64_t at = fq_rec(n0 / FQ_NTILE + c / FQ_NTILE, kblock, ntiles, j * 16 + c % FQ_NTILE);
        uint32_t* dst = codes + at * RW;                 // record of column c; the next one follows it
        if constexpr (BITS == 3) {
            // 24 bytes, 8-byte aligned (c is even)
            *reinterpret_cast<uint2*>(dst) = make_uint2(rec0[0], rec0[1]);
            *reinterpret_cast<uint2*>(dst + 2) = make_uint2(rec0[2], rec1[0]);
            *reinterpret_cast<uint2*>(dst + 4) = make_uint2(rec1[1], rec1[2]);
        } else {
            *reinterpret_cast<uint4*>(dst) = make_uint4(rec0[0], rec0[1], rec0[2], rec0[3]);
            *reinterpret_cast<uint4*>(dst + 4) = make_uint4(rec1[0], rec1[1], rec1[2], rec1[3]);
        }
    }
}

// ---------------------------------------------------------------------------------
// Unpack: one thread per logical element, writes are coalesced along N.
// ---------------------------------------------------------------------------------
template <int BITS>
__global__ __launch_bounds__(256) void fq_unpack_kernel(const uint32_t* __restrict__ codes, int64_t K,
                                                        int64_t N, int8_t* __restrict__ q) {
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    for (int64_t k = blockIdx.y; k < K; k += gridDim.y) {
        const fq_pos p = fq_locate(k, n, N, BITS);
        int v;
        if (BITS == 4) {
            const uint32_t w = codes[p.rec * 4 + p.t];
            v = (int)((w >> (4 * fq_nibble_slot(p.e))) & 0xfu) - 8;
        } else if (BITS == 3) {
            v = (int)fq_get3(codes + p.rec * 3, p.t, p.e) - 4;
        } else {
            const uint32_t w = codes[p.rec * 4 + 2 * p.t + (p.e >> 2)];
            v = (int)((w >> (8 * (p.e & 3))) & 0xffu) - 128;
        }
        q[k * N + n] = (int8_t)v;
    }
}

// ---------------------------------------------------------------------------------
// Heuristic (section 3.3).  Pass 1: abs-max of the finest blocks (f rows) -> fine[K/f, N]
// as binary16 bit patterns.  Pass 2: one thread per (column, coarsest group) folds the
// fine values pairwise, level by level, and sets flag[level] when the smaller child is
// below thr * parent.  The host then walks the flags from the coarsest level down.
// ---------------------------------------------------------------------------------
// Adds a thread's flags.  (Both words live at the memory's point of coherence, where device-wide atomics are performed; an
// atomic that has returned its old value has been performed.  That order is all publish_flags needs: a __threadfence() in
// every block, which writes the caches back, made the call 15 us longer on 8192 x 28672.)
__device__ inline void add_flags(uint32_t* flags, uint32_t hits) {
    uint32_t old = *(volatile uint32_t*)flags;
    if (hits & ~old) old = atomicOr(flags, hits);
    asm volatile("" : : "v"(old) : "memory");
}
// The last block to end hands the flags to the host: flags[1] counts the blocks whose flags have been added.  (Copied back by
// a transfer of their own they cost a call another 10 us.)  Called by one thread, behind the block's add_flags.
__device__ inline void publish_flags(uint32_t* flags, uint32_t blocks, uint32_t* host) {
    if (atomicAdd(flags + 1, 1u) == blocks - 1) *host = atomicOr(flags, 0u);
}

// levels = number of halvings covered; a top group spans 2^levels fine blocks.
// Bit l of *flags (l = 0 is the coarsest transition g_start -> g_start/2; fq_fine_absmax_kernel clears the word and the count
// behind it) is set when any parent at that level has min(child) < thr * parent.  One word, and a block or wave that has nothing to
// add leaves it alone: every block setting one word per level cost 28 us on 8192 x 28672, nearly all of it atomics
// waiting for each other (now 15 us).
__global__ __launch_bounds__(256) void fq_halving_flags_kernel(const uint16_t* __restrict__ fine,
                                                               int64_t N, int64_t tops, int levels,
                                                               float thr, uint32_t* __restrict__ flags,
                                                               uint32_t* __restrict__ host) {
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t top = blockIdx.y;                      // < tops: the grid's height
    const int64_t span = (int64_t)1 << levels;
    const uint16_t* col = fine + (top * span) * N + (n < N ? n : 0);
    // Level d = blockIdx.z (d = levels - 1 is the finest transition): parents are pairs of nodes of
    // 2^(levels-1-d) fine blocks, recomputed from the fine array, so a thread reads span values; one
    // grid layer per level keeps enough threads in flight when there are few top groups.
    const int d = blockIdx.z;
    const int64_t child = span >> (d + 1);     // fine blocks per child at this level
    bool hit = false;
    // one pass over the column's fine values (independent loads, several in flight): `node` collects the
    // child under way, `prev` is its left sibling once that one is complete
    uint32_t node = 0, prev = 0;
#pragma unroll 8
    for (int64_t q = 0; q < span; ++q) {
        const uint32_t a = col[q * N];
        node = a > node ? a : node;
        if (((q + 1) & (child - 1)) == 0) {            // a child ends here
            if (((q + 1) & (2 * child - 1)) == 0) {    // ... and it is the right one of its pair
                const float lo = half_bits_to_float((uint16_t)(prev < node ? prev : node));
                const float hi = half_bits_to_float((uint16_t)(prev < node ? node : prev));
                hit = hit || (lo < __fmul_rn(thr, hi));
            }
            prev = node;
            node = 0;
        }
    }
    if (hit) add_flags(flags, 1u << d);
    __syncthreads();
    if (threadIdx.x == 0) publish_flags(flags, gridDim.x * gridDim.y * gridDim.z, host);
}

// The same test with every fine value read from memory once (a top group of at most 1024 fine blocks).  An item is one top
// group of 8 * 2^lu columns; a thread takes eight neighbouring columns of R = 2^LR neighbouring fine blocks (16-byte loads, all
// in flight), folds those in registers, and the rest of the tree by exchange with the thread whose number differs in one bit:
// inside a wave by shuffles, between waves through LDS.  Both partners form the same parent.  (Packed 16-bit minima and
// maxima: magnitudes of binary16 order like their bit patterns.)
// Bound by the count that each block adds to at its end, on one address: about 40 ns a block.  So blocks are large and walk
// the items, at most FQ_TREE_BLOCKS of them.  With a block of 256 threads per 64 columns and the fold in LDS level by
// level: 1536 x 37408 down to g = 96 (585 blocks) 23 us, 8192 x 28672 down to 64 (448 blocks) 22 us;
// now 6 and 10 us (blocks of 256 threads 6 and 12, of 1024 threads 8 and 10.5).
constexpr int FQ_TREE_THREADS = 512;
constexpr int FQ_TREE_BLOCKS = 256;
template <int LR>
__global__ __launch_bounds__(FQ_TREE_THREADS) void fq_halving_tree_kernel(const uint16_t* __restrict__ fine, int64_t N,
                                                                          int levels, int lu, float thr, int64_t items_n,
                                                                          int64_t items, uint32_t* __restrict__ flags,
                                                                          uint32_t* __restrict__ host) {
    constexpr int R = 1 << LR;
    __shared__ uint4 other[FQ_TREE_THREADS];
    __shared__ uint32_t wave_hits[FQ_TREE_THREADS / 64];
    const int tid = threadIdx.x;
    const int unit = tid & ((1 << lu) - 1);
    const int64_t row = (int64_t)(tid >> lu) * R;
    uint32_t hits = 0;                                          // (the same in every lane of a wave)
    auto fold = [&](uint4& a, const uint4& b, bool& hit) {
        uint32_t x[4] = {a.x, a.y, a.z, a.w};
        const uint32_t y[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u16x2_t p = __builtin_bit_cast(u16x2_t, x[i]), q = __builtin_bit_cast(u16x2_t, y[i]);
            const u16x2_t lo = __builtin_elementwise_min(p, q), hi = __builtin_elementwise_max(p, q);
            hit = hit || (half_bits_to_float(lo[0]) < __fmul_rn(thr, half_bits_to_float(hi[0])));
            hit = hit || (half_bits_to_float(lo[1]) < __fmul_rn(thr, half_bits_to_float(hi[1])));
            x[i] = __builtin_bit_cast(uint32_t, hi);
        }
        a = make_uint4(x[0], x[1], x[2], x[3]);
    };
    for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
        const int64_t n = (((item % items_n) << lu) + unit) * 8;
        uint4 m[R];
#pragma unroll
        for (int r = 0; r < R; ++r) m[r] = make_uint4(0u, 0u, 0u, 0u);
        if (n < N) {                                            // N is a multiple of 16: whole units
            const uint16_t* base = fine + (((item / items_n) << levels) + row) * N + n;
#pragma unroll
            for (int r = 0; r < R; ++r) m[r] = *reinterpret_cast<const uint4*>(base + (int64_t)r * N);
        }
#pragma unroll
        for (int s = 0; s < LR; ++s) {                          // halving step levels - 1 - s
            bool hit = false;
#pragma unroll
            for (int r = 0; r < R; r += 2 << s) fold(m[r], m[r + (1 << s)], hit);
            if (__any(hit)) hits |= 1u << (levels - 1 - s);
        }
        for (int s = LR; s < levels; ++s) {
            const int bit = 1 << (lu + s - LR);
            uint4 o;
            if (bit < 64) {
                o = make_uint4(__shfl_xor(m[0].x, bit), __shfl_xor(m[0].y, bit), __shfl_xor(m[0].z, bit),
                               __shfl_xor(m[0].w, bit));
            } else {
                __syncthreads();                                // what was written before has been read
                other[tid] = m[0];
                __syncthreads();
                o = other[tid ^ bit];
            }
            bool hit = false;
            fold(m[0], o, hit);
            if (__any(hit)) hits |= 1u << (levels - 1 - s);
        }
    }
    if ((tid & 63) == 0) wave_hits[tid >> 6] = hits;
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int i = 1; i < FQ_TREE_THREADS / 64; ++i) hits |= wave_hits[i];
        if (hits) add_flags(flags, hits);
        publish_flags(flags, gridDim.x, host);
    }
}

// ---------------------------------------------------------------------------------
// Round-trip error (section 3.2, figure 2a: mean squared error between the weights and their
// dequantised codes, Appendix A: dequantised value = q * s).  binary64 throughout: w, q * s and
// their difference are exact, the squares are added with one rounding each, and the sums are taken in a fixed
// order (thread strip -> tree over the wave -> the block's waves -> one block over the per-block partials), so the
// result is deterministic.  part[0 .. nblk) holds the sums, part[nblk .. 2 nblk) the maxima.
// ---------------------------------------------------------------------------------
// A block takes panels of 128 rows x 128 columns: the weights are staged in LDS with coalesced 16-byte loads, and a
// thread walks the lane records of two neighbouring columns (adjacent in memory) against them, one 4-byte LDS read
// per row serving both.  The next panel's weights are in flight (in registers) while the present one is worked on.
// (Looking every weight's code up by its position instead reads the packed buffer four bytes at a time and computes
// a record address per weight.)  Bound by HBM next to its own instructions: 8192 x 28672, int4
// g = 64: 146 -> 125 us (4.8 TB/s) with the final sum.

// q of element e of the 32-row step t of a record as binary32, divided by CODE_UNIT<BITS> (a power of two: exact)
template <int BITS>
constexpr float CODE_UNIT = BITS == 4 ? 16.0f : 1.0f;
template <int BITS>
__device__ inline uint32_t step_word(const uint32_t (&d)[4], int t) {   // 3 and 4 bits: the step's eight nibbles
    if constexpr (BITS == 4) {
        return d[t] ^ 0x88888888u;                       // q in two's complement
    } else {
        return t < 3 ? d[t] : ((d[0] >> 3) & 0x11111111u) | ((d[1] >> 2) & 0x22222222u) | ((d[2] >> 1) & 0x44444444u);
    }
}
template <int BITS>
__device__ inline float code_value(const uint32_t (&d)[4], uint32_t w, int t, int e) {
    if constexpr (BITS == 8) {
        return (float)(int8_t)((d[2 * t + (e >> 2)] ^ 0x80808080u) >> (8 * (e & 3)));
    } else if constexpr (BITS == 4) {
        return __builtin_amdgcn_cvt_off_f32_i4(w >> (4 * fq_nibble_slot(e)));   // low nibble / 16
    } else {
        return (float)((w >> (4 * fq_nibble_slot(e))) & 7u) - 4.0f;
    }
}

template <int BITS, bool EXACT32>
__global__ __launch_bounds__(256) void fq_quant_error_kernel(const uint16_t* __restrict__ W,
                                                             const uint32_t* __restrict__ codes,
                                                             const uint16_t* __restrict__ scales, int64_t K,
                                                             int64_t N, int g, int sfmt,
                                                             double* __restrict__ part, int64_t nblk) {
    __shared__ __align__(16) uint16_t panel[FQ_QP_ROWS * FQ_QP_PITCH];
    __shared__ double sh_s[4];
    __shared__ double sh_m[4];
    constexpr int KBLK = fq_kblk(BITS);
    constexpr int STEPS = KBLK / FQ_KSTEP;
    constexpr int RW = fq_rec_bytes(BITS) / 4;                 // dwords per lane record
    constexpr int NL = FQ_QP_ROWS / 16;
    const int tid = threadIdx.x;
    const int64_t panels_n = (N + FQ_QP_COLS - 1) / FQ_QP_COLS;
    const int64_t panels = panels_n * ((K + FQ_QP_ROWS - 1) / FQ_QP_ROWS);
    const int64_t ntiles = N / FQ_NTILE;
    double sse = 0.0, mx = 0.0;
    float mxf = 0.0f;
    // With binary16 scales the error w - q s of one weight is formed in binary32, where it is exact: q s has at
    // most 19 significant bits, and when q != 0, |w| >= s / 2, so w, q s and their difference are multiples of
    // 2^(exponent of s - 11) below 2^(exponent of s + 8): 19 bits.  (q = 0: the error is w itself.)  Only its
    // square is accumulated in binary64; the largest magnitude is a binary32 maximum.  A third of the binary64
    // instructions per weight that the all-binary64 form needs, with the same bits in both results.
    const int lr = tid >> 4, c8 = (tid & 15) * 8;              // staging: rows lr + 16 i, eight columns
    const int c = (tid & 63) * 2, j = tid >> 6;                // work: columns c, c + 1, lane group j
    uint4 v[NL];
    auto load_panel = [&](int64_t pnl) {
        const int64_t n = (pnl % panels_n) * FQ_QP_COLS + c8, k = (pnl / panels_n) * FQ_QP_ROWS + lr;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            v[i] = make_uint4(0u, 0u, 0u, 0u);
            // (N is a multiple of 16: whole units)
            if (n < N && k + 16 * i < K) v[i] = *reinterpret_cast<const uint4*>(W + (k + 16 * i) * N + n);
        }
    };
    // a block walks panels blockIdx.x, blockIdx.x + gridDim.x, ... (one partial result per block)
    int64_t pnl = blockIdx.x;
    if (pnl < panels) load_panel(pnl);
    for (; pnl < panels; pnl += gridDim.x) {
        const int64_t n0 = (pnl % panels_n) * FQ_QP_COLS;
        const int64_t k0 = (pnl / panels_n) * FQ_QP_ROWS;
        __syncthreads();                                       // the previous panel has been read
#pragma unroll
        for (int i = 0; i < NL; ++i) *reinterpret_cast<uint4*>(&panel[(lr + 16 * i) * FQ_QP_PITCH + c8]) = v[i];
        __syncthreads();
        if (pnl + gridDim.x < panels) load_panel(pnl + gridDim.x);
        if (n0 + c >= N) continue;                             // (the barriers above are reached by every thread)
#pragma unroll
        for (int kbl = 0; kbl < FQ_QP_ROWS / KBLK; ++kbl) {
            const int64_t kb = k0 / KBLK + kbl;
            if (kb * KBLK >= K) break;
            const uint32_t* rec = codes + fq_rec((n0 + c) / FQ_NTILE, kb, ntiles, j * 16 + c % FQ_NTILE) * RW;
            uint32_t d0[4] = {0u, 0u, 0u, 0u}, d1[4] = {0u, 0u, 0u, 0u};
            if constexpr (BITS == 3) {
                // 24 bytes, 8-byte aligned (c is even)
                const uint2 x = *reinterpret_cast<const uint2*>(rec), y = *reinterpret_cast<const uint2*>(rec + 2),
                            u = *reinterpret_cast<const uint2*>(rec + 4);
                d0[0] = x.x; d0[1] = x.y; d0[2] = y.x; d1[0] = y.y; d1[1] = u.x; d1[2] = u.y;
            } else {
                const uint4 x = *reinterpret_cast<const uint4*>(rec), y = *reinterpret_cast<const uint4*>(rec + 4);
                d0[0] = x.x; d0[1] = x.y; d0[2] = x.z; d0[3] = x.w;
                d1[0] = y.x; d1[1] = y.y; d1[2] = y.z; d1[3] = y.w;
            }
#pragma unroll
            for (int t = 0; t < STEPS; ++t) {
                const int krel = kbl * KBLK + FQ_KSTEP * t + 8 * j;
                const uint32_t s2 = *reinterpret_cast<const uint32_t*>(scales + ((k0 + krel) / g) * N + n0 + c);
                const float f0 = scale_bits_to_float((uint16_t)s2, sfmt), f1 = scale_bits_to_float((uint16_t)(s2 >> 16), sfmt);
                const uint32_t w0 = BITS == 8 ? 0u : step_word<BITS>(d0, t), w1 = BITS == 8 ? 0u : step_word<BITS>(d1, t);
                const float u0 = CODE_UNIT<BITS> * f0, u1 = CODE_UNIT<BITS> * f1;   // exact (binary16 scales)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t w2 = *reinterpret_cast<const uint32_t*>(&panel[(krel + e) * FQ_QP_PITCH + c]);
                    const float wf0 = half_bits_to_float((uint16_t)w2), wf1 = half_bits_to_float((uint16_t)(w2 >> 16));
                    const float q0 = code_value<BITS>(d0, w0, t, e), q1 = code_value<BITS>(d1, w1, t, e);
                    if constexpr (EXACT32) {
                        const float e0 = __builtin_fmaf(-q0, u0, wf0), e1 = __builtin_fmaf(-q1, u1, wf1);
                        sse = __builtin_fma((double)e0, (double)e0, sse);
                        sse = __builtin_fma((double)e1, (double)e1, sse);
                        mxf = fmaxf(mxf, fmaxf(fabsf(e0), fabsf(e1)));
                    } else {
                        // (the products and differences are exact in binary64; a bfloat16 scale may reach 2^127)
                        const double e0 = __builtin_fma(-(double)(CODE_UNIT<BITS> * q0), (double)f0, (double)wf0);
                        const double e1 = __builtin_fma(-(double)(CODE_UNIT<BITS> * q1), (double)f1, (double)wf1);
                        sse = __builtin_fma(e0, e0, sse);
                        sse = __builtin_fma(e1, e1, sse);
                        mx = fmax(mx, fmax(fabs(e0), fabs(e1)));
                    }
                }
            }
        }
    }
    mx = fmax(mx, (double)mxf);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sse += __shfl_xor(sse, o, 64);
        mx = fmax(mx, __shfl_xor(mx, o, 64));
    }
    if ((tid & 63) == 0) {
        sh_s[tid >> 6] = sse;
        sh_m[tid >> 6] = mx;
    }
    __syncthreads();
    if (tid == 0) {
        part[blockIdx.x] = (sh_s[0] + sh_s[1]) + (sh_s[2] + sh_s[3]);
        part[nblk + blockIdx.x] = fmax(fmax(sh_m[0], sh_m[1]), fmax(sh_m[2], sh_m[3]));
    }
}

// (one block of 1024 threads: at most two partial results per thread, all of them in flight at once)
__global__ __launch_bounds__(1024) void fq_quant_error_final_kernel(const double* __restrict__ part, int64_t nblk,
                                                                    double* __restrict__ out) {
    __shared__ double sh_s[16];
    __shared__ double sh_m[16];
    double sse = 0.0, mx = 0.0;
    for (int64_t i = threadIdx.x; i < nblk; i += 1024) {
        sse += part[i];
        mx = fmax(mx, part[nblk + i]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sse += __shfl_xor(sse, o, 64);
        mx = fmax(mx, __shfl_xor(mx, o, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        sh_s[threadIdx.x >> 6] = sse;
        sh_m[threadIdx.x >> 6] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) {
            sse += sh_s[w];
            mx = fmax(mx, sh_m[w]);
        }
        out[0] = sse;
        out[1] = mx;
    }
}

}  // namespace

// ---------------------------------------------------------------------------------
// Measurement helper: reads a buffer and nothing else (16 bytes per lane, four non-temporal loads in
// flight per lane, grid-stride), one checksum word per block so that the loads cannot be dropped.
// Launched as 256 blocks of 768 threads, the shape of the small-M product kernel; of the shapes tried
// (256 ... 2048 blocks of 256 ... 1024 threads, 2 ... 8 loads in flight) this is among the fastest
// (7.1 - 7.3 TB/s), whereas grids whose stride between a lane's loads is 4 or 8 MiB lose 15 - 20 %, and
// ordinary (temporal) loads 10 %.
// ---------------------------------------------------------------------------------
typedef uint32_t probe_u32x4 __attribute__((ext_vector_type(4)));
#define FQ_PROBE_BLOCKS 256
#define FQ_PROBE_THREADS 768
__global__ __launch_bounds__(FQ_PROBE_THREADS) void fq_stream_read_kernel(const probe_u32x4* __restrict__ buf,
                                                                          size_t units,
                                                                          uint32_t* __restrict__ sink) {
    const size_t stride = (size_t)gridDim.x * FQ_PROBE_THREADS;
    size_t i = (size_t)blockIdx.x * FQ_PROBE_THREADS + threadIdx.x;
    probe_u32x4 acc = {0u, 0u, 0u, 0u};
    for (; i + 3 * stride < units; i += 4 * stride) {
        const probe_u32x4 a = __builtin_nontemporal_load(buf + i);
        const probe_u32x4 b = __builtin_nontemporal_load(buf + i + stride);
        const probe_u32x4 c = __builtin_nontemporal_load(buf + i + 2 * stride);
        const probe_u32x4 d = __builtin_nontemporal_load(buf + i + 3 * stride);
        acc ^= a ^ b ^ c ^ d;
    }
    for (; i < units; i += stride) acc ^= __builtin_nontemporal_load(buf + i);
    uint32_t x = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x ^= (uint32_t)__shfl_xor((int)x, o, 64);
    __shared__ uint32_t red[FQ_PROBE_THREADS / 64];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t y = 0;
        for (int w = 0; w < FQ_PROBE_THREADS / 64; ++w) y ^= red[w];
        sink[blockIdx.x] = y;
    }
}

// ----------------------------------------------------------------------------- launchers
namespace {
// Results that a call hands back to the host (a word of flags, two sums) are written by its last kernel into pinned host
// memory instead of being copied there behind it: a copy adds 8 - 12 us (fq_choose_group of 1792 x 2464 33 -> 22 us,
// fq_quant_error 35 -> 23; with fq_quantize between them 85 -> 60, on 8192 x 28672 454 -> 436).
// One page for the process, allocated by the first such call, in 64 slots of 64 bytes; a call holds one from before its
// launches until its stream has been waited for, whatever the thread, stream or device.  With all slots taken, or without the
// page, results go to the workspace and are copied.
constexpr int HOST_SLOTS = 64, HOST_SLOT_BYTES = 64;
std::mutex g_slots_mutex;
char* g_slots = nullptr;
bool g_slots_tried = false;
uint64_t g_slots_taken = 0;

struct host_slot {
    char* ptr = nullptr;
    host_slot() {
        std::lock_guard<std::mutex> lock(g_slots_mutex);
        if (!g_slots_tried) {
            g_slots_tried = true;
            // (another thread may be capturing a graph: this thread's allocation is none of its business)
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
            const bool exchanged = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
            void* p = nullptr;
            if (hipHostMalloc(&p, HOST_SLOTS * HOST_SLOT_BYTES, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess)
                g_slots = (char*)p;
            if (exchanged) (void)hipThreadExchangeStreamCaptureMode(&mode);
            (void)hipGetLastError();
        }
        if (!g_slots || g_slots_taken == ~(uint64_t)0) return;
        const int i = __builtin_ctzll(~g_slots_taken);
        g_slots_taken |= (uint64_t)1 << i;
        ptr = g_slots + i * HOST_SLOT_BYTES;
    }
    host_slot(const host_slot&) = delete;
    ~host_slot() {
        if (!ptr) return;
        std::lock_guard<std::mutex> lock(g_slots_mutex);
        g_slots_taken &= ~((uint64_t)1 << ((ptr - g_slots) / HOST_SLOT_BYTES));
    }
    // waits for the stream and takes the result from `out` (the slot, or device memory)
    int read(void* to, const void* out, size_t bytes, hipStream_t stream) {
        const bool launched = hipGetLastError() == hipSuccess;
        bool copied = true;
        if (launched && !ptr) copied = hipMemcpyAsync(to, out, bytes, hipMemcpyDeviceToHost, stream) == hipSuccess;
        if (hipStreamSynchronize(stream) != hipSuccess) {
            ptr = nullptr;          // a kernel may still write there: the slot is not given back
            return FQ_ERR_HIP;
        }
        if (!launched || !copied) return FQ_ERR_HIP;
        if (ptr) memcpy(to, ptr, bytes);
        return FQ_OK;
    }
};
}  // namespace

int fq_launch_stream_read_probe(const void* buf, size_t bytes, void* sink, hipStream_t stream) {
    hipLaunchKernelGGL(fq_stream_read_kernel, dim3(FQ_PROBE_BLOCKS), dim3(FQ_PROBE_THREADS), 0, stream, (const probe_u32x4*)buf, bytes / 16,
                       (uint32_t*)sink);
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

#define FQ_LAUNCH_PANEL(OWN)                                                                                  \
    do {                                                                                                      \
        if (bits == 3)                                                                                        \
            hipLaunchKernelGGL((fq_quantize_panel_kernel<3, OWN>), grid, dim3(256), 0, stream,                \
                               (const uint16_t*)W, K, N, g, L, sfmt, (uint16_t*)scales, (uint32_t*)codes);    \
        else if (bits == 4)                                                                                   \
            hipLaunchKernelGGL((fq_quantize_panel_kernel<4, OWN>), grid, dim3(256), 0, stream,                \
                               (const uint16_t*)W, K, N, g, L, sfmt, (uint16_t*)scales, (uint32_t*)codes);    \
        else                                                                                                  \
            hipLaunchKernelGGL((fq_quantize_panel_kernel<8, OWN>), grid, dim3(256), 0, stream,                \
                               (const uint16_t*)W, K, N, g, L, sfmt, (uint16_t*)scales, (uint32_t*)codes);    \
    } while (0)

int fq_launch_quantize(const void* W, int64_t K, int64_t N, int bits, int g, int sfmt, void* codes, void* scales,
                       hipStream_t stream) {
    const float L = (float)((1 << bits) - 1);
    if (g == 32 || g == 64 || g == 128) {
        dim3 grid((unsigned)((N + FQ_QP_COLS - 1) / FQ_QP_COLS), (unsigned)((K + FQ_QP_ROWS - 1) / FQ_QP_ROWS));
        FQ_LAUNCH_PANEL(true);
        return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
    }
    if (g >= 1024 && g % 128 == 0) {
        // two stages; the block maxima (K / 128 x N binary16 = K * N / 64 bytes) are parked in the
        // code buffer, which is only written by the encoding pass below
        uint16_t* fine = (uint16_t*)codes;
        dim3 block(16, 16);
        dim3 grid((unsigned)((N + 127) / 128), (unsigned)(K / 128));
        hipLaunchKernelGGL(fq_fine_absmax_kernel<256>, grid, block, 0, stream, (const uint16_t*)W, N, 128, fine, (uint32_t*)nullptr);
        dim3 grid2((unsigned)((N + 255) / 256), (unsigned)(K / g));
        hipLaunchKernelGGL(fq_scales_fold_kernel, grid2, dim3(256), 0, stream, (const uint16_t*)fine, N, g / 128, L,
                           sfmt, (uint16_t*)scales);
    } else {
        dim3 block(16, 16);
        dim3 grid((unsigned)((N + 127) / 128), (unsigned)(K / g));
        hipLaunchKernelGGL(fq_scales_kernel, grid, block, 0, stream, (const uint16_t*)W, K, N, g, L, sfmt,
                           (uint16_t*)scales);
    }
    {
        // encoding pass from LDS panels, with the scales just written
        dim3 grid((unsigned)((N + FQ_QP_COLS - 1) / FQ_QP_COLS), (unsigned)((K + FQ_QP_ROWS - 1) / FQ_QP_ROWS));
        FQ_LAUNCH_PANEL(false);
    }
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

int fq_launch_unpack(const void* codes, int64_t K, int64_t N, int bits, int8_t* q, hipStream_t stream) {
    dim3 block(256);
    dim3 grid((unsigned)((N + 255) / 256), (unsigned)(K < 16384 ? K : 16384));
    if (bits == 3)
        hipLaunchKernelGGL(fq_unpack_kernel<3>, grid, block, 0, stream, (const uint32_t*)codes, K, N, q);
    else if (bits == 4)
        hipLaunchKernelGGL(fq_unpack_kernel<4>, grid, block, 0, stream, (const uint32_t*)codes, K, N, q);
    else
        hipLaunchKernelGGL(fq_unpack_kernel<8>, grid, block, 0, stream, (const uint32_t*)codes, K, N, q);
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

int fq_launch_choose_group(const void* W, int64_t K, int64_t N, int g_top, int levels, float alpha,
                           uint32_t* flags_host, void* workspace, hipStream_t stream) {
    // workspace: [flags: flags, blocks that are done, copy for the host; 256 bytes][fine: (K / f) * N binary16]
    uint32_t* flags = (uint32_t*)workspace;
    host_slot slot;
    uint32_t* out = slot.ptr ? (uint32_t*)slot.ptr : flags + 2;
    uint16_t* fine = (uint16_t*)((char*)workspace + 256);
    const int f = g_top >> levels;
    {
        dim3 block(16, 16);
        dim3 grid((unsigned)((N + 127) / 128), (unsigned)(K / f));
        hipLaunchKernelGGL(fq_fine_absmax_kernel<256>, grid, block, 0, stream, (const uint16_t*)W, N, f, fine, flags);
    }
    {
        const float thr = 1.0f - alpha;
        if (levels <= 10) {
            // threads * R values per item: 8 * 2^lu columns of 2^levels fine blocks
            const int lr = levels < 3 ? levels : 3;
            int lu = lr - levels;
            while ((1 << (lu - lr + levels)) < FQ_TREE_THREADS) ++lu;
            const int64_t items_n = (N + ((int64_t)8 << lu) - 1) / ((int64_t)8 << lu), items = items_n * (K / g_top);
            const dim3 grid((unsigned)(items < FQ_TREE_BLOCKS ? items : FQ_TREE_BLOCKS));
#define FQ_TREE_GO(LR_)                                                                                               \
    hipLaunchKernelGGL(fq_halving_tree_kernel<LR_>, grid, dim3(FQ_TREE_THREADS), 0, stream, (const uint16_t*)fine, N, \
                       levels, lu, thr, items_n, items, flags, out)
            if (lr == 1) FQ_TREE_GO(1);
            else if (lr == 2) FQ_TREE_GO(2);
            else FQ_TREE_GO(3);
#undef FQ_TREE_GO
        } else {
            dim3 block(256);
            dim3 grid((unsigned)((N + 255) / 256), (unsigned)(K / g_top), (unsigned)levels);   // levels >= 1
            hipLaunchKernelGGL(fq_halving_flags_kernel, grid, block, 0, stream, (const uint16_t*)fine, N,
                               K / g_top, levels, thr, flags, out);
        }
    }
    return slot.read(flags_host, out, sizeof(uint32_t), stream);
}

int64_t fq_quant_error_blocks(int64_t K, int64_t N) {
    const int64_t panels = ((N + FQ_QP_COLS - 1) / FQ_QP_COLS) * ((K + FQ_QP_COLS - 1) / FQ_QP_COLS);
    return panels < 2048 ? panels : 2048;
}

int fq_launch_quant_error(const void* W, int64_t K, int64_t N, int bits, int g, int sfmt, const void* codes,
                          const void* scales, double* out_host2, void* workspace, hipStream_t stream) {
    // workspace: [out: 2 doubles][partials: 2 * nblk doubles]
    double* part = (double*)workspace + 2;
    host_slot slot;
    double* out = slot.ptr ? (double*)slot.ptr : (double*)workspace;
    const int64_t nblk = fq_quant_error_blocks(K, N);
    dim3 grid((unsigned)nblk);
#define FQ_QE_GO(B_, X_)                                                                                    \
    hipLaunchKernelGGL((fq_quant_error_kernel<B_, X_>), grid, dim3(256), 0, stream, (const uint16_t*)W,     \
                       (const uint32_t*)codes, (const uint16_t*)scales, K, N, g, sfmt, part, nblk)
    const bool x32 = sfmt == FQ_SCALE_F16;
    if (bits == 3) { if (x32) FQ_QE_GO(3, true); else FQ_QE_GO(3, false); }
    else if (bits == 4) { if (x32) FQ_QE_GO(4, true); else FQ_QE_GO(4, false); }
    else { if (x32) FQ_QE_GO(8, true); else FQ_QE_GO(8, false); }
#undef FQ_QE_GO
    hipLaunchKernelGGL(fq_quant_error_final_kernel, dim3(1), dim3(1024), 0, stream, (const double*)part, nblk, out);
    return slot.read(out_host2, out, sizeof(double) * 2, stream);
}
