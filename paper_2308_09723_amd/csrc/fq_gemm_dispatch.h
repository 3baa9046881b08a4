// Host-side dispatch templates of the product kernels (included by the per-type translation
// units fq_gemm_f16_4.hip ... so that they compile in parallel).
#ifndef FQ_GEMM_DISPATCH_H_
#define FQ_GEMM_DISPATCH_H_

#include <math.h>
#include <stdint.h>

#include "fq_gemm_config.h"
#include "fq_gemm_kernels.h"
#include "fq_lds_limit.h"

namespace fqd {

using namespace fqk;

template <int ACT, int BITS, int NT, int DEPTH, int MAXW, int AU>
int launch_skinny(const void* A, int64_t M, int64_t N, int64_t K, const void* codes, const void* scales, int g,
                  void* C, float* partial, const fq_gemm_plan& plan, uint64_t tag, hipStream_t stream) {
    const int kblk = fq_kblk(BITS);
    // scale rows per k-block: 1, KBLK / g, or one per 32-row step when g does not divide KBLK
    const int sr = (g % kblk) == 0 ? 1 : ((kblk % g) == 0 ? kblk / g : kblk / 32);
    const int ntiles = (int)(N / FQ_NTILE);
    const int ngroups = (ntiles + NT - 1) / NT;
    const int bgroups = (ngroups + plan.gp - 1) / plan.gp;
    const int kc = kblk / 8;
    const size_t lds_act = (size_t)2 * plan.kw * kc * FQ_SK_PITCH * 16;
    const size_t lds_red = (size_t)plan.gp * plan.kw * NT * 64 * 16;
    const size_t lds = lds_act > lds_red ? lds_act : lds_red;
    const uint32_t g32 = (uint32_t)(g / 32);
    const uint32_t g32_recip = (uint32_t)((((uint64_t)1 << 32) + g32 - 1) / g32);   // unused when g32 == 1
    constexpr int STEPS = fq_kblk(BITS) / FQ_KSTEP;
    auto kern = sr == 1 ? fq_gemm_skinny_kernel<ACT, BITS, NT, DEPTH, 1, MAXW, AU>
                        : (sr == 2 ? fq_gemm_skinny_kernel<ACT, BITS, NT, DEPTH, 2, MAXW, AU>
                                   : fq_gemm_skinny_kernel<ACT, BITS, NT, DEPTH, STEPS, MAXW, AU>);
    if (lds > 65536) {
        // more than the default dynamic LDS limit: raise it for this kernel (up to the 160 KiB of a CU)
        if (lds > 160 * 1024) return FQ_ERR_UNSUPPORTED;
        static std::atomic<uint64_t> raised[3];   // per instantiation: [scale rows per k-block]
        if (raise_lds_limit((const void*)kern, raised[sr == 1 ? 0 : (sr == 2 ? 1 : 2)]) != FQ_OK) return FQ_ERR_HIP;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(bgroups * plan.splits)), dim3((unsigned)(plan.gp * plan.kw * 64)),
                       lds, stream, (const uint16_t*)A, (const u32x4*)codes, (const uint16_t*)scales,
                       (uint16_t*)C, partial, (int)M, (int)N, (int)K, g32, g32_recip, plan.gp, plan.kw,
                       plan.splits, tag, fq_no_items{});
    return FQ_OK;
}

template <int ACT, int BITS, int NT, int DEPTH, int MAXW>
int launch_skinny_au(const void* A, int64_t M, int64_t N, int64_t K, const void* codes, const void* scales,
                     int g, void* C, float* partial, const fq_gemm_plan& plan, uint64_t tag, hipStream_t stream) {
    switch (plan.au) {
        case 1: return launch_skinny<ACT, BITS, NT, DEPTH, MAXW, 1>(A, M, N, K, codes, scales, g, C, partial, plan, tag, stream);
        case 2: return launch_skinny<ACT, BITS, NT, DEPTH, MAXW, 2>(A, M, N, K, codes, scales, g, C, partial, plan, tag, stream);
        default: return launch_skinny<ACT, BITS, NT, DEPTH, MAXW, 4>(A, M, N, K, codes, scales, g, C, partial, plan, tag, stream);
    }
}

// Mid-M streaming kernel (plan.kind == 2)
template <int ACT, int BITS, int NT, int MT, int MAXW>
int launch_mid(const void* A, int64_t M, int64_t N, int64_t K, const void* codes, const void* scales, int g, void* C,
               float* partial, const fq_gemm_plan& plan, uint64_t tag, hipStream_t stream) {
    constexpr int kblk = fq_kblk(BITS);
    constexpr int STEPS = kblk / FQ_KSTEP;
    const int sr = (g % kblk) == 0 ? 1 : ((kblk % g) == 0 ? kblk / g : STEPS);
    const int ngroups = (int)((N / FQ_NTILE + NT - 1) / NT);
    const int bgroups = (ngroups + plan.gp - 1) / plan.gp;
    const size_t lds_act = (size_t)mid_bufs(MT) * plan.kw * MT * 16 * (kblk / 8) * 16;
    const size_t lds_red = (size_t)plan.gp * plan.kw * NT * MT * 64 * 16;
    const size_t lds = lds_act > lds_red ? lds_act : lds_red;
    if (lds > 160 * 1024) return FQ_ERR_UNSUPPORTED;
    const uint32_t g32 = (uint32_t)(g / 32);
    const uint32_t g32_recip = (uint32_t)((((uint64_t)1 << 32) + g32 - 1) / g32);   // unused when g32 == 1
    auto kern = sr == 1 ? fq_gemm_mid_kernel<ACT, BITS, NT, MT, 1, MAXW>
                        : (sr == 2 ? fq_gemm_mid_kernel<ACT, BITS, NT, MT, 2, MAXW>
                                   : fq_gemm_mid_kernel<ACT, BITS, NT, MT, STEPS, MAXW>);
    if (lds > 65536) {
        static std::atomic<uint64_t> raised[3];   // per instantiation: [scale rows per k-block]
        if (raise_lds_limit((const void*)kern, raised[sr == 1 ? 0 : (sr == 2 ? 1 : 2)]) != FQ_OK) return FQ_ERR_HIP;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(bgroups * plan.splits)), dim3((unsigned)(plan.gp * plan.kw * 64)), lds, stream,
                       (const uint16_t*)A, (const u32x4*)codes, (const uint16_t*)scales, (uint16_t*)C, partial, (int)M,
                       (int)N, (int)K, g32, g32_recip, plan.gp, plan.kw, plan.splits, tag);
    return FQ_OK;
}

// Tiles of up to 48 rows of a grouped product: the mid-M kernel, no split of K over the grid.
template <int ACT, int BITS, int NT>
int launch_mid_items(const void* A, const fq_small_items& items, int count, int rows_max, const fq_small_shape& sh, int64_t N,
                     int64_t K, const void* codes, const void* scales, int g, void* C, hipStream_t stream) {
    constexpr int MAXW = 12;
    constexpr int kblk = fq_kblk(BITS);
    constexpr int STEPS = kblk / FQ_KSTEP;
    const int sr = (g % kblk) == 0 ? 1 : ((kblk % g) == 0 ? kblk / g : STEPS);
    const int ngroups = (int)((N / FQ_NTILE + NT - 1) / NT);
    // (three tiles of 32 rows hold as much as two of 48, and more than what lower items take)
    const int mt = rows_max <= 16 ? 1 : 2;
    const size_t lds_act = (size_t)mid_bufs(mt) * sh.kw * mt * 16 * (kblk / 8) * 16;
    const size_t lds_red = (size_t)sh.gp * sh.kw * NT * ((rows_max + 15) / 16) * 64 * 16;
    const size_t lds = lds_act > lds_red ? lds_act : lds_red;
    if (lds > 160 * 1024 || sh.gp * sh.kw > MAXW) return FQ_ERR_UNSUPPORTED;
    const uint32_t g32 = (uint32_t)(g / 32);
    const uint32_t g32_recip = (uint32_t)((((uint64_t)1 << 32) + g32 - 1) / g32);   // unused when g32 == 1
    auto kern = sr == 1 ? fq_gemm_mid_items_kernel<ACT, BITS, NT, 1, MAXW>
                        : (sr == 2 ? fq_gemm_mid_items_kernel<ACT, BITS, NT, 2, MAXW>
                                   : fq_gemm_mid_items_kernel<ACT, BITS, NT, STEPS, MAXW>);
    if (lds > 65536) {
        static std::atomic<uint64_t> raised[3];   // per instantiation: [scale rows per k-block]
        if (raise_lds_limit((const void*)kern, raised[sr == 1 ? 0 : (sr == 2 ? 1 : 2)]) != FQ_OK) return FQ_ERR_HIP;
    }
    const int64_t blocks = (int64_t)((ngroups + sh.gp - 1) / sh.gp) * count;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3((unsigned)(sh.gp * sh.kw * 64)), lds, stream, (const uint16_t*)A,
                       (const u32x4*)codes, (const uint16_t*)scales, (uint16_t*)C, (int)N, (int)K, g32, g32_recip, sh.gp, sh.kw,
                       items);
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

// rows whose units of 8 values fit four waves' registers take those, longer ones sixteen waves
// SCALES: the `count` bfloat16 scales are searched for their largest in the same launch
template <bool SCALES>
inline void launch_rows_to_f16(const void* A, int64_t M, int64_t K, uint16_t* A16, float* rowscale, const void* scales,
                               int64_t count, hipStream_t stream) {
    const bool small = K <= 256 * ROW_UNITS * 8;
    auto kern = small ? fq_rows_to_f16_kernel<256, SCALES> : fq_rows_to_f16_kernel<1024, SCALES>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(M + (SCALES ? FQ_SCALE_PARTS : 0))), dim3(small ? 256 : 1024), 0, stream,
                       (const uint16_t*)A, (int)K, A16, rowscale, (const uint16_t*)scales, count / 8,
                       (uint32_t*)(rowscale + M + 2));
}

template <int ACT, int BITS>
int launch_typed(const void* A, int64_t M, int64_t N, int64_t K, const void* codes, const void* scales,
                 int g, void* C, void* workspace, const fq_gemm_plan& plan, hipStream_t stream) {
    const int ntiles = (int)(N / FQ_NTILE);
    float* partial = (float*)workspace;
    // The streaming kernels add a split of K themselves where a tile's partial sums are few enough for one block; not where
    // the ticket in C would be misaligned, nor where C lies on what other blocks still read (a product written over its own
    // activations: the separate sum writes once everything is read), nor where C or the scratch is not the
    // device's own memory.
    const int tile_cols = plan.gp * FQ_NTILE * (plan.kind == 0 ? SKINNY_VARIANTS[plan.variant].nt : plan.nt);
    const bool sums = plan.kind != 1 && fq_sums_splits((int)M, tile_cols, plan.splits, C) &&
                      !fq_overlaps(C, (size_t)(M * N * 2), {{A, (size_t)(M * K * 2)}, {codes, (size_t)(K * N * BITS / 8)},
                                   {scales, (size_t)(K / g * N * 2)}, {partial, fq_partial_bytes(plan, M, N)}}) &&
                      fq_counts_tickets(C, partial, stream);
    const uint64_t tag = sums ? fq_next_tag() : 0;
    if (plan.kind == 0) {
        int st;
        switch (plan.variant) {
            case 0: st = launch_skinny_au<ACT, BITS, 3, 2, 12>(A, M, N, K, codes, scales, g, C, partial, plan, tag, stream); break;
            case 1: st = launch_skinny_au<ACT, BITS, 3, 3, 8>(A, M, N, K, codes, scales, g, C, partial, plan, tag, stream); break;
            case 2: st = launch_skinny_au<ACT, BITS, 1, 4, 12>(A, M, N, K, codes, scales, g, C, partial, plan, tag, stream); break;
            default: st = launch_skinny_au<ACT, BITS, 2, 3, 12>(A, M, N, K, codes, scales, g, C, partial, plan, tag, stream); break;
        }
        if (st != FQ_OK) return st;
    } else if (plan.kind == 2) {
        int st;
#define FQ_MID_LAUNCH(NT_, MT_) st = launch_mid<ACT, BITS, NT_, MT_, 12>(A, M, N, K, codes, scales, g, C, partial, plan, tag, stream)
        if (plan.nt == 1 && plan.mt == 2) FQ_MID_LAUNCH(1, 2);
        else if (plan.nt == 1) FQ_MID_LAUNCH(1, 3);
        else if (plan.mt == 2) FQ_MID_LAUNCH(MMA_NT, 2);
        else FQ_MID_LAUNCH(MMA_NT, 3);
#undef FQ_MID_LAUNCH
        if (st != FQ_OK) return st;
    } else if (plan.kind == 3) {
        // row blocks of the mid-M kernel: as few as 48 rows allow, of nearly equal height, all without a bias
        fq_small_items items;
        items.codes_stride16 = items.scales_stride = 0;
        int count = 0;
        for (int32_t r = 0, take = 0; r < M; r += take) {
            take = fq_mid_rows((int32_t)M - r);
            items.row0[count] = r;
            items.rows[count] = (uint8_t)(take | FQ_ITEM_EXACT);
            items.expert[count] = 0;
            ++count;
        }
        const int st = plan.nt == 1 ? launch_mid_items<ACT, BITS, 1>(A, items, count, 48, {plan.gp, plan.kw}, N, K, codes, scales, g, C, stream)
                                    : launch_mid_items<ACT, BITS, MMA_NT>(A, items, count, 48, {plan.gp, plan.kw}, N, K, codes, scales, g, C, stream);
        if (st != FQ_OK) return st;
    } else {
        // rows of K per k-block of this block shape (two layout blocks at a time for 8-bit codes in the
        // 8-wave shapes of 80 rows and more), and the scale rows such a k-block spans: 1, kblk / g, or one per 32-row step
        const int kblk = fq_mma_kblk(BITS, plan.mt, plan.waves, K, g);
        const bool wide = kblk != fq_kblk(BITS);
        const int sr = (g % kblk) == 0 ? 1 : ((kblk % g) == 0 ? kblk / g : kblk / 32);
        const int bm = plan.mt * 16;
        const int nblocks_n = (ntiles + plan.waves * plan.nt - 1) / (plan.waves * plan.nt);
        const int nblocks_m = (int)((M + bm - 1) / bm);
        // ring depth of the pipelined form per block shape (0 = two-buffer form); must match the
        // instantiations below
        const bool flexible = fq_flexible(plan);
        const int ring = plan.mt >= 5 ? (plan.waves == 8 ? 2 : 0) : (plan.mt == 4 ? FQ_RING_MT4 : FQ_RING_MT2);
        // (an LDS tile of the flexible shapes is a whole number of rounds of their eight waves' direct loads)
        const int units = flexible ? ((kblk / 8) * bm + 511) / 512 * 512 : (kblk / 8) * bm;
        const size_t lds = (size_t)(ring ? ring + 1 : 2) * units * 16;
        const int64_t tiles = (int64_t)nblocks_n * nblocks_m;
        dim3 grid((unsigned)(plan.tail_tiles > 0 ? tiles - plan.tail_tiles + (int64_t)plan.tail_tiles * plan.tail_splits
                                                 : tiles * plan.splits));
        fq_group_items none;
        none.count = 0;
#define FQ_MMA_LAUNCH_SR(ACT_, A_, RS_, MT_, W_, PIPE_, SR_, KREC_)                                       \
    FQ_MMA_LAUNCH_NT(ACT_, A_, RS_, MT_, MMA_NT, W_, PIPE_, SR_, use_post(ACT_, BITS, MT_, SR_, PIPE_), KREC_)
#define FQ_MMA_LAUNCH_NT(ACT_, A_, RS_, MT_, NT_, W_, PIPE_, SR_, POST_, KREC_)                           \
    do {                                                                                                \
        auto kern = fq_gemm_mma_kernel<ACT_, BITS, MT_, NT_, W_, SR_, false, PIPE_, POST_, KREC_>;      \
        if (lds > 65536) {                                                                              \
            static std::atomic<uint64_t> raised;                                                        \
            if (raise_lds_limit((const void*)kern, raised) != FQ_OK) return FQ_ERR_HIP;                 \
        }                                                                                               \
        hipLaunchKernelGGL(kern, grid, dim3(W_ * 64), lds, stream, (const uint16_t*)(A_),               \
                           (const u32x4*)codes, (const uint16_t*)scales, (uint16_t*)C, partial, (int)M, \
                           (int)N, (int)K, g, plan.kb_per_split, plan.splits, nblocks_n, nblocks_m,     \
                           (int64_t)0, (int64_t)0, none, plan.tail_tiles, plan.tail_splits,             \
                           plan.tail_kbs, (const float*)(RS_));                                         \
    } while (0)
#define FQ_MMA_LAUNCH_ACT(ACT_, A_, RS_, MT_, W_, PIPE_)                                                \
    do {                                                                                                \
        if (sr == 1) FQ_MMA_LAUNCH_SR(ACT_, A_, RS_, MT_, W_, PIPE_, 1, 1);                             \
        else if (sr == 2) FQ_MMA_LAUNCH_SR(ACT_, A_, RS_, MT_, W_, PIPE_, 2, 1);                        \
        else if constexpr (BITS != 8) FQ_MMA_LAUNCH_SR(ACT_, A_, RS_, MT_, W_, PIPE_, 4, 1);            \
    } while (0)
// the 128-row, 8-wave shape: 8-bit codes take two layout k-blocks per k-block where K allows it
#define FQ_MMA_LAUNCH_BIG(ACT_, A_, RS_)                                                                \
    do {                                                                                                \
        if constexpr (BITS == 8) {                                                                      \
            if (wide) { /* (one scale row per k-block by construction) */                              \
                FQ_MMA_LAUNCH_SR(ACT_, A_, RS_, 8, 8, 2, 1, 2);                                         \
            } else {                                                                                    \
                FQ_MMA_LAUNCH_ACT(ACT_, A_, RS_, 8, 8, 2);                                              \
            }                                                                                           \
        } else {                                                                                        \
            FQ_MMA_LAUNCH_ACT(ACT_, A_, RS_, 8, 8, 2);                                                  \
        }                                                                                               \
    } while (0)
// the flexible shapes
#define FQ_MMA_LAUNCH_FLEX(ACT_, A_, RS_, MT_, NT_)                                                     \
    do {                                                                                                \
        if constexpr (BITS == 8) {                                                                      \
            if (wide) FQ_MMA_LAUNCH_NT(ACT_, A_, RS_, MT_, NT_, 8, 2, 1, false, 2);                     \
            else if (sr == 1) FQ_MMA_LAUNCH_NT(ACT_, A_, RS_, MT_, NT_, 8, 2, 1, false, 1);             \
            else FQ_MMA_LAUNCH_NT(ACT_, A_, RS_, MT_, NT_, 8, 2, 2, false, 1);                          \
        } else {                                                                                        \
            if (sr == 1) FQ_MMA_LAUNCH_NT(ACT_, A_, RS_, MT_, NT_, 8, 2, 1, true, 1);                   \
            else if (sr == 2) FQ_MMA_LAUNCH_NT(ACT_, A_, RS_, MT_, NT_, 8, 2, 2, false, 1);             \
            else FQ_MMA_LAUNCH_NT(ACT_, A_, RS_, MT_, NT_, 8, 2, 4, false, 1);                          \
        }                                                                                               \
    } while (0)
#define FQ_MMA_LAUNCH_FLEXIBLE(ACT_, A_, RS_)                                                           \
    do {                                                                                                \
        if (plan.nt == 2 && plan.mt == 5) FQ_MMA_LAUNCH_FLEX(ACT_, A_, RS_, 5, 2);                      \
        else if (plan.nt == 2 && plan.mt == 6) FQ_MMA_LAUNCH_FLEX(ACT_, A_, RS_, 6, 2);                 \
        else if (plan.nt == 2 && plan.mt == 7) FQ_MMA_LAUNCH_FLEX(ACT_, A_, RS_, 7, 2);                 \
        else if (plan.nt == 2 && plan.mt == 8) FQ_MMA_LAUNCH_FLEX(ACT_, A_, RS_, 8, 2);                 \
        else if (plan.nt == 3 && plan.mt == 5) FQ_MMA_LAUNCH_FLEX(ACT_, A_, RS_, 5, 3);                 \
        else return FQ_ERR_UNSUPPORTED;                                                                 \
    } while (0)
#define FQ_MMA_LAUNCH(MT_, W_, PIPE_) FQ_MMA_LAUNCH_ACT(ACT, A, nullptr, MT_, W_, PIPE_)
        bool launched = false;
        if constexpr (ACT == FQ_BF16) {
            if (fq_via_f16(FQ_BF16, FQ_SCALE_F16, plan, N)) {
                // bf16 activations on the fp16 matrix path: rows rewritten as binary16 first (the
                // buffers sit behind the split-K partials in the workspace)
                char* extra = (char*)workspace + fq_partial_bytes(plan, M, N);
                uint16_t* A16 = (uint16_t*)extra;
                float* rs = (float*)(extra + fq_a16_bytes(M, K));
                launch_rows_to_f16<false>(A, M, K, A16, rs, nullptr, 0, stream);
                if (flexible) FQ_MMA_LAUNCH_FLEXIBLE(FQ_BF16_VIA_F16, A16, rs);
                else if (plan.waves == 8) FQ_MMA_LAUNCH_BIG(FQ_BF16_VIA_F16, A16, rs);
                else FQ_MMA_LAUNCH_ACT(FQ_BF16_VIA_F16, A16, rs, 8, 4, 0);
                launched = true;
            }
        }
        if constexpr (ACT == FQ_BF16_BS) {
            if (fq_via_f16(FQ_BF16, FQ_SCALE_BF16, plan, N)) {
                // the same with bfloat16 scales: their common power of two is searched in the same launch
                char* extra = (char*)workspace + fq_partial_bytes(plan, M, N);
                uint16_t* A16 = (uint16_t*)extra;
                float* rs = (float*)(extra + fq_a16_bytes(M, K));
                launch_rows_to_f16<true>(A, M, K, A16, rs, scales, (K / g) * N, stream);
                if (flexible) FQ_MMA_LAUNCH_FLEXIBLE(FQ_BF16S_VIA_F16, A16, rs);
                else if (plan.waves == 8) FQ_MMA_LAUNCH_BIG(FQ_BF16S_VIA_F16, A16, rs);
                else FQ_MMA_LAUNCH_ACT(FQ_BF16S_VIA_F16, A16, rs, 8, 4, 0);
                launched = true;
            }
        }
        if (launched) {
        } else if (flexible) {
            // (bf16 activations take these shapes on the fp16 matrix path only)
            if constexpr (ACT == FQ_F16) FQ_MMA_LAUNCH_FLEXIBLE(ACT, A, nullptr);
            else return FQ_ERR_UNSUPPORTED;
        } else if (plan.waves == 8) {
            if (plan.mt == 2) FQ_MMA_LAUNCH(2, 8, FQ_RING_MT2);
            else if (plan.mt == 4) FQ_MMA_LAUNCH(4, 8, FQ_RING_MT4);
            else FQ_MMA_LAUNCH_BIG(ACT, A, nullptr);
        } else {
            if (plan.mt == 2) FQ_MMA_LAUNCH(2, 4, FQ_RING_MT2);
            else if (plan.mt == 4) FQ_MMA_LAUNCH(4, 4, FQ_RING_MT4);
            else FQ_MMA_LAUNCH(8, 4, 0);
        }
#undef FQ_MMA_LAUNCH
#undef FQ_MMA_LAUNCH_BIG
#undef FQ_MMA_LAUNCH_ACT
#undef FQ_MMA_LAUNCH_SR
#undef FQ_MMA_LAUNCH_NT
#undef FQ_MMA_LAUNCH_FLEX
#undef FQ_MMA_LAUNCH_FLEXIBLE
    }
    if (plan.kind == 1 && plan.tail_tiles > 0) {
        const int bm = plan.mt * 16;
        const int bn_cols = plan.waves * plan.nt * FQ_NTILE;
        const int nblocks_n = (ntiles + plan.waves * plan.nt - 1) / (plan.waves * plan.nt);
        const int nblocks_m = (int)((M + bm - 1) / bm);
        hipLaunchKernelGGL(fq_reduce_tail_kernel<(ACT == FQ_F16 ? FQ_F16 : FQ_BF16)>, dim3((unsigned)plan.tail_tiles, (unsigned)plan.mt), dim3(256), 0, stream,
                           (const float*)partial, plan.tail_splits, (int)M, (int)N, nblocks_n, nblocks_m,
                           nblocks_n * nblocks_m - plan.tail_tiles, bm, bn_cols, (uint16_t*)C);
    }
    if (plan.splits > 1 && !sums) {
        const int64_t MN = M * N;
        dim3 grid((unsigned)((MN / 4 + 255) / 256));
        hipLaunchKernelGGL(fq_reduce_kernel<(ACT == FQ_F16 ? FQ_F16 : FQ_BF16)>, grid, dim3(256), 0, stream, (const float*)partial,
                           plan.splits, MN, (uint16_t*)C);
    }
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

// The experts with few rows of a grouped product: the small-M kernel, items of 1 .. 16 rows.  Block shape: gp column
// groups (of three tiles) x kw k-workers, gp * kw waves; gp is at least what lets one activation unit per lane hold a
// super-block's slice of the tallest item (more units per lane spill registers).
template <int ACT, int BITS>
int launch_grouped_small(const void* A, const fq_small_items& items, int count, int rows_max, int64_t N, int64_t K,
                         const void* codes, const void* scales, int g, void* C, hipStream_t stream) {
    constexpr int NT = 3, DEPTH = 2, MAXW = 12;
    constexpr int kblk = fq_kblk(BITS);
    constexpr int STEPS = kblk / FQ_KSTEP;
    const int sr = (g % kblk) == 0 ? 1 : ((kblk % g) == 0 ? kblk / g : STEPS);
    const int KB = (int)(K / kblk);
    const int ngroups = (int)((N / FQ_NTILE + NT - 1) / NT);
    const fq_small_shape sh = fq_plan_grouped_small(count, rows_max * (kblk / 8), ngroups, KB);
    const size_t lds_act = (size_t)2 * sh.kw * (kblk / 8) * FQ_SK_PITCH * 16;
    const size_t lds_red = (size_t)sh.gp * sh.kw * NT * 64 * 16;
    const size_t lds = lds_act > lds_red ? lds_act : lds_red;       // at most 52 KiB (gp >= 2)
    const uint32_t g32 = (uint32_t)(g / 32);
    const uint32_t g32_recip = (uint32_t)((((uint64_t)1 << 32) + g32 - 1) / g32);   // unused when g32 == 1
    auto kern = sr == 1 ? fq_gemm_skinny_kernel<ACT, BITS, NT, DEPTH, 1, MAXW, 1, fq_small_items>
                        : (sr == 2 ? fq_gemm_skinny_kernel<ACT, BITS, NT, DEPTH, 2, MAXW, 1, fq_small_items>
                                   : fq_gemm_skinny_kernel<ACT, BITS, NT, DEPTH, STEPS, MAXW, 1, fq_small_items>);
    const int64_t blocks = (int64_t)((ngroups + sh.gp - 1) / sh.gp) * count;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3((unsigned)(sh.gp * sh.kw * 64)), lds, stream, (const uint16_t*)A,
                       (const u32x4*)codes, (const uint16_t*)scales, (uint16_t*)C, (float*)nullptr, 0, (int)N, (int)K, g32,
                       g32_recip, sh.gp, sh.kw, 1, (uint64_t)0, items);
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
}

// Grouped (per-expert) product.  Every expert's rows are cut into row tiles (fq_next_tile), and the tiles of each class go
// to the kernel instantiated for it: experts with few rows then stream their weights through small tiles instead of
// multiplying mostly padding.  Experts without rows produce no tile.
template <int ACT, int BITS>
int launch_grouped_typed(const void* A, const int32_t* offsets, int E, const fq_grouped_plan& plan, int64_t N, int64_t K,
                         const void* codes, const void* scales, int g, void* C, const hipStream_t* streams) {
    const int ntiles = (int)(N / FQ_NTILE);
    const int64_t codes_stride16 = (int64_t)(K * N * BITS / 8) / 16;
    const int64_t scales_stride = (K / g) * N;
    fq_group_items items;
    for (int cls = FQ_TILE_128; cls <= FQ_TILE_64; ++cls) {
        const int mt = cls == FQ_TILE_128 ? 8 : 4;
        const int bm = mt * 16;
        // 8-wave blocks (384 columns), measured 1 - 5 % faster than 4-wave ones also for the 64-row tiles (64 experts of
        // 4096 x 16384 / 16384 x 4096)
        const int waves = 8;
        const hipStream_t stream = streams[cls];
        const int nblocks_n = (ntiles + waves * MMA_NT - 1) / (waves * MMA_NT);
        const int ring = mt == 8 ? 2 : FQ_RING_MT4;
        // rows of K per k-block of this tile size (8-bit codes: two layout blocks at a time in the 128-row
        // shape where K and g allow it) and the scale rows such a k-block spans
        const int kblk = fq_mma_kblk(BITS, mt, waves, K, g);
        const bool wide = kblk != fq_kblk(BITS);
        const int sr = (g % kblk) == 0 ? 1 : ((kblk % g) == 0 ? kblk / g : kblk / 32);
        const int KB = (int)(K / kblk);
        const size_t lds = (size_t)(ring ? ring + 1 : 2) * (kblk / 8) * bm * 16;
        items.count = 0;
        auto flush_items = [&]() -> int {
            if (items.count == 0) return FQ_OK;
            dim3 grid((unsigned)((int64_t)nblocks_n * items.count));
#define FQ_GROUPED_LAUNCH_SR(MT_, W_, PIPE_, SR_, KREC_)                                                 \
    do {                                                                                                \
        auto kern = fq_gemm_mma_kernel<ACT, BITS, MT_, MMA_NT, W_, SR_, true, PIPE_,                   \
                                       use_post(ACT, BITS, MT_, SR_, PIPE_), KREC_>;                    \
        if (lds > 65536) {                                                                              \
            static std::atomic<uint64_t> raised;                                                        \
            if (raise_lds_limit((const void*)kern, raised) != FQ_OK) return FQ_ERR_HIP;                 \
        }                                                                                               \
        hipLaunchKernelGGL(kern, grid, dim3(W_ * 64), lds, stream, (const uint16_t*)A,                  \
                           (const u32x4*)codes, (const uint16_t*)scales, (uint16_t*)C, (float*)nullptr, \
                           0, (int)N, (int)K, g, KB, 1, nblocks_n, items.count, codes_stride16,         \
                           scales_stride, items, 0, 1, 0, (const float*)nullptr);                       \
    } while (0)
#define FQ_GROUPED_LAUNCH(MT_, W_, PIPE_)                                                               \
    do {                                                                                                \
        if (sr == 1) FQ_GROUPED_LAUNCH_SR(MT_, W_, PIPE_, 1, 1);                                        \
        else if (sr == 2) FQ_GROUPED_LAUNCH_SR(MT_, W_, PIPE_, 2, 1);                                   \
        else if constexpr (BITS != 8) FQ_GROUPED_LAUNCH_SR(MT_, W_, PIPE_, 4, 1);                       \
    } while (0)
            if (mt == 8) {
                if constexpr (BITS == 8) {
                    if (wide) FQ_GROUPED_LAUNCH_SR(8, 8, 2, 1, 2);
                    else FQ_GROUPED_LAUNCH(8, 8, 2);
                } else {
                    FQ_GROUPED_LAUNCH(8, 8, 2);
                }
            }
            else FQ_GROUPED_LAUNCH(4, 8, FQ_RING_MT4);
#undef FQ_GROUPED_LAUNCH
#undef FQ_GROUPED_LAUNCH_SR
            items.count = 0;
            return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_HIP;
        };
        for (int e = 0; e < E; ++e) {
            for (int32_t r = offsets[e], take = 0; r < offsets[e + 1]; r += take) {
                if (fq_next_tile(plan, offsets[e + 1] - r, &take) != cls) continue;
                const int i = items.count++;
                items.row0[i] = r;
                items.rows[i] = (int16_t)take;
                items.expert[i] = (int16_t)e;
                if (items.count == 256) {
                    const int st = flush_items();
                    if (st != FQ_OK) return st;
                }
            }
        }
        const int st = flush_items();
        if (st != FQ_OK) return st;
    }
    fq_small_items small;
    small.codes_stride16 = codes_stride16;
    small.scales_stride = scales_stride;
    int count = 0, rows_max = 0;
    auto flush_small = [&](bool mid) -> int {
        const int n = count, most = rows_max;
        count = rows_max = 0;
        if (n == 0) return FQ_OK;
        if (mid) return launch_mid_items<ACT, BITS, MMA_NT>(A, small, n, most, plan.mid, N, K, codes, scales, g, C, streams[FQ_TILE_MID]);
        return launch_grouped_small<ACT, BITS>(A, small, n, most, N, K, codes, scales, g, C, streams[FQ_TILE_SMALL]);
    };
    // the tallest tiles of the mid-M kernel first, those of the small-M kernel last
    for (int height = 48; height >= 0; height -= 16) {
        const int cls = height > 0 ? FQ_TILE_MID : FQ_TILE_SMALL;
        for (int e = 0; e < E; ++e) {
            for (int32_t r = offsets[e], take = 0; r < offsets[e + 1]; r += take) {
                if (fq_next_tile(plan, offsets[e + 1] - r, &take) != cls || (height > 0 && (take + 15) / 16 * 16 != height)) continue;
                small.row0[count] = r;
                // (an expert of up to 48 rows, and what 128- or 64-row tiles leave over, keep the operands, biased ones in
                // bfloat16, that a product of as many rows has)
                const bool exact = plan.cut == FQ_CUT_MID && offsets[e + 1] - offsets[e] > 48;
                small.rows[count] = (uint8_t)(take | (exact ? FQ_ITEM_EXACT : 0));
                small.expert[count] = (uint8_t)e;
                const int32_t as = exact && take <= 16 ? 17 : take;      // (an exact item takes two row tiles at least)
                rows_max = as > rows_max ? as : rows_max;
                if (++count == 256) {
                    const int st = flush_small(height > 0);
                    if (st != FQ_OK) return st;
                }
            }
        }
        if (height > 16) continue;          // (one launch for all heights)
        const int st = flush_small(height > 0);
        if (st != FQ_OK) return st;
    }
    return FQ_OK;
}


}  // namespace fqd

// Explicitly instantiated once per (activation type, code width) in its own translation unit.
#define FQ_INSTANTIATE_GEMM(ACT, BITS)                                                                     \
    int fq_launch_typed_##ACT##_##BITS(const void* A, int64_t M, int64_t N, int64_t K, const void* codes,  \
                                       const void* scales, int g, void* C, void* workspace,                \
                                       const fq_gemm_plan& plan, hipStream_t stream) {                     \
        return fqd::launch_typed<ACT, BITS>(A, M, N, K, codes, scales, g, C, workspace, plan, stream);     \
    }                                                                                                      \
    int fq_launch_grouped_typed_##ACT##_##BITS(const void* A, const int32_t* offsets, int E,               \
                                               const fq_grouped_plan& plan, int64_t N, int64_t K,          \
                                               const void* codes, const void* scales, int g, void* C,      \
                                               const hipStream_t* streams) {                               \
        return fqd::launch_grouped_typed<ACT, BITS>(A, offsets, E, plan, N, K, codes, scales, g, C,        \
                                                    streams);                                              \
    }

#endif  // FQ_GEMM_DISPATCH_H_
