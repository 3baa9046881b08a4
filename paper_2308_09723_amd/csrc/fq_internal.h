// Internal launcher declarations shared by the translation units of libfq.
#ifndef FQ_INTERNAL_H_
#define FQ_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <initializer_list>
#include <stddef.h>
#include <stdint.h>

#include "../../include/fq.h"

// quantiser side (sfmt: an fq_scale_format)
int fq_launch_quantize(const void* W, int64_t K, int64_t N, int bits, int g, int sfmt, void* codes, void* scales,
                       hipStream_t stream);
int fq_launch_unpack(const void* codes, int64_t K, int64_t N, int bits, int8_t* q, hipStream_t stream);
int64_t fq_quant_error_blocks(int64_t K, int64_t N);
int fq_launch_quant_error(const void* W, int64_t K, int64_t N, int bits, int g, int sfmt, const void* codes,
                          const void* scales, double* out_host2, void* workspace, hipStream_t stream);
int fq_launch_choose_group(const void* W, int64_t K, int64_t N, int g_top, int levels, float alpha,
                           uint32_t* flags_host, void* workspace, hipStream_t stream);

// measurement helper: a kernel that only reads a buffer
int fq_launch_stream_read_probe(const void* buf, size_t bytes, void* sink, hipStream_t stream);
size_t fq_mfma_probe_operand_bytes();
size_t fq_mfma_probe_sink_bytes();
double fq_mfma_probe_flops(int iterations, int int8);
int fq_launch_mfma_rate_probe(const void* operands, void* sink, int iterations, int lds_reads, int int8,
                              hipStream_t stream);

// A tag for the tickets of one call (fq_split_sum.h); never 0.
uint64_t fq_next_tag();
// Whether C is memory that tickets can be counted in and the blocks of one kernel can hand each other partial sums through
// `partial`: both allocated on the stream's device, in no special way.
bool fq_counts_tickets(const void* C, const void* partial, hipStream_t stream);
// Whether `bytes` bytes from C on share memory with one of the buffers that a call reads.
struct fq_span {
    const void* p;
    size_t bytes;
};
inline bool fq_overlaps(const void* C, size_t bytes, std::initializer_list<fq_span> read) {
    for (const fq_span& r : read)
        if ((uintptr_t)C < (uintptr_t)r.p + r.bytes && (uintptr_t)r.p < (uintptr_t)C + bytes) return true;
    return false;
}

// product side
struct fq_gemm_plan {
    int kind;      // 0 = skinny (M <= 16), 1 = tiled, 2 = mid-M streaming (17 <= M <= 48), 3 = its row blocks (M > 48)
    int mt;        // row tiles of 16 per block (tiled and mid-M kernel)
    int nt;        // column tiles of 16 per wave: tiled kernel 3, or 2 in the flexible shapes; mid-M kernel 3 or 1
    int waves;     // waves per block
    int variant;   // small-M kernel: which compiled variant (NT, ring depth, register class)
    int gp, kw;    // small-M and mid-M kernel: column groups x k-workers per block
    int au;        // small-M kernel: activation units a lane stages per super-block (1, 2 or 4)
    int splits;    // split-K factor (>= 1)
    int kb_per_split;   // k-blocks per grid split (tiled) or per wave (small-M)
    // tiled kernel, splits == 1 only: the last `tail_tiles` output tiles (the partly filled last round
    // of blocks) are split `tail_splits` ways along K so that they fill the idle compute units
    int tail_tiles, tail_splits, tail_kbs;
};
// Block shapes of the tiled kernel beside 32, 64 and 128 rows x 3 column tiles per wave (see fq_plan_flexible)
inline bool fq_flexible(const fq_gemm_plan& p) { return p.kind == 1 && p.mt >= 5 && !(p.mt == 8 && p.nt == 3); }
// act_dtype: FQ_F16 or FQ_BF16; the plans differ in the block shape alone (see fq_plan_flexible), not in the scratch
fq_gemm_plan fq_plan_gemm(int64_t M, int64_t N, int64_t K, int bits, int g, int act_dtype);
// Rows of the next tile of the mid-M kernel when `left` are left: as few tiles as 48 rows allow, of nearly equal height.
inline int32_t fq_mid_rows(int32_t left) {
    if (left > 96) return 48;        // (three tiles and more of nearly equal height are 48 rows high)
    const int32_t n = (left + 47) / 48;
    const int32_t even = ((left + n - 1) / n + 15) / 16 * 16;
    return left < even ? left : even;
}
// Grouped product.  Every expert's rows are cut into tiles, and the tiles of one class share a launch: 128 or 64 rows of the
// tiled kernel, up to 48 of the mid-M one, up to 16 of the small-M one.
enum fq_tile_class { FQ_TILE_128, FQ_TILE_64, FQ_TILE_MID, FQ_TILE_SMALL, FQ_TILE_CLASSES };
enum fq_cut { FQ_CUT_SMALL, FQ_CUT_MID, FQ_CUT_TALL };
struct fq_small_shape { int gp, kw; };   // column groups (of three tiles) x k-workers per block
struct fq_grouped_plan {
    fq_cut cut;                  // all tiles small; all for the mid-M kernel; 128 and 64 rows, and the mid-M kernel below 49
    bool fork;                   // each class on a stream of its own
    fq_small_shape mid;          // block shape of the mid-M kernel
};
fq_grouped_plan fq_plan_grouped(const int32_t* offsets, int E, int64_t N, int64_t K, int bits, int g);
// The next tile of an expert that has `left` rows left.
inline fq_tile_class fq_next_tile(const fq_grouped_plan& p, int32_t left, int32_t* take) {
    if (p.cut == FQ_CUT_SMALL) {
        *take = left < 16 ? left : 16;
        return FQ_TILE_SMALL;
    }
    if (p.cut == FQ_CUT_TALL && left > 48) {
        const int32_t tall = left > 64 ? 128 : 64;
        *take = left < tall ? left : tall;
        return tall == 128 ? FQ_TILE_128 : FQ_TILE_64;
    }
    *take = fq_mid_rows(left);
    return FQ_TILE_MID;
}
// Block shape of the small-M kernel for `count` items of a grouped product (at most 16 rows each);
// units = activation units (16 bytes) of a k-block in the tallest of them, ngroups = groups of three column tiles.
fq_small_shape fq_plan_grouped_small(int count, int units, int ngroups, int KB);
// compute units of the device (asked once per process; 256 without a device)
int fq_cu_count();
// Rows of K per k-block of the tiled kernel for a block shape (the unit of kb_per_split and tail_kbs):
// the layout's k-block, except that the 8-wave shapes of 80 rows and more take two 64-row blocks of 8-bit codes at a
// time when K allows it and such a k-block lies inside one scale group (with two scale rows the wider
// kernel spills and gains nothing, with four it loses).
inline int fq_mma_kblk(int bits, int mt, int waves, int64_t K, int g) {
    return (bits == 8 && mt >= 5 && waves == 8 && K % 128 == 0 && g % 128 == 0) ? 128 : (bits == 8 ? 64 : 128);
}
// Workspace layout of fq_gemm: [split-K partial tiles][bf16 activations rewritten as binary16][their M row scales,
// two unused words, then (bfloat16 scales) FQ_SCALE_PARTS words of the search for the largest scale's exponent]
inline size_t fq_partial_bytes(const fq_gemm_plan& p, int64_t M, int64_t N) {
    const int parts = p.splits > 1 ? p.splits : (p.tail_tiles > 0 ? p.tail_splits : 0);
    return (size_t)parts * (size_t)M * (size_t)N * sizeof(float);
}
inline size_t fq_a16_bytes(int64_t M, int64_t K) { return (((size_t)M * (size_t)K * 2) + 255) / 256 * 256; }
#define FQ_SCALE_PARTS 256
inline size_t fq_rowscale_bytes(int64_t M) { return ((size_t)M + 2 + FQ_SCALE_PARTS) * sizeof(float); }
// bf16 activations (binary16 or bfloat16 scales) take the fp16 matrix path for the 128-row shapes of wide matrices and the
// shapes of 80 rows and more that fq_plan_flexible puts in their place: the rewrite of the rows costs 4 M K bytes of traffic against 2 M N K flops
inline bool fq_via_f16(int act_dtype, int scale_format, const fq_gemm_plan& p, int64_t N) {
    (void)scale_format;
    return act_dtype == FQ_BF16 && p.kind == 1 && p.mt >= 5 && N >= 8192;
}
// act: FQ_F16, FQ_BF16, or 2 = bf16 activations with bf16 scales
// plan: fq_plan_gemm's for these sizes (made once per call: on small matrices making it is a tenth of the call)
int fq_launch_gemm(const fq_gemm_plan& plan, const void* A, int act, int64_t M, int64_t N, int64_t K, const void* codes,
                   const void* scales, int bits, int g, void* C, void* workspace, hipStream_t stream);
int fq_launch_gemm_grouped(const void* A, int act, const int32_t* offsets, int E, int64_t N, int64_t K,
                           const void* codes, const void* scales, int bits, int g, void* C,
                           hipStream_t stream);

#endif  // FQ_INTERNAL_H_
