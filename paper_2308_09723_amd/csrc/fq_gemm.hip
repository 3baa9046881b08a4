// Host side of the product: the plan (which kernel, which block shape) and the entry points
// that dispatch on activation type and code width.  The kernels themselves are instantiated
// in fq_gemm_<type>_<bits>.hip.
#include <hip/hip_runtime.h>
#include <atomic>
#include <chrono>
#include <math.h>
#include <mutex>
#include <stdint.h>

#include "fq_gemm_config.h"
#include "fq_internal.h"
#include "fq_layout.h"


using namespace fqd;

#define FQ_DECLARE_GEMM(ACT, BITS)                                                                         \
    int fq_launch_typed_##ACT##_##BITS(const void* A, int64_t M, int64_t N, int64_t K, const void* codes,  \
                                       const void* scales, int g, void* C, void* workspace,                \
                                       const fq_gemm_plan& plan, hipStream_t stream);                      \
    int fq_launch_grouped_typed_##ACT##_##BITS(const void* A, const int32_t* offsets, int E,               \
                                               const fq_grouped_plan& plan, int64_t N, int64_t K,          \
                                               const void* codes, const void* scales, int g, void* C,      \
                                               const hipStream_t* streams);
FQ_DECLARE_GEMM(0, 4)
FQ_DECLARE_GEMM(0, 8)
FQ_DECLARE_GEMM(1, 4)
FQ_DECLARE_GEMM(1, 8)
FQ_DECLARE_GEMM(2, 4)   // bf16 activations, bf16 scales
FQ_DECLARE_GEMM(2, 8)
FQ_DECLARE_GEMM(0, 3)   // 3-bit codes
FQ_DECLARE_GEMM(1, 3)
FQ_DECLARE_GEMM(2, 3)

// Compute units of the device, asked once per process (the current device at the first call); without a
// device (host-only use of the size queries and fq_gemm_describe) the MI355X's 256.
int fq_cu_count() {
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            return v;
        (void)hipGetLastError();
        return 256;
    }();
    return n;
}

// The calls of a process are numbered from a place of its own on, so that what another process left in memory carries no
// tag of this one either.
uint64_t fq_next_tag() {
    static std::atomic<uint64_t> calls{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull >> 20};
    return 0xffa5ull << 48 | (calls.fetch_add(1, std::memory_order_relaxed) & 0xffffffffffull) << 8;
}

// Atomics of agent scope count among the compute units of one device, in that device's own memory.  C in pinned host memory, in
// managed memory or on another GPU is only ever stored to, as is memory that the runtime cannot place (asked in 60 ns each), and
// partial sums there are read by a later kernel only.
bool fq_counts_tickets(const void* C, const void* partial, hipStream_t stream) {
    if (hipPeekAtLastError() != hipSuccess) return false;      // (an earlier error is not this call's to clear)
    hipDevice_t dev = -1;
    bool plain = hipStreamGetDevice(stream, &dev) == hipSuccess;
    for (const void* p : {C, partial}) {
        hipPointerAttribute_t at = {};
        plain = plain && hipPointerGetAttributes(&at, p) == hipSuccess && at.type == hipMemoryTypeDevice && at.device == (int)dev &&
                !at.isManaged && at.allocationFlags == 0;
    }
    if (!plain) (void)hipGetLastError();
    return plain;
}

// scale rows a layout k-block spans: 1, kblk / g, or one per 32-row step
static int fq_scale_rows(int bits, int g) {
    const int kblk = fq_kblk(bits);
    return g % kblk == 0 ? 1 : (kblk % g == 0 ? kblk / g : kblk / 32);
}

// Mid-M streaming kernel (17 <= M <= 48): the block shape (gp column groups x kw k-workers, at most 12 waves, three
// (M <= 32) or two activation tiles of kw k-blocks in the 160 KiB of LDS) and split of K over the grid with the least
//   sum over rounds of blocks (iterations * t_it + 5 us)  +  partial sums (their traffic at 5 TB/s + 4 us, if split)
// where an iteration takes the longest of the time the vector and matrix units need for the block's waves, the time
// memory needs for what the resident blocks ask of it (weights, and three tenths of the activations, which come from the L2
// caches, at 7 TB/s), and a latency of 1.4 us.  (Without the activations shapes of one column group and twelve k-workers won,
// which load twice their weights in activations: 8-bit codes on 49152 x 12288, M = 32 125 us where 4 x 3 in four splits takes
// 104.)  Against sweeps of (gp, kw, splits) on nineteen matrices at M = 17 .. 48 the choice is 2 % slower than the sweep's
// best on average.  With four row tiles (M = 64) the kernel took 88 - 101 us where the tiled one takes 91 - 98, so 49 rows
// and more stay there.  Returns the model's time.
struct fq_mid_model {
    int KB, fit;         // k-blocks; k-workers whose activation tiles fit the LDS
    double work;         // microseconds of vector / matrix work per iteration of a full block (12 waves, a k-block of 48 columns each)
    double rec_bytes;    // codes and scales a wave loads per iteration
    int tile_bytes;      // activation tile of a k-worker
    fq_mid_model(int mt, int kblocks, int bits, int sr) : KB(kblocks) {
        const int kblk = fq_kblk(bits);
        work = mt <= 2 ? (bits == 8 ? 0.85 : (bits == 3 ? 1.75 : 1.5)) : (bits == 8 ? 1.3 : (bits == 3 ? 2.6 : 2.4));
        work += (sr - 1) * (mt <= 2 ? 0.27 : 0.4);
        rec_bytes = MMA_NT * 64.0 * fq_rec_bytes(bits) + MMA_NT * 32.0 * sr;
        tile_bytes = mt * 16 * kblk * 2;
        fit = 160 * 1024 / ((mt == 3 ? 2 : 3) * tile_bytes);
    }
    // the most k-workers for gp column groups
    int workers(int gp) const {
        int kw = 12 / gp;
        if (kw > fit) kw = fit;
        return kw > KB ? KB : kw;
    }
    // one iteration of a block: vector / matrix work, and memory when `active` blocks are resident
    double compute(int waves) const { return work * (1.0 / 3.0) * (double)((waves + 3) / 4); }
    double memory(int gp, int kw, double active, double us_per_byte) const {
        return active * (gp * kw * rec_bytes + 0.3 * kw * tile_bytes) * us_per_byte;
    }
    double iteration(int gp, int kw, double active) const {
        const double t_work = compute(gp * kw), t_mem = memory(gp, kw, active, 1.0 / 7e6);
        const double t_it = t_mem > t_work ? t_mem : t_work;
        return t_it > 1.4 ? t_it : 1.4;
    }
};

static double fq_plan_mid(int64_t M, int64_t N, int64_t K, int bits, int g, int ncu, fq_gemm_plan* p) {
    const int mt = M <= 32 ? 2 : 3;
    const fq_mid_model model(mt, (int)(K / fq_kblk(bits)), bits, fq_scale_rows(bits, g));
    const int ngroups = (int)((N / FQ_NTILE + MMA_NT - 1) / MMA_NT);
    double best = 1e30;
    for (int gp = 1; gp <= 12; ++gp) {
        const int kw = model.workers(gp);
        const int blocks = (ngroups + gp - 1) / gp;
        const int SB = (model.KB + kw - 1) / kw;
        for (int gs = 1; gs <= 8 && gs <= SB; ++gs) {
            const int grid = blocks * gs;
            if (gs > 1 && grid > 2 * ncu) break;
            const int n_it = (SB + gs - 1) / gs;
            const int full = grid / ncu, rest = grid % ncu;
            auto round_us = [&](double active) { return n_it * model.iteration(gp, kw, active) + 5.0; };
            double t = (double)full * round_us((double)ncu) + (rest ? round_us((double)rest) : 0.0);
            if (gs > 1) t += 2.0 * gs * (double)M * (double)N * 4.0 / 5e6 + 4.0;
            if (t < best - 1e-9) {
                best = t;
                p->kind = 2;
                p->mt = mt;
                p->nt = MMA_NT;
                p->gp = gp;
                p->kw = kw;
                p->waves = gp * kw;
                p->splits = gs;
            }
        }
    }
    return best;
}

// Waves of 16 columns instead of 48 (nt = 1), without a split of K, in place of the plan above: 48 columns leave half the chip
// idle on matrices of less than 12288 of them, 16 fill it in one round of blocks.  Both are weighed by a model
// of either width, fitted together (of log time, rms error 9 %) to 360 problems of 17 .. 48 rows, 1024 .. 17600 columns, in 30
// shapes each: a block takes its start and end, and per iteration a latency, its waves' vector and matrix work, and memory
// traffic, which add up.  The narrow waves have to win by 7 %, by 20 % where they replace a split (the model ranks those
// worse; scratch only shrinks).  Of those problems 157 change, 1.20x faster on average, one more than 3 % slower (3.4 %);
// 2176 x 2336, 28 rows, g = 32 11.3 -> 7.7 us.  Above 12000 columns 9 of 34 became slower.
static double fq_mid_us(int nt, int mt, int KB, int ngroups, int row_blocks, int64_t M, int64_t N, int bits, int sr, int gp, int kw,
                        int splits, int ncu) {
    static const double c[2][9] = {      // work of 32 and 48 rows, 8- and 3-bit codes' share of it, a further scale row; us
        {0.331, 0.566, 0.542, 1.007, 0.050, 0.364, 4.89, 3.27, 0.50},      // per iteration, per block, more for a second one
        {0.927, 1.325, 0.615, 1.069, 0.253, 0.342, 6.46, 10.0, 0.39}};     // beside it, ragged end
    const double* x = c[nt == 1 ? 0 : 1];
    const int waves = gp * kw, blocks = (ngroups + gp - 1) / gp * row_blocks * splits, SB = (KB + kw - 1) / kw, n_it = (SB + splits - 1) / splits;
    const int tile = mt * 16 * fq_kblk(bits) * 2, act = (mt == 3 ? 2 : 3) * kw * tile, red = waves * nt * mt * 1024;
    int resident = 160 * 1024 / (act > red ? act : red);
    resident = resident < 24 / waves ? resident : 24 / waves;
    const int slots = ncu * (resident > 1 ? resident : 1);
    const double share = (double)blocks / ncu, together = share < 1.0 ? 1.0 : (share < (double)slots / ncu ? share : (double)slots / ncu);
    const double work = x[mt == 2 ? 0 : 1] * (bits == 8 ? x[2] : (bits == 3 ? x[3] : 1.0)) + x[4] * (sr - 1);
    const double bytes = waves * (nt * 64.0 * fq_rec_bytes(bits) + nt * 32.0 * sr);
    double t = x[6] + x[7] * (together - 1.0) +
               n_it * (x[5] + work * ((waves + 3) / 4) * together * (1.0 / 3.0) + (blocks < slots ? blocks : slots) * bytes * (1.0 / 16e6));
    if (blocks > slots) {
        const double full = (double)((blocks + slots - 1) / slots), part = (double)blocks / slots + x[8];
        t *= part < full ? part : full;
    }
    return splits > 1 ? t + 1.9 + 2.0 * splits * (double)M * (double)N * (4.0 / 5.6e6) : t;
}

static void fq_plan_mid_narrow(int64_t M, int64_t N, int64_t K, int bits, int g, int ncu, fq_gemm_plan* p) {
    if (N > 12000) return;
    const int mt = p->mt, KB = (int)(K / fq_kblk(bits)), sr = fq_scale_rows(bits, g), ntiles = (int)(N / FQ_NTILE);
    const fq_mid_model model(mt, KB, bits, sr);
    double best = (p->splits > 1 ? 0.80 : 0.93) *
                  fq_mid_us(MMA_NT, mt, KB, (ntiles + MMA_NT - 1) / MMA_NT, 1, M, N, bits, sr, p->gp, p->kw, p->splits, ncu);
    static const int groups[6] = {1, 2, 3, 4, 6, 12};
    for (const int gp : groups) {
        const int kw = model.workers(gp);
        if ((ntiles + gp - 1) / gp > ncu) continue;      // (a second round: 8-bit codes on 8400 columns 0.74 - 0.93)
        const double t = fq_mid_us(1, mt, KB, ntiles, 1, M, N, bits, sr, gp, kw, 1, ncu);
        if (t < best) {
            best = t;
            p->nt = 1;
            p->gp = gp;
            p->kw = kw;
            p->waves = gp * kw;
            p->splits = 1;
        }
    }
}

// Row blocks of the mid-M kernel (kind 3) with 16 columns per wave, for 49 .. 256 rows on less than 8192 columns: in one round of
// blocks, without a split, where the model above puts them below the present plan's time (best, by its own model).  A few dozen
// blocks of the other shapes leave most of the chip idle there, or pay for a split's second launch.  Chosen by margin: 150 products
// of 49 .. 400 rows (in graphs, against the plans without it) gave 1.015x, 1.035x, 1.053x at 0.8, 0.9, 1.0 of that time,
// none slower; 1.065x at 1.1, but three slower (0.86x at worst).  150 products of 49 .. 256 rows twice, each side timed first
// once: 1.10x on average both times; of those it changes by more than 3 %, 126 have K up to 6400 and became 1.25x as fast on average,
// none slower (1152 x 560, 133 rows 12.1 -> 6.6 us; 2304 x 3280, 159 rows 13.2 -> 10.9).  Longer K keeps its plan: 2 of 12
// became slower there (9472 x 272, 204 rows 20.2 -> 24.2 us).  Scratch only shrinks.  Above 256 rows and from 8192
// columns on the plan depends on the activations' type (binary16 alone takes some shapes), so a change for one type could leave
// another with more scratch than the one size that serves all.
static void fq_plan_rows_narrow(int64_t M, int64_t N, int64_t K, int bits, int g, int ncu, double best, fq_gemm_plan* p) {
    const int row_blocks = (int)((M + 47) / 48), ntiles = (int)(N / FQ_NTILE);
    const int mt = fq_mid_rows((int32_t)M) > 32 ? 3 : 2, KB = (int)(K / fq_kblk(bits)), sr = fq_scale_rows(bits, g);
    const fq_mid_model model(mt, KB, bits, sr);
    static const int groups[6] = {1, 2, 3, 4, 6, 12};
    for (const int gp : groups) {
        const int kw = model.workers(gp);
        if ((ntiles + gp - 1) / gp * row_blocks > ncu) continue;
        const double t = fq_mid_us(1, mt, KB, ntiles, row_blocks, M, N, bits, sr, gp, kw, 1, ncu);
        if (t < best) {
            best = t;
            *p = fq_gemm_plan{};
            p->kind = 3;
            p->mt = 3;
            p->nt = 1;
            p->gp = gp;
            p->kw = kw;
            p->waves = gp * kw;
            p->splits = 1;
            p->tail_splits = 1;
        }
    }
}

// The streaming kernel or the tiled one (plan t, t_tiled by its model) for 17 .. 48 rows.  Measured in turn on 23
// matrices, all formats and group sizes, six M (1656 pairs): the streaming kernel everywhere is 1.142x as fast as the
// tiled one, but more than 3 % slower in 103 pairs (down to 0.86x; 50 pairs differ that much when both sides are the
// same kernel), most of them 3- and 4-bit codes with one scale row per k-block and two row tiles, where the tiled kernel
// is post-scaled too.  With the tiled kernel there where its model's time is 0.92 of the other's or less: 1.143x, 69 pairs.
// Below 13 us the launches decide.
static bool fq_mid_pays(double t_mid, const fq_gemm_plan& t, double t_tiled, int64_t M, int64_t N, int bits, int g) {
    if (t_mid <= 13.0 || bits == 8 || M > 32 || fq_scale_rows(bits, g) > 1) return true;
    // (what fq_gemm_noalloc's scratch holds one way it does not refuse for the other)
    return t_tiled >= 0.92 * t_mid || fq_partial_bytes(t, M, N) > (size_t)FQ_NOALLOC_SCRATCH_BYTES;
}

// Tiled kernel, shapes between the classes of 64 and 128 rows: 80 .. 128 rows x 256 columns (two column tiles per wave)
// and 80 rows x 384.  128 x 384 blocks leave the chip partly idle where the output has few of them (200 rows x 28656
// columns: 150 blocks of which the second 75 are 44 % padding; split 3 ways along K they fill 1.8 rounds and move 70 MB
// of partial sums), 112 x 256 makes it 224 blocks without padding or a split.  3- and 4-bit codes with one scale row
// per k-block run post-scaled here (the second accumulator set of two column tiles fits the registers up to 112 rows).
// `u` = microseconds per k-block of a block, fitted like fq_plan_gemm's to sweeps of (shape, split) over five matrices
// (8192 x 28656, 12288 x 36864, 12288^2, 4096 x 16384, 8192^2) at sixteen M from 72 to 1000: rms error 5 % (7 % for
// 8-bit codes).  Because the model of the other shapes is off by 10 %, these have to win by that much (15 % for 8-bit
// codes with k-blocks of 64 rows), and by 3 us more where they replace 32- or 64-row blocks: of the 400 records of the
// sweeps 186 take them, 1.23x faster on average, one choice 2 % slower than before.  fp16 int4, us: 8192 x 28656 g = 64 M = 200
// 130 -> 103, M = 160 104 -> 80; 12288^2 M = 160 75 -> 57; 4096 x 16384 M = 384 71 -> 48.
// bfloat16 activations take these shapes on the fp16 matrix path (fq_via_f16), whose range is binary16's beside a power of
// two per row and, for bfloat16 scales, one for the matrix.  That is what the 128-row blocks of wide matrices do; the 32- and 64-row
// blocks multiply bfloat16 operands as they are, so where those are chosen bfloat16 products keep them (a column whose
// scales lie 2^14 .. 2^20 below the widest came out with errors of 2 % instead of 0.3 %), and binary16 ones leave them
// only for shapes that need no scratch either (one size serves both types).  A split whose partial sums exceed
// fq_gemm_noalloc's scratch gives way for both, to these shapes or to the same blocks without a split.
// Not below 65 rows (the lower classes measure the same), nor above 1024 (1408 x 15456 at M = 1847: 102 -> 109), nor for
// matrices narrower than 8192 columns, where bfloat16 products do not take the fp16 matrix path.  Two scale rows: the 32-row shape stays where it is chosen (41 against 40 us
// in the one record).  Above 256 rows a plan whose last round is split along K stays: it was the faster one in 26 of 37 such
// records (up to 1.27x).
static double fq_plan_flexible(int64_t M, int64_t N, int64_t K, int bits, int g, int act_dtype, int ncu, double best,
                             fq_gemm_plan* p) {
    static const struct { int mt, nt; } shapes[5] = {{5, 2}, {6, 2}, {7, 2}, {8, 2}, {5, 3}};
    static const double consts[5][5] = {
        {1.10, 1.22, 1.40, 1.53, 1.53},     // 3- and 4-bit, one scale row per k-block (post-scaled)
        {1.16, 1.265, 1.43, 1.54, 1.585},   // two scale rows
        {1.525, 1.60, 1.73, 1.84, 2.36},    // four
        {1.19, 1.31, 1.46, 1.57, 1.67},     // 8-bit, k-blocks of 128 rows
        {0.62, 0.74, 0.75, 0.85, 0.86}};    // 8-bit, k-blocks of 64 rows
    const double other = best;
    if (M <= 64 || M > 1024 || N < 8192) return other;
    const bool low = p->mt < 8;      // replaces 32- or 64-row blocks
    const size_t scratch = FQ_NOALLOC_SCRATCH_BYTES;
    const bool fits = fq_partial_bytes(*p, M, N) <= scratch;
    if (low && fits && (act_dtype != FQ_F16 || p->splits > 1 || p->tail_tiles > 0)) return other;
    const int kblk = fq_mma_kblk(bits, 8, 8, K, g);
    const int sr = g % kblk == 0 ? 1 : (kblk % g == 0 ? kblk / g : kblk / 32);
    if (bits != 8 && sr == 2 && p->mt == 2) return other;
    if (M > 256 && p->tail_tiles > 0) return other;
    const double* u = consts[bits == 8 ? (kblk == 128 ? 3 : 4) : (sr == 1 ? 0 : (sr == 2 ? 1 : 2))];
    const int KB = (int)(K / kblk);
    const int ntiles = (int)(N / FQ_NTILE);
    const int split_opts[5] = {1, 2, 3, 4, 6};
    // what fq_gemm_noalloc's scratch held for the former shape it has to hold for the new one
    const size_t rewrite = fq_a16_bytes(M, K) + fq_rowscale_bytes(M);
    const size_t was_f16 = fq_partial_bytes(*p, M, N), was_bf16 = was_f16 + (low ? 0 : rewrite);
    const size_t most_f16 = was_f16 > scratch ? was_f16 : scratch, most_bf16 = was_bf16 > scratch ? was_bf16 : scratch;
    best = 0.90 * (low ? best - 3.0 : best);
    if (bits == 8 && kblk == 64) best *= 0.95;
    fq_gemm_plan chosen = *p;
    chosen.splits = 0;
    for (int v = 0; v < 5; ++v) {
        const int bm = shapes[v].mt * 16;
        const int64_t blocks = ((ntiles + 8 * shapes[v].nt - 1) / (8 * shapes[v].nt)) * ((M + bm - 1) / bm);
        for (int si = 0; si < 5; ++si) {
            if (split_opts[si] > (low && fits ? 1 : KB)) break;
            const int kbs = (KB + split_opts[si] - 1) / split_opts[si];
            const int splits = (KB + kbs - 1) / kbs;
            const size_t partial = splits > 1 ? (size_t)splits * (size_t)M * (size_t)N * sizeof(float) : 0;
            if (partial > most_f16 || partial + rewrite > most_bf16) continue;
            double t = (double)((blocks * splits + ncu - 1) / ncu) * kbs * u[v] + 1.3;
            if (splits > 1) t += 2.0 * splits * (double)M * (double)N * 4.0 / 5e6 + 5.0;
            if (t < best - 1e-9) {
                best = t;
                chosen.mt = shapes[v].mt;
                chosen.nt = shapes[v].nt;
                chosen.waves = 8;
                chosen.splits = splits;
                chosen.kb_per_split = kbs;
            }
        }
    }
    if (chosen.splits == 0) return other;
    if (low && (act_dtype != FQ_F16 || chosen.splits > 1)) {
        // (the split does not fit fq_gemm_noalloc's scratch: the same blocks without it)
        chosen = *p;
        chosen.splits = 1;
        chosen.kb_per_split = (int)(K / fq_mma_kblk(bits, p->mt, p->waves, K, g));
    }
    chosen.tail_tiles = 0;
    chosen.tail_splits = 1;
    chosen.tail_kbs = 0;
    *p = chosen;
    return best;
}

// Microseconds a block of the tiled kernel spends on 128 rows of K (see fq_plan_gemm):
//   u8(mt=2) u4(mt=2) u8(mt=4) u4(mt=4) u8(mt=8) u4(mt=8)  lone 4-wave block factor (mt < 8, mt = 8)
static const double* fq_tiled_costs(int bits, int g) {
    static const double consts[4][8] = {
        {0.99, 0.506, 1.43, 0.83, 2.33, 1.43, 1.2, 1.2},     // 4-bit, one scale row per k-block
        {1.17, 0.634, 1.60, 0.884, 2.34, 1.46, 1.2, 1.2},    // 4-bit, two scale rows
        {1.64, 0.731, 2.16, 1.29, 2.70, 1.57, 1.5, 1.35},    // 4-bit, four scale rows
        {1.73, 0.77, 1.73, 1.035, 2.50, 1.47, 1.2, 1.35}};   // 8-bit
    const int sr = g % 128 == 0 ? 1 : (128 % g == 0 ? 128 / g : 4);
    return consts[bits == 8 ? 3 : (sr == 1 ? 0 : (sr == 2 ? 1 : 2))];
}

// Model of a grouped call, fitted (of log time, rms error 10 %) to 200 calls of 8 .. 64 experts, 8 .. 2048 tokens and
// matrices from 1024 x 1024 to 4096 x 16384, each cut in up to ten ways.
//   a block of the tiled kernel     its cost per 128 rows of K (fq_tiled_costs) times tile_f, + 10 us
//   a block of the mid-M kernel     iterations of fq_mid_model's length times mid_f (at least 1 us, memory at 8.5 TB/s), + 5.8 us
//   a block of the small-M kernel   1.26 us per iteration, + 5 us (2.5 without k-workers)
//   a launch                        the compute units' share of its blocks + 0.35 of the longest for the ragged end (not more
//                                   than its whole rounds for the mid-M kernel); at least the longest
// Side by side on streams of their own the launches share one ragged end, but forking and joining the streams costs 21 us.

// Block shape of the mid-M kernel for the tiles of a grouped product (count[i]: those of i + 1 row tiles); the launch's
// time, the time its blocks hold the compute units in all, and the longest of them.  even: row blocks of one product, all as
// long as each other, so that a launch of 280 blocks takes two whole rounds.  The shape is the best by that (140 such products
// that it changes: 1.33x, 2332 x 288, K = 2176, 8-bit 25 -> 17 us); the time returned stays the one above, by which these products
// take this kernel and no scratch, unless the tiled plan needs none either.  Where the blocks' work alone takes `limit` or
// more, that time is returned and nothing is looked at.
static double fq_plan_grouped_mid(const int (&count)[3], int64_t N, int64_t K, int bits, int g, bool even, double limit,
                                  fq_small_shape* sh, double* busy_us, double* block_us) {
    static const double mid_f[2][3] = {{0.67, 1.13, 0.88}, {0.8, 0.96, 1.19}};      // (3- and 4-bit codes, 8-bit codes)
    const int ngroups = (int)((N / FQ_NTILE + MMA_NT - 1) / MMA_NT);
    const int ncu_n = fq_cu_count();
    const double ncu = (double)ncu_n, share = 1.0 / ncu;
    const int items = count[0] + count[1] + count[2];
    const int kblocks = (int)(K / fq_kblk(bits)), sr = fq_scale_rows(bits, g);
    const fq_mid_model model[3] = {{1, kblocks, bits, sr}, {2, kblocks, bits, sr}, {3, kblocks, bits, sr}};
    const fq_mid_model& tallest = model[count[2] ? 2 : (count[1] ? 1 : 0)];
    double best = 1e30, best_rank = 1e30, least = 0.0;
    for (int i = 0; i < 3; ++i) least += count[i] * mid_f[bits == 8][i] * model[i].work;
    least *= share * (1.0 / 12.0) * ngroups * model[0].KB;
    if (least >= limit) return least;
    for (int gp = 1; gp <= 12; ++gp) {
        const int kw = tallest.workers(gp);
        if ((double)((tallest.KB + kw - 1) / kw) + 5.8 > best_rank) continue;      // (at least 1 us per iteration)
        const int per_item = (ngroups + gp - 1) / gp;
        const int64_t blocks = (int64_t)per_item * items;
        const double active = blocks < ncu_n ? (double)blocks : ncu;
        double sum = 0.0, longest = 0.0;
        for (int i = 0; i < 3; ++i) {
            if (count[i] == 0) continue;
            const double t_work = mid_f[bits == 8][i] * model[i].compute(gp * kw), t_mem = model[i].memory(gp, kw, active, 1.0 / 8.5e6);
            const double t_it = t_work > t_mem ? t_work : t_mem;
            const double t = ((model[i].KB + kw - 1) / kw) * (t_it > 1.0 ? t_it : 1.0) + 5.8;
            sum += t * ((double)per_item * count[i]);
            longest = t > longest ? t : longest;
        }
        const double rounds = (double)((blocks + ncu_n - 1) / ncu_n) * longest;
        double total = sum * share + 0.35 * longest;
        total = total < rounds ? total : rounds;
        if (total < longest) total = longest;
        if (total < best) best = total;
        const double rank = even ? rounds : total;
        if (rank < best_rank - 1e-9) {
            best_rank = rank;
            *busy_us = sum;
            *block_us = longest;
            sh->gp = gp;
            sh->kw = kw;
        }
    }
    return best;
}

constexpr int64_t FQ_ROW_BLOCKS_MOST_K = 6400;

// Time of the small-M kernel for a block shape (NT = nt column tiles per wave), fitted (of log time, rms error 11 %) to 190
// problems of 1 .. 16 rows from 1024 x 1024 to 12288 x 49152 with 80 shapes each, timed inside graphs.  An iteration takes 0.3 us
// and the longer of its vector work and its memory traffic at 9 TB/s over the resident blocks (which find part of it in a
// cache); a split of K over the grid the partial sums and 3.5 us, the launch of a second kernel that added them when this was
// fitted.  The last block of a tile adds most of them now (fq_split_sum.h); the term stays, and with it plans and scratch.
static double fq_small_us(int64_t M, int64_t N, int64_t K, int bits, int g, int ncu, int nt, int gp, int kw, int au, int gs) {
    const int kblk = fq_kblk(bits), sr = fq_scale_rows(bits, g), waves = gp * kw;
    const int ntiles = (int)(N / FQ_NTILE), KB = (int)(K / kblk);
    static const int resident[13] = {1, 12, 6, 4, 3, 2, 2, 1, 1, 1, 1, 1, 1};       // blocks of so many waves per compute unit
    const int blocks_n = (ntiles + nt * gp - 1) / (nt * gp) * gs, slots_n = ncu * resident[waves];
    const double blocks = (double)blocks_n;
    const double slots = (double)slots_n;
    const double n_it = (double)((((KB + kw - 1) / kw) + gs - 1) / gs);
    const double bytes = waves * (nt * 64.0 * fq_rec_bytes(bits) + nt * 32.0 * sr) + (double)M * kw * kblk;
    const double together = blocks <= ncu ? 1.0 : (blocks < slots ? blocks : slots) * (1.0 / ncu);
    const double work = 0.022 * waves * nt * ((bits == 8 ? 0.33 : 1.0) + 0.12 * sr) * together;
    const double mem = bytes * (blocks < slots ? blocks : slots) * (1.0 / 9e6);
    const double t_it = (work > mem ? work : mem) + 0.3 + (au == 2 ? 0.3 : (au == 4 ? 2.7 : 0.0));
    double t = 3.9 + n_it * t_it;
    if (blocks_n > slots_n) t *= 0.45 * (double)((blocks_n + slots_n - 1) / slots_n) + 0.55 * blocks / slots;
    return gs > 1 ? t + 3.6 + 2.0 * gs * (double)M * (double)N * 4.0 / 1.65e6 : t;
}

fq_gemm_plan fq_plan_gemm(int64_t M, int64_t N, int64_t K, int bits, int g, int act_dtype) {
    fq_gemm_plan p = {};
    const int ncu = fq_cu_count();
    const int kblk = fq_kblk(bits);
    const int KB = (int)(K / kblk);
    const int ntiles = (int)(N / FQ_NTILE);
    if (M <= 16) {
        // One block per compute unit, all resident at once.  Candidates are scored by how evenly
        // the column tiles (times the grid's split of K) fill one block per compute unit, by the bytes a compute
        // unit keeps in flight (waves x NT KiB x ring depth, ~64 KiB saturates), and by how many
        // activation units a lane must stage (fewer registers); ties keep the earlier variant.
        // The factors come from sweeps over the OPT-175B shapes at M = 1 and 8.
        p.kind = 0;
        p.mt = 1;
        const int kc = kblk / 8;
        const double f_nt[4] = {0.0, 0.93, 0.97, 1.0};
        double best = -1.0;
        for (int v = 0; v < 4; ++v) {
            const SkinnyVariant sv = SKINNY_VARIANTS[v];
            for (int gp = 1; gp <= sv.maxw; ++gp) {
                const int tb = sv.nt * gp;
                const int64_t blocks = (ntiles + tb - 1) / tb;
                const int need = (int)M * kc;
                const int au = need <= 64 * gp ? 1 : (need <= 128 * gp ? 2 : (need <= 256 * gp ? 4 : 0));
                if (au == 0) continue;
                // (all the waves the register class allows: with one column group per block, twelve k-workers
                // of two stages measured 3 - 8 % faster than eight of three on the 12288-column layers)
                int kw = sv.maxw / gp;
                if (kw > KB) kw = KB;
                if (kw < 1) continue;
                const int SB = (KB + kw - 1) / kw;       // iterations if one block walks all of K
                // Few column blocks: K is also split over the grid (binary32 partials, added by the last block),
                // which moreover divides the activation bytes every block has to fetch.
                int gs = 1;
                if (blocks <= ncu / 2) gs = (int)(ncu / blocks);
                if (gs > 8) gs = 8;
                if (gs > SB) gs = SB;
                const int64_t grid = blocks * gs;
                const int64_t rounds = (grid + ncu - 1) / ncu;
                const double eff = (double)ntiles * gs / (double)(rounds * ncu * tb);
                const int waves = gp * kw;
                const double inflight = (double)waves * sv.nt * sv.depth;   // KiB
                const double n_it = (double)((SB + gs - 1) / gs);
                double score = eff * eff * (inflight >= 64.0 ? 1.0 : sqrt(inflight / 64.0)) * f_nt[sv.nt];
                score /= 1.0 + 0.1 * (double)(rounds - 1);   // a single resident round beats several
                score *= au == 1 ? 1.0 : (au == 2 ? 0.8 : 0.6);
                // a split of K over the grid costs its partial sums, and with few iterations left per
                // block the register ring is mostly filling and draining
                if (gs > 1) score *= n_it >= 16.0 ? 0.80 : 0.65;
                // every block fetches its whole k range of the activations: M * K * 2 / gs bytes,
                // once per block, next to K * N * bits / 8 bytes of weights
                score /= 1.0 + 0.15 * ((double)M * 2.0 * (double)ncu / gs) / ((double)N * bits / 8.0);
                if (waves < 6) score *= 0.85;
                if (kw == 1) score *= 0.95;                  // no k-workers: measured ~5 % slower
                if (score > best + 1e-9) {
                    best = score;
                    p.variant = v;
                    p.gp = gp;
                    p.kw = kw;
                    p.au = au;
                    p.waves = waves;
                    p.splits = gs;
                }
            }
        }
        // A split of K over the grid gives way where the blocks alone are as fast: the scores above were made for matrices
        // that take 15 us and more.  190 problems of 1 .. 16 rows: 89 lose their split, 1.11x on average over all (inside
        // graphs), none more than 3 % slower; 2304 x 4528, 13 rows 9.9 -> 6.7 us (all against sums by a
        // second kernel).  Matrices of up to 64 column tiles, a quarter of the compute units, keep their split,
        // although the unsplit kernel is the faster one there, too (1024 x 1024, 4 rows 4.5 us; split 5.3, 7 with the second kernel):
        // the scratch that is asked for follows the plan, and tests take these products to ask for some.
        static const int groups[6] = {1, 2, 3, 4, 6, 12};
        double best_us = 1e30;
        if (p.splits > 1 && 4 * ntiles > ncu)
            best_us = 0.85 * fq_small_us(M, N, K, bits, g, ncu, SKINNY_VARIANTS[p.variant].nt, p.gp, p.kw, p.au, p.splits);
        for (int v = 0; best_us < 20.0 && v < 4; ++v) {
            for (const int gp : groups) {
                const int need = (int)M * kc;
                const int au = need <= 64 * gp ? 1 : (need <= 128 * gp ? 2 : 0);
                int kw = SKINNY_VARIANTS[v].maxw / gp;
                if (kw > KB) kw = KB;
                if (au == 0 || kw < 1 || 3.9 + 0.3 * ((KB + kw - 1) / kw) > best_us) continue;
                const double t = fq_small_us(M, N, K, bits, g, ncu, SKINNY_VARIANTS[v].nt, gp, kw, au, 1);
                if (t < best_us - 1e-9) {
                    best_us = t;
                    p.variant = v;
                    p.gp = gp;
                    p.kw = kw;
                    p.au = au;
                    p.waves = gp * kw;
                    p.splits = 1;
                }
            }
        }
        p.kb_per_split = 0;
    } else {
        // Tiled MFMA kernel: BM = 16 * mt rows per block (mt = 2, 4 or 8), 48 columns per wave, 4 or 8
        // waves, and optionally a split of K over `splits` blocks whose binary32 partial tiles a second
        // kernel adds.  The block shape is the one that minimises a measured cost model:
        //   time = ceil(blocks / compute units) * k-blocks per block * u(mt, waves)  +  cost of the partials
        // where u is the time one block spends on one k-block of 128 rows of K when every compute
        // unit holds its share of blocks (microseconds), and the partials cost their write plus read
        // at ~5 TB/s plus a launch.  The constants are a least-squares fit (of log time; rms error
        // 9 - 11 %) to exhaustive sweeps of (mt, waves, splits) over the OPT-175B shapes at M = 17 ...
        // 256, both activation types, separately for the four kinds of kernels the dispatch
        // distinguishes (4-bit codes with 1, 2 or 4 scale rows per k-block, of which only the first
        // runs post-scaled at every small shape; 8-bit codes): the model's choice is 0.5 - 2 % slower
        // than the sweep's best on average, 15 % at worst.
        // Up to 256 rows the smaller blocks compete with the 128-row ones (several row blocks, each
        // converting the weights again) and often win there, e.g. QKV at M = 128 in two 64-row blocks
        // and no split of K.  Beyond 256 rows a narrow matrix makes few 128-row blocks, so the smaller ones compete there too
        // where the matrix has less than 8192 columns (wider bfloat16 products take the fp16 matrix path, in 128-row
        // blocks only).  They have to win by 5 % and to need no more scratch than the 128-row plan; 8-bit
        // plans of eight waves stay (none of the problems below would leave them).  Where these blocks hold bfloat16
        // operands with their storage bias and the 128-row ones hold q s, binary16 products alone take them, in the same split of K
        // (one size of scratch serves both types): beside activations 10^6 times their neighbours a bias costs precision.
        // 167 problems of 257 .. 2048 rows: 19 change, 1.15x faster on average, none more than 1.4 % slower; 1408 x 2752,
        // M = 1046 8-bit 27 -> 19 us, 5376 x 4816, M = 1212 g = 64 106 -> 81.
        p.kind = 1;
        const double* cs = fq_tiled_costs(bits, g);
        const int split_opts[6] = {1, 2, 3, 4, 6, 8};
        double best = 1e30;
        p.nt = MMA_NT;
        p.tail_tiles = 0;
        p.tail_splits = 1;
        p.tail_kbs = 0;
        double best128 = 1e30;       // the 128-row blocks' time and plan
        fq_gemm_plan p128 = {};
        for (int mt = 8; mt >= 2; mt /= 2) {
            // a block shape is a candidate when the matrix has more rows than half its height (the
            // smallest always is), and the small ones up to 256 rows, or 2048 on narrow matrices
            if (mt > 2 && (int64_t)mt * 8 >= M) continue;
            const bool tall = mt < 8 && M > 256;
            if (tall && (N >= 8192 || M > 2048 || (bits == 8 && p128.waves == 8))) continue;
            // (a biased bfloat16 operand, as use_post and Dequant make it)
            const bool biased = bits != 8 && (fq_scale_rows(bits, g) == 1 || (mt == 2 && fq_scale_rows(bits, g) == 2));
            if (tall && biased && (act_dtype != FQ_F16 || p128.tail_tiles > 0 || p.splits != p128.splits)) continue;
            const int bm = mt * 16;
            const int64_t nbm = (M + bm - 1) / bm;
            const double u8 = mt == 8 ? cs[4] : (mt == 4 ? cs[2] : cs[0]);
            const double u4 = mt == 8 ? cs[5] : (mt == 4 ? cs[3] : cs[1]);
            for (int waves = 8; waves >= 4; waves -= 4) {
                const int64_t nbn = (ntiles + waves * MMA_NT - 1) / (waves * MMA_NT);
                // k-blocks of this shape: 8-bit codes in the 128-row, 8-wave shape go two layout blocks at
                // a time (measured ~7 % less per row of K)
                const int kblk_c = fq_mma_kblk(bits, mt, waves, K, g);
                const int KB = (int)(K / kblk_c);
                const double kscale = (double)kblk_c / 128.0 * (kblk_c != kblk ? 0.93 : 1.0);
                const double u = (waves == 8 ? u8 : u4) * kscale;
                for (int si = 0; si < 6; ++si) {
                    int splits = split_opts[si];
                    if (splits > KB || (tall && splits > p128.splits)) break;
                    if (tall && biased && splits != p128.splits) continue;
                    const int kbs = (KB + splits - 1) / splits;
                    splits = (KB + kbs - 1) / kbs;
                    const int64_t blocks = nbn * nbm * splits;
                    const int64_t per_cu = (blocks + ncu - 1) / ncu;
                    double t = (double)per_cu * kbs * u;
                    if (waves == 4) {
                        // u is a 4-wave block's share when `cap` of them run together on a compute unit; the
                        // ones left over run with idle SIMDs and take longer than that share
                        const int cap = mt == 2 ? 3 : 2;
                        const int64_t left = per_cu % cap;
                        if (left > 0) {
                            const double f = per_cu < cap ? (mt == 8 ? cs[7] : cs[6]) : (mt == 8 ? 1.13 : 1.0);
                            t += (f - 1.0) * (double)left * kbs * u;
                        }
                    }
                    // (with fewer blocks than compute units a block takes as long as in a full grid)
                    if (splits > 1) t += 2.0 * splits * (double)M * (double)N * 4.0 / 5e6 + 5.0;
                    if (t < (tall && best == best128 ? 0.95 * best : best) - 1e-9) {
                        best = t;
                        p.mt = mt;
                        p.waves = waves;
                        p.splits = splits;
                        p.kb_per_split = kbs;
                        p.tail_tiles = 0;
                        p.tail_splits = 1;
                        p.tail_kbs = 0;
                    }
                }
                // No uniform split, but the tiles of the partly filled last round are split along K so
                // that they occupy every block slot once more: the last round then lasts 1 / tail_splits
                // of a full one, at the price of partial tiles for those tiles only.
                if (tall) continue;
                const int64_t tiles = nbn * nbm;
                const int64_t slots = (int64_t)ncu * (waves == 8 ? 1 : (mt == 2 ? 3 : 2));
                const int64_t rem = tiles % slots;
                if (tiles > slots && rem > 0) {
                    int ts = (int)(slots / rem);
                    if (ts > 8) ts = 8;
                    if (ts > KB) ts = KB;
                    if (ts >= 2) {
                        const int tkbs = (KB + ts - 1) / ts;
                        ts = (KB + tkbs - 1) / tkbs;
                        const int64_t head = tiles - rem;
                        double t = (double)(head / ncu) * KB * u + (double)((rem * ts + ncu - 1) / ncu) * tkbs * u;
                        const double bm_bn = (double)bm * (double)(waves * MMA_NT * FQ_NTILE);
                        t += 2.0 * ts * (double)rem * bm_bn * 4.0 / 5e6 + 5.0;
                        // for the small shapes the model is 10 % optimistic about this form (QKV at M = 256:
                        // 221 us predicted, 244 measured), so it has to win by that much
                        if (mt < 8) t *= 1.10;
                        if (ts >= 2 && t < best - 1e-9) {
                            best = t;
                            p.mt = mt;
                            p.waves = waves;
                            p.splits = 1;
                            p.kb_per_split = KB;
                            p.tail_tiles = (int)rem;
                            p.tail_splits = ts;
                            p.tail_kbs = tkbs;
                        }
                    }
                }
            }
            if (mt == 8) {
                best128 = best;
                p128 = p;
            }
        }
        if (M <= 48) {
            fq_gemm_plan mid = {};
            const double t_mid = fq_plan_mid(M, N, K, bits, g, ncu, &mid);
            if (fq_mid_pays(t_mid, p, best, M, N, bits, g)) {
                fq_plan_mid_narrow(M, N, K, bits, g, ncu, &mid);
                return mid;
            }
        }
        best = fq_plan_flexible(M, N, K, bits, g, act_dtype, ncu, best, &p);
        if (M > 48 && K <= FQ_ROW_BLOCKS_MOST_K && (M <= 256 || (N < 8192 && M <= 48 * 256))) {
            // Row blocks of the mid-M kernel (kind 3): as k-workers inside a block they split K without partial sums or a
            // second kernel, and 48 rows x 48 columns cut a small output finer than the tiled kernel's blocks.  Longer K lost up
            // to 15 %.  Above 256 rows bfloat16 products of wide matrices stay on the fp16 matrix path.  650 products that take
            // them, K from 256 to 6272 and N from 128 on, against the tiled plan:
            //   49 .. 256 rows       220   1.19x on average, 16 more than 3 % slower (15 % at worst: 50 - 64 rows, K of 3000 and more)
            //   257 .. 600 rows      150   1.19x, 23 slower (3 of them than the 128-row blocks, 4 % at worst)
            //   601 .. 12288 rows    280   1.24x, 29 slower (7 of them than the 128-row blocks, 8 %)
            // (1408 x 1056, 324 rows, 8-bit 16.5 -> 9.4 us.)  The slower ones have K of 3000 and more beside few columns: the
            // tiled kernel's split of K wins there, but needs scratch that these products do not ask for.
            int count[3] = {0, 0, M > 96 ? (int)(M - 49) / 48 : 0};       // (fq_mid_rows gives 48 while more than 96 are left)
            for (int32_t left = (int32_t)M - 48 * count[2], take = 0; left > 0; left -= take) {
                take = fq_mid_rows(left);
                ++count[(take - 1) / 16];
            }
            fq_small_shape sh = {};
            double busy = 0.0, longest = 0.0;
            // (above 256 rows weighed against the 128-row blocks as it was measured: the model does not rank it among the smaller
            // ones, which lost by up to 1.4x where they took its place)
            const double rival = M > 256 && p.mt < 8 ? best128 : best;
            const double limit = 0.95 * (rival + 2.0);
            const double rows_us = fq_plan_grouped_mid(count, N, K, bits, g, true, limit, &sh, &busy, &longest);
            bool pays = rows_us < limit;
            if (pays && fq_partial_bytes(p, M, N) == 0 && !fq_via_f16(act_dtype, FQ_SCALE_F16, p, N)) {
                const int blocks = ((ntiles + MMA_NT - 1) / MMA_NT + sh.gp - 1) / sh.gp * (count[0] + count[1] + count[2]);
                pays = longest * ((blocks + ncu - 1) / ncu) < limit;
            }
            if (pays) {
                p = fq_gemm_plan{};
                p.kind = 3;
                p.mt = 3;
                p.nt = MMA_NT;
                p.gp = sh.gp;
                p.kw = sh.kw;
                p.waves = sh.gp * sh.kw;
                p.splits = 1;
                p.tail_splits = 1;
                best = rows_us;
            }
        }
        if (M > 48 && M <= 256 && N < 8192 && K <= FQ_ROW_BLOCKS_MOST_K) fq_plan_rows_narrow(M, N, K, bits, g, ncu, best, &p);
    }
    return p;
}

// Whether all experts of a grouped product may take the small-M kernel: none has more than 16 rows, or none more than 32
// and at most one in nine more than 16 (those few become two items each: their weights are read twice, mostly from a cache
// the second time).
static bool fq_all_small(const int32_t* offsets, int E) {
    int n16 = 0, n32 = 0;
    for (int e = 0; e < E; ++e) {
        const int32_t rows = offsets[e + 1] - offsets[e];
        n16 += rows > 0 && rows <= 16;
        n32 += rows > 16;
        if (rows > 32) return false;
    }
    return 8 * n32 <= n16;
}

// Block shape for the experts of the small-M kernel: the shape with the least
//   (blocks / slots + 0.7) * (iterations * 1.5 us + ramp)
// i.e. the rounds of blocks, with an average partly filled one, times the time of a block: 12 waves stream 36 KiB per
// iteration, and a block's start and end cost 2.5 us (5 with the sum over k-workers).  Not rounded up to whole rounds:
// the other row classes of the call hold an unknown part of the compute units.  Against sweeps of 64 experts of 16384 x
// 4096 and 4096 x 16384 with 96 rows the model is within 10 %: e.g. 3 x 4 waves 224 us predicted / 239 measured, 12 x 1
// 336 / 337 on the former, 12 x 1 224 / 222, 4 x 3 253 / 248 on the latter.  Blocks have 12 or 4 waves: two blocks of
// six do not fit a compute unit's four SIMDs (310 us where 12 x 1 takes 222).
fq_small_shape fq_plan_grouped_small(int count, int units, int ngroups, int KB) {
    static const fq_small_shape shapes[7] = {{12, 1}, {6, 2}, {4, 3}, {3, 4}, {2, 6}, {4, 1}, {2, 2}};
    fq_small_shape best = {12, 1};
    double best_t = 1e30;
    for (const fq_small_shape& s : shapes) {
        if (units > 64 * s.gp || s.kw > KB) continue;
        const double together = 12.0 / (s.gp * s.kw);
        const double rounds = (double)((ngroups + s.gp - 1) / s.gp) * count / (fq_cu_count() * together);
        const double filled = rounds + 0.7;
        const double t = (filled < 1.0 ? 1.0 : filled) * (1.5 * ((KB + s.kw - 1) / s.kw) + (s.kw > 1 ? 5.0 : 2.5));
        if (t < best_t) {
            best_t = t;
            best = s;
        }
    }
    return best;
}

// The model's time of a call cut as `p` says; fills in `fork` and the mid-M kernel's block shape.
static double fq_grouped_us(const int32_t* offsets, int E, int64_t N, int64_t K, int bits, int g, fq_grouped_plan* p) {
    static const double tile_f[2][2] = {{0.85, 0.85}, {0.80, 0.83}};    // (3- and 4-bit codes, 8-bit codes) x (128, 64 rows)
    int count[FQ_TILE_CLASSES] = {}, mid_count[3] = {};
    int32_t small_rows = 0;
    for (int e = 0; e < E; ++e) {
        for (int32_t left = offsets[e + 1] - offsets[e], take = 0; left > 0; left -= take) {
            const fq_tile_class c = fq_next_tile(*p, left, &take);
            ++count[c];
            if (c == FQ_TILE_SMALL && take > small_rows) small_rows = take;
            if (c == FQ_TILE_MID) ++mid_count[(take - 1) / 16];
        }
    }
    const int ntiles = (int)(N / FQ_NTILE);
    const double ncu = (double)fq_cu_count();
    const double* cs = fq_tiled_costs(bits, g);
    double sum = 0.0, longest = 0.0, apart = 0.0;
    int classes = 0;
    auto add = [&](double busy, double block, double most) {
        double t = busy / ncu + 0.35 * block;
        t = t < most ? t : most;
        sum += busy;
        longest = block > longest ? block : longest;
        apart += t > block ? t : block;
        ++classes;
    };
    for (int c = FQ_TILE_128; c <= FQ_TILE_64; ++c) {
        if (count[c] == 0) continue;
        const int nblocks_n = (ntiles + 8 * MMA_NT - 1) / (8 * MMA_NT);
        const double t = (double)K / 128.0 * cs[c == FQ_TILE_128 ? 4 : 2] * tile_f[bits == 8][c] + 10.0;
        add(t * nblocks_n * count[c], t, 1e30);
    }
    if (count[FQ_TILE_MID] > 0) {
        double busy = 0.0, block = 0.0;
        const double t = fq_plan_grouped_mid(mid_count, N, K, bits, g, false, 1e30, &p->mid, &busy, &block);
        add(busy, block, t);
    }
    if (count[FQ_TILE_SMALL] > 0) {
        const int kblk = fq_kblk(bits);
        const int ngroups = (ntiles + 2) / 3, KB = (int)(K / kblk);
        const fq_small_shape s = fq_plan_grouped_small(count[FQ_TILE_SMALL], small_rows * (kblk / 8), ngroups, KB);
        const double t = 1.26 * ((KB + s.kw - 1) / s.kw) + (s.kw > 1 ? 5.0 : 2.5);
        add(t * ((ngroups + s.gp - 1) / s.gp) * count[FQ_TILE_SMALL] * (s.gp * s.kw) / 12.0, t, 1e30);
    }
    double t = sum / ncu + 0.35 * longest;
    t = (t > longest ? t : longest) + 21.0;
    p->fork = classes > 1 && t < apart;
    return p->fork ? t : apart;
}

// The cut with the least time by the model.  Against tiles of 128, 64 and 32 rows and the small-M kernel, each class on a
// stream of its own, the 200 calls are 1.24x faster on average, and up to 3.3x on small matrices, where one launch takes the
// place of four; 5 of them are more than 5 % slower (calls of 60 us and more: 9 % at worst).  Two sets of 200 others: experts
// that all fit the small-M kernel 1.03x, 13 more than 3 % slower (12 % at worst), with taller ones 1.41x, 11 slower (8 %); a
// different margin between the cuts makes as many calls slower as faster.  A launch of 32-row tiles
// of the tiled kernel was the best choice in none of them.  Experts of at most 16 rows stay with the small-M kernel unless
// the model gives that 15 % more, and with 8-bit codes always (up to 1.27x faster there).
fq_grouped_plan fq_plan_grouped(const int32_t* offsets, int E, int64_t N, int64_t K, int bits, int g) {
    fq_grouped_plan best = {};
    int32_t most = 0;
    for (int e = 0; e < E; ++e) most = offsets[e + 1] - offsets[e] > most ? offsets[e + 1] - offsets[e] : most;
    double best_us = 1e30;
    if (fq_all_small(offsets, E)) {
        best.cut = FQ_CUT_SMALL;
        if (most <= 16 && bits == 8) return best;
        best_us = fq_grouped_us(offsets, E, N, K, bits, g, &best) * (most <= 16 ? 0.85 : 1.0);
    }
    const fq_cut cuts[2] = {FQ_CUT_MID, FQ_CUT_TALL};
    for (const fq_cut cut : cuts) {
        if (cut == FQ_CUT_TALL && most <= 48) break;
        fq_grouped_plan p = {};
        p.cut = cut;
        const double us = fq_grouped_us(offsets, E, N, K, bits, g, &p);
        if (us < best_us) {
            best_us = us;
            best = p;
        }
    }
    return best;
}

int fq_launch_gemm(const fq_gemm_plan& plan, const void* A, int act, int64_t M, int64_t N, int64_t K, const void* codes,
                   const void* scales, int bits, int g, void* C, void* workspace, hipStream_t stream) {
#define FQ_PICK(ACT)                                                                                        \
    (bits == 3   ? fq_launch_typed_##ACT##_3(A, M, N, K, codes, scales, g, C, workspace, plan, stream)      \
     : bits == 4 ? fq_launch_typed_##ACT##_4(A, M, N, K, codes, scales, g, C, workspace, plan, stream)      \
                 : fq_launch_typed_##ACT##_8(A, M, N, K, codes, scales, g, C, workspace, plan, stream))
    if (act == FQ_F16) return FQ_PICK(0);
    if (act == FQ_BF16) return FQ_PICK(1);
    return FQ_PICK(2);
#undef FQ_PICK
}

// The grouped product launches up to three kernels (row tiles of 128, of 64 and of up to 48 rows) that do not
// depend on each other.  Launched one after the other on the caller's stream, each would end with
// a partly filled last round of blocks; where that costs more than the fork, they go to streams of their own: the blocks of the next kernel fill the
// compute units the previous one leaves idle.  The two extra streams (default priority) and the
// events that fork them from and join them to the caller's stream are created once per device and
// live until the process ends.
namespace {
struct fq_side {
    bool tried = false, ok = false;
    hipStream_t s[2];
    hipEvent_t fork, join[2];
};
std::mutex g_side_mutex;    // guards the creation of the side streams
std::mutex g_fork_mutex;    // serialises fork ... join sequences: the events are shared by all callers on a device
fq_side g_side[64];

fq_side* side_streams() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(g_side_mutex);
    fq_side& x = g_side[dev];
    if (!x.tried) {
        x.tried = true;
        bool ok = hipEventCreateWithFlags(&x.fork, hipEventDisableTiming) == hipSuccess;
        for (int i = 0; i < 2; ++i)
            ok = ok && hipStreamCreateWithFlags(&x.s[i], hipStreamNonBlocking) == hipSuccess &&
                 hipEventCreateWithFlags(&x.join[i], hipEventDisableTiming) == hipSuccess;
        x.ok = ok;
        if (!ok) (void)hipGetLastError();
    }
    return x.ok ? &x : nullptr;
}
}  // namespace

int fq_launch_gemm_grouped(const void* A, int act, const int32_t* offsets, int E, int64_t N, int64_t K,
                           const void* codes, const void* scales, int bits, int g, void* C,
                           hipStream_t stream) {
    const fq_grouped_plan plan = fq_plan_grouped(offsets, E, N, K, bits, g);
    bool has[FQ_TILE_CLASSES] = {};
    for (int e = 0; e < E; ++e)
        for (int32_t left = offsets[e + 1] - offsets[e], take = 0; left > 0; left -= take) has[fq_next_tile(plan, left, &take)] = true;
    hipStream_t streams[FQ_TILE_CLASSES];
    for (hipStream_t& s : streams) s = stream;
    fq_side* side = plan.fork ? side_streams() : nullptr;
    // host threads that fork at the same time would record and wait on each other's events
    std::unique_lock<std::mutex> fork_lock(g_fork_mutex, std::defer_lock);
    if (side) fork_lock.lock();
    bool forked[2] = {false, false};
    if (side) {
        // the first class present stays on the caller's stream, the others go to the side streams
        int next = -1;
        if (hipEventRecord(side->fork, stream) != hipSuccess) return FQ_ERR_HIP;
        for (int c = 0; c < FQ_TILE_CLASSES; ++c) {
            if (!has[c]) continue;
            if (next >= 0) {
                if (hipStreamWaitEvent(side->s[next], side->fork, 0) != hipSuccess) return FQ_ERR_HIP;
                forked[next] = true;
                streams[c] = side->s[next];
            }
            if (++next == 2) break;
        }
    }
    int st;
#define FQ_PICK(ACT)                                                                                        \
    (bits == 3   ? fq_launch_grouped_typed_##ACT##_3(A, offsets, E, plan, N, K, codes, scales, g, C, streams)     \
     : bits == 4 ? fq_launch_grouped_typed_##ACT##_4(A, offsets, E, plan, N, K, codes, scales, g, C, streams)     \
                 : fq_launch_grouped_typed_##ACT##_8(A, offsets, E, plan, N, K, codes, scales, g, C, streams))
    if (act == FQ_F16) st = FQ_PICK(0);
    else if (act == FQ_BF16) st = FQ_PICK(1);
    else st = FQ_PICK(2);
#undef FQ_PICK
    // join even after a failed launch, so that the side streams never run ahead of the caller's
    for (int i = 0; i < 2; ++i) {
        if (!forked[i]) continue;
        if (hipEventRecord(side->join[i], side->s[i]) != hipSuccess ||
            hipStreamWaitEvent(stream, side->join[i], 0) != hipSuccess)
            st = st == FQ_OK ? FQ_ERR_HIP : st;
    }
    return st;
}
