// The sum of a split of K over the grid, made by the kernel that makes the partial sums.
//
// Every block writes its binary32 (or int32) partial sums through to memory and then takes a ticket of its output tile;
// the block that takes the last one adds the tile's partial sums, split 0 + split 1 + ..., in the order of the separate
// sum kernel, and stores the result.  No block waits for another.  What this saves is a second launch: 2.7 us of the
// host's time and 3 - 5 us on the GPU, of products that take 7 - 20.
//
// The ticket is a 64-bit word in the output itself: the first four 16-bit results of the tile's row 0, which nobody but
// the last block writes and which hold anything before the call.  It needs no clearing and no memory beside the caller's
// (the scratch of a product is exactly its partial sums): a block counts in a word that carries the call's tag, and tags
// the word first where it does not.  A tag is used by one call only (fq_next_tag) and is gone when the call ends, since
// the results take its place, so that a captured call may be replayed with the tag that it was captured with.  Its upper
// 16 bits are a NaN in either 16-bit type, 0xffa5; results could hold that one too (a NaN's payload may pass through a
// conversion), but not with the call's 40 bits beside it.
//
// So C must be the call's own while it runs: a second call that counted in the same words at the same time would replace the
// tag, and neither would find its last block.  (A word elsewhere would have to be the library's: the scratch that callers hand
// over holds the partial sums and nothing else.)  Where C lies on an input, or C or the scratch is not the device's own memory, the separate sum
// kernel adds, as it does for outputs that are not aligned.
//
// Memory: partial sums and tickets are read and written with accesses of agent scope, which pass by the L2 caches (one
// per XCD, not coherent with each other within a kernel); a block's ticket is taken after its stores have completed.
#ifndef FQ_SPLIT_SUM_H_
#define FQ_SPLIT_SUM_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fqk {

constexpr int FQ_MOST_FUSED_SPLITS = 8;      // partial sums that a lane of the last block has in flight

// Whether a block adds the splits of its tile (rows x cols, partial sums of 32 bits): not where the word in C would not be
// aligned, nor above 80 KiB of partial sums per tile, which one block reads in 5 us and more where the sum kernel's blocks
// share them.  Timed inside graphs, where a launch costs the host nothing, one kernel against two, 570 products of 1 - 48 rows
// and of the integer path: up to 24 KiB 1.09x on average (219, worst 0.98x; 5248 x 1920, 9 rows 9.4 -> 8.0 us), 24 - 80 KiB 1.03x
// (307; six of them more than 3 % slower, 5 % at worst, most with blocks of six waves and 40 KiB or more: 3584 x 400, 44 rows
// 8.2 -> 8.6; 8576 x 21120, 13 rows, seven waves 34.0 -> 35.3), 80 - 110 KiB 0.99x (44, six slower), above 0.92 - 1.02x
// (3968 x 4240, 36 rows, 162 KiB 13.2 -> 15.5; 8192 x 28672, 16 rows, 180 KiB 43.5 -> 44.9).  KiB per wave predict the slower
// ones no better.  A call on its own also saves the launch: 1024 x 1024, 4 rows 10.1 -> 6.5 us.
inline bool fq_sums_splits(int rows, int cols, int splits, const void* C) {
    return splits > 1 && splits <= FQ_MOST_FUSED_SPLITS && ((uintptr_t)C & 7) == 0 && (int64_t)rows * cols * 4 * splits <= 80 * 1024;
}

// Bits of the 64-bit word: 0xffa5 | 40 bits that count the calls of the process | 8 bits that count blocks.
__device__ inline uint64_t ticket_peek(const uint64_t* word) {
    return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Tags the word that held `seen`.  The exchange fails only where another block of the call has tagged it since.
__device__ inline void ticket_tag(uint64_t* word, uint64_t seen, uint64_t tag) {
    if ((seen ^ tag) >> 8)
        __hip_atomic_compare_exchange_strong(word, &seen, tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Called by every thread of a block once its partial sums are stored: true in the block that is the tile's last.  `flag`
// is LDS that the block no longer reads.
__device__ inline bool ticket_last(uint64_t* word, int splits, uint64_t tag, uint32_t* flag) {
    uint64_t seen = 0;
    if (threadIdx.x == 0) seen = ticket_peek(word);      // (beside the last stores: no wait of its own)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's stores have reached memory
    __syncthreads();
    if (threadIdx.x == 0) {
        ticket_tag(word, seen, tag);
        *flag = (uint32_t)__hip_atomic_fetch_add(word, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xffu;
    }
    __syncthreads();
    return *flag == (uint32_t)(splits - 1);
}

// Four partial sums (V: a vector of four 32-bit values, 16-byte aligned).  through: with agent scope (sc1), for a block of
// this kernel to read; the separate kernel finds plain stores in the caches (8192 x 28672, 16 rows 42.1 us, 43.2 with sc1).
// The compiler's atomic stores end at eight bytes, and two of them cost the streaming kernels registers that they do not
// have.  (The wait states: a store of more than eight bytes reads its data after it has issued.)
template <typename V>
__device__ inline void store_partial(void* p, const V& v, bool through) {
    static_assert(sizeof(V) == 16, "");
    if (through) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
    else *reinterpret_cast<V*>(p) = v;
}
template <typename V>
__device__ inline V load_partial(const void* p) {
    typedef uint64_t u64x2v __attribute__((ext_vector_type(2)));
    u64x2v b;
    b[0] = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    b[1] = __hip_atomic_load((const uint64_t*)p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_bit_cast(V, b);
}
// split 0 + split 1 + ... of the four sums at p, `stride` values apart; all of them in flight at once
template <typename V, typename T>
__device__ inline V sum_partials(const T* p, int64_t stride, int splits) {
    V part[FQ_MOST_FUSED_SPLITS];
#pragma unroll
    for (int s = 0; s < FQ_MOST_FUSED_SPLITS; ++s)
        if (s < splits) part[s] = load_partial<V>(p + s * stride);
    V v = part[0];
#pragma unroll
    for (int s = 1; s < FQ_MOST_FUSED_SPLITS; ++s)
        if (s < splits) {
            v[0] += part[s][0]; v[1] += part[s][1]; v[2] += part[s][2]; v[3] += part[s][3];
        }
    return v;
}

// The end of a block of a split that its kernel sums (tag != 0): if the block is the last of its tile, rows x cols of C from
// column n0 on (C and partial at the tile's row 0, splits `stride` values apart), it hands every four sums to
// store(row, column, sums), neighbouring lanes in the same row.
template <typename V, typename T, typename STORE>
__device__ __forceinline__ void finish_split_sums(void* lds, const T* partial, int64_t stride, int splits, uint16_t* C, int rows,
                                                  int N, int n0, int cols, uint64_t tag, STORE store) {
    if (tag == 0 || !ticket_last(reinterpret_cast<uint64_t*>(C + n0), splits, tag, reinterpret_cast<uint32_t*>(lds))) return;
    const int quads = (cols < N - n0 ? cols : N - n0) / 4;
    for (int q = threadIdx.x; q < rows * quads; q += blockDim.x) {
        const int m = q / quads, n = n0 + (q - m * quads) * 4;
        store(m, n, sum_partials<V>(partial + (int64_t)m * N + n, stride, splits));
    }
}

}  // namespace fqk

#endif  // FQ_SPLIT_SUM_H_
