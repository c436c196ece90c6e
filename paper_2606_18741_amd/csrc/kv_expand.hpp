// Block-table expansion into per-block descriptors, and the bucket sort of the new
// descriptors by physical block.
// Included by migrate.hip only (one translation unit holds every kernel).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kv_device.hpp"

namespace remp {

// ---------------------------------------------------------------------------
// expansion: block tables -> one descriptor per live block
// ---------------------------------------------------------------------------

// Bucket of a physical block for the descriptor sort of the new tables (see
// below): nb buckets spread evenly over [0, num_blocks).
constexpr int kDescsPerBucket = 4;   // buckets = ceil(live blocks / 4): order kept at ~4-block granularity

__device__ __forceinline__ uint32_t block_bucket(int32_t block, int64_t num_blocks, uint32_t nb) {
    const int64_t b = static_cast<int64_t>(block > 0 ? block : 0) * nb / num_blocks;
    return static_cast<uint32_t>(b < nb ? b : nb - 1);
}

// Exclusive prefix sums of tokens and of blocks per sequence (one workgroup,
// wave64 shuffle scans combined through LDS, carried across chunks of 1024).
__global__ __launch_bounds__(kScanThreads) void expand_scan(const int32_t* __restrict__ lens, int32_t S,
                                                           int32_t bs, int32_t reset_flag, int32_t* __restrict__ flag,
                                                           int32_t* __restrict__ tok_off,
                                                           int32_t* __restrict__ blk_off,
                                                           int32_t* __restrict__ bucket, uint32_t nb) {
    __shared__ int64_t wave_tok[kScanThreads / 64];
    __shared__ int64_t wave_blk[kScanThreads / 64];
    __shared__ int64_t carry[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) {
        carry[0] = 0;
        carry[1] = 0;
        if (reset_flag) *flag = 0;
    }
    if (bucket)   // counters of the descriptor sort, filled by expand_emit
        for (uint32_t i = tid; i < nb; i += kScanThreads) bucket[i] = 0;
    __syncthreads();
    bool bad = false;
    for (int32_t base = 0; base < S; base += kScanThreads) {
        const int32_t s = base + tid;
        int64_t n = s < S ? lens[s] : 0;
        if (n < 0) {
            n = 0;
            bad = true;
        }
        const int64_t nb = (n + bs - 1) / bs;
        int64_t it = n, ib = nb;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t a = __shfl_up(it, d, 64);
            const int64_t b = __shfl_up(ib, d, 64);
            if (lane >= d) {
                it += a;
                ib += b;
            }
        }
        if (lane == 63) {
            wave_tok[wave] = it;
            wave_blk[wave] = ib;
        }
        __syncthreads();
        if (wave == 0) {
            const int nw = kScanThreads / 64;
            int64_t wt = lane < nw ? wave_tok[lane] : 0;
            int64_t wb = lane < nw ? wave_blk[lane] : 0;
#pragma unroll
            for (int d = 1; d < nw; d <<= 1) {
                const int64_t a = __shfl_up(wt, d, 64);
                const int64_t b = __shfl_up(wb, d, 64);
                if (lane >= d) {
                    wt += a;
                    wb += b;
                }
            }
            if (lane < nw) {   // exclusive totals of preceding waves
                wave_tok[lane] = wt;
                wave_blk[lane] = wb;
            }
        }
        __syncthreads();
        const int64_t pre_t = carry[0] + (wave ? wave_tok[wave - 1] : 0);
        const int64_t pre_b = carry[1] + (wave ? wave_blk[wave - 1] : 0);
        if (s < S) {
            const int64_t et = pre_t + it - n, eb = pre_b + ib - nb;
            if (et > INT32_MAX || eb > INT32_MAX) bad = true;
            tok_off[s] = static_cast<int32_t>(et < INT32_MAX ? et : INT32_MAX);
            blk_off[s] = static_cast<int32_t>(eb < INT32_MAX ? eb : INT32_MAX);
        }
        __syncthreads();
        if (tid == kScanThreads - 1) {
            carry[0] = pre_t + it;
            carry[1] = pre_b + ib;
        }
        __syncthreads();
    }
    if (tid == 0) {
        tok_off[S] = static_cast<int32_t>(carry[0] < INT32_MAX ? carry[0] : INT32_MAX);
        blk_off[S] = static_cast<int32_t>(carry[1] < INT32_MAX ? carry[1] : INT32_MAX);
    }
    if (bad) *flag = kFlagTables;
}

// One thread per live block: locate its sequence by binary search over the
// block offsets, then read its id from the table row.  Every index is bounded
// by the host-side sizes; an inconsistency yields an empty descriptor and sets
// the flag instead of an out-of-bounds access.
__global__ __launch_bounds__(256) void expand_emit(const int32_t* __restrict__ lens,
                                                   const int32_t* __restrict__ row_off,
                                                   const int32_t* __restrict__ ids, int32_t S, int32_t bs,
                                                   const int32_t* __restrict__ tok_off,
                                                   const int32_t* __restrict__ blk_off, int64_t nnz,
                                                   int64_t num_blocks, int64_t total_tokens, int64_t n_desc,
                                                   BlockDesc* __restrict__ desc, int32_t* __restrict__ flag,
                                                   int32_t* __restrict__ bucket, uint32_t nb,
                                                   uint64_t* __restrict__ stamp_at, uint64_t stamp) {
    const int64_t b = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (b == 0 && stamp_at) *stamp_at = stamp;   // the descriptors are complete once this kernel is
    if (b >= n_desc) return;
    int32_t lo = 0, hi = S;   // last s in [0, S] with blk_off[s] <= b
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (blk_off[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    BlockDesc d{0, 0, 0, 0};
    bool ok = lo < S;
    if (ok) {
        const int32_t s = lo;
        const int64_t j = b - blk_off[s];
        const int64_t n = lens[s];
        const int64_t r = static_cast<int64_t>(row_off[s]) + j;
        ok = r >= 0 && r < nnz;
        if (ok) {
            const int64_t id = ids[r];
            const int64_t tok = static_cast<int64_t>(tok_off[s]) + j * bs;
            const int64_t rest = n - j * bs;
            const int64_t cnt = rest < bs ? rest : bs;
            ok = id >= 0 && id < num_blocks && cnt > 0 && tok >= 0 && tok + cnt <= total_tokens;
            if (ok) d = BlockDesc{static_cast<int32_t>(id), static_cast<int32_t>(tok), static_cast<int32_t>(cnt), s};
        }
    }
    if (!ok) *flag = kFlagTables;
    desc[b] = d;
    if (bucket) atomicAdd(&bucket[block_bucket(d.block, num_blocks > 0 ? num_blocks : 1, nb)], 1);
}

// ---------------------------------------------------------------------------
// ordering of the new descriptors by physical block
// ---------------------------------------------------------------------------

// The new tables come from a serving engine's free list, so consecutive live
// blocks sit at scattered physical addresses, and an unpack in descriptor
// order writes the pool in random 4-64 KiB pieces.  On MI355X random writes
// cost more than random reads (measured, 4 KiB pieces: 5.6 TB/s scattered
// writes against 6.1 TB/s scattered reads), so the new descriptors are
// bucket-sorted by block id first: the expansion clears and counts the
// buckets, then an exclusive scan and a scatter.  Order inside a bucket is
// whatever the atomics give; every order yields the same bytes.

// Exclusive scan of cnt[0, nb) in place (one workgroup, 4 consecutive counters
// per thread, carried over chunks of 4096).
constexpr int kSortScanPerThread = 4;

__global__ __launch_bounds__(kScanThreads) void sort_scan(int32_t* __restrict__ cnt, uint32_t nb) {
    __shared__ int32_t wave_sum[kScanThreads / 64];
    __shared__ int32_t carry;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (uint32_t base = 0; base < nb; base += kScanThreads * kSortScanPerThread) {
        const uint32_t i0 = base + tid * kSortScanPerThread;
        int32_t c[kSortScanPerThread];
        int32_t v = 0;
#pragma unroll
        for (int k = 0; k < kSortScanPerThread; ++k) {
            c[k] = i0 + k < nb ? cnt[i0 + k] : 0;
            v += c[k];
        }
        int32_t x = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t a = __shfl_up(x, d, 64);
            if (lane >= d) x += a;
        }
        if (lane == 63) wave_sum[wave] = x;
        __syncthreads();
        if (wave == 0) {
            const int nw = kScanThreads / 64;
            int32_t w = lane < nw ? wave_sum[lane] : 0;
#pragma unroll
            for (int d = 1; d < nw; d <<= 1) {
                const int32_t a = __shfl_up(w, d, 64);
                if (lane >= d) w += a;
            }
            if (lane < nw) wave_sum[lane] = w;
        }
        __syncthreads();
        int32_t run = carry + (wave ? wave_sum[wave - 1] : 0) + x - v;   // exclusive prefix of counter i0
#pragma unroll
        for (int k = 0; k < kSortScanPerThread; ++k) {
            if (i0 + k < nb) cnt[i0 + k] = run;
            run += c[k];
        }
        const int32_t pre = carry + (wave ? wave_sum[wave - 1] : 0);
        __syncthreads();
        if (tid == kScanThreads - 1) carry = pre + x;
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void sort_scatter(const BlockDesc* __restrict__ desc, int32_t n, int64_t num_blocks,
                                                    uint32_t nb, int32_t* __restrict__ next,
                                                    BlockDesc* __restrict__ out, uint64_t* __restrict__ stamp_at,
                                                    uint64_t stamp) {
    const int32_t i = static_cast<int32_t>(blockIdx.x * 256 + threadIdx.x);
    if (i == 0 && stamp_at) *stamp_at = stamp;   // the sorted descriptors are complete once this kernel is
    if (i < n) {
        const BlockDesc d = desc[i];
        const int32_t pos = atomicAdd(&next[block_bucket(d.block, num_blocks, nb)], 1);
        if (pos >= 0 && pos < n) out[pos] = d;
    }
}

// ---------------------------------------------------------------------------
// expansion and ordering of few blocks by one workgroup
// ---------------------------------------------------------------------------

// expand_scan, expand_emit and, with bucket, sort_scan and sort_scatter in one launch, for at most kSmallSeqs sequences
// and kSmallBlocks live blocks: the offsets and the bucket counters stay in LDS.  Bound by latency: each launch that it
// saves takes 2-5 us, and every 1024 blocks take one workgroup 6-7 us more a call pair.  Measured on MI355X (us, pack and
// unpack, by several launches / by this one): 64 blocks 33.4 / 19.4, 512 33.6 / 21.8, 1024 33.6 / 28.1, 2048 45.5 / 41.6, 3072 56.9 /
// 54.5, 4096 67.8 / 69.0, 6000 86.8 / 92.7, 9000 118.6 / 133.2.
constexpr int32_t kSmallSeqs = kScanThreads;
constexpr int64_t kSmallBlocks = 4096;
constexpr int kSmallBuckets = kSmallBlocks / kDescsPerBucket;

// Exclusive prefix sum of v over the workgroup's threads and the total; wave: one value per wave, in LDS.
template <typename T>
__device__ __forceinline__ T block_prefix(T v, T* wave, T* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    T x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T a = __shfl_up(x, d, 64);
        if (lane >= d) x += a;
    }
    if (lane == 63) wave[w] = x;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < kScanThreads / 64; ++k) {
        if (k < w) before += wave[k];
        all += wave[k];
    }
    *total = all;
    return before + x - v;
}

__global__ __launch_bounds__(kScanThreads) void expand_small(
    const int32_t* __restrict__ lens, const int32_t* __restrict__ row_off, const int32_t* __restrict__ ids, int32_t S,
    int32_t bs, int64_t nnz, int64_t num_blocks, int64_t total_tokens, int32_t n_desc, int32_t reset_flag,
    int32_t* __restrict__ flag, int32_t* __restrict__ tok_off, int32_t* __restrict__ blk_off,
    BlockDesc* __restrict__ desc, int32_t* __restrict__ bucket, uint32_t nb, BlockDesc* __restrict__ sorted,
    uint64_t* __restrict__ stamp_at, uint64_t stamp) {
    __shared__ int64_t wave_tok[kScanThreads / 64], wave_blk[kScanThreads / 64];
    __shared__ int32_t wave_cnt[kScanThreads / 64];
    __shared__ int32_t s_len[kSmallSeqs], s_row[kSmallSeqs], s_tok[kSmallSeqs], s_blk[kSmallSeqs + 1];
    __shared__ int32_t s_cnt[kSmallBuckets];
    __shared__ int32_t s_bad;
    const int tid = threadIdx.x;
    if (tid == 0) s_bad = 0;
    if (bucket)
        for (uint32_t k = tid; k < nb; k += kScanThreads) s_cnt[k] = 0;
    bool bad = false;
    const int64_t len = tid < S ? lens[tid] : 0;
    if (tid < S) {
        s_len[tid] = static_cast<int32_t>(len);
        s_row[tid] = row_off[tid];
    }
    if (len < 0) bad = true;
    const int64_t n = len < 0 ? 0 : len;
    int64_t tokens, blocks;
    const int64_t et = block_prefix<int64_t>(n, wave_tok, &tokens);
    const int64_t eb = block_prefix<int64_t>((n + bs - 1) / bs, wave_blk, &blocks);
    if (tid < S) {
        if (et > INT32_MAX || eb > INT32_MAX) bad = true;
        s_tok[tid] = static_cast<int32_t>(et < INT32_MAX ? et : INT32_MAX);
        s_blk[tid] = static_cast<int32_t>(eb < INT32_MAX ? eb : INT32_MAX);
        tok_off[tid] = s_tok[tid];
        blk_off[tid] = s_blk[tid];
    }
    if (tid == 0) {
        s_blk[S] = static_cast<int32_t>(blocks < INT32_MAX ? blocks : INT32_MAX);
        tok_off[S] = static_cast<int32_t>(tokens < INT32_MAX ? tokens : INT32_MAX);
        blk_off[S] = s_blk[S];
    }
    __syncthreads();

    const int64_t nblk = num_blocks > 0 ? num_blocks : 1;
#pragma unroll 4
    for (int32_t b = tid; b < n_desc; b += kScanThreads) {   // as expand_emit
        int32_t lo = 0, hi = S;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (s_blk[mid] <= b) lo = mid;
            else hi = mid - 1;
        }
        BlockDesc d{0, 0, 0, 0};
        bool ok = lo < S;
        if (ok) {
            const int64_t j = b - s_blk[lo];
            const int64_t r = static_cast<int64_t>(s_row[lo]) + j;
            ok = r >= 0 && r < nnz;
            if (ok) {
                const int64_t id = ids[r];
                const int64_t tok = static_cast<int64_t>(s_tok[lo]) + j * bs;
                const int64_t rest = s_len[lo] - j * bs;
                const int64_t cnt = rest < bs ? rest : bs;
                ok = id >= 0 && id < num_blocks && cnt > 0 && tok >= 0 && tok + cnt <= total_tokens;
                if (ok)
                    d = BlockDesc{static_cast<int32_t>(id), static_cast<int32_t>(tok), static_cast<int32_t>(cnt), lo};
            }
        }
        if (!ok) bad = true;
        desc[b] = d;
        if (bucket) atomicAdd(&s_cnt[block_bucket(d.block, nblk, nb)], 1);
    }
    if (bad) s_bad = 1;
    __syncthreads();
    if (tid == 0) {
        if (s_bad) *flag = kFlagTables;
        else if (reset_flag) *flag = 0;
        if (stamp_at) *stamp_at = stamp;   // the descriptors are complete once this kernel is
    }
    if (!bucket) return;

    constexpr int kPer = kSmallBuckets / kScanThreads;   // counters per thread, scanned in place
    int32_t c[kPer], sum = 0, total;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t i = tid * kPer + k;
        c[k] = i < nb ? s_cnt[i] : 0;
        sum += c[k];
    }
    int32_t at = block_prefix<int32_t>(sum, wave_cnt, &total);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t i = tid * kPer + k;
        if (i < nb) s_cnt[i] = at;
        at += c[k];
    }
    __syncthreads();
#pragma unroll 4
    for (int32_t b = tid; b < n_desc; b += kScanThreads) {   // each thread's own descriptors
        const BlockDesc d = desc[b];
        const int32_t pos = atomicAdd(&s_cnt[block_bucket(d.block, nblk, nb)], 1);
        if (pos >= 0 && pos < n_desc) sorted[pos] = d;
    }
    __syncthreads();
    for (uint32_t k = tid; k < nb; k += kScanThreads) bucket[k] = s_cnt[k];
}

}  // namespace remp
