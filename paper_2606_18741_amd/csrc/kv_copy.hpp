// The pack / unpack copy kernel (copy_runs) and the NHD local copies (copy_local, copy_local_rows).
// Included by migrate.hip only (one translation unit holds every kernel).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kv_device.hpp"

namespace remp {

// ---------------------------------------------------------------------------
// pack / unpack copy
// ---------------------------------------------------------------------------


// One launch copies the same part of several slices (grid y) for K and V (grid z); grid x numbers the
// words of a slice's live blocks, block after block, and a wave takes 1 KiB of them.  Bound by HBM.
// Of aligned 16-byte words the waves are as short as they can be: with one vector in
// flight per lane the chip already has 8 MiB in flight at full occupancy, and more loads per lane or
// longer workgroups only spread the accesses over more DRAM rows at a time (kRunThreads has the rates).
// Nothing passes through LDS and no wave waits for another.  K and V are separate runs of the grid, not
// alternating units: +1.2% on 4 KiB units, +3.2% on 32 KiB units.
// Measured on MI355X against the kernel before it (128 threads x 4 vectors per 8 KiB, descriptors through
// LDS, flat loads): random 4 KiB blocks packed 5.99 -> 6.29 TB/s, 32 KiB blocks 5.90 -> 6.40 TB/s.
// Rows that are not whole vectors, or not aligned, go by words of V = 8 bytes, K to a lane, or (V = 0) by 16 bytes at any
// address and smaller parts at the end of a row (run_words has the rates).
// What a wave's words are:
//   kRuns     of whole paged rows, so a block's live rows are one run of bytes on both sides
//   kCutRows  of parts of rows, row after row, cut wherever the wave's words end
//   kRows     the same, but of the whole rows that fit into the wave, K and V by turns
enum RunShape { kRuns, kCutRows, kRows };

template <bool PACK, int N, RunShape SHAPE, int V, int K, int ITEMS>
__global__ __launch_bounds__(kMaxRunThreads) void copy_runs(const CopyArgs<ITEMS> args) {
    constexpr uint32_t W = V ? V : kVecBytes;   // bytes of a word
    if (stale_descriptors(args.check)) return;
    const CopyItem& it = args.items[blockIdx.y];
    const uint32_t row_bytes = it.row_bytes, lane = threadIdx.x & 63u;
    const uint32_t vpr = (row_bytes + W - 1) / W;
    WaveUnits<N> units;
    uint32_t kv = blockIdx.z, first;
    if (SHAPE == kRows) {
        kv = blockIdx.x & 1u;
        first = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(
                    static_cast<int>(((blockIdx.x >> 1) * blockDim.x + threadIdx.x) / 64))) * it.rows;
    } else {
        first = wave_first(args.xcd) * K;
    }
    if (!units.load(args.desc, args.n_desc, first, it.vpu, it.vpu_magic, it.vpu_shift)) return;
    Moved<V> word[K];
    uint64_t dst[K];
    uint32_t left[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        left[k] = 0;
        BlockDesc d;
        uint32_t r, i = k * 64 + lane, c = 0;
        if (SHAPE == kRows) {
            const uint32_t j = fast_div(i, it.vpr_magic, it.vpr_shift);
            if (j >= it.rows) continue;
            c = i - j * vpr;
            i = j;
        }
        if (!units.pick(args.desc, args.n_desc, i, it.vpu, it.vpu_magic, it.vpu_shift, &d, &r)) continue;
        const uint32_t n = static_cast<uint32_t>(d.n);
        uint64_t paged = (kv ? it.paged_v : it.paged_k) + static_cast<uint64_t>(static_cast<uint32_t>(d.block)) *
                                                              static_cast<uint64_t>(args.block_stride);
        uint64_t stage =
            it.stage + (static_cast<uint64_t>(kv) * args.total_tokens + static_cast<uint32_t>(d.tok)) * row_bytes;
        uint32_t off = r * W, len = n * row_bytes;
        if (SHAPE != kRuns) {
            const uint32_t row = SHAPE == kRows ? r : fast_div(r, it.vpr_magic, it.vpr_shift);
            if (SHAPE == kCutRows) c = r - row * vpr;
            paged += static_cast<uint64_t>(row) * args.row_stride;
            stage += static_cast<uint64_t>(row) * row_bytes;
            off = c * W;
            len = row < n ? row_bytes : 0;
        }
        if (off >= len) continue;
        left[k] = len - off;
        dst[k] = (PACK ? stage : paged) + off;
        word[k].load((PACK ? paged : stage) + off, left[k]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (left[k]) word[k].store(dst[k], left[k]);
}


// Local copy (a slice whose old and new owner is the same rank): the new pool's live blocks are walked as
// in copy_runs, and each row's source is found through the old descriptors.  A new block's first token
// lies t0 tokens into its sequence, whose old blocks start at descriptor b0; both come by scalar loads
// behind the block's own descriptor, and behind them the M old descriptors that the wave's rows of the block can come
// from.  Where those are more than two, or the wave meets many blocks, each lane loads its row's (M = 0, N = 0).
// Bound by HBM.  Measured on MI355X: the chain of scalar loads costs 2% (4 KiB blocks 6.12 TB/s, 6.24 with the old
// block ids at hand); the rows of 16 KiB resolved into LDS first, by 256 threads x 2 vectors, ran at 5.5, and a look-up
// per lane between block sizes at 4.9 (256-byte rows, blocks of 64 to 20, us: LDS 652, by lane 713, so 620).
constexpr int kMaxLocalItems = 8;     // local slices per launch (few per launch measured faster, as for kMaxItems)
constexpr int kMaxLocalRows = 1024;   // largest new block size of the local copies

struct LocalItem {
    uint64_t src_k, src_v;   // old storage of the layer, offset to the slice's first head
    uint64_t dst_k, dst_v;   // new storage of the layer, offset to the slice's first head
    uint32_t row_bytes;
    uint32_t vpr_magic;      // fast division by words per row
    uint32_t vpu;            // words per (new block, K or V) unit
    uint32_t vpu_magic;
    uint16_t vpr_shift;
    uint16_t vpu_shift;
    uint32_t pad;
};

struct LocalArgs {
    const BlockDesc* new_desc;
    const BlockDesc* old_desc;
    const int32_t* tok_off;       // first token of each sequence on the token axis
    const int32_t* old_blk_off;   // first old descriptor of each sequence
    int32_t* flag;
    int64_t old_block_stride, new_block_stride;
    uint32_t n_new_desc, n_old_desc;
    uint32_t old_row_stride, new_row_stride;
    uint32_t old_block_size, new_block_size;
    uint32_t bo_magic, bo_shift;  // fast division by the old block size
    uint32_t bn_magic, bn_shift;  // and by the new one
    uint32_t xcd;                 // as in CopyArgs
    StampCheck check;
    LocalItem items[kMaxLocalItems];
};
static_assert(sizeof(LocalArgs) < 4096, "local copy kernel arguments must stay below 4 KiB");

// What the lanes of a wave need to know of one new block: its id, live tokens and sequence, its first token's index in its
// sequence (negative when the device tables disagree), the sequence's first old descriptor and the M (0: none) old
// blocks from number b0 + q on that hold its rows from `row` on, as (id, live tokens; 0: not of this sequence).
struct OldBlock {
    int32_t block, n;
};

template <int M>
struct LocalUnit {
    int32_t block, n, seq;
    int32_t t0, b0;
    uint32_t q;
    Values<OldBlock, M> o;
};

__device__ __forceinline__ void choose(bool yes, const OldBlock& v, OldBlock* own) {
    own->block = yes ? v.block : own->block;
    own->n = yes ? v.n : own->n;
}

template <typename T>
__device__ __forceinline__ void choose(bool, const Values<T, 0>&, Values<T, 0>*) {}

template <typename T, int N>
__device__ __forceinline__ void choose(bool yes, const Values<T, N>& v, Values<T, N>* own) {
    choose(yes, v.v, &own->v);
    choose(yes, v.next, &own->next);
}

template <int M>
__device__ __forceinline__ void choose(bool yes, const LocalUnit<M>& v, LocalUnit<M>* own) {
    own->block = yes ? v.block : own->block;
    own->n = yes ? v.n : own->n;
    own->seq = yes ? v.seq : own->seq;
    own->t0 = yes ? v.t0 : own->t0;
    own->b0 = yes ? v.b0 : own->b0;
    own->q = yes ? v.q : own->q;
    choose(yes, v.o, &own->o);
}

template <int M, typename Args, typename Table, typename Ints>
__device__ __forceinline__ LocalUnit<M> load_local_unit(const Args& a, const Table* new_desc, const Table* old_desc,
                                                        const Ints* tok_off, const Ints* blk_off, uint32_t u,
                                                        uint32_t row) {
    const Int4 v = new_desc[u];
    LocalUnit<M> x;
    x.block = v.x;
    x.n = v.z;
    x.seq = v.w;
    x.t0 = v.y - tok_off[v.w];
    x.b0 = blk_off[v.w];
    x.q = 0;
    if (M) {
        const int64_t t = static_cast<int64_t>(x.t0) + row;
        x.q = fast_div(static_cast<uint32_t>(t < 0 ? 0 : t), a.bo_magic, a.bo_shift);
    }
    x.o.fill([&](uint32_t m) {
        const int64_t b = static_cast<int64_t>(x.b0) + x.q + m;
        const bool in = b >= 0 && b < a.n_old_desc;
        const Int4 o = old_desc[in ? b : 0];
        return OldBlock{o.x, in && o.w == v.w ? o.z : 0};
    });
    return x;
}

// Old block and slot of a row of the unit; false when it has no source.
template <int M, typename Args>
__device__ __forceinline__ bool find_source(const Args& a, const LocalUnit<M>& x, uint32_t row, int32_t* block,
                                            uint32_t* slot) {
    // token within its sequence: the new expansion's token offset less the old one's, so device tables
    // that disagree can make it negative; such a row has no source
    const int32_t t = x.t0 + static_cast<int32_t>(row);
    if (t < 0) return false;
    uint32_t s = static_cast<uint32_t>(t) - x.q * a.old_block_size, passed = 0;
    OldBlock o;
    if constexpr (M > 0) {
        o = x.o.v;
        x.o.next.advance(a.old_block_size, &s, &passed, &o);
    }
    if (M == 0 || s >= a.old_block_size) {   // with M: only where the device tables disagree about the sequence's start
        const uint32_t q = fast_div(static_cast<uint32_t>(t), a.bo_magic, a.bo_shift);
        const int64_t ob = static_cast<int64_t>(x.b0) + q;
        if (ob < 0 || ob >= a.n_old_desc) return false;
        s = static_cast<uint32_t>(t) - q * a.old_block_size;
        const BlockDesc d = a.old_desc[ob];
        o = OldBlock{d.block, d.seq == x.seq ? d.n : 0};
    }
    *slot = s;
    *block = o.block;
    return s < static_cast<uint32_t>(o.n);
}

template <int N, int M, int V, int K>
__global__ __launch_bounds__(kMaxRunThreads) void copy_local(const LocalArgs args) {
    constexpr uint32_t W = V ? V : kVecBytes;   // as in copy_runs
    if (stale_descriptors(args.check)) return;
    const LocalItem& it = args.items[blockIdx.y];
    const uint32_t kv = blockIdx.z, w0 = wave_first(args.xcd) * K, lane = threadIdx.x & 63u, vpu = it.vpu;
    const uint32_t vpr = (it.row_bytes + W - 1) / W;
    Values<LocalUnit<M>, N> units;
    uint32_t u0 = 0;
    if constexpr (N > 0) {
        const REMP_CONSTANT Int4* nd = (const REMP_CONSTANT Int4*)(reinterpret_cast<uint64_t>(args.new_desc));
        const REMP_CONSTANT Int4* od = (const REMP_CONSTANT Int4*)(reinterpret_cast<uint64_t>(args.old_desc));
        const REMP_CONSTANT int32_t* to = (const REMP_CONSTANT int32_t*)(reinterpret_cast<uint64_t>(args.tok_off));
        const REMP_CONSTANT int32_t* bo = (const REMP_CONSTANT int32_t*)(reinterpret_cast<uint64_t>(args.old_blk_off));
        u0 = fast_div(w0, it.vpu_magic, it.vpu_shift);
        if (u0 >= args.n_new_desc) return;
        const uint32_t row = M ? fast_div(w0 - u0 * vpu, it.vpr_magic, it.vpr_shift) : 0;
        units.fill([&](uint32_t k) {
            return load_local_unit<M>(args, nd, od, to, bo, min(u0 + k, args.n_new_desc - 1), k ? 0 : row);
        });
    }
    LocalUnit<M> own[K];
    uint32_t at[K];
    bool in[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if constexpr (N == 0) {   // as in pick_unit: small units, every lane by itself
            const uint32_t w = w0 + k * 64 + lane, u = fast_div(w, it.vpu_magic, it.vpu_shift);
            in[k] = u < args.n_new_desc;
            at[k] = w - u * vpu;
            own[k] = load_local_unit<M>(args, reinterpret_cast<const Int4*>(args.new_desc),
                                        reinterpret_cast<const Int4*>(args.old_desc), args.tok_off, args.old_blk_off,
                                        min(u, args.n_new_desc - 1), fast_div(at[k], it.vpr_magic, it.vpr_shift));
        } else {
            uint32_t u = u0;
            at[k] = w0 - u0 * vpu + k * 64 + lane;
            own[k] = units.v;
            units.next.advance(vpu, &at[k], &u, &own[k]);
            in[k] = u < args.n_new_desc;
        }
    }
    Moved<V> word[K];
    uint64_t dst[K];
    uint32_t left[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        left[k] = 0;
        if (!in[k]) continue;
        const LocalUnit<M>& x = own[k];
        const uint32_t r = at[k];
        const uint32_t row = fast_div(r, it.vpr_magic, it.vpr_shift);
        if (row >= static_cast<uint32_t>(x.n)) continue;
        int32_t block;
        uint32_t slot;
        if (!find_source(args, x, row, &block, &slot)) {
            *args.flag = kFlagTables;
            continue;
        }
        const uint32_t off = (r - row * vpr) * W;
        const uint64_t src = (kv ? it.src_v : it.src_k) +
                             static_cast<uint64_t>(static_cast<uint32_t>(block)) * static_cast<uint64_t>(args.old_block_stride) +
                             static_cast<uint64_t>(slot) * args.old_row_stride + off;
        dst[k] = (kv ? it.dst_v : it.dst_k) +
                 static_cast<uint64_t>(static_cast<uint32_t>(x.block)) * static_cast<uint64_t>(args.new_block_stride) +
                 static_cast<uint64_t>(row) * args.new_row_stride + off;
        left[k] = it.row_bytes - off;
        word[k].load(src, left[k]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (left[k]) word[k].store(dst[k], left[k]);
}

// The same for aligned rows of 64 bytes and more in new blocks of less than 1 KiB: a wave of copy_local meets three blocks or
// more, whose look-ups cost more than its 1 KiB.  Here it takes 4 KiB: each lane looks up one of its rows, and the
// lanes that move a row's vectors get its two addresses from that lane.  Bound by HBM and the look-ups' latency.  Measured on
// MI355X (us, rows resolved into LDS / copy_local / so): 64-byte rows in blocks of 5 535 / 596 / 515, of 12 465 / 502 / 435, of 128
// bytes in blocks of 5 467 / 502 / 437, blocks of 16 to 6 459 / 512 / 432, 256 bytes, blocks of 16 to 1 378 / 410 / 360.  One
// wave to a workgroup instead of four 391 in the last.  Not where a wave of copy_local meets two blocks at most (256 bytes in blocks of
// 2 200 / 205, 512 bytes in blocks of 1 97 / 105), not where rows end inside lines that others go on in (64 of 128 bytes in blocks
// of 4 294 / 266 / 307, of 1 186 / 183 / 218), and not in blocks that end inside 64 bytes, or are no more (80 bytes 928 / 876 / 956, 336
// bytes 610 / 551 / 658, 64 bytes 784 / 813 / 838).
constexpr int kLookupThreads = 256, kLookupVectors = 4;
constexpr uint32_t kLookupMinRow = 64;     // so that a wave has no more rows than lanes
constexpr uint32_t kLookupMinBlock = 128;

__global__ __launch_bounds__(kMaxRunThreads) void copy_local_rows(const LocalArgs args) {
    constexpr int K = kLookupVectors;
    if (stale_descriptors(args.check)) return;
    const LocalItem& it = args.items[blockIdx.y];
    const uint32_t kv = blockIdx.z, lane = threadIdx.x & 63u, w0 = wave_first(args.xcd) * K;
    const uint32_t vpr = it.row_bytes / kVecBytes;
    // rows of all blocks are numbered one after another; the wave's first one, its last and the lane's
    const uint32_t g0 = fast_div(w0, it.vpr_magic, it.vpr_shift);
    const uint32_t end = min(fast_div(w0 + 64 * K - 1, it.vpr_magic, it.vpr_shift), args.n_new_desc * args.new_block_size - 1);
    const uint32_t g = min(g0 + lane, end);
    const uint32_t u = fast_div(g, args.bn_magic, args.bn_shift), row = g - u * args.new_block_size;
    const LocalUnit<1> x = load_local_unit<1>(args, reinterpret_cast<const Int4*>(args.new_desc),
                                              reinterpret_cast<const Int4*>(args.old_desc), args.tok_off,
                                              args.old_blk_off, u, row);
    uint64_t src = 0, dst = 0;
    if (g0 + lane <= end && row < static_cast<uint32_t>(x.n)) {
        int32_t block;
        uint32_t slot;
        if (find_source(args, x, row, &block, &slot)) {
            src = (kv ? it.src_v : it.src_k) +
                  static_cast<uint64_t>(static_cast<uint32_t>(block)) * static_cast<uint64_t>(args.old_block_stride) +
                  static_cast<uint64_t>(slot) * args.old_row_stride;
            dst = (kv ? it.dst_v : it.dst_k) +
                  static_cast<uint64_t>(static_cast<uint32_t>(x.block)) * static_cast<uint64_t>(args.new_block_stride) +
                  static_cast<uint64_t>(row) * args.new_row_stride;
        } else {
            *args.flag = kFlagTables;
        }
    }
    Vec16 val[K];
    uint64_t to[K];
    bool on[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t w = w0 + k * 64 + lane, t = fast_div(w, it.vpr_magic, it.vpr_shift);
        const uint32_t off = (w - t * vpr) * kVecBytes;
        const uint64_t from = __shfl(src, static_cast<int>(t - g0), 64);
        to[k] = __shfl(dst, static_cast<int>(t - g0), 64) + off;
        on[k] = from != 0;
        if (on[k]) val[k] = __builtin_nontemporal_load((const REMP_GLOBAL Vec16*)(from + off));
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (on[k]) __builtin_nontemporal_store(val[k], (REMP_GLOBAL Vec16*)to[k]);
}

}  // namespace remp
