// Head-tile kernels for HND and ROCm pools: copy_head_rows, copy_strips and copy_tile_groups (pack / unpack),
// copy_local_strips and copy_local_tiles (local copy between any layouts).
// Included by migrate.hip only (one translation unit holds every kernel).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kv_copy.hpp"     // kMaxLocalRows
#include "kv_device.hpp"

namespace remp {

// ---------------------------------------------------------------------------
// head-tile copies, for pools whose token rows are not contiguous
// ---------------------------------------------------------------------------
//
// Layouts other than NHD keep each (block, head) as one contiguous tile of
// block_size * head_dim elements: HND stores it token-major ([slot][dim]);
// the ROCm paged-attention cache stores K as [dim / x][slot][x] (x = the
// elements in 16 bytes) and V as [dim][slot].  The staging side is always
// token-major.

enum : int32_t { kLayoutNHD = 0, kLayoutHND = 1, kLayoutRocmSplit = 2 };
constexpr int kTileThreads = 256;
constexpr int kTileLdsBytes = 32 * 1024;   // dynamic LDS per workgroup, at most
constexpr int64_t kTileWgBytes = 16 * 1024; // payload bytes a tile workgroup aims to move
constexpr int kStripLanes = 256;           // lanes of a strip (copy_strips), where the columns can be split so
constexpr int kMaxStripThreads = 1024;     // and at most: one column of the largest block

// Slices of one layer that hold 2-4 KiB of each block are copied side by side, block by block: one after another,
// each pass writes (or reads) every other 2 KiB of the pool, which the memory takes slower (MI355X, 70B
// GQA fp8, two sources' 2 KiB head tiles, pack and unpack, us one after another / side by side: HND 2100 / 1968, ROCm 2114 / 2022;
// 3 KiB ROCm 1222 / 1199; over less memory, 2 to 3.5 KiB, 0-1% either way).  Larger pieces are
// no faster so (two of 4 KiB: 1926 / 1943), and pieces of 1.25 KiB lose 2-6%.
constexpr uint64_t kPeerMinBytes = 2048, kPeerEndBytes = 4096;

struct TileItem {
    uint64_t paged_k, paged_v;   // the slice's first head tile of the layer's block 0
    uint64_t stage;              // first byte of the slice in its staging buffer (K part)
    uint32_t row_bytes;          // a staging row
    uint32_t heads;              // heads in the slice, or in the part of it that this item is
    uint32_t strips;             // strips per block (copy_strips)
    uint32_t last;               // columns of a block's last strip (copy_strips)
    uint32_t unit;               // vectors per unit (copy_head_rows)
    uint32_t strips_magic, unit_magic, last_magic, heads_magic, row_magic;   // division by strips, unit, last,
    uint16_t strips_shift, unit_shift, last_shift, heads_shift, row_shift;   // heads, vectors of a staging row
};

struct TileArgs {
    const BlockDesc* desc;
    int64_t block_stride;        // paged bytes per block
    int64_t total_tokens;
    uint32_t n_desc;
    uint32_t block_size;
    uint32_t head_bytes;         // head_dim * elem_bytes
    uint32_t strip;              // columns (16 bytes of a staging row) per strip
    uint32_t peers;              // slices of one layer: items y * peers .. are copied side by side
    uint32_t run;                // workgroups of one of them in a row
    uint32_t strip_magic, head_magic, bs_magic, vd_magic;   // division by strip, the vectors of a head row,
    uint16_t strip_shift, head_shift, bs_shift, vd_shift;   // block_size, the vectors of a V dim,
    uint32_t run_magic, peers_magic;                        // run, peers
    uint16_t run_shift, peers_shift;
    StampCheck check;
    TileItem items[kMaxItems];
};
static_assert(sizeof(TileArgs) < 4096, "tile kernel arguments must stay below 4 KiB");

__device__ __forceinline__ BlockDesc load_desc_scalar(const BlockDesc* desc, uint32_t i) {
    const Int4 v = ((const REMP_CONSTANT Int4*)(reinterpret_cast<uint64_t>(desc)))[i];
    return BlockDesc{v.x, v.y, v.z, v.w};
}

// The item of a workgroup and its position among that item's workgroups.
__device__ __forceinline__ const TileItem& tile_item(const TileArgs& a, uint32_t* pos) {
    const uint32_t wg = xcd_position(blockIdx.x);
    const uint32_t q = fast_div(wg, a.run_magic, a.run_shift);
    const uint32_t g = fast_div(q, a.peers_magic, a.peers_shift);
    *pos = g * a.run + (wg - q * a.run);
    return a.items[blockIdx.y * a.peers + (q - g * a.peers)];
}

// pick_unit for units that are one of `heads` tiles of a live block: also the tile's number j in its block.
template <int N>
__device__ __forceinline__ bool pick_tile(const BlockDesc* desc, uint32_t n_desc, uint32_t w0, uint32_t lane,
                                          const TileItem& it, uint32_t heads, BlockDesc* d, uint32_t* r, uint32_t* j) {
    const uint32_t u0 = fast_div(N == 0 ? w0 + lane : w0, it.unit_magic, it.unit_shift);
    const uint32_t i0 = heads == 1 ? u0 : fast_div(u0, it.heads_magic, it.heads_shift);
    if (i0 >= n_desc) return false;
    *r = w0 + lane - u0 * it.unit;
    *j = u0 - i0 * heads;
    if (N == 0) {
        *d = desc[i0];
        return true;
    }
    *d = load_desc_scalar(desc, i0);
    uint32_t i = i0, jn = *j;
    bool ok = true;
#pragma unroll
    for (int k = 1; k < N; ++k) {
        if (++jn == heads) {
            jn = 0;
            ++i;
        }
        const BlockDesc next = load_desc_scalar(desc, min(i, n_desc - 1));
        if (*r >= it.unit) {
            *r -= it.unit;
            *j = jn;
            *d = next;
            ok = i < n_desc;
        }
    }
    return ok;
}

// Move the elements of one 16-byte vector (consecutive slots of one dim) to or
// from LDS rows `lrow` bytes apart.
template <typename E>
__device__ __forceinline__ void scatter_t(const unsigned int __attribute__((ext_vector_type(4))) & val,
                                          unsigned char* p, uint32_t lrow) {
    const E* e = reinterpret_cast<const E*>(&val);
#pragma unroll
    for (int k = 0; k < 16 / static_cast<int>(sizeof(E)); ++k) *reinterpret_cast<E*>(p + k * lrow) = e[k];
}

template <typename E>
__device__ __forceinline__ unsigned int __attribute__((ext_vector_type(4))) gather_t(const unsigned char* p,
                                                                                      uint32_t lrow) {
    unsigned int __attribute__((ext_vector_type(4))) val;
    E* e = reinterpret_cast<E*>(&val);
#pragma unroll
    for (int k = 0; k < 16 / static_cast<int>(sizeof(E)); ++k) e[k] = *reinterpret_cast<const E*>(p + k * lrow);
    return val;
}

template <int EB>
__device__ __forceinline__ void scatter_dim(const Vec16& val, unsigned char* p, uint32_t lrow) {
    if (EB == 2) scatter_t<unsigned short>(val, p, lrow);
    else if (EB == 4) scatter_t<unsigned int>(val, p, lrow);
    else scatter_t<unsigned char>(val, p, lrow);
}

template <int EB>
__device__ __forceinline__ Vec16 gather_dim(const unsigned char* p, uint32_t lrow) {
    if (EB == 2) return gather_t<unsigned short>(p, lrow);
    if (EB == 4) return gather_t<unsigned int>(p, lrow);
    return gather_t<unsigned char>(p, lrow);
}

__device__ __forceinline__ void scatter_dim(const unsigned int __attribute__((ext_vector_type(4))) & val,
                                            unsigned char* p, uint32_t lrow, int32_t eb) {
    if (eb == 2) scatter_t<unsigned short>(val, p, lrow);
    else if (eb == 4) scatter_t<unsigned int>(val, p, lrow);
    else scatter_t<unsigned char>(val, p, lrow);
}

__device__ __forceinline__ unsigned int __attribute__((ext_vector_type(4))) gather_dim(const unsigned char* p,
                                                                                        uint32_t lrow, int32_t eb) {
    if (eb == 2) return gather_t<unsigned short>(p, lrow);
    if (eb == 4) return gather_t<unsigned int>(p, lrow);
    return gather_t<unsigned char>(p, lrow);
}

// Store the first `nbytes` bytes of a vector (whole elements of eb bytes) at a 16-byte aligned dst.
// The vector stays in registers: whole words first, then the elements of the last partial word.  Taking
// the vector's address instead (store_prefix_bytes) puts it in scratch memory on every pass of the
// caller's loop, also for whole vectors; in the head-tile unpack that cost 3-9% (MI355X, same process,
// ROCm pools: 7B MHA unpack +9.1% with this form, 70B GQA +3.0%, 13B MHA +3.2%).
__device__ __forceinline__ void store_prefix(const unsigned int __attribute__((ext_vector_type(4))) & val,
                                             void* dst, int32_t nbytes, int32_t eb) {
    unsigned int* o = reinterpret_cast<unsigned int*>(dst);
    const int32_t nw = nbytes >> 2;   // whole 4-byte words
    if (nw > 0) o[0] = val.x;
    if (nw > 1) o[1] = val.y;
    if (nw > 2) o[2] = val.z;
    if (nw > 3) o[3] = val.w;
    const int32_t rest = nbytes & 3;   // 2 (eb 2) or 1-3 (eb 1); eb 4 leaves none
    if (rest == 0) return;
    const unsigned int w = nw == 0 ? val.x : nw == 1 ? val.y : nw == 2 ? val.z : val.w;
    unsigned char* ob = reinterpret_cast<unsigned char*>(o + nw);
    if (eb == 2) {
        *reinterpret_cast<unsigned short*>(ob) = static_cast<unsigned short>(w);
    } else {
        ob[0] = static_cast<unsigned char>(w);
        if (rest > 1) ob[1] = static_cast<unsigned char>(w >> 8);
        if (rest > 2) ob[2] = static_cast<unsigned char>(w >> 16);
    }
}

// The same through the vector's bytes in memory.  The local head-tile copy keeps this form: with the
// register form its ROCm-pool local copies ran 1-3% slower (MI355X, same process, 13B MHA and 70B GQA
// shares), although both forms store the same bytes.
__device__ __forceinline__ void store_prefix_bytes(const unsigned int __attribute__((ext_vector_type(4))) & val,
                                                   void* dst, int32_t nbytes, int32_t eb) {
    const unsigned char* b = reinterpret_cast<const unsigned char*>(&val);
    unsigned char* o = reinterpret_cast<unsigned char*>(dst);
    if (eb == 4) {
        for (int q = 0; q < nbytes; q += 4)
            *reinterpret_cast<unsigned int*>(o + q) = *reinterpret_cast<const unsigned int*>(b + q);
    } else if (eb == 2) {
        for (int q = 0; q < nbytes; q += 2)
            *reinterpret_cast<unsigned short*>(o + q) = *reinterpret_cast<const unsigned short*>(b + q);
    } else {
        for (int q = 0; q < nbytes; ++q) o[q] = b[q];
    }
}

// HND tiles: a head's rows lie one after another in token order in the pool, so every 16-byte vector of a
// tile has one vector of a staging row, and no LDS is needed.  Grid as copy_runs; the vectors are numbered
// in the destination's order, so that every store is part of a contiguous run: a pack takes block after block
// in staging order (slot, head, dim), an unpack tile after tile in the pool's (block, head, slot, dim).  Bound by HBM.
// Measured on MI355X against tiles staged in LDS, 16 KiB to 256 lanes: 70B GQA unpack 5.85 -> 6.2 TB/s, 7B MHA pack
// and unpack 5.88 -> 6.05, 160-byte heads in blocks of 12 and 20 5.1 -> 5.5.
template <bool PACK, int N>
__global__ __launch_bounds__(kRunThreads) void copy_head_rows(const TileArgs a) {
    if (stale_descriptors(a.check)) return;
    uint32_t pos;
    const TileItem& it = tile_item(a, &pos);
    const uint32_t kv = blockIdx.z, hb = a.head_bytes, heads = PACK ? 1 : it.heads;
    BlockDesc d;
    uint32_t r, j, row, c;
    if (!pick_tile<N>(a.desc, a.n_desc, pos * kRunThreads, threadIdx.x & 63u, it, heads, &d, &r, &j)) return;
    if (PACK) {
        row = fast_div(r, it.row_magic, it.row_shift);
        c = r - row * it.heads * (hb / kVecBytes);
        j = fast_div(c, a.head_magic, a.head_shift);
        c -= j * (hb / kVecBytes);
    } else {
        row = fast_div(r, a.head_magic, a.head_shift);
        c = r - row * (hb / kVecBytes);
    }
    if (row >= static_cast<uint32_t>(d.n)) return;
    const uint64_t paged = (kv ? it.paged_v : it.paged_k) +
                           static_cast<uint64_t>(static_cast<uint32_t>(d.block)) * static_cast<uint64_t>(a.block_stride) +
                           static_cast<uint64_t>(j * a.block_size + row) * hb;
    const uint64_t stage =
        it.stage + (static_cast<uint64_t>(kv) * a.total_tokens + static_cast<uint32_t>(d.tok) + row) * it.row_bytes +
        static_cast<uint64_t>(j) * hb;
    move_vector<false>(PACK ? paged : stage, PACK ? stage : paged, c * kVecBytes, hb);
}

// ROCm tiles.  A slice's staging row is a run of 16-byte columns; in the pool, where head tiles follow one
// another, column x of a block is the 16 * block_size bytes at x * 16 * block_size whatever head it is of
// (K: that column of every slot; V: its dims, each with every slot).  So a workgroup takes a strip of columns for all
// slots of a block, one vector per lane: contiguous in the pool, runs of strip * 16 bytes in staging.  The
// lanes load in the source's order, exchange through LDS (token-major rows, padded by 16 bytes against bank
// conflicts) and store in the destination's.  Bound by HBM.  Measured on MI355X against 256 lanes that took 16 KiB
// of tiles in turn (copy_tile_groups): 70B GQA fp8 pack 5.7 -> 6.1 TB/s, unpack 4.8 -> 5.95; 32 heads of 160
// bytes, 32-token blocks, pack 4.2 -> 6.1, unpack 4.7 -> 5.75; 7B MHA bf16 5.84 -> 5.88 for both.
template <bool PACK, int EB>
__global__ __launch_bounds__(kMaxStripThreads) void copy_strips(const TileArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr uint32_t M = kVecBytes / EB;   // elements per vector
    if (stale_descriptors(a.check)) return;
    const uint32_t v = threadIdx.x;
    uint32_t u;
    const TileItem& it = tile_item(a, &u);
    const uint32_t kv = blockIdx.z, bs = a.block_size;
    const uint32_t i = fast_div(u, it.strips_magic, it.strips_shift), s = u - i * it.strips;
    if (i >= a.n_desc) return;
    const BlockDesc d = load_desc_scalar(a.desc, i);
    const uint32_t n = static_cast<uint32_t>(d.n);
    const bool tail = s == it.strips - 1;
    const uint32_t cols = tail ? it.last : a.strip, c0 = s * a.strip;
    const uint32_t lrow = (a.strip + 1) * kVecBytes;
    // in staging: column `col` of row `row`
    const uint32_t row = fast_div(v, tail ? it.last_magic : a.strip_magic, tail ? it.last_shift : a.strip_shift);
    const uint32_t col = v - row * cols;
    const uint64_t stage =
        it.stage + (static_cast<uint64_t>(kv) * a.total_tokens + static_cast<uint32_t>(d.tok) + row) * it.row_bytes +
        (c0 + col) * kVecBytes;
    // in the pool: the strip's v-th vector, K: column x of slot y, V: slots y.. of dim x
    const uint64_t paged = (kv ? it.paged_v : it.paged_k) +
                           static_cast<uint64_t>(static_cast<uint32_t>(d.block)) * static_cast<uint64_t>(a.block_stride) +
                           (static_cast<uint64_t>(c0) * bs + v) * kVecBytes;
    uint32_t x, y;
    if (kv == 0) {
        x = fast_div(v, a.bs_magic, a.bs_shift);
        y = v - x * bs;
    } else {
        x = fast_div(v, a.vd_magic, a.vd_shift);
        y = (v - x * (bs / M)) * M;
    }
    const bool in_pool = x < (kv ? cols * M : cols) && y < n, in_stage = row < n;
    unsigned char* cell = lds + y * lrow + x * (kv ? EB : kVecBytes);
    unsigned char* line = lds + row * lrow + col * kVecBytes;
    if (PACK) {
        if (in_pool) {
            const Vec16 val = __builtin_nontemporal_load((const REMP_GLOBAL Vec16*)paged);
            if (kv == 0) *reinterpret_cast<Vec16*>(cell) = val;
            else scatter_dim<EB>(val, cell, lrow);
        }
        __syncthreads();
        if (in_stage) __builtin_nontemporal_store(*reinterpret_cast<const Vec16*>(line), (REMP_GLOBAL Vec16*)stage);
    } else {
        if (in_stage) *reinterpret_cast<Vec16*>(line) = __builtin_nontemporal_load((const REMP_GLOBAL Vec16*)stage);
        __syncthreads();
        if (!in_pool) return;
        if (kv == 0) {
            __builtin_nontemporal_store(*reinterpret_cast<const Vec16*>(cell), (REMP_GLOBAL Vec16*)paged);
            return;
        }
        const Vec16 val = gather_dim<EB>(cell, lrow);
        if (y + M <= n) __builtin_nontemporal_store(val, (REMP_GLOBAL Vec16*)paged);
        else store_prefix(val, reinterpret_cast<void*>(paged), static_cast<int32_t>((n - y) * EB), EB);   // only the live slots
    }
}

// ROCm tiles whose strip would be a whole row of a few columns that leaves many lanes of its waves idle
// (strips_fill): a workgroup of 256 lanes takes several (block, K or V, head) tiles, 16 KiB, vector
// after vector, through LDS.  Measured on MI355X, one fp8 head a rank, blocks of 16 (us by strips / so, pack and unpack): of the
// strip's lanes 62% busy 448 / 421 and 238 / 208, 75% 396 / 414 and 221 / 218 (of 192 lanes 403 / 403 and 217 / 204), 81% 365 / 375 and
// 196 / 197, 83% 380 / 385 and 206 / 202, 87% 362 / 417 and 200 / 212, 92% 367 / 395 and 198 / 204, 94% 356 / 395 and 189 / 196.
struct GroupItem {
    uint64_t paged_k, paged_v, stage;   // as TileItem
    uint32_t row_bytes;
};

struct GroupArgs {
    const BlockDesc* desc;
    int64_t block_stride;      // paged bytes per block
    int64_t total_tokens;
    int32_t n_desc;
    int32_t tiles_per_wg;
    int32_t block_size;
    int32_t head_bytes;        // head_dim * elem_bytes
    int32_t elem_bytes;
    int32_t lds_row;           // head_bytes + 16
    uint32_t vpt_magic, vpt_shift;   // division by vectors per tile
    uint32_t vph_magic, vph_shift;   // division by vectors per head row
    uint32_t bs_magic, bs_shift;     // division by block_size
    StampCheck check;
    GroupItem items[kMaxItems];       // paged_k/v: the slice's first head tile of the layer's block 0
};
static_assert(sizeof(GroupArgs) < 4096, "tile-group kernel arguments must stay below 4 KiB");


template <bool PACK>
__global__ __launch_bounds__(kTileThreads) void copy_tile_groups(const GroupArgs args) {
    typedef unsigned int V4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ uint64_t s_paged[kMaxUnitsPerWg];
    __shared__ uint64_t s_stage[kMaxUnitsPerWg];
    __shared__ int32_t s_n[kMaxUnitsPerWg];
    __shared__ int32_t s_kv[kMaxUnitsPerWg];

    const bool stale = stamps_differ(args.check);   // acted on after the descriptor prologue
    const GroupItem& it = args.items[blockIdx.y];
    const int32_t hc = static_cast<int32_t>(it.row_bytes) / args.head_bytes;   // heads in the slice
    const int64_t ntiles = static_cast<int64_t>(args.n_desc) * 2 * hc;
    const int64_t g0 = static_cast<int64_t>(blockIdx.x) * args.tiles_per_wg;
    if (g0 >= ntiles) return;
    const int32_t nt = static_cast<int32_t>(min(static_cast<int64_t>(args.tiles_per_wg), ntiles - g0));
    const int tid = threadIdx.x;
    const int32_t bs = args.block_size, hb = args.head_bytes;
    const uint64_t tile_bytes = static_cast<uint64_t>(bs) * hb;
    const uint64_t kv_stride = static_cast<uint64_t>(args.total_tokens) * it.row_bytes;

    for (int i = tid; i < nt; i += kTileThreads) {
        const int64_t g = g0 + i;
        const int64_t d = g / (2 * hc);
        const int32_t r = static_cast<int32_t>(g - d * 2 * hc);
        const int32_t kv = r / hc, j = r - (r / hc) * hc;
        const BlockDesc bd = args.desc[d];
        s_paged[i] = (kv ? it.paged_v : it.paged_k) + static_cast<uint64_t>(bd.block) * args.block_stride +
                     static_cast<uint64_t>(j) * tile_bytes;
        s_stage[i] = it.stage + kv * kv_stride + static_cast<uint64_t>(bd.tok) * it.row_bytes +
                     static_cast<uint64_t>(j) * hb;
        s_n[i] = bd.n;
        s_kv[i] = kv;
    }
    __syncthreads();
    if (stale) {
        report_stale(args.check);
        return;
    }

    const uint32_t vpt = static_cast<uint32_t>(tile_bytes / 16);     // 16-byte vectors per tile
    const uint32_t vph = static_cast<uint32_t>(hb / 16);             // 16-byte vectors per head row
    const uint32_t total = static_cast<uint32_t>(nt) * vpt;
    const uint32_t lrow = static_cast<uint32_t>(args.lds_row);
    const int32_t m = 16 / args.elem_bytes;                          // elements per vector
    const uint32_t tile_lds = static_cast<uint32_t>(bs) * lrow;

    // phase 1: fill LDS (token-major)
    for (uint32_t x = tid; x < total; x += kTileThreads) {
        const uint32_t i = fast_div(x, args.vpt_magic, args.vpt_shift);
        const uint32_t v = x - i * vpt;
        unsigned char* tl = lds + i * tile_lds;
        if (PACK) {
            const V4* src = reinterpret_cast<const V4*>(s_paged[i] + uint64_t(v) * 16);
            if (s_kv[i] == 0) {                                    // [dim / x][slot][x]
                const uint32_t c = fast_div(v, args.bs_magic, args.bs_shift);
                const uint32_t srow = v - c * bs;
                if (static_cast<int32_t>(srow) < s_n[i])
                    *reinterpret_cast<V4*>(tl + srow * lrow + c * 16) = __builtin_nontemporal_load(src);
            } else {                                                      // [dim][slot]
                const uint32_t e0 = v * m;
                const uint32_t dim = fast_div(e0, args.bs_magic, args.bs_shift);
                const uint32_t s0 = e0 - dim * bs;
                if (static_cast<int32_t>(s0) < s_n[i])
                    scatter_dim(__builtin_nontemporal_load(src), tl + s0 * lrow + dim * args.elem_bytes, lrow,
                                args.elem_bytes);
            }
        } else {
            const uint32_t srow = fast_div(v, args.vph_magic, args.vph_shift);
            const uint32_t cb = v - srow * vph;
            if (static_cast<int32_t>(srow) < s_n[i]) {
                const V4 val = __builtin_nontemporal_load(
                    reinterpret_cast<const V4*>(s_stage[i] + uint64_t(srow) * it.row_bytes + cb * 16));
                *reinterpret_cast<V4*>(tl + srow * lrow + cb * 16) = val;
            }
        }
    }
    __syncthreads();

    // phase 2: drain LDS
    for (uint32_t x = tid; x < total; x += kTileThreads) {
        const uint32_t i = fast_div(x, args.vpt_magic, args.vpt_shift);
        const uint32_t v = x - i * vpt;
        const unsigned char* tl = lds + i * tile_lds;
        if (PACK) {
            const uint32_t srow = fast_div(v, args.vph_magic, args.vph_shift);
            const uint32_t cb = v - srow * vph;
            if (static_cast<int32_t>(srow) < s_n[i])
                __builtin_nontemporal_store(*reinterpret_cast<const V4*>(tl + srow * lrow + cb * 16),
                                            reinterpret_cast<V4*>(s_stage[i] + uint64_t(srow) * it.row_bytes + cb * 16));
        } else {
            V4* dst = reinterpret_cast<V4*>(s_paged[i] + uint64_t(v) * 16);
            if (s_kv[i] == 0) {
                const uint32_t c = fast_div(v, args.bs_magic, args.bs_shift);
                const uint32_t srow = v - c * bs;
                if (static_cast<int32_t>(srow) < s_n[i])
                    __builtin_nontemporal_store(*reinterpret_cast<const V4*>(tl + srow * lrow + c * 16), dst);
            } else {
                const uint32_t e0 = v * m;
                const uint32_t dim = fast_div(e0, args.bs_magic, args.bs_shift);
                const uint32_t s0 = e0 - dim * bs;
                const int32_t live = min(m, s_n[i] - static_cast<int32_t>(s0));
                if (live <= 0) continue;
                const V4 val = gather_dim(tl + s0 * lrow + dim * args.elem_bytes, lrow, args.elem_bytes);
                if (live == m) {
                    __builtin_nontemporal_store(val, dst);
                } else {                                                  // only the live slots
                    store_prefix(val, dst, live * args.elem_bytes, args.elem_bytes);
                }
            }
        }
    }
}


// Leading slots that have a source among the m (4, 8 or 16) consecutive one-byte flags at p (1: the
// row has a source), p aligned to m bytes: a ROCm V vector's slots in one or two LDS reads instead of
// one per slot.
__device__ __forceinline__ int32_t leading_sources(const uint8_t* p, int32_t m) {
    if (m == 4) {
        const uint32_t z = ~*reinterpret_cast<const uint32_t*>(p) & 0x01010101u;
        return z ? static_cast<int32_t>(__builtin_ctz(z) >> 3) : 4;
    }
    const uint64_t z0 = ~*reinterpret_cast<const uint64_t*>(p) & 0x0101010101010101ull;
    if (z0 || m == 8) return z0 ? static_cast<int32_t>(__builtin_ctzll(z0) >> 3) : 8;
    const uint64_t z1 = ~*reinterpret_cast<const uint64_t*>(p + 8) & 0x0101010101010101ull;
    return z1 ? 8 + static_cast<int32_t>(__builtin_ctzll(z1) >> 3) : 16;
}

// ---------------------------------------------------------------------------
// local copy between pools of any layouts (not both NHD), one head tile at a time
// ---------------------------------------------------------------------------
//
// A unit is one (new block, K or V, head of the slice) tile.  The prologue
// resolves each of its rows to the old (block, slot) through the old
// descriptors.  When both pools have the same layout, every 16-byte vector of
// a new tile has one 16-byte source vector in an old tile and is copied
// directly.  Otherwise the tile goes through LDS: phase 1 reads every live
// row's head vectors from the old pool in its layout into LDS (token-major;
// ROCm V tiles, where a token's elements of one head lie block_size elements
// apart, as vectors of m rows of one dim, stored element by element); phase 2
// writes the tile into the new pool in its layout, live slots only.

constexpr int kMaxLocalTileItems = 8;

// Dynamic LDS of copy_local_tiles: `tiles` head tiles of bn rows of lds_row bytes, then per row an
// 8-byte source base, a 4-byte slot and a 1-byte flag, then a 1-byte flag per tile.
inline int64_t local_tile_lds_bytes(int64_t tiles, int64_t bn, int64_t lds_row) {
    return tiles * bn * lds_row + tiles * bn * 13 + tiles;
}

struct LocalTileItem {
    uint64_t src_k, src_v;   // old storage of the layer at the slice's first head (block 0)
    uint64_t dst_k, dst_v;   // new storage of the layer at the slice's first head (block 0)
    int32_t heads;           // heads in the slice
    int32_t pad;
};

struct LocalTileArgs {
    const BlockDesc* new_desc;
    const BlockDesc* old_desc;
    const int32_t* tok_off;       // first token of each sequence on the token axis
    const int32_t* old_blk_off;   // first old descriptor of each sequence
    int32_t* flag;
    int64_t old_block_stride, new_block_stride;   // bytes per block (all local heads)
    int32_t n_new_desc, n_old_desc;
    int32_t tiles_per_wg;
    int32_t old_block_size, new_block_size;
    int32_t head_bytes, elem_bytes;
    int32_t old_layout, new_layout;
    int32_t old_row_stride, new_row_stride;       // NHD: bytes per token row of all local heads
    int32_t old_head_step, new_head_step;         // bytes from one head's data to the next at block 0
    int32_t lds_row;                              // head_bytes + 16
    uint32_t vph_magic, vph_shift;                // division by vectors per head row
    uint32_t rows_magic, rows_shift;              // division by new_block_size * vectors per head row
    uint32_t bn_magic, bn_shift;                  // division by the new block size
    StampCheck check;
    LocalTileItem items[kMaxLocalTileItems];
};
static_assert(sizeof(LocalTileArgs) < 4096, "local tile kernel arguments must stay below 4 KiB");

__global__ __launch_bounds__(kTileThreads) void copy_local_tiles(const LocalTileArgs a) {
    typedef unsigned int V4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ uint64_t s_dst[kMaxUnitsPerWg];
    __shared__ int32_t s_n[kMaxUnitsPerWg];
    __shared__ int32_t s_kv[kMaxUnitsPerWg];

    if (stale_descriptors(a.check)) return;
    const LocalTileItem& it = a.items[blockIdx.y];
    const int32_t hc = it.heads;
    const int64_t ntiles = static_cast<int64_t>(a.n_new_desc) * 2 * hc;
    const int64_t g0 = static_cast<int64_t>(blockIdx.x) * a.tiles_per_wg;
    if (g0 >= ntiles) return;
    const int32_t nt = static_cast<int32_t>(min(static_cast<int64_t>(a.tiles_per_wg), ntiles - g0));
    const int tid = threadIdx.x;
    const int32_t bn = a.new_block_size, bo = a.old_block_size, hb = a.head_bytes, eb = a.elem_bytes;
    // per-(unit, row) arrays behind the tiles in the dynamic LDS, sized by the launch for tiles_per_wg
    // units (local_tile_lds_bytes), so that the workgroup holds only what its units need
    const uint32_t rows_cap = static_cast<uint32_t>(a.tiles_per_wg) * bn;
    unsigned char* rows_lds = lds + static_cast<uint32_t>(a.tiles_per_wg) * bn * static_cast<uint32_t>(a.lds_row);
    uint64_t* s_src = reinterpret_cast<uint64_t*>(rows_lds);               // old tile base of each row, 0: none
    int32_t* s_slot = reinterpret_cast<int32_t*>(rows_lds + rows_cap * 8);  // its old slot
    uint8_t* s_has = reinterpret_cast<uint8_t*>(rows_lds + rows_cap * 12);  // 1: the row has a source
    uint8_t* s_full = s_has + rows_cap;       // per tile, 1: every row live and with a source

    for (int i = tid; i < nt; i += kTileThreads) {
        const int64_t g = g0 + i;
        const int64_t d = g / (2 * hc);
        const int32_t r = static_cast<int32_t>(g - d * 2 * hc);
        const int32_t kv = r / hc, j = r - (r / hc) * hc;
        const BlockDesc nd = a.new_desc[d];
        s_dst[i] = (kv ? it.dst_v : it.dst_k) + static_cast<uint64_t>(nd.block) * a.new_block_stride +
                   static_cast<uint64_t>(j) * a.new_head_step;
        s_n[i] = nd.n;
        s_kv[i] = kv;
        s_full[i] = nd.n == bn;
    }
    __syncthreads();
    for (int x = tid; x < nt * bn; x += kTileThreads) {
        const int32_t i = x / bn, r = x - (x / bn) * bn;
        const int64_t g = g0 + i;
        const int64_t d = g / (2 * hc);
        const int32_t rr = static_cast<int32_t>(g - d * 2 * hc);
        const int32_t kv = rr / hc, j = rr - (rr / hc) * hc;
        const BlockDesc nd = a.new_desc[d];
        uint64_t base = 0;
        int32_t slot = 0;
        if (r < nd.n) {
            // token within its sequence (negative when the device tables disagree: no source)
            const int32_t t = nd.tok - a.tok_off[nd.seq] + r;
            const int32_t ob = a.old_blk_off[nd.seq] + t / bo;
            slot = t - (t / bo) * bo;
            bool ok = t >= 0 && ob >= 0 && ob < a.n_old_desc;
            BlockDesc od{0, 0, 0, 0};
            if (ok) {
                od = a.old_desc[ob];
                ok = od.seq == nd.seq && slot < od.n;
            }
            if (ok)
                base = (kv ? it.src_v : it.src_k) + static_cast<uint64_t>(od.block) * a.old_block_stride +
                       static_cast<uint64_t>(j) * a.old_head_step;
            else
                *a.flag = kFlagTables;
        }
        s_src[x] = base;
        s_slot[x] = slot;
        s_has[x] = base != 0;
        if (base == 0) s_full[i] = 0;
    }
    __syncthreads();

    const uint32_t vph = static_cast<uint32_t>(hb / 16);
    const uint32_t per_tile = static_cast<uint32_t>(bn) * vph;
    const uint32_t total = static_cast<uint32_t>(nt) * per_tile;
    const uint32_t lrow = static_cast<uint32_t>(a.lds_row);
    const uint32_t tile_lds = static_cast<uint32_t>(bn) * lrow;
    const int32_t m = 16 / eb;                                      // elements per vector

    if (a.old_layout == a.new_layout && bo == bn) {
        // Same tile layout and block size: a new block holds the same tokens at the same slots as one
        // old block (blocks start at sequence starts), so each tile is copied vector for vector in
        // its own order, live slots only, without LDS.
        for (uint32_t x = tid; x < total; x += kTileThreads) {
            const uint32_t i = fast_div(x, a.rows_magic, a.rows_shift);
            const uint32_t v = x - i * per_tile;
            const int32_t n = s_n[i];
            const uint64_t src0 = s_src[i * bn];
            if (src0 == 0) continue;
            const V4* src = reinterpret_cast<const V4*>(src0 + uint64_t(v) * 16);
            V4* dst = reinterpret_cast<V4*>(s_dst[i] + uint64_t(v) * 16);
            if (s_full[i]) {                                            // every vector of the tile is live
                __builtin_nontemporal_store(__builtin_nontemporal_load(src), dst);
            } else if (a.new_layout == kLayoutHND || s_kv[i] == 0) {
                uint32_t r;
                if (a.new_layout == kLayoutHND) {
                    r = fast_div(v, a.vph_magic, a.vph_shift);
                } else {                                                 // [dim / x][slot][x]
                    const uint32_t c = fast_div(v, a.bn_magic, a.bn_shift);
                    r = v - c * bn;
                }
                if (static_cast<int32_t>(r) < n && s_src[i * bn + r] != 0)
                    __builtin_nontemporal_store(__builtin_nontemporal_load(src), dst);
            } else {                                                     // [dim][slot]
                const uint32_t e0 = v * m;
                const uint32_t dim = fast_div(e0, a.bn_magic, a.bn_shift);
                const uint32_t s0 = e0 - dim * bn;
                const int32_t live = min(min(m, n - static_cast<int32_t>(s0)), leading_sources(s_has + i * bn + s0, m));
                if (live <= 0) continue;
                const V4 val = __builtin_nontemporal_load(src);
                if (live == m) __builtin_nontemporal_store(val, dst);
                else store_prefix_bytes(val, dst, live * eb, eb);
            }
        }
        return;
    }

    if (a.old_layout == a.new_layout) {
        // Same tile layout, block sizes that differ: token t of a sequence sits at row t mod bn of its new
        // block and at slot t mod bo of its old one, and both sizes are multiples of m (16 bytes of
        // elements), so a 16-byte vector of a new tile, part of one row (HND, ROCm K) or m rows of one dim
        // starting at a multiple of m (ROCm V), has one 16-byte source vector in an old tile: each is
        // copied directly, without LDS.  A V vector is read at its first row's source; one whose slot is
        // not a multiple of m (only when the device tables disagree with the host's) is not copied.
        for (uint32_t x = tid; x < total; x += kTileThreads) {
            const uint32_t i = fast_div(x, a.rows_magic, a.rows_shift);
            const uint32_t v = x - i * per_tile;
            const int32_t n = s_n[i];
            V4* dst = reinterpret_cast<V4*>(s_dst[i] + uint64_t(v) * 16);
            if (a.new_layout == kLayoutHND || s_kv[i] == 0) {
                uint32_t r;
                uint64_t off;                                            // within the old tile, but the slot
                uint32_t slot_bytes;
                if (a.new_layout == kLayoutHND) {                        // [slot][dim]
                    r = fast_div(v, a.vph_magic, a.vph_shift);
                    off = uint64_t(v - r * vph) * 16;
                    slot_bytes = static_cast<uint32_t>(hb);
                } else {                                                 // [dim / x][slot][x]
                    const uint32_t c = fast_div(v, a.bn_magic, a.bn_shift);
                    r = v - c * bn;
                    off = uint64_t(c) * bo * 16;
                    slot_bytes = 16;
                }
                if (static_cast<int32_t>(r) >= n || !s_has[i * bn + r]) continue;
                const uint64_t src = s_src[i * bn + r] + off + uint64_t(s_slot[i * bn + r]) * slot_bytes;
                __builtin_nontemporal_store(__builtin_nontemporal_load(reinterpret_cast<const V4*>(src)), dst);
            } else {                                                     // [dim][slot]
                const uint32_t e0 = v * m;
                const uint32_t dim = fast_div(e0, a.bn_magic, a.bn_shift);
                const uint32_t s0 = e0 - dim * bn;
                const int32_t live = min(min(m, n - static_cast<int32_t>(s0)), leading_sources(s_has + i * bn + s0, m));
                if (live <= 0) continue;
                const uint32_t slot = static_cast<uint32_t>(s_slot[i * bn + s0]);
                if (slot & static_cast<uint32_t>(m - 1)) continue;
                const V4 val = __builtin_nontemporal_load(reinterpret_cast<const V4*>(
                    s_src[i * bn + s0] + uint64_t(dim) * bo * eb + uint64_t(slot) * eb));
                if (live == m) __builtin_nontemporal_store(val, dst);
                else store_prefix_bytes(val, dst, live * eb, eb);
            }
        }
        return;
    }

    // phase 1: live rows of every tile from the old pool into LDS, token-major
    for (uint32_t x = tid; x < total; x += kTileThreads) {
        const uint32_t i = fast_div(x, a.rows_magic, a.rows_shift);
        const uint32_t rem = x - i * per_tile;
        if (a.old_layout == kLayoutRocmSplit && s_kv[i] == 1) {
            // [dim][slot] V tiles: vector rem holds m rows s0.. of one dim, whose old slots run on from a
            // multiple of m in one old block (as in the same-layout copy), so it is read as one 16-byte vector
            // at its first row's source and stored to LDS element by element; live rows outside that run
            // (only when the device tables disagree with the host's) are read element by element
            const uint32_t e0 = rem * m;
            const uint32_t dim = fast_div(e0, a.bn_magic, a.bn_shift);
            const uint32_t s0 = e0 - dim * bn;
            const int32_t nl = min(m, s_n[i] - static_cast<int32_t>(s0));    // live rows of the vector
            if (nl <= 0) continue;
            unsigned char* t0 = lds + i * tile_lds + s0 * lrow + dim * eb;
            const uint32_t slot0 = static_cast<uint32_t>(s_slot[i * bn + s0]);
            const int32_t run = (slot0 & static_cast<uint32_t>(m - 1)) ? 0 : leading_sources(s_has + i * bn + s0, m);
            if (run > 0)
                scatter_dim(__builtin_nontemporal_load(reinterpret_cast<const V4*>(
                                s_src[i * bn + s0] + uint64_t(dim) * bo * eb + uint64_t(slot0) * eb)),
                            t0, lrow, eb);
            for (int32_t k = run; k < nl; ++k) {
                const uint32_t row = s0 + static_cast<uint32_t>(k);
                if (!s_has[i * bn + row]) continue;
                const unsigned char* e = reinterpret_cast<const unsigned char*>(s_src[i * bn + row]) +
                                         uint64_t(dim) * bo * eb + uint64_t(s_slot[i * bn + row]) * eb;
                unsigned char* o = t0 + k * lrow;
                if (eb == 2) *reinterpret_cast<unsigned short*>(o) = *reinterpret_cast<const unsigned short*>(e);
                else if (eb == 4) *reinterpret_cast<unsigned int*>(o) = *reinterpret_cast<const unsigned int*>(e);
                else *o = *e;
            }
            continue;
        }
        const uint32_t r = fast_div(rem, a.vph_magic, a.vph_shift);
        const uint32_t c = rem - r * vph;
        const uint64_t base = s_src[i * bn + r];
        if (static_cast<int32_t>(r) >= s_n[i] || base == 0) continue;
        const uint32_t slot = static_cast<uint32_t>(s_slot[i * bn + r]);
        V4 val;
        if (a.old_layout == kLayoutNHD) {
            val = __builtin_nontemporal_load(reinterpret_cast<const V4*>(base + uint64_t(slot) * a.old_row_stride + c * 16));
        } else if (a.old_layout == kLayoutHND) {
            val = __builtin_nontemporal_load(reinterpret_cast<const V4*>(base + uint64_t(slot) * hb + c * 16));
        } else {                                                         // [dim / x][slot][x] (K)
            val = __builtin_nontemporal_load(reinterpret_cast<const V4*>(base + uint64_t(c) * bo * 16 + slot * 16));
        }
        *reinterpret_cast<V4*>(lds + i * tile_lds + r * lrow + c * 16) = val;
    }
    __syncthreads();

    // phase 2: every tile into the new pool in its layout, live slots only
    for (uint32_t x = tid; x < total; x += kTileThreads) {
        const uint32_t i = fast_div(x, a.rows_magic, a.rows_shift);
        const uint32_t v = x - i * per_tile;                            // vector of the tile in its own order
        const unsigned char* tl = lds + i * tile_lds;
        const int32_t n = s_n[i];
        const bool full = s_full[i];
        if (a.new_layout == kLayoutNHD) {
            const uint32_t r = fast_div(v, a.vph_magic, a.vph_shift);
            const uint32_t c = v - r * vph;
            if (full || (static_cast<int32_t>(r) < n && s_src[i * bn + r] != 0))
                __builtin_nontemporal_store(*reinterpret_cast<const V4*>(tl + r * lrow + c * 16),
                                            reinterpret_cast<V4*>(s_dst[i] + uint64_t(r) * a.new_row_stride + c * 16));
            continue;
        }
        V4* dst = reinterpret_cast<V4*>(s_dst[i] + uint64_t(v) * 16);
        if (a.new_layout == kLayoutHND) {
            const uint32_t r = fast_div(v, a.vph_magic, a.vph_shift);
            if (full || (static_cast<int32_t>(r) < n && s_src[i * bn + r] != 0))
                __builtin_nontemporal_store(*reinterpret_cast<const V4*>(tl + r * lrow + (v - r * vph) * 16), dst);
        } else if (s_kv[i] == 0) {                                       // [dim / x][slot][x]
            const uint32_t c = fast_div(v, a.bn_magic, a.bn_shift);
            const uint32_t r = v - c * bn;
            if (full || (static_cast<int32_t>(r) < n && s_src[i * bn + r] != 0))
                __builtin_nontemporal_store(*reinterpret_cast<const V4*>(tl + r * lrow + c * 16), dst);
        } else {                                                         // [dim][slot]
            const uint32_t e0 = v * m;
            const uint32_t dim = fast_div(e0, a.bn_magic, a.bn_shift);
            const uint32_t s0 = e0 - dim * bn;
            // rows without a source stay untouched
            const int32_t live =
                full ? m : min(min(m, n - static_cast<int32_t>(s0)), leading_sources(s_has + i * bn + s0, m));
            if (live <= 0) continue;
            const V4 val = gather_dim(tl + s0 * lrow + dim * eb, lrow, eb);
            if (live == m) __builtin_nontemporal_store(val, dst);
            else store_prefix_bytes(val, dst, live * eb, eb);
        }
    }
}

// Between a ROCm pool and one of another layout, with one block size on both sides: copy_strips with the other
// pool's rows in the place of staging.  A new block holds the tokens of one old block, slot for slot; where the device
// tables say otherwise the flag is set and each row is looked up (copy_strip_rows).  Bound by HBM.  Measured on MI355X against
// copy_local_tiles (us with the expansion): 7B MHA ROCm -> NHD 1090 -> 919, NHD -> ROCm 1083 -> 922, 70B GQA ROCm -> NHD
// 975 -> 803, fp8 NHD -> ROCm 584 -> 479.
struct LocalStripItem {
    uint64_t src_k, src_v, dst_k, dst_v;   // as LocalTileItem
    uint32_t strips, last;                 // as TileItem
    uint32_t strips_magic, last_magic;
    uint16_t strips_shift, last_shift;
    uint32_t pad;
};

struct LocalStripArgs {
    const BlockDesc* new_desc;
    const BlockDesc* old_desc;
    const int32_t* tok_off;       // first token of each sequence on the token axis
    const int32_t* old_blk_off;   // first old descriptor of each sequence
    int32_t* flag;
    int64_t old_block_stride, new_block_stride;
    uint32_t n_new_desc, n_old_desc;
    uint32_t old_block_size;      // and the new one
    uint32_t strip;               // columns per strip
    uint32_t head_vecs;           // columns of a head row
    uint32_t row_step;            // the other pool: bytes from a row to the next, NHD of all heads, HND of one
    uint32_t head_step;           // and from a head's row to the next head's
    uint32_t bo_magic, bo_shift;  // division by the block size
    uint32_t strip_magic, head_magic, vd_magic;
    uint16_t strip_shift, head_shift, vd_shift;
    StampCheck check;
    LocalStripItem items[kMaxLocalTileItems];
};
static_assert(sizeof(LocalStripArgs) < 4096, "local strip kernel arguments must stay below 4 KiB");

template <int EB> struct ElemT;
template <> struct ElemT<1> { typedef uint8_t type; };
template <> struct ElemT<2> { typedef uint16_t type; };
template <> struct ElemT<4> { typedef uint32_t type; };

// A strip of a block whose rows do not lie in one old block slot for slot: every lane takes a column of a row, from wherever
// that row's source is; rows without one are left alone.  It loads the unit again and divides by itself: what it shares
// with copy_local_strips is computed before the branch, and waited for there (7B MHA ROCm -> NHD 920 -> 957 us).
template <bool TO_ROCM, int EB>
__device__ __forceinline__ void copy_strip_rows(const LocalStripArgs& a, const LocalStripItem& it, uint32_t kv, uint32_t i,
                                                uint32_t c0, uint32_t cols) {
    typedef typename ElemT<EB>::type E;
    constexpr uint32_t M = kVecBytes / EB;
    const uint32_t bs = a.old_block_size, row = threadIdx.x / cols, col = c0 + threadIdx.x % cols;
    const uint32_t j = col / a.head_vecs;
    const LocalUnit<0> b = load_local_unit<0>(a, reinterpret_cast<const Int4*>(a.new_desc),
                                                 reinterpret_cast<const Int4*>(a.old_desc), a.tok_off, a.old_blk_off, i, 0);
    int32_t block;
    uint32_t slot;
    if (row >= static_cast<uint32_t>(b.n) || !find_source(a, b, row, &block, &slot)) return;
    const uint64_t src = (kv ? it.src_v : it.src_k) +
                         static_cast<uint64_t>(static_cast<uint32_t>(block)) * static_cast<uint64_t>(a.old_block_stride);
    const uint64_t dst = (kv ? it.dst_v : it.dst_k) +
                         static_cast<uint64_t>(static_cast<uint32_t>(b.block)) * static_cast<uint64_t>(a.new_block_stride);
    const uint32_t at = TO_ROCM ? slot : row, cell_at = TO_ROCM ? row : slot;   // in the other pool, in the ROCm pool
    const uint64_t line = (TO_ROCM ? src : dst) + static_cast<uint64_t>(at) * a.row_step +
                          static_cast<uint64_t>(j) * a.head_step + (col - j * a.head_vecs) * kVecBytes;
    const uint64_t cell = (TO_ROCM ? dst : src) + static_cast<uint64_t>(col) * bs * kVecBytes;
    if (kv == 0) {
        const uint64_t k = cell + cell_at * kVecBytes;
        *(REMP_GLOBAL Vec16*)(TO_ROCM ? k : line) = *(const REMP_GLOBAL Vec16*)(TO_ROCM ? line : k);
        return;
    }
    for (uint32_t e = 0; e < M; ++e) {
        const uint64_t v = cell + (e * bs + cell_at) * EB;
        *(REMP_GLOBAL E*)(TO_ROCM ? v : line + e * EB) = *(const REMP_GLOBAL E*)(TO_ROCM ? line + e * EB : v);
    }
}

template <bool TO_ROCM, int EB>
__global__ __launch_bounds__(kMaxStripThreads) void copy_local_strips(const LocalStripArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr uint32_t M = kVecBytes / EB;
    if (stale_descriptors(a.check)) return;
    const LocalStripItem& it = a.items[blockIdx.y];
    const uint32_t kv = blockIdx.z, bs = a.old_block_size, v = threadIdx.x, u = xcd_position(blockIdx.x);
    const uint32_t i = fast_div(u, it.strips_magic, it.strips_shift), s = u - i * it.strips;
    if (i >= a.n_new_desc) return;
    const LocalUnit<1> b = load_local_unit<1>(
        a, (const REMP_CONSTANT Int4*)(reinterpret_cast<uint64_t>(a.new_desc)),
        (const REMP_CONSTANT Int4*)(reinterpret_cast<uint64_t>(a.old_desc)),
        (const REMP_CONSTANT int32_t*)(reinterpret_cast<uint64_t>(a.tok_off)),
        (const REMP_CONSTANT int32_t*)(reinterpret_cast<uint64_t>(a.old_blk_off)), i, 0);
    const bool same = b.t0 >= 0 && b.q * bs == static_cast<uint32_t>(b.t0) && b.o.v.n >= b.n;
    const bool tail = s == it.strips - 1;
    const uint32_t cols = tail ? it.last : a.strip, c0 = s * a.strip;
    if (__builtin_expect(!same, 0)) {
        if (v == 0) *a.flag = kFlagTables;
        copy_strip_rows<TO_ROCM, EB>(a, it, kv, i, c0, cols);
        return;
    }
    const uint32_t n = static_cast<uint32_t>(b.n);
    const uint32_t lrow = (a.strip + 1) * kVecBytes;
    const uint64_t src = (kv ? it.src_v : it.src_k) + static_cast<uint64_t>(static_cast<uint32_t>(b.o.v.block)) *
                                                         static_cast<uint64_t>(a.old_block_stride);
    const uint64_t dst = (kv ? it.dst_v : it.dst_k) +
                         static_cast<uint64_t>(static_cast<uint32_t>(b.block)) * static_cast<uint64_t>(a.new_block_stride);
    // in the other pool: column c0 + col of row `row`
    const uint32_t row = fast_div(v, tail ? it.last_magic : a.strip_magic, tail ? it.last_shift : a.strip_shift);
    const uint32_t col = v - row * cols, j = fast_div(c0 + col, a.head_magic, a.head_shift);
    const uint64_t line_at = (TO_ROCM ? src : dst) + static_cast<uint64_t>(row) * a.row_step +
                             static_cast<uint64_t>(j) * a.head_step + (c0 + col - j * a.head_vecs) * kVecBytes;
    // in the ROCm pool, as in copy_strips
    const uint64_t cell_at = (TO_ROCM ? dst : src) + (static_cast<uint64_t>(c0) * bs + v) * kVecBytes;
    uint32_t x, y;
    if (kv == 0) {
        x = fast_div(v, a.bo_magic, a.bo_shift);
        y = v - x * bs;
    } else {
        x = fast_div(v, a.vd_magic, a.vd_shift);
        y = (v - x * (bs / M)) * M;
    }
    const bool in_rocm = x < (kv ? cols * M : cols) && y < n, in_rows = row < n;
    unsigned char* cell = lds + y * lrow + x * (kv ? EB : kVecBytes);
    unsigned char* line = lds + row * lrow + col * kVecBytes;
    if (TO_ROCM) {
        if (in_rows) *reinterpret_cast<Vec16*>(line) = __builtin_nontemporal_load((const REMP_GLOBAL Vec16*)line_at);
        __syncthreads();
        if (!in_rocm) return;
        if (kv == 0) {
            __builtin_nontemporal_store(*reinterpret_cast<const Vec16*>(cell), (REMP_GLOBAL Vec16*)cell_at);
            return;
        }
        const Vec16 val = gather_dim<EB>(cell, lrow);
        if (y + M <= n) __builtin_nontemporal_store(val, (REMP_GLOBAL Vec16*)cell_at);
        else store_prefix(val, reinterpret_cast<void*>(cell_at), static_cast<int32_t>((n - y) * EB), EB);
    } else {
        if (in_rocm) {
            const Vec16 val = __builtin_nontemporal_load((const REMP_GLOBAL Vec16*)cell_at);
            if (kv == 0) *reinterpret_cast<Vec16*>(cell) = val;
            else scatter_dim<EB>(val, cell, lrow);
        }
        __syncthreads();
        if (in_rows) __builtin_nontemporal_store(*reinterpret_cast<const Vec16*>(line), (REMP_GLOBAL Vec16*)line_at);
    }
}

}  // namespace remp
