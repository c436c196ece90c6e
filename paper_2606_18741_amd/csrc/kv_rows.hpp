// Copies of whole paged rows split among several staging slices (copy_rows, copy_pieces).
// Included by migrate.hip only (one translation unit holds every kernel).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kv_device.hpp"

namespace remp {

// ---------------------------------------------------------------------------
// whole paged rows
// ---------------------------------------------------------------------------
//
// When a new rank receives a layer's heads from several sources, the plain
// unpack writes each source's head range as its own pass over the new blocks,
// so every block row is opened once per source; likewise the plain pack reads
// an old block's rows once per destination when several destinations split
// its heads.  This variant walks the paged blocks once, with all nseg equal
// shares of a row (one per staging slice, consecutive heads), in one of two
// orders:
//   kByRow    the block's vectors in paged order, each lane picking its share's staging slice;
//   kByShare  consecutive workgroups take the same 1 KiB of one share after another.
// All layers of a call share the split of the row into slices.  Which of the two, or the plain
// per-slice copy, is fastest depends on how wide the rows are (rows_order).

constexpr int kMaxMergeSegs = 4;     // slices per row (copy_rows)
constexpr int kMaxPieceSegs = 8;     // the same of copy_pieces
constexpr int kMaxMergeGroups = 8;   // layers per launch

enum RowsOrder { kBySlice, kByRow, kByShare };   // kBySlice: not here, each slice by copy_runs

// Measured on MI355X (16-token blocks, blocks at random, TB/s by slice / by row / by share; the row order of
// packs with 256 threads, the others 64):
//   pack    2 x 256 B 6.23 / 6.07 / 6.11   2 x 512 B 6.16 / 6.11 / 6.09   2 x 1 KiB 6.14 / 6.19 / 6.23
//           2 x 2 KiB 5.75 / 6.14 / 6.61   2 x 4 KiB 6.52 / 6.03 / 6.65
//           4 x 128 B 6.23 / 6.67 / 5.82   4 x 256 B 6.25 / 6.71 / 5.93   4 x 512 B 6.17 / 6.72 / 6.04
//           4 x 1 KiB 5.60 / 7.04 / 6.45   4 x 2 KiB 5.90 / 7.16 / 6.50
//   unpack  2 x 256 B 6.07 / 5.82 / 5.87   2 x 512 B 6.04 / 5.83 / 5.85   2 x 1 KiB 6.36 / 5.96 / 6.24
//           2 x 2 KiB 5.55 / 5.92 / 6.32   2 x 4 KiB 6.57 / 6.14 / 6.68
//           4 x 128 B 5.81 / 6.04 / 5.59   4 x 256 B 5.73 / 6.09 / 5.59   4 x 512 B 6.16 / 6.10 / 5.82
//           4 x 1 KiB 5.59 / 5.83 / 6.20   4 x 2 KiB 5.68 / 5.92 / 6.30
// and three shares (us):
//   pack    3 x 64 B 1399 / 946 / 1421   3 x 256 B 920 / 917 / 910   3 x 512 B 870 / 887 / 873   3 x 2 KiB 722 / 748 / 727
//   unpack  3 x 64 B 1250 / 961 / 1143   3 x 256 B 997 / 902 / 910   3 x 512 B 908 / 859 / 869   3 x 2 KiB 744 / 713 / 721
// So: packs with three or four shares by row; rows of 4 KiB and more by share; rows of three or four shares
// of up to 256 B unpacked by row; the rest by slice (of three shares of 512 B to 1 KiB that costs 4-6% unpacked, and by row 1-3%
// packed).  Shares that are not whole vectors go by copy_pieces, or by row if
// they are less than a vector: by slice each would write parts of the same 64-byte sectors at different times.
constexpr uint32_t kByShareMinRow = 4096;
constexpr uint32_t kUnpackByRowMaxShare = 256;

inline RowsOrder rows_order(bool pack, uint32_t nseg, uint32_t seg_bytes, bool odd) {
    if (odd) return kByRow;
    if (pack && nseg > 2) return kByRow;
    if (static_cast<uint64_t>(nseg) * seg_bytes >= kByShareMinRow) return kByShare;
    if (nseg > 2 && seg_bytes <= kUnpackByRowMaxShare) return kByRow;
    return kBySlice;
}

struct MergeArgs {
    const BlockDesc* desc;
    int64_t block_stride;
    int64_t total_tokens;
    uint32_t n_desc;
    uint32_t row_stride;      // full paged row (all local heads)
    uint32_t nseg;            // shares per row
    uint32_t seg_bytes;       // bytes of one share of a row (= row_stride / nseg)
    uint32_t vpu;                      // vectors per (block, K/V) unit: of all shares (by row), of one (by share)
    uint32_t vpu_magic, vpu_shift;
    uint32_t vpr_magic, vpr_shift;     // division by the vectors of a row: of all shares (by row), of one (by share)
    uint32_t vps_magic, vps_shift;     // division by the vectors of a share of a row (by row)
    uint32_t seg_magic, seg_shift;     // division by nseg (by share; copy_pieces)
    uint32_t piece_magic, piece_shift; // division by seg_bytes (copy_pieces)
    uint32_t xcd;                      // as in CopyArgs (by row)
    StampCheck check;
    uint64_t paged_k[kMaxMergeGroups];
    uint64_t paged_v[kMaxMergeGroups];
    uint64_t stage[kMaxMergeGroups][kMaxPieceSegs];
};
static_assert(sizeof(MergeArgs) < 4096, "whole-row kernel arguments must stay below 4 KiB");

// Grid as copy_runs, with a layer per grid y.  By share, grid x counts the shares fastest.
template <bool PACK, int N, bool BY_ROW, bool ODD>
__global__ __launch_bounds__(kMaxRunThreads) void copy_rows(const MergeArgs args) {
    if (stale_descriptors(args.check)) return;
    const uint32_t g = blockIdx.y, kv = blockIdx.z;
    uint32_t w0, sg = 0;
    if (BY_ROW) {
        w0 = wave_first(args.xcd);
    } else {   // 64-thread workgroups: the division is uniform
        const uint32_t q = fast_div(blockIdx.x, args.seg_magic, args.seg_shift);
        sg = blockIdx.x - q * args.nseg;
        w0 = q * 64;
    }
    BlockDesc d;
    uint32_t r;
    if (!pick_unit<N>(args.desc, args.n_desc, w0, threadIdx.x & 63u, args.vpu, args.vpu_magic, args.vpu_shift, &d, &r))
        return;
    const uint32_t vps = (args.seg_bytes + kVecBytes - 1) / kVecBytes;   // vectors per share of a row
    const uint32_t row = fast_div(r, args.vpr_magic, args.vpr_shift);
    if (row >= static_cast<uint32_t>(d.n)) return;
    uint32_t c = r - row * (BY_ROW ? args.nseg * vps : vps);
    uint64_t base;
    if (BY_ROW) {
        sg = fast_div(c, args.vps_magic, args.vps_shift);
        c -= sg * vps;
        // selected from uniform values: a per-lane index into the arguments would be a load of its own
        const uint64_t st0 = args.stage[g][0], st1 = args.stage[g][1], st2 = args.stage[g][2], st3 = args.stage[g][3];
        base = sg == 0 ? st0 : sg == 1 ? st1 : sg == 2 ? st2 : st3;
    } else {
        base = args.stage[g][sg];
    }
    const uint64_t paged = (kv ? args.paged_v[g] : args.paged_k[g]) +
                           static_cast<uint64_t>(static_cast<uint32_t>(d.block)) * static_cast<uint64_t>(args.block_stride) +
                           static_cast<uint64_t>(row) * args.row_stride + sg * args.seg_bytes;
    const uint64_t stage =
        base + (static_cast<uint64_t>(kv) * args.total_tokens + static_cast<uint32_t>(d.tok) + row) * args.seg_bytes;
    move_vector<ODD>(PACK ? paged : stage, PACK ? stage : paged, c * kVecBytes, args.seg_bytes);
}

// Bytes [s, s + 16) of the 32 bytes lo, hi (s = 0..15).
__device__ __forceinline__ Vec16Any join_bytes(Vec16Any lo, Vec16Any hi, uint32_t s) {
    const uint32_t x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    uint32_t y[6], z[5];
#pragma unroll
    for (int i = 0; i < 6; ++i) y[i] = s & 8 ? x[i + 2] : x[i];
#pragma unroll
    for (int i = 0; i < 5; ++i) z[i] = s & 4 ? y[i + 1] : y[i];
    Vec16Any r;
    r.x = __builtin_amdgcn_alignbyte(z[1], z[0], s & 3);
    r.y = __builtin_amdgcn_alignbyte(z[2], z[1], s & 3);
    r.z = __builtin_amdgcn_alignbyte(z[3], z[2], s & 3);
    r.w = __builtin_amdgcn_alignbyte(z[4], z[3], s & 3);
    return r;
}

// The same for shares of 16 bytes or more that are not whole vectors (or not aligned).  Where each lane moves a
// vector of a share and the share's last part in words, stores end inside a line at every share; here a lane
// makes 16 consecutive bytes of the destination instead, from the one or two shares of a row (unpack: the block's rows
// are one run of the pool) or rows of a share (pack: they are one run of staging) that these lie in.  Only the
// last part of a run is moved in smaller parts.  A pack takes the shares of 8 waves in turn, eight workgroups
// apart, so that one XCD reads the lines that shares have in common.
// Measured on MI355X against rows_order's by row with the parts in words, 100-byte shares of 16-token blocks (us,
// pack + unpack): two shares packed 1204 -> 738, unpacked (blocks of 20) 1534 -> 680; four 1862 -> 1170 and
// 2687 -> 1018.
template <bool PACK, int N>
__global__ __launch_bounds__(64) void copy_pieces(const MergeArgs args) {
    if (stale_descriptors(args.check)) return;
    const uint32_t g = blockIdx.y, kv = blockIdx.z, seg = args.seg_bytes, nseg = args.nseg;
    uint32_t w0, share = 0;
    if (PACK) {
        const uint32_t l = blockIdx.x >> 3, q = fast_div(l, args.seg_magic, args.seg_shift);
        share = l - q * nseg;
        w0 = (q * 8 + (blockIdx.x & 7u)) * 64;
    } else {
        w0 = xcd_position(blockIdx.x) * 64;
    }
    BlockDesc d;
    uint32_t r;
    if (!pick_unit<N>(args.desc, args.n_desc, w0, threadIdx.x, args.vpu, args.vpu_magic, args.vpu_shift, &d, &r)) return;
    const uint32_t len = static_cast<uint32_t>(d.n) * (PACK ? seg : args.row_stride), off = r * kVecBytes;
    if (off >= len) return;
    const uint32_t q = fast_div(off, args.piece_magic, args.piece_shift), c = off - q * seg;
    const uint64_t paged = (kv ? args.paged_v[g] : args.paged_k[g]) +
                           static_cast<uint64_t>(static_cast<uint32_t>(d.block)) * static_cast<uint64_t>(args.block_stride);
    const uint64_t tok = static_cast<uint64_t>(kv) * args.total_tokens + static_cast<uint32_t>(d.tok);
    uint64_t dst, src, next;   // the run, and the pieces q and q + 1 that it is made of
    if (PACK) {
        dst = args.stage[g][share] + tok * seg;
        src = paged + share * seg + static_cast<uint64_t>(q) * args.row_stride;
        next = src + args.row_stride;
    } else {
        const uint32_t row = fast_div(q, args.seg_magic, args.seg_shift), sg = q - row * nseg;
        const uint32_t wrap = sg + 1 == nseg, sn = wrap ? 0 : sg + 1;
        dst = paged;
        src = args.stage[g][0];   // selected from uniform values, as in copy_rows
        next = src;
#pragma unroll
        for (uint32_t k = 1; k < kMaxPieceSegs; ++k) {
            src = sg == k ? args.stage[g][k] : src;
            next = sn == k ? args.stage[g][k] : next;
        }
        src += (tok + row) * seg;
        next += (tok + row + wrap) * seg;
    }
    if (off + kVecBytes > len) {   // inside the last piece
        move_vector<true>(src, dst + static_cast<uint64_t>(q) * seg, c, seg);
        return;
    }
    const uint32_t start = min(c, seg - kVecBytes);
    const Vec16Any lo = __builtin_nontemporal_load((const REMP_GLOBAL Vec16Any*)(src + start));
    Vec16Any hi = {0, 0, 0, 0};
    if (start < c) hi = __builtin_nontemporal_load((const REMP_GLOBAL Vec16Any*)next);
    __builtin_nontemporal_store(join_bytes(lo, hi, c - start), (REMP_GLOBAL Vec16Any*)(dst + off));
}

}  // namespace remp
