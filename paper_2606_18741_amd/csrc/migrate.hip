// GPU side of the KV-cache migration for gfx950: the host launch code and the
// C entry points (pack, unpack, local copy).  The kernels are in kv_expand.hpp
// (block-table expansion, descriptor sort), kv_copy.hpp (pack / unpack copy,
// NHD local copy), kv_tiles.hpp (head tiles of HND and ROCm pools)
// and kv_rows.hpp (whole-row unpack); all of them build in this one unit.
//
// The copy is pure data movement (no arithmetic on the payload), so it is
// bound by HBM bandwidth.  The layout makes every 16-byte vector of a slice
// have exactly one source and one destination:
//   paged side   [block][slot][local head][head_dim]  (a row run of head_count*head_dim
//                elements at a stride of H_loc*head_dim)
//   staging side [kv][token][head of the overlap][head_dim] (contiguous per block)
// so both directions are coalesced row copies.  A wave takes 64 consecutive
// vectors of one slice's live blocks and moves them with one load and one store
// per lane.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <unordered_set>
#include <vector>

#include "device_util.hpp"
#include "kv_copy.hpp"
#include "kv_device.hpp"
#include "kv_expand.hpp"
#include "kv_rows.hpp"
#include "kv_tiles.hpp"
#include "plan.hpp"

namespace remp {

// ---------------------------------------------------------------------------
// host launch code
// ---------------------------------------------------------------------------

static thread_local hipEvent_t g_trace_start = nullptr;
static thread_local hipEvent_t g_trace_stop = nullptr;

// Bound on the vectors of one unit.
constexpr uint64_t kMaxUnitVectors = uint64_t(1) << 31;

// Head tiles: slices with more vectors than this in a block go by ranges of heads, so that a launch can number a block's
// (units_per_launch).  1 GiB of one block: no layout in use comes near.
constexpr uint64_t kMaxTileVectors = uint64_t(1) << 26;

// A dispatch counts its work-items in 32 bits per grid dimension.
static remp_status check_grid(int64_t gx, int64_t gy, int threads, const char* what) {
    if (gx * threads >= (int64_t(1) << 32) || gx * gy >= (int64_t(1) << 32))
        return fail(REMP_E_UNSUPPORTED, std::string(what) + ": too many workgroups for one launch");
    return REMP_OK;
}

struct HostSlice {
    uint64_t paged_k, paged_v, stage;
    uint32_t row_bytes;
    int32_t layer = 0;        // global layer
    int32_t head_local = 0;   // first head of the slice within the paged rank's heads
    int32_t head_count = 0;
    uint64_t layer_k = 0, layer_v = 0;   // the layer's storage (no head offset)
};


// Descriptor stamps.  The old descriptors are a function of the plan alone
// (its old tables), the new ones of the plan and the new tables given to the
// call, so a stamp is a 64-bit hash of those (never 0, which no expansion
// writes).  Combination step after Boost's hash_combine, finished with the
// SplitMix64 output function (Steele, Lea and Flood, 2014).
static uint64_t mix64(uint64_t h, uint64_t v) { return h ^ (v + 0x9e3779b97f4a7c15ull + (h << 6) + (h >> 2)); }

static uint64_t finish64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    return z ? z : 1;
}

static uint64_t old_stamp(const remp_kv_plan_t& p) { return finish64(mix64(mix64(0, p.serial), 1)); }

static StampCheck no_check(int32_t* flag) {
    StampCheck c;
    c.at[0] = c.at[1] = nullptr;
    c.want[0] = c.want[1] = 0;
    c.flag = flag;
    return c;
}

static uint32_t sort_buckets(int64_t n_desc) {
    return static_cast<uint32_t>((std::max<int64_t>(n_desc, 1) + kDescsPerBucket - 1) / kDescsPerBucket);
}

// Enqueue expansion of `tables` into the workspace areas at scan_off / desc_off;
// `flag` is the status flag (reset first if reset_flag).  With bucket_off >= 0
// the expansion also clears and fills the bucket counters of the descriptor
// sort (new tables only).  A non-NULL stamp_at receives `stamp` in the same
// launch that writes the descriptors.
static remp_status launch_expand_many(const remp_kv_plan_t& p, const remp_dev_tables& dt, int32_t bs, int64_t nnz,
                                      int64_t num_blocks, int64_t n_desc, char* ws, int32_t* flag, int64_t scan_off,
                                      int64_t desc_off, bool reset_flag, hipStream_t stream, int64_t bucket_off,
                                      uint64_t* stamp_at, uint64_t stamp) {
    if (n_desc >= (int64_t(1) << 30)) return fail(REMP_E_UNSUPPORTED, "more than 2^30 live blocks in one call");
    int32_t* tok_off = reinterpret_cast<int32_t*>(ws + scan_off);
    int32_t* blk_off = tok_off + (p.num_seqs + 1);
    BlockDesc* desc = reinterpret_cast<BlockDesc*>(ws + desc_off);
    int32_t* bucket = bucket_off >= 0 ? reinterpret_cast<int32_t*>(ws + bucket_off) : nullptr;
    const uint32_t nb = bucket ? sort_buckets(n_desc) : 0;
    hipLaunchKernelGGL(expand_scan, dim3(1), dim3(kScanThreads), 0, stream, dt.seq_lens, p.num_seqs, bs,
                       reset_flag ? 1 : 0, flag, tok_off, blk_off, bucket, nb);
    if (remp_status st = hip_check(hipGetLastError(), "expand_scan launch")) return st;
    if (n_desc > 0) {
        const int64_t blocks = (n_desc + 255) / 256;
        hipLaunchKernelGGL(expand_emit, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, stream, dt.seq_lens,
                           dt.row_offsets, dt.block_ids, p.num_seqs, bs, tok_off, blk_off, nnz, num_blocks,
                           p.total_tokens, n_desc, desc, flag, bucket, nb, stamp_at, stamp);
        if (remp_status st = hip_check(hipGetLastError(), "expand_emit launch")) return st;
    }
    return REMP_OK;
}

// Finish the bucket sort of the n_desc new descriptors at desc_off (counted by
// the expansion into bucket_off) into sorted_off; stamp_at receives `stamp`.
static remp_status launch_sort_new(int64_t n_desc, int64_t num_blocks, char* ws, int64_t desc_off,
                                   int64_t bucket_off, int64_t sorted_off, uint64_t* stamp_at, uint64_t stamp,
                                   hipStream_t stream) {
    if (n_desc <= 0) return REMP_OK;
    const uint32_t nb = sort_buckets(n_desc);
    const uint32_t grid = static_cast<uint32_t>((n_desc + 255) / 256);
    const BlockDesc* desc = reinterpret_cast<const BlockDesc*>(ws + desc_off);
    int32_t* cnt = reinterpret_cast<int32_t*>(ws + bucket_off);
    BlockDesc* out = reinterpret_cast<BlockDesc*>(ws + sorted_off);
    const int64_t nblk = num_blocks > 0 ? num_blocks : 1;
    hipLaunchKernelGGL(sort_scan, dim3(1), dim3(kScanThreads), 0, stream, cnt, nb);
    hipLaunchKernelGGL(sort_scatter, dim3(grid), dim3(256), 0, stream, desc, static_cast<int32_t>(n_desc), nblk, nb,
                       cnt, out, stamp_at, stamp);
    return hip_check(hipGetLastError(), "descriptor sort launch");
}

// Expansion of one side's tables: with sorted_off >= 0 (the new side) also the descriptor sort into it, with its counters
// at bucket_off.  stamp_at receives `stamp` with the descriptors that the copies read.
static remp_status launch_expand(const remp_kv_plan_t& p, const remp_dev_tables& dt, int32_t bs, int64_t nnz,
                                 int64_t num_blocks, int64_t n_desc, char* ws, int32_t* flag, int64_t scan_off,
                                 int64_t desc_off, bool reset_flag, hipStream_t stream, int64_t bucket_off,
                                 int64_t sorted_off, uint64_t* stamp_at, uint64_t stamp) {
    const bool sort = sorted_off >= 0;
    if (p.num_seqs <= kSmallSeqs && n_desc > 0 && n_desc <= kSmallBlocks) {
        int32_t* tok_off = reinterpret_cast<int32_t*>(ws + scan_off);
        hipLaunchKernelGGL(expand_small, dim3(1), dim3(kScanThreads), 0, stream, dt.seq_lens, dt.row_offsets,
                           dt.block_ids, p.num_seqs, bs, nnz, num_blocks, p.total_tokens,
                           static_cast<int32_t>(n_desc), reset_flag ? 1 : 0, flag, tok_off, tok_off + (p.num_seqs + 1),
                           reinterpret_cast<BlockDesc*>(ws + desc_off),
                           sort ? reinterpret_cast<int32_t*>(ws + bucket_off) : nullptr, sort_buckets(n_desc),
                           sort ? reinterpret_cast<BlockDesc*>(ws + sorted_off) : nullptr, stamp_at, stamp);
        return hip_check(hipGetLastError(), "expand_small launch");
    }
    if (remp_status st = launch_expand_many(p, dt, bs, nnz, num_blocks, n_desc, ws, flag, scan_off, desc_off,
                                            reset_flag, stream, sort ? bucket_off : -1, sort ? nullptr : stamp_at, stamp))
        return st;
    return sort ? launch_sort_new(n_desc, num_blocks, ws, desc_off, bucket_off, sorted_off, stamp_at, stamp, stream)
                : REMP_OK;
}

// Threads of a pack / unpack workgroup: `builtin`, or one per 16 bytes of the tuning override's target.
static int run_threads(const remp_kv_plan_t& p, int builtin) {
    if (p.wg_bytes <= 0) return builtin;
    const int64_t waves = p.wg_bytes / (64 * static_cast<int64_t>(kVecBytes));
    return 64 * static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(waves, kMaxRunThreads / 64)));
}

// Workgroups of a grid whose kernel numbers them by xcd_position.
static uint64_t xcd_grid(uint64_t wgs) { return (wgs + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun); }

// Whether rows of `row` bytes, `stride` apart, or blocks of `block` bytes of whole rows, end inside lines of the L2 (128 bytes) that
// others go on in, or `odd` addresses make them: then the workgroups are numbered by xcd_position (MI355X, us, without / with: shares of
// 400 bytes 1317 / 1262, of 160 362 / 349; whole rows unpacked, blocks of 336 bytes 664 / 500, of 528 610 / 481, of 320 470 / 453, 1008
// bytes copied locally 533 / 450; where no line is shared it costs 0.7-1.5%).
static uint32_t shares_lines(uint64_t row, uint64_t stride, uint64_t block, bool odd) {
    return odd || (row == stride ? block : row | stride) % 128 != 0;
}

// Units of `vpu` vectors that one launch can number: a dispatch counts its work-items in 32 bits, and `shares`
// lanes of the grid take each vector number.
static uint32_t units_per_launch(int64_t n_desc, uint64_t vpu, uint32_t shares) {
    const uint64_t most = ((uint64_t(1) << 32) - 4 * kMaxRunThreads * uint64_t(8 * kXcdRun)) / (vpu * shares);
    return static_cast<uint32_t>(std::min<uint64_t>(static_cast<uint64_t>(n_desc), most));
}

// Bytes of the words that rows of at most `row` bytes go by when they are not whole vectors, all aligned: 8, or 0, which is
// 16 at any address.  Words leave no odd part at a row's end, which is an instruction of its own; longer rows have few
// of those, and 4-byte words take too many instructions (rates at the callers).
static int odd_words(uint64_t bits, uint32_t row, uint32_t most) { return bits % 8 == 0 && row <= most ? 8 : 0; }

// Slices per launch of copy_runs: kMaxItems, or as many as bring a launch to kLaunchBytes where slices are small, in
// equal launches.
static size_t items_per_launch(size_t slices, uint64_t slice_bytes, bool odd) {
    if (odd || slices <= kMaxItems || slice_bytes * kMaxItems >= kLaunchBytes) return kMaxItems;
    const size_t most = std::min<uint64_t>(kMaxSmallItems, kLaunchBytes / std::max<uint64_t>(1, slice_bytes));
    const size_t launches = (slices + most - 1) / most;
    return (slices + launches - 1) / launches;
}

template <bool PACK, int N>
static void launch_runs_n(const CopyArgs<kMaxSmallItems>& big, dim3 grid, int threads, RunShape shape, int vec,
                          hipStream_t stream) {
    if (grid.y > kMaxItems) {   // always of whole vectors (items_per_launch)
        if (shape == kRuns)
            hipLaunchKernelGGL((copy_runs<PACK, N, kRuns, 16, 1, kMaxSmallItems>), grid, dim3(threads), 0, stream, big);
        else
            hipLaunchKernelGGL((copy_runs<PACK, N, kCutRows, 16, 1, kMaxSmallItems>), grid, dim3(threads), 0, stream, big);
        return;
    }
    CopyArgs<kMaxItems> a;
    static_assert(offsetof(CopyArgs<kMaxItems>, items) == offsetof(CopyArgs<kMaxSmallItems>, items), "same head");
    std::memcpy(&a, &big, sizeof(a));
    if (shape == kRuns && vec == 16)
        hipLaunchKernelGGL((copy_runs<PACK, N, kRuns, 16, 1, kMaxItems>), grid, dim3(threads), 0, stream, a);
    else if (shape == kRuns)
        hipLaunchKernelGGL((copy_runs<PACK, N, kRuns, 0, 1, kMaxItems>), grid, dim3(threads), 0, stream, a);
    else if (vec == 16)
        hipLaunchKernelGGL((copy_runs<PACK, N, kCutRows, 16, 1, kMaxItems>), grid, dim3(threads), 0, stream, a);
    else if (vec == 8)
        hipLaunchKernelGGL((copy_runs<PACK, N, PACK ? kCutRows : kRows, 8, 2, kMaxItems>), grid, dim3(threads), 0, stream, a);
    else if (PACK || shape == kCutRows)
        hipLaunchKernelGGL((copy_runs<PACK, N, kCutRows, 0, 1, kMaxItems>), grid, dim3(threads), 0, stream, a);
    else
        hipLaunchKernelGGL((copy_runs<PACK, N, PACK ? kCutRows : kRows, 0, 1, kMaxItems>), grid, dim3(threads), 0, stream, a);
}

template <bool PACK>
static remp_status launch_copy(const remp_kv_plan_t& p, const std::vector<HostSlice>& slices, int64_t n_desc,
                               int32_t bs, int64_t block_stride, int32_t row_stride, const char* ws,
                               int64_t desc_off, const StampCheck& check, hipStream_t stream) {
    if (slices.empty() || n_desc == 0) return REMP_OK;
    if (n_desc >= (int64_t(1) << 30)) return fail(REMP_E_UNSUPPORTED, "more than 2^30 live blocks in one call");
    uint64_t bits = static_cast<uint64_t>(block_stride) | static_cast<uint64_t>(row_stride);
    uint32_t max_row = 0;
    bool contig = true;   // every slice takes whole rows
    for (const HostSlice& s : slices) {
        bits |= s.paged_k | s.paged_v | s.stage | s.row_bytes |
                (static_cast<uint64_t>(p.total_tokens) * s.row_bytes);
        max_row = std::max(max_row, s.row_bytes);
        contig &= static_cast<int64_t>(s.row_bytes) == row_stride;
    }
    const bool odd = bits % kVecBytes != 0;
    // a contiguous block is indexed by its bytes in 32 bits
    contig &= static_cast<uint64_t>(bs) * max_row < (uint64_t(1) << 31);
    // Parts of rows that are not whole vectors.  Unpacked, their ends are parts of lines that no other wave should
    // write: whole rows to a wave.  MI355X, blocks of 16, half of each row (us; before: LDS descriptors, aligned words):
    //   pack    72 B before 997, 8-byte words 985, any 1047    136 B 1062 / 948 / 990     520 B 768 / 726 / 707
    //           36 B before 1275, any 1121                     100 B 1325 / 1039          260 B 1198 / 834
    //   unpack  72 B before 1685, whole rows by 8-byte words 1599, any 1894, cut rows by words 1675
    //           136 B 1609 / 1679 / 1737 / 1768    200 B 1402 / 1381 / 1385 / 1447    328 B 1087 / 1106 / 1055 / 1180
    //           36 B before 2052, whole rows any 1744, cut any 1776    100 B 1890 / 1949 / 1956    260 B 1453 / 1234 / 1331
    //           520 B before 941, cut any 935, whole rows 938
    const int vec = !odd ? 16 : contig ? 0 : odd_words(bits, max_row, PACK ? kPackWordRow : kUnpackWordRow);
    const uint32_t word = vec ? vec : kVecBytes, words = kVecBytes / word;   // bytes of a word; words of a lane
    const uint32_t max_vpr = (max_row + word - 1) / word;
    const RunShape shape = contig ? kRuns : !PACK && odd && 2 * max_vpr <= 64 * words ? kRows : kCutRows;
    const auto vectors = [&](uint32_t row) {
        return contig ? (static_cast<uint64_t>(bs) * row + kVecBytes - 1) / kVecBytes
                      : static_cast<uint64_t>(bs) * ((row + word - 1) / word);
    };
    const uint64_t max_vpu = vectors(max_row);
    if (max_vpu >= kMaxUnitVectors) return fail(REMP_E_UNSUPPORTED, "a block of one slice exceeds 2^31 vectors");
    const int threads = run_threads(p, kRunThreads);

    CopyArgs<kMaxSmallItems> a;
    std::memset(&a, 0, sizeof(a));
    a.block_stride = block_stride;
    a.total_tokens = p.total_tokens;
    a.row_stride = static_cast<uint32_t>(row_stride);
    a.check = check;
    for (const HostSlice& s : slices)
        a.xcd |= shares_lines(s.row_bytes, a.row_stride, static_cast<uint64_t>(bs) * s.row_bytes, odd);
    const BlockDesc* desc = reinterpret_cast<const BlockDesc*>(ws + desc_off);
    const uint32_t per_launch = units_per_launch(n_desc, max_vpu, 1);
    if (g_trace_start) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_start, stream), "trace start event")) return st;
    }
    const size_t per = items_per_launch(slices.size(), 2 * static_cast<uint64_t>(p.total_tokens) * max_row, odd);
    for (size_t first = 0; first < slices.size(); first += per) {
        const size_t cnt = std::min<size_t>(per, slices.size() - first);
        int n = 1;   // units that a wave can meet: 1, 2, 4, 8, or any number (0)
        for (size_t i = 0; i < cnt; ++i) {
            const HostSlice& s = slices[first + i];
            CopyItem& c = a.items[i];
            c.paged_k = s.paged_k;
            c.paged_v = s.paged_v;
            c.stage = s.stage;
            c.row_bytes = s.row_bytes;
            c.vpu = static_cast<uint32_t>(vectors(s.row_bytes));
            int m = units_per_wave(c.vpu, 64 * words);
            if (shape == kRows) {   // numbered in rows instead of words
                c.rows = 64 * words / ((s.row_bytes + word - 1) / word);
                c.vpu = static_cast<uint32_t>(bs);
                m = units_per_wave(c.vpu, c.rows);
            }
            const FastDiv fv = make_fastdiv((s.row_bytes + word - 1) / word);
            const FastDiv fu = make_fastdiv(c.vpu);
            c.vpr_magic = fv.magic;
            c.vpr_shift = static_cast<uint16_t>(fv.shift);
            c.vpu_magic = fu.magic;
            c.vpu_shift = static_cast<uint16_t>(fu.shift);
            n = n == 0 || m == 0 ? 0 : std::max(n, m);
        }
        for (int64_t d0 = 0; d0 < n_desc; d0 += per_launch) {
            a.desc = desc + d0;
            a.n_desc = static_cast<uint32_t>(std::min<int64_t>(per_launch, n_desc - d0));
            dim3 grid(0, static_cast<uint32_t>(cnt), 2);
            if (shape == kRows) {
                const uint64_t rows = static_cast<uint64_t>(64 * words / max_vpr) * (threads / 64);   // of a workgroup
                grid.x = static_cast<uint32_t>(2 * ((a.n_desc * static_cast<uint64_t>(bs) + rows - 1) / rows));
                grid.z = 1;
            } else {
                const uint64_t wgs = (a.n_desc * max_vpu + threads * words - 1) / (threads * words);
                grid.x = static_cast<uint32_t>(a.xcd ? xcd_grid(wgs) : wgs);
            }
            switch (n) {
                case 1: launch_runs_n<PACK, 1>(a, grid, threads, shape, vec, stream); break;
                case 2: launch_runs_n<PACK, 2>(a, grid, threads, shape, vec, stream); break;
                case 4: launch_runs_n<PACK, 4>(a, grid, threads, shape, vec, stream); break;
                case 8: launch_runs_n<PACK, 8>(a, grid, threads, shape, vec, stream); break;
                default: launch_runs_n<PACK, 0>(a, grid, threads, shape, vec, stream); break;
            }
            if (remp_status st = hip_check(hipGetLastError(), PACK ? "pack launch" : "unpack launch")) return st;
        }
    }
    if (g_trace_stop) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_stop, stream), "trace stop event")) return st;
    }
    return REMP_OK;
}


// Columns per strip of ROCm tiles with `bs` slots and staging rows of at most `cols` columns (copy_strips):
// whole rows up to kStripLanes lanes, else runs of 128 bytes where rows are a multiple of that (a line of
// the L2, which then no other workgroup writes a part of), else equal strips.  Where rows are what is written
// (to_rows), longer runs are the better ones, as long as they divide the row and a workgroup has no more
// than 2 * kStripLanes lanes (MI355X, ROCm -> NHD kept slices, 4 KiB rows, runs of 128 / 256 / 512 / 1024 bytes:
// 1024 / 975 / 914 / 945 us; ROCm -> HND in 32-token blocks 128 / 256 / 512: 528 / 449 / 530).
static uint32_t strip_columns(uint32_t bs, uint32_t cols, bool to_rows) {
    const uint32_t most = std::max<uint32_t>(1, kStripLanes / bs);
    if (cols <= most) return cols;
    if (cols % 8 == 0) {
        uint32_t g = std::min<uint32_t>(8, kMaxStripThreads / bs);
        while (to_rows && cols % (2 * g) == 0 && bs * 2 * g <= 2 * kStripLanes) g *= 2;
        return g;
    }
    const uint32_t strips = (cols + most - 1) / most;
    return (cols + strips - 1) / strips;
}

// Whether strips of whole rows fill the lanes of their waves to 85%.
static bool strips_fill(uint32_t bs, uint32_t strip, uint32_t cols) {
    const uint32_t unit = bs * strip;
    return strip < cols || unit * 100 >= (unit + 63) / 64 * 64 * 85;
}

template <bool PACK>
static void launch_strips(const TileArgs& a, dim3 grid, int threads, size_t lds, int32_t eb, hipStream_t stream) {
    if (eb == 1) hipLaunchKernelGGL((copy_strips<PACK, 1>), grid, dim3(threads), lds, stream, a);
    else if (eb == 2) hipLaunchKernelGGL((copy_strips<PACK, 2>), grid, dim3(threads), lds, stream, a);
    else hipLaunchKernelGGL((copy_strips<PACK, 4>), grid, dim3(threads), lds, stream, a);
}

template <bool PACK>
static void launch_head_rows(const TileArgs& a, dim3 grid, int units, hipStream_t stream) {
    switch (units) {
        case 1: hipLaunchKernelGGL((copy_head_rows<PACK, 1>), grid, dim3(kRunThreads), 0, stream, a); break;
        case 2: hipLaunchKernelGGL((copy_head_rows<PACK, 2>), grid, dim3(kRunThreads), 0, stream, a); break;
        case 4: hipLaunchKernelGGL((copy_head_rows<PACK, 4>), grid, dim3(kRunThreads), 0, stream, a); break;
        case 8: hipLaunchKernelGGL((copy_head_rows<PACK, 8>), grid, dim3(kRunThreads), 0, stream, a); break;
        default: hipLaunchKernelGGL((copy_head_rows<PACK, 0>), grid, dim3(kRunThreads), 0, stream, a); break;
    }
}

// Slices of one layer when every layer of the call has that many, one after another, and a launch holds them; else 1.
static uint32_t layer_slices(const std::vector<HostSlice>& slices) {
    size_t n = 1;
    while (n < slices.size() && slices[n].layer == slices[0].layer) ++n;
    if (n > kMaxItems || slices.size() % n) return 1;
    for (size_t i = 0; i < slices.size(); ++i)
        if (slices[i].layer != slices[i - i % n].layer || (i % n == 0 && i && slices[i].layer == slices[i - 1].layer))
            return 1;
    return static_cast<uint32_t>(n);
}

// Calls add(first head, heads) for the ranges of `heads` heads that have at most kMaxTileVectors in a block, `tile` each.
template <typename F>
static void head_ranges(uint32_t heads, uint64_t tile, const F& add) {
    const uint32_t most = static_cast<uint32_t>(std::max<uint64_t>(1, kMaxTileVectors / tile));
    for (uint32_t h = 0; h < heads; h += most) add(h, std::min(most, heads - h));
}

template <bool PACK>
static remp_status launch_tile_groups(const remp_kv_plan_t& p, const std::vector<HostSlice>& slices, int64_t n_desc,
                                      int32_t bs, int64_t block_stride, int32_t max_hc, const char* ws,
                                      int64_t desc_off, const StampCheck& check, hipStream_t stream) {
    const int32_t eb = p.shape.elem_bytes;
    const int64_t hb = static_cast<int64_t>(p.shape.head_dim) * eb;
    const int64_t tile_bytes = bs * hb, lrow = hb + 16, tile_lds = bs * lrow;
    const int32_t tpw = static_cast<int32_t>(std::max<int64_t>(
        1, std::min<int64_t>({kTileWgBytes / tile_bytes, kTileLdsBytes / tile_lds, int64_t(kMaxUnitsPerWg)})));
    const int64_t gx = (n_desc * 2 * max_hc + tpw - 1) / tpw;
    if (remp_status st = check_grid(gx, kMaxItems, kTileThreads, "head tiles")) return st;

    GroupArgs a;
    std::memset(&a, 0, sizeof(a));
    a.desc = reinterpret_cast<const BlockDesc*>(ws + desc_off);
    a.block_stride = block_stride;
    a.total_tokens = p.total_tokens;
    a.n_desc = static_cast<int32_t>(n_desc);
    a.tiles_per_wg = tpw;
    a.block_size = bs;
    a.head_bytes = static_cast<int32_t>(hb);
    a.elem_bytes = eb;
    a.lds_row = static_cast<int32_t>(lrow);
    const FastDiv fvpt = make_fastdiv(static_cast<uint32_t>(tile_bytes / 16));
    const FastDiv fvph = make_fastdiv(static_cast<uint32_t>(hb / 16));
    const FastDiv fbs = make_fastdiv(static_cast<uint32_t>(bs));
    a.vpt_magic = fvpt.magic;
    a.vpt_shift = fvpt.shift;
    a.vph_magic = fvph.magic;
    a.vph_shift = fvph.shift;
    a.bs_magic = fbs.magic;
    a.bs_shift = fbs.shift;
    a.check = check;
    if (g_trace_start) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_start, stream), "trace start event")) return st;
    }
    for (size_t first = 0; first < slices.size(); first += kMaxItems) {
        const size_t cnt = std::min<size_t>(kMaxItems, slices.size() - first);
        for (size_t i = 0; i < cnt; ++i) {
            const HostSlice& s = slices[first + i];
            a.items[i] = GroupItem{s.paged_k, s.paged_v, s.stage, s.row_bytes};
        }
        const dim3 grid(static_cast<uint32_t>(gx), static_cast<uint32_t>(cnt));
        hipLaunchKernelGGL((copy_tile_groups<PACK>), grid, dim3(kTileThreads), static_cast<size_t>(tpw * tile_lds), stream, a);
        if (remp_status st = hip_check(hipGetLastError(), PACK ? "pack tile launch" : "unpack tile launch")) return st;
    }
    if (g_trace_stop) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_stop, stream), "trace stop event")) return st;
    }
    return REMP_OK;
}

template <bool PACK>
static remp_status launch_tiles(const remp_kv_plan_t& p, const std::vector<HostSlice>& whole, int64_t n_desc,
                                int32_t bs, int64_t block_stride, int32_t layout, const char* ws, int64_t desc_off,
                                const StampCheck& check, hipStream_t stream) {
    if (whole.empty() || n_desc == 0) return REMP_OK;
    if (n_desc >= (int64_t(1) << 30)) return fail(REMP_E_UNSUPPORTED, "more than 2^30 live blocks in one call");
    const int32_t eb = p.shape.elem_bytes;
    const int64_t hb = static_cast<int64_t>(p.shape.head_dim) * eb;
    std::vector<HostSlice> slices;
    for (const HostSlice& s : whole)
        head_ranges(static_cast<uint32_t>(s.head_count), static_cast<uint64_t>(bs) * hb / kVecBytes, [&](uint32_t h, uint32_t n) {
            HostSlice part = s;
            part.paged_k += static_cast<uint64_t>(h) * bs * hb;
            part.paged_v += static_cast<uint64_t>(h) * bs * hb;
            part.stage += static_cast<uint64_t>(h) * hb;
            part.head_count = static_cast<int32_t>(n);
            slices.push_back(part);
        });
    uint64_t bits = static_cast<uint64_t>(block_stride) | static_cast<uint64_t>(hb);
    uint32_t max_hc = 1;
    for (const HostSlice& s : slices) {
        bits |= s.paged_k | s.paged_v | s.stage;
        max_hc = std::max(max_hc, static_cast<uint32_t>(s.head_count));
    }
    if (bits & 15) return fail(REMP_E_ALIGN, "head-tile layouts need 16-byte aligned storage, staging and head rows");
    if (bs * (hb + 16) > kTileLdsBytes) return fail(REMP_E_UNSUPPORTED, "a (block, head) tile does not fit in LDS");

    TileArgs a;
    std::memset(&a, 0, sizeof(a));
    a.block_stride = block_stride;
    a.total_tokens = p.total_tokens;
    a.block_size = static_cast<uint32_t>(bs);
    a.head_bytes = static_cast<uint32_t>(hb);
    a.check = check;
    const auto set = [](auto* magic, uint16_t* shift, uint32_t divisor) {
        const FastDiv f = make_fastdiv(divisor);
        *magic = f.magic;
        *shift = static_cast<uint16_t>(f.shift);
    };
    const uint32_t head_vecs = static_cast<uint32_t>(hb / kVecBytes);
    const bool rocm = layout == kLayoutRocmSplit;
    const uint32_t max_cols = max_hc * head_vecs;
    a.strip = rocm ? strip_columns(a.block_size, max_cols, PACK) : 1;
    if (rocm && !strips_fill(a.block_size, a.strip, max_cols))
        return launch_tile_groups<PACK>(p, slices, n_desc, bs, block_stride, max_hc, ws, desc_off, check, stream);
    set(&a.strip_magic, &a.strip_shift, a.strip);
    set(&a.head_magic, &a.head_shift, head_vecs);
    set(&a.bs_magic, &a.bs_shift, a.block_size);
    set(&a.vd_magic, &a.vd_shift, rocm ? static_cast<uint32_t>(a.block_size * eb / kVecBytes) : 1);
    // lanes, and live blocks that one launch can number (work-items are counted in 32 bits)
    const int threads = rocm ? static_cast<int>((a.block_size * a.strip + 63) / 64 * 64) : kRunThreads;
    const uint64_t max_strips = (max_cols + a.strip - 1) / a.strip, max_vectors = static_cast<uint64_t>(bs) * max_cols;
    const uint64_t lanes = rocm ? max_strips * threads : max_vectors;   // per live block, at most
    const uint64_t piece = static_cast<uint64_t>(bs) * max_hc * hb;   // a slice's bytes of one block
    a.peers = piece >= kPeerMinBytes && piece < kPeerEndBytes ? layer_slices(slices) : 1;
    a.run = rocm ? static_cast<uint32_t>(max_strips)
                 : static_cast<uint32_t>(std::max<uint64_t>(1, static_cast<uint64_t>(bs) * head_vecs / kRunThreads));
    set(&a.run_magic, &a.run_shift, a.run);
    set(&a.peers_magic, &a.peers_shift, a.peers);
    const int64_t per_launch = units_per_launch(n_desc, lanes, 2 * a.peers);
    const uint32_t groups = kMaxItems / a.peers;   // layers per launch
    const size_t lds = static_cast<size_t>(bs) * (a.strip + 1) * kVecBytes;
    const BlockDesc* desc = reinterpret_cast<const BlockDesc*>(ws + desc_off);
    if (g_trace_start) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_start, stream), "trace start event")) return st;
    }
    for (size_t first = 0; first < slices.size(); first += groups * a.peers) {
        const size_t cnt = std::min<size_t>(groups * a.peers, slices.size() - first);
        int units = 1;   // units that a wave can meet, as in launch_copy (copy_head_rows)
        for (size_t i = 0; i < cnt; ++i) {
            const HostSlice& s = slices[first + i];
            const uint32_t heads = static_cast<uint32_t>(s.head_count), cols = heads * head_vecs;
            TileItem& t = a.items[i];
            t.paged_k = s.paged_k;
            t.paged_v = s.paged_v;
            t.stage = s.stage;
            t.row_bytes = s.row_bytes;
            t.heads = heads;
            t.strips = (cols + a.strip - 1) / a.strip;
            t.last = cols - (t.strips - 1) * a.strip;
            t.unit = a.block_size * (PACK ? cols : head_vecs);
            set(&t.strips_magic, &t.strips_shift, t.strips);
            set(&t.last_magic, &t.last_shift, t.last);
            set(&t.unit_magic, &t.unit_shift, t.unit);
            set(&t.heads_magic, &t.heads_shift, heads);
            set(&t.row_magic, &t.row_shift, cols);
            const int m = units_per_wave(t.unit);
            units = units == 0 || m == 0 ? 0 : std::max(units, m);
        }
        for (int64_t d0 = 0; d0 < n_desc; d0 += per_launch) {
            a.desc = desc + d0;
            a.n_desc = static_cast<uint32_t>(std::min<int64_t>(per_launch, n_desc - d0));
            const uint64_t gx = rocm ? a.n_desc * max_strips : (a.n_desc * max_vectors + threads - 1) / threads;
            const uint64_t wgs = (gx + a.run - 1) / a.run * a.run * a.peers;
            const dim3 grid(static_cast<uint32_t>(xcd_grid(wgs)), static_cast<uint32_t>(cnt / a.peers), 2);
            if (rocm) launch_strips<PACK>(a, grid, threads, lds, eb, stream);
            else launch_head_rows<PACK>(a, grid, units, stream);
            if (remp_status st = hip_check(hipGetLastError(), PACK ? "pack tile launch" : "unpack tile launch"))
                return st;
        }
    }
    if (g_trace_stop) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_stop, stream), "trace stop event")) return st;
    }
    return REMP_OK;
}

// Whole paged rows, when every layer of the call splits its rows the same way
// into 2..kMaxPieceSegs staging slices of equal head counts that cover all of
// the rank's heads.  Returns false if not applicable.
static bool merged_rows_apply(const std::vector<HostSlice>& slices, int32_t heads_per_rank,
                              std::vector<std::vector<const HostSlice*>>& groups) {
    std::vector<int32_t> layers;
    for (const HostSlice& s : slices)
        if (std::find(layers.begin(), layers.end(), s.layer) == layers.end()) layers.push_back(s.layer);
    groups.clear();
    for (int32_t l : layers) {
        std::vector<const HostSlice*> g;
        for (const HostSlice& s : slices)
            if (s.layer == l) g.push_back(&s);
        std::sort(g.begin(), g.end(), [](const HostSlice* a, const HostSlice* b) { return a->head_local < b->head_local; });
        if (g.size() < 2 || g.size() > static_cast<size_t>(kMaxPieceSegs)) return false;
        int32_t next = 0;                                 // equal slices tile the rank's heads exactly
        for (const HostSlice* s : g) {
            if (s->head_local != next || s->head_count != g.front()->head_count) return false;
            next += s->head_count;
        }
        if (next != heads_per_rank) return false;
        if (!groups.empty()) {                            // same split in every layer
            const auto& f = groups.front();
            if (g.size() != f.size()) return false;
            for (size_t i = 0; i < g.size(); ++i)
                if (g[i]->head_local != f[i]->head_local || g[i]->head_count != f[i]->head_count) return false;
        }
        groups.push_back(g);
    }
    return !groups.empty();
}

template <bool PACK, int N>
static void launch_rows_n(const MergeArgs& a, dim3 grid, int threads, RowsOrder order, bool odd, bool pieces,
                          hipStream_t stream) {
    if (pieces)
        hipLaunchKernelGGL((copy_pieces<PACK, N>), grid, dim3(threads), 0, stream, a);
    else if (order == kByShare)   // never odd (rows_order)
        hipLaunchKernelGGL((copy_rows<PACK, N, false, false>), grid, dim3(threads), 0, stream, a);
    else if (!odd)
        hipLaunchKernelGGL((copy_rows<PACK, N, true, false>), grid, dim3(threads), 0, stream, a);
    else
        hipLaunchKernelGGL((copy_rows<PACK, N, true, true>), grid, dim3(threads), 0, stream, a);
}

// The call's slices as whole paged rows; *done is false, and nothing is enqueued, when they do not form
// whole rows or are faster by slice (rows_order).
template <bool PACK>
static remp_status launch_rows(const remp_kv_plan_t& p, const std::vector<HostSlice>& slices, int32_t heads_per_rank,
                               int64_t n_desc, int32_t bs, int64_t block_stride, int32_t row_stride, const char* ws,
                               int64_t desc_off, const StampCheck& check, hipStream_t stream, bool* done) {
    *done = false;
    std::vector<std::vector<const HostSlice*>> groups;
    if (n_desc == 0 || n_desc >= (int64_t(1) << 30) || !merged_rows_apply(slices, heads_per_rank, groups)) return REMP_OK;
    // merged_rows_apply admits only equal shares that tile the row: nseg * seg_bytes == row_stride
    const uint32_t nseg = static_cast<uint32_t>(groups.front().size());
    const uint32_t seg_bytes = groups.front().front()->row_bytes;
    uint64_t bits = static_cast<uint64_t>(block_stride) | static_cast<uint64_t>(row_stride) | seg_bytes |
                    (static_cast<uint64_t>(p.total_tokens) * seg_bytes);
    for (const auto& g : groups)
        for (const HostSlice* s : g) bits |= s->layer_k | s->layer_v | s->stage;
    const bool odd = bits % kVecBytes != 0;
    const bool pieces = odd && seg_bytes >= kVecBytes;   // copy_pieces
    const RowsOrder order = rows_order(PACK, nseg, seg_bytes, odd);
    if (order == kBySlice || (nseg > kMaxMergeSegs && !pieces)) return REMP_OK;
    const uint64_t vps = (seg_bytes + kVecBytes - 1) / kVecBytes;
    const uint64_t vpr = order == kByRow ? nseg * vps : vps;
    const uint64_t vpu = pieces ? (static_cast<uint64_t>(bs) * (PACK ? seg_bytes : row_stride) + kVecBytes - 1) / kVecBytes
                                : static_cast<uint64_t>(bs) * vpr;
    if (vpu * nseg >= kMaxUnitVectors / (pieces ? kVecBytes : 1)) return REMP_OK;   // pieces: bytes in 32 bits
    *done = true;

    MergeArgs a;
    std::memset(&a, 0, sizeof(a));
    a.block_stride = block_stride;
    a.total_tokens = p.total_tokens;
    a.row_stride = static_cast<uint32_t>(row_stride);
    a.nseg = nseg;
    a.seg_bytes = seg_bytes;
    a.vpu = static_cast<uint32_t>(vpu);
    a.check = check;
    const FastDiv fu = make_fastdiv(a.vpu), fr = make_fastdiv(static_cast<uint32_t>(vpr));
    const FastDiv fv = make_fastdiv(static_cast<uint32_t>(vps)), fs = make_fastdiv(nseg);
    a.vpu_magic = fu.magic;
    a.vpu_shift = fu.shift;
    a.vpr_magic = fr.magic;
    a.vpr_shift = fr.shift;
    a.vps_magic = fv.magic;
    a.vps_shift = fv.shift;
    a.seg_magic = fs.magic;
    a.seg_shift = fs.shift;
    const FastDiv fp = make_fastdiv(seg_bytes);
    a.piece_magic = fp.magic;
    a.piece_shift = fp.shift;
    a.xcd = order == kByRow ? shares_lines(seg_bytes, row_stride, 0, odd) : 0;
    const bool wave = order == kByShare || pieces;
    const int threads = wave ? 64 : run_threads(p, PACK || odd ? kRowsPackThreads : kRunThreads);
    const uint32_t shares = order == kByShare || (pieces && PACK) ? nseg : 1;
    const BlockDesc* desc = reinterpret_cast<const BlockDesc*>(ws + desc_off);
    const uint32_t per_launch = units_per_launch(n_desc, vpu, shares);
    if (g_trace_start) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_start, stream), "trace start event")) return st;
    }
    for (size_t f = 0; f < groups.size(); f += kMaxMergeGroups) {
        const size_t cnt = std::min<size_t>(kMaxMergeGroups, groups.size() - f);
        for (size_t i = 0; i < cnt; ++i) {
            const auto& g = groups[f + i];
            a.paged_k[i] = g.front()->layer_k;
            a.paged_v[i] = g.front()->layer_v;
            for (size_t k = 0; k < g.size(); ++k) a.stage[i][k] = g[k]->stage;
        }
        for (int64_t d0 = 0; d0 < n_desc; d0 += per_launch) {
            a.desc = desc + d0;
            a.n_desc = static_cast<uint32_t>(std::min<int64_t>(per_launch, n_desc - d0));
            uint64_t wgs = (a.n_desc * vpu + threads - 1) / threads;
            if (pieces && PACK) wgs = (wgs + 7) / 8 * 8;
            else if (a.xcd) wgs = xcd_grid(wgs);
            const dim3 grid(static_cast<uint32_t>(wgs * shares), static_cast<uint32_t>(cnt), 2);
            switch (units_per_wave(a.vpu)) {
                case 1: launch_rows_n<PACK, 1>(a, grid, threads, order, odd, pieces, stream); break;
                case 2: launch_rows_n<PACK, 2>(a, grid, threads, order, odd, pieces, stream); break;
                case 4: launch_rows_n<PACK, 4>(a, grid, threads, order, odd, pieces, stream); break;
                case 8: launch_rows_n<PACK, 8>(a, grid, threads, order, odd, pieces, stream); break;
                default: launch_rows_n<PACK, 0>(a, grid, threads, order, odd, pieces, stream); break;
            }
            if (remp_status st = hip_check(hipGetLastError(), PACK ? "pack rows launch" : "unpack rows launch"))
                return st;
        }
    }
    if (g_trace_stop) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_stop, stream), "trace stop event")) return st;
    }
    return REMP_OK;
}

static bool aligned(const void* p, int64_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

static remp_status check_window(const remp_kv_plan_t* plan, int32_t l0, int32_t l1) {
    if (l0 < 0 || l1 < l0 || l1 > plan->shape.num_layers)
        return fail(REMP_E_RANGE, "layer window [" + std::to_string(l0) + ", " + std::to_string(l1) +
                                      ") outside [0, " + std::to_string(plan->shape.num_layers) + "]");
    return REMP_OK;
}

static remp_status check_pool(const remp_kv_plan_t* plan, const remp_kv_pool* pool, int32_t layers_per_rank,
                              int32_t block_size, const char* what) {
    if (!pool) return fail(REMP_E_INVALID, std::string(what) + " pool is NULL");
    if (pool->layout != kLayoutNHD && pool->layout != kLayoutHND && pool->layout != kLayoutRocmSplit)
        return fail(REMP_E_INVALID, std::string(what) + " pool has an unknown layout");
    const int64_t hb = static_cast<int64_t>(plan->shape.head_dim) * plan->shape.elem_bytes;
    if (pool->layout != kLayoutNHD && hb % 16 != 0)
        return fail(REMP_E_UNSUPPORTED, std::string(what) + " pool layout needs head_dim * elem_bytes % 16 == 0");
    if (pool->layout == kLayoutRocmSplit && (static_cast<int64_t>(block_size) * plan->shape.elem_bytes) % 16 != 0)
        return fail(REMP_E_UNSUPPORTED, std::string(what) + " pool layout needs block_size * elem_bytes % 16 == 0");
    if (pool->num_layers != layers_per_rank)
        return fail(REMP_E_INVALID, std::string(what) + " pool has " + std::to_string(pool->num_layers) +
                                        " layers, the rank holds " + std::to_string(layers_per_rank));
    if (!pool->k || !pool->v) return fail(REMP_E_INVALID, std::string(what) + " pool pointer arrays are NULL");
    return REMP_OK;
}

// A (block, head) tile of block_size rows of head_dim * elem_bytes bytes, each padded by 16 bytes, must fit
// the head-tile kernels' LDS budget; checked with the other arguments, before anything is enqueued.  Pack and unpack of HND pools
// need no LDS, but the header states the limit for both layouts, and the local copy between layouts needs it.
static remp_status check_tile_fits(const remp_kv_plan_t* plan, int32_t block_size, const char* what) {
    const int64_t hb = static_cast<int64_t>(plan->shape.head_dim) * plan->shape.elem_bytes;
    if (static_cast<int64_t>(block_size) * (hb + 16) > kTileLdsBytes)
        return fail(REMP_E_UNSUPPORTED, std::string(what) + ": a (block, head) tile of " + std::to_string(block_size) +
                                            " rows does not fit the LDS budget of the head-tile kernels");
    return REMP_OK;
}

static remp_status check_workspace(const remp_kv_plan_t* plan, void* ws, int64_t ws_bytes) {
    if (!ws) return fail(REMP_E_INVALID, "workspace is NULL");
    if (!aligned(ws, 256)) return fail(REMP_E_ALIGN, "workspace is not 256-byte aligned");
    if (ws_bytes < workspace_bytes(*plan))
        return fail(REMP_E_SIZE, "workspace has " + std::to_string(ws_bytes) + " bytes, needs " +
                                     std::to_string(workspace_bytes(*plan)));
    return REMP_OK;
}

static remp_status check_dev_tables(const remp_kv_plan_t* plan, const remp_dev_tables* dt, int64_t nnz,
                                    const char* what) {
    if (!dt) return fail(REMP_E_INVALID, std::string("device ") + what + " tables are NULL");
    if (plan->num_seqs > 0 && (!dt->seq_lens || !dt->row_offsets))
        return fail(REMP_E_INVALID, std::string("device ") + what + " table arrays are NULL");
    if (nnz > 0 && !dt->block_ids) return fail(REMP_E_INVALID, std::string("device ") + what + " block ids are NULL");
    return REMP_OK;
}

// New tables describe the planned sequences, every row is long enough, every
// live id is in range and used once, and the pool can hold the live cache.
static remp_status check_new_tables(const remp_kv_plan_t* plan, const remp_block_tables* nt,
                                    const remp_kv_pool* dst, int64_t* nnz_out, uint64_t* stamp_out) {
    if (!nt) return fail(REMP_E_INVALID, "new tables are NULL");
    const remp_block_tables& t = *nt;
    const remp_kv_shape& sh = plan->shape;
    if (t.num_seqs != plan->num_seqs)
        return fail(REMP_E_INVALID, "new tables describe a different number of sequences");
    if (t.num_seqs > 0 && (!t.seq_lens || !t.row_offsets)) return fail(REMP_E_INVALID, "new table arrays are NULL");
    if (t.num_blocks < 0 || t.num_blocks > INT32_MAX) return fail(REMP_E_INVALID, "new num_blocks out of range");
    if (plan->new_live_blocks > t.num_blocks)
        return fail(REMP_E_CAPACITY, "the live cache needs " + std::to_string(plan->new_live_blocks) +
                                         " blocks, the new pool has " + std::to_string(t.num_blocks));
    if (dst->num_blocks < t.num_blocks) return fail(REMP_E_SIZE, "destination pool smaller than its tables");
    int64_t nnz = 0;
    if (t.num_seqs > 0) {
        if (t.row_offsets[0] < 0) return fail(REMP_E_INVALID, "new row_offsets[0] < 0");
        nnz = t.row_offsets[t.num_seqs];
        if (nnz > 0 && !t.block_ids) return fail(REMP_E_INVALID, "new block_ids is NULL");
    }
    std::vector<uint8_t> used(static_cast<size_t>(t.num_blocks), 0);
    // the new descriptors depend on the plan, the pool size (bounds and sort buckets), the table
    // length and the ids the expansion reads
    uint64_t h = mix64(mix64(mix64(mix64(0, plan->serial), 2), static_cast<uint64_t>(t.num_blocks)),
                       static_cast<uint64_t>(nnz));
    for (int32_t q = 0; q < t.num_seqs; ++q) {
        if (t.seq_lens[q] != plan->seq_lens[q])
            return fail(REMP_E_INVALID, "new tables give sequence " + std::to_string(q) + " length " +
                                            std::to_string(t.seq_lens[q]) + ", planned " +
                                            std::to_string(plan->seq_lens[q]));
        const int32_t a = t.row_offsets[q], b = t.row_offsets[q + 1];
        if (b < a) return fail(REMP_E_INVALID, "new row_offsets decrease at sequence " + std::to_string(q));
        const int64_t need = ceil_div(t.seq_lens[q], sh.new_block_size);
        if (b - a < need) return fail(REMP_E_INVALID, "new table row of sequence " + std::to_string(q) + " too short");
        h = mix64(h, static_cast<uint32_t>(a));
        for (int64_t j = 0; j < need; ++j) {
            const int32_t id = t.block_ids[a + j];
            if (id < 0 || id >= t.num_blocks)
                return fail(REMP_E_RANGE, "new block id " + std::to_string(id) + " outside [0, " +
                                              std::to_string(t.num_blocks) + ")");
            if (used[id]) return fail(REMP_E_INVALID, "new block id " + std::to_string(id) + " used twice");
            used[id] = 1;
            h = mix64(h, static_cast<uint32_t>(id));
        }
    }
    *nnz_out = nnz;
    *stamp_out = finish64(h);
    return REMP_OK;
}

// Slices of the window for one side; fills `out`.  `pack`: items of old rank
// `rank`; else items of new rank `rank`.  skip_local leaves out the slices
// whose peer is the same global rank.
static remp_status collect_slices(const remp_kv_plan_t& p, bool pack, int32_t rank, int32_t l0, int32_t l1,
                                  const remp_kv_pool& pool, const remp_buffer* staging, bool skip_local,
                                  std::vector<HostSlice>& out) {
    const Ownership& mine = pack ? p.own_old : p.own_new;
    const int64_t hrow = static_cast<int64_t>(p.shape.head_dim) * p.shape.elem_bytes;
    const int32_t eb = p.shape.elem_bytes;
    for (const Item& it : p.items) {
        if ((pack ? it.src : it.dst) != rank || it.layer < l0 || it.layer >= l1) continue;
        const int32_t peer = pack ? it.dst : it.src;
        if (skip_local && peer == rank) continue;
        const Pair& pr = p.pairs[it.pair];
        const int32_t ws0 = std::max(l0, pr.layer_begin), ws1 = std::min(l1, pr.layer_end);
        const remp_buffer& sb = staging[peer];
        const int64_t need = static_cast<int64_t>(ws1 - ws0) * pr.slice_bytes;
        if (need > 0) {
            if (!sb.ptr)
                return fail(REMP_E_INVALID, std::string("staging buffer for ") + (pack ? "destination " : "source ") +
                                                std::to_string(peer) + " is NULL");
            if (sb.bytes < need)
                return fail(REMP_E_SIZE, "staging buffer for rank " + std::to_string(peer) + " has " +
                                             std::to_string(sb.bytes) + " bytes, the window needs " +
                                             std::to_string(need));
            if (!aligned(sb.ptr, eb)) return fail(REMP_E_ALIGN, "staging buffer not element aligned");
        }
        const int32_t li = it.layer - mine.first_layer(rank);
        void* k = pool.k[li];
        void* v = pool.v[li];
        if (!k || !v)
            return fail(REMP_E_INVALID, "pool storage of layer " + std::to_string(it.layer) + " is NULL");
        if (!aligned(k, eb) || !aligned(v, eb)) return fail(REMP_E_ALIGN, "pool storage not element aligned");
        const int64_t hstep = pool.layout == kLayoutNHD
                                  ? hrow
                                  : hrow * (pack ? p.shape.old_block_size : p.shape.new_block_size);
        const int64_t hoff = static_cast<int64_t>(it.head_begin - mine.first_head(rank)) * hstep;
        HostSlice s;
        s.paged_k = reinterpret_cast<uint64_t>(k) + hoff;
        s.paged_v = reinterpret_cast<uint64_t>(v) + hoff;
        s.stage = reinterpret_cast<uint64_t>(sb.ptr) + static_cast<uint64_t>(it.layer - ws0) * pr.slice_bytes;
        s.row_bytes = static_cast<uint32_t>(it.head_count * hrow);
        s.layer = it.layer;
        s.head_local = it.head_begin - mine.first_head(rank);
        s.head_count = it.head_count;
        s.layer_k = reinterpret_cast<uint64_t>(k);
        s.layer_v = reinterpret_cast<uint64_t>(v);
        out.push_back(s);
    }
    return REMP_OK;
}

// In an HND pool the rows of one head's tile are contiguous and in token
// order, so a slice of a single head has the staging slice's byte order: it is
// copied like an NHD slice whose rows are one head long.  Used for pack.  Measured on MI355X against copy_head_rows (us, so / by it):
// 256-byte rows in blocks of 16 1033 / 1040, of 64 1024 / 1037, of 1 521 / 529, 512 bytes 1023 / 1038, 1152 bytes 997 / 1014; only 160
// bytes in blocks of 20, which end inside lines, 1130 / 1084.  Unpacked the two are as close (529 / 534; 160 bytes 594 / 562).
static bool hnd_single_heads(int32_t layout, const std::vector<HostSlice>& slices) {
    if (layout != kLayoutHND) return false;
    for (const HostSlice& s : slices)
        if (s.head_count != 1) return false;
    return true;
}

// ---------------------------------------------------------------------------
// local copy: old pool -> new pool for slices that stay on the same rank
// ---------------------------------------------------------------------------

struct HostLocal {
    uint64_t src_k, src_v, dst_k, dst_v;
    uint32_t row_bytes;
};

template <int N, int M>
static void launch_local_n(const LocalArgs& a, dim3 grid, int threads, int vec, int words, hipStream_t stream) {
    if (vec == 16)
        hipLaunchKernelGGL((copy_local<N, M, 16, 1>), grid, dim3(threads), 0, stream, a);
    else if (vec == 8 && words == 2)
        hipLaunchKernelGGL((copy_local<N, M, 8, 2>), grid, dim3(threads), 0, stream, a);
    else if (vec == 8)
        hipLaunchKernelGGL((copy_local<N, M, 8, kLocalWords>), grid, dim3(threads), 0, stream, a);
    else
        hipLaunchKernelGGL((copy_local<N, M, 0, 1>), grid, dim3(threads), 0, stream, a);
}

template <bool TO_ROCM>
static void launch_local_strips_t(const LocalStripArgs& a, dim3 grid, int threads, size_t lds, int32_t eb,
                                  hipStream_t stream) {
    if (eb == 1) hipLaunchKernelGGL((copy_local_strips<TO_ROCM, 1>), grid, dim3(threads), lds, stream, a);
    else if (eb == 2) hipLaunchKernelGGL((copy_local_strips<TO_ROCM, 2>), grid, dim3(threads), lds, stream, a);
    else hipLaunchKernelGGL((copy_local_strips<TO_ROCM, 4>), grid, dim3(threads), lds, stream, a);
}

// Local copy between a ROCm pool and one of another layout, block sizes equal (copy_local_strips).
static remp_status launch_local_strips(const remp_kv_plan_t& p, const std::vector<HostLocal>& whole, uint32_t strip,
                                       uint32_t max_cols, int32_t old_layout, int32_t new_layout, const char* ws,
                                       const StampCheck& check, hipStream_t stream) {
    const remp_kv_shape& sh = p.shape;
    const WorkspaceLayout L = workspace_layout(p);
    const int64_t n_desc = p.new_live_blocks;
    const int32_t eb = sh.elem_bytes, bs = sh.new_block_size;
    const int64_t hb = static_cast<int64_t>(sh.head_dim) * eb;
    const int64_t orow = p.own_old.heads_per_rank() * hb, nrow = p.own_new.heads_per_rank() * hb;
    const bool to_rocm = new_layout == kLayoutRocmSplit;
    const int32_t other = to_rocm ? old_layout : new_layout;
    const uint64_t ostep = old_layout == kLayoutNHD ? hb : hb * bs, nstep = new_layout == kLayoutNHD ? hb : hb * bs;
    std::vector<HostLocal> items;
    for (const HostLocal& h : whole)
        head_ranges(static_cast<uint32_t>(h.row_bytes / hb), static_cast<uint64_t>(bs) * hb / kVecBytes, [&](uint32_t first, uint32_t n) {
            items.push_back(HostLocal{h.src_k + first * ostep, h.src_v + first * ostep, h.dst_k + first * nstep,
                                      h.dst_v + first * nstep, static_cast<uint32_t>(n * hb)});
        });
    max_cols = std::min<uint32_t>(max_cols, static_cast<uint32_t>(std::max<uint64_t>(hb / kVecBytes, kMaxTileVectors / bs)));
    const auto set = [](auto* magic, auto* shift, uint32_t divisor) {
        const FastDiv f = make_fastdiv(divisor);
        *magic = f.magic;
        *shift = static_cast<std::remove_reference_t<decltype(*shift)>>(f.shift);
    };

    LocalStripArgs a;
    std::memset(&a, 0, sizeof(a));
    a.old_desc = reinterpret_cast<const BlockDesc*>(ws + L.desc_old);
    a.tok_off = reinterpret_cast<const int32_t*>(ws + L.scan_old);
    a.old_blk_off = reinterpret_cast<const int32_t*>(ws + L.scan_old) + (p.num_seqs + 1);
    a.flag = reinterpret_cast<int32_t*>(const_cast<char*>(ws));
    a.old_block_stride = orow * bs;
    a.new_block_stride = nrow * bs;
    a.n_old_desc = static_cast<uint32_t>(p.old_live_blocks);
    a.old_block_size = static_cast<uint32_t>(bs);
    a.strip = strip;
    a.head_vecs = static_cast<uint32_t>(hb / kVecBytes);
    a.row_step = static_cast<uint32_t>(other == kLayoutHND ? hb : to_rocm ? orow : nrow);
    a.head_step = static_cast<uint32_t>(other == kLayoutHND ? hb * bs : hb);
    set(&a.bo_magic, &a.bo_shift, a.old_block_size);
    set(&a.strip_magic, &a.strip_shift, strip);
    set(&a.head_magic, &a.head_shift, a.head_vecs);
    set(&a.vd_magic, &a.vd_shift, static_cast<uint32_t>(bs * eb / kVecBytes));
    a.check = check;
    const int threads = static_cast<int>((a.old_block_size * strip + 63) / 64 * 64);
    const uint64_t max_strips = (max_cols + strip - 1) / strip;
    const int64_t per_launch = units_per_launch(n_desc, max_strips * threads, 1);
    const size_t lds = static_cast<size_t>(bs) * (strip + 1) * kVecBytes;
    const BlockDesc* desc = reinterpret_cast<const BlockDesc*>(ws + L.sorted_new);
    if (g_trace_start) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_start, stream), "trace start event")) return st;
    }
    for (size_t first = 0; first < items.size(); first += kMaxLocalTileItems) {
        const size_t cnt = std::min<size_t>(kMaxLocalTileItems, items.size() - first);
        for (size_t i = 0; i < cnt; ++i) {
            const HostLocal& h = items[first + i];
            LocalStripItem& c = a.items[i];
            const uint32_t cols = static_cast<uint32_t>(h.row_bytes / kVecBytes);
            c.src_k = h.src_k;
            c.src_v = h.src_v;
            c.dst_k = h.dst_k;
            c.dst_v = h.dst_v;
            c.strips = (cols + strip - 1) / strip;
            c.last = cols - (c.strips - 1) * strip;
            set(&c.strips_magic, &c.strips_shift, c.strips);
            set(&c.last_magic, &c.last_shift, c.last);
        }
        for (int64_t d0 = 0; d0 < n_desc; d0 += per_launch) {
            a.new_desc = desc + d0;
            a.n_new_desc = static_cast<uint32_t>(std::min<int64_t>(per_launch, n_desc - d0));
            const dim3 grid(static_cast<uint32_t>(xcd_grid(a.n_new_desc * max_strips)), static_cast<uint32_t>(cnt), 2);
            if (to_rocm) launch_local_strips_t<true>(a, grid, threads, lds, eb, stream);
            else launch_local_strips_t<false>(a, grid, threads, lds, eb, stream);
            if (remp_status st = hip_check(hipGetLastError(), "copy_local_strips launch")) return st;
        }
    }
    if (g_trace_stop) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_stop, stream), "trace stop event")) return st;
    }
    return REMP_OK;
}

// Local copy when either pool is not NHD: head tiles through LDS.  items carry
// the slice's first-head offsets in each pool's own layout.
static remp_status launch_local_tiles(const remp_kv_plan_t& p, const std::vector<HostLocal>& items,
                                      int32_t old_layout, int32_t new_layout, const char* ws,
                                      const StampCheck& check, hipStream_t stream) {
    const remp_kv_shape& sh = p.shape;
    const WorkspaceLayout L = workspace_layout(p);
    const int64_t n_desc = p.new_live_blocks;
    if (items.empty() || n_desc == 0) return REMP_OK;
    if (n_desc >= (int64_t(1) << 28)) return fail(REMP_E_UNSUPPORTED, "more than 2^28 live blocks in one call");
    const int32_t eb = sh.elem_bytes;
    const int64_t hb = static_cast<int64_t>(sh.head_dim) * eb;
    if (hb % 16 != 0) return fail(REMP_E_UNSUPPORTED, "head tiles need head_dim * elem_bytes % 16 == 0");
    const int32_t bo = sh.old_block_size, bn = sh.new_block_size;
    if (bn > kMaxLocalRows) return fail(REMP_E_UNSUPPORTED, "new block size above the local-copy row limit");
    const int64_t lds_row = hb + 16;
    const int64_t tile_lds = bn * lds_row;
    if (tile_lds > kTileLdsBytes) return fail(REMP_E_UNSUPPORTED, "a head tile does not fit the LDS budget");
    if (bo == bn && (old_layout == kLayoutRocmSplit) != (new_layout == kLayoutRocmSplit)) {
        uint32_t cols = 1;
        for (const HostLocal& h : items) cols = std::max(cols, static_cast<uint32_t>(h.row_bytes / kVecBytes));
        const uint32_t strip = strip_columns(static_cast<uint32_t>(bn), cols, new_layout != kLayoutRocmSplit);
        if (strips_fill(static_cast<uint32_t>(bn), strip, cols))
            return launch_local_strips(p, items, strip, cols, old_layout, new_layout, ws, check, stream);
    }
    int64_t T = std::max<int64_t>(1, kTileWgBytes / (bn * hb));
    T = std::min<int64_t>({T, kTileLdsBytes / tile_lds, kMaxLocalRows / bn, kMaxUnitsPerWg});
    const int64_t orow = p.own_old.heads_per_rank() * hb, nrow = p.own_new.heads_per_rank() * hb;

    LocalTileArgs a;
    std::memset(&a, 0, sizeof(a));
    a.new_desc = reinterpret_cast<const BlockDesc*>(ws + L.sorted_new);
    a.old_desc = reinterpret_cast<const BlockDesc*>(ws + L.desc_old);
    a.tok_off = reinterpret_cast<const int32_t*>(ws + L.scan_old);
    a.old_blk_off = reinterpret_cast<const int32_t*>(ws + L.scan_old) + (p.num_seqs + 1);
    a.flag = reinterpret_cast<int32_t*>(const_cast<char*>(ws));
    a.old_block_stride = orow * bo;
    a.new_block_stride = nrow * bn;
    a.n_new_desc = static_cast<int32_t>(n_desc);
    a.n_old_desc = static_cast<int32_t>(p.old_live_blocks);
    a.tiles_per_wg = static_cast<int32_t>(T);
    a.old_block_size = bo;
    a.new_block_size = bn;
    a.head_bytes = static_cast<int32_t>(hb);
    a.elem_bytes = eb;
    a.old_layout = old_layout;
    a.new_layout = new_layout;
    a.old_row_stride = static_cast<int32_t>(orow);
    a.new_row_stride = static_cast<int32_t>(nrow);
    a.old_head_step = static_cast<int32_t>(old_layout == kLayoutNHD ? hb : hb * bo);
    a.new_head_step = static_cast<int32_t>(new_layout == kLayoutNHD ? hb : hb * bn);
    a.lds_row = static_cast<int32_t>(lds_row);
    const FastDiv fv = make_fastdiv(static_cast<uint32_t>(hb / 16));
    const FastDiv fr = make_fastdiv(static_cast<uint32_t>(bn * (hb / 16)));
    const FastDiv fb = make_fastdiv(static_cast<uint32_t>(bn));
    a.vph_magic = fv.magic;
    a.vph_shift = fv.shift;
    a.rows_magic = fr.magic;
    a.rows_shift = fr.shift;
    a.bn_magic = fb.magic;
    a.bn_shift = fb.shift;
    a.check = check;
    if (g_trace_start) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_start, stream), "trace start event")) return st;
    }
    for (size_t first = 0; first < items.size(); first += kMaxLocalTileItems) {
        const size_t cnt = std::min<size_t>(kMaxLocalTileItems, items.size() - first);
        int32_t max_hc = 1;
        for (size_t i = 0; i < cnt; ++i) {
            const HostLocal& h = items[first + i];
            LocalTileItem& c = a.items[i];
            c.src_k = h.src_k;
            c.src_v = h.src_v;
            c.dst_k = h.dst_k;
            c.dst_v = h.dst_v;
            c.heads = static_cast<int32_t>(h.row_bytes / hb);
            max_hc = std::max(max_hc, c.heads);
        }
        const int64_t gx = (n_desc * 2 * max_hc + T - 1) / T;
        if (remp_status st = check_grid(gx, kMaxLocalTileItems, kTileThreads, "local head tiles")) return st;
        // 32-bit vector indices per workgroup: T tiles of bn rows of hb / 16 vectors
        hipLaunchKernelGGL(copy_local_tiles, dim3(static_cast<uint32_t>(gx), static_cast<uint32_t>(cnt)),
                           dim3(kTileThreads), static_cast<size_t>(local_tile_lds_bytes(T, bn, lds_row)), stream, a);
        if (remp_status st = hip_check(hipGetLastError(), "copy_local_tiles launch")) return st;
    }
    if (g_trace_stop) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_stop, stream), "trace stop event")) return st;
    }
    return REMP_OK;
}

static remp_status launch_local(const remp_kv_plan_t& p, const std::vector<HostLocal>& items, const char* ws,
                                const StampCheck& check, hipStream_t stream) {
    const remp_kv_shape& sh = p.shape;
    const WorkspaceLayout L = workspace_layout(p);
    const int64_t n_desc = p.new_live_blocks;
    if (items.empty() || n_desc == 0) return REMP_OK;
    if (n_desc >= (int64_t(1) << 30)) return fail(REMP_E_UNSUPPORTED, "more than 2^30 live blocks in one call");
    const int64_t hrow = static_cast<int64_t>(sh.head_dim) * sh.elem_bytes;
    const int64_t orow = p.own_old.heads_per_rank() * hrow, nrow = p.own_new.heads_per_rank() * hrow;
    const int32_t bo = sh.old_block_size, bn = sh.new_block_size;
    uint64_t bits = static_cast<uint64_t>(orow) | static_cast<uint64_t>(nrow);
    uint32_t max_row = 0, min_row = items[0].row_bytes;
    for (const HostLocal& it : items) {
        bits |= it.src_k | it.src_v | it.dst_k | it.dst_v | it.row_bytes;
        max_row = std::max(max_row, it.row_bytes);
        min_row = std::min(min_row, it.row_bytes);
    }
    // Rows that are not whole vectors (MI355X, us; before: rows resolved into LDS, aligned words): 200 of 400 bytes in
    // blocks of 20, before 719, 8-byte words (4 to a lane) 690, any 779; in blocks of 64 706 / 666 / 757; blocks of 64 to
    // 20 718 / 704 / 776; 520 of 1040 bytes 857 / 756 / 746; any for rows of 4-byte words, 100 of 200 bytes 1268 / 1095.
    const bool odd = bits % kVecBytes != 0;
    const int vec = odd ? odd_words(bits, max_row, kLocalWordRow) : 16;
    const uint32_t word = vec ? vec : kVecBytes;   // bytes of a word
    const auto vectors = [&](uint32_t row) { return static_cast<uint64_t>(bn) * ((row + word - 1) / word); };
    const uint64_t max_vpu = vectors(max_row);
    uint32_t xcd = 0;
    // copy_local_rows: where waves of copy_local meet more than two blocks
    bool lookup = !odd && min_row >= kLookupMinRow && static_cast<uint64_t>(bn) * min_row >= kLookupMinBlock &&
                  static_cast<uint64_t>(bn) * nrow % 64 == 0;
    for (const HostLocal& it : items) {
        const uint32_t rows = shares_lines(it.row_bytes, orow, 0, odd) | shares_lines(it.row_bytes, nrow, 0, odd);
        const int u = units_per_wave(static_cast<uint32_t>(vectors(it.row_bytes)));
        lookup &= !rows && u != 1 && u != 2;
        xcd |= rows | shares_lines(it.row_bytes, nrow, static_cast<uint64_t>(bn) * nrow, odd);
    }
    if (lookup) xcd = 0;
    const uint32_t words = lookup ? kLookupVectors : vec != 8 ? 1 : max_vpu >= 64 * kLocalWords ? kLocalWords : 2;   // of a lane
    if (bn > kMaxLocalRows) return fail(REMP_E_UNSUPPORTED, "new block size above the local-copy row limit");
    if (max_vpu >= kMaxUnitVectors) return fail(REMP_E_UNSUPPORTED, "a block of one slice exceeds 2^31 vectors");
    const int threads = run_threads(p, lookup ? kLookupThreads : kRunThreads);

    LocalArgs a;
    std::memset(&a, 0, sizeof(a));
    a.old_desc = reinterpret_cast<const BlockDesc*>(ws + L.desc_old);
    a.tok_off = reinterpret_cast<const int32_t*>(ws + L.scan_old);
    a.old_blk_off = reinterpret_cast<const int32_t*>(ws + L.scan_old) + (p.num_seqs + 1);
    a.flag = reinterpret_cast<int32_t*>(const_cast<char*>(ws));
    a.old_block_stride = orow * bo;
    a.new_block_stride = nrow * bn;
    a.n_old_desc = static_cast<uint32_t>(p.old_live_blocks);
    a.old_row_stride = static_cast<uint32_t>(orow);
    a.new_row_stride = static_cast<uint32_t>(nrow);
    a.old_block_size = static_cast<uint32_t>(bo);
    const FastDiv fo = make_fastdiv(static_cast<uint32_t>(bo));
    a.bo_magic = fo.magic;
    a.bo_shift = fo.shift;
    const FastDiv fn = make_fastdiv(static_cast<uint32_t>(bn));
    a.new_block_size = static_cast<uint32_t>(bn);
    a.bn_magic = fn.magic;
    a.bn_shift = fn.shift;
    a.check = check;
    a.xcd = xcd;
    const BlockDesc* desc = reinterpret_cast<const BlockDesc*>(ws + L.sorted_new);
    const uint32_t per_launch = units_per_launch(n_desc, max_vpu, 1);
    if (g_trace_start) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_start, stream), "trace start event")) return st;
    }
    for (size_t first = 0; first < items.size(); first += kMaxLocalItems) {
        const size_t cnt = std::min<size_t>(kMaxLocalItems, items.size() - first);
        int n = 1;        // units that a wave can meet, as in launch_copy
        uint32_t m = 1;   // old blocks that the rows of one of them can come from
        for (size_t i = 0; i < cnt; ++i) {
            const HostLocal& h = items[first + i];
            LocalItem& c = a.items[i];
            c.src_k = h.src_k;
            c.src_v = h.src_v;
            c.dst_k = h.dst_k;
            c.dst_v = h.dst_v;
            c.row_bytes = h.row_bytes;
            c.vpu = static_cast<uint32_t>(vectors(h.row_bytes));
            const uint32_t vpr = (h.row_bytes + word - 1) / word;
            const FastDiv fv = make_fastdiv(vpr);
            const FastDiv fu = make_fastdiv(c.vpu);
            c.vpr_magic = fv.magic;
            c.vpr_shift = static_cast<uint16_t>(fv.shift);
            c.vpu_magic = fu.magic;
            c.vpu_shift = static_cast<uint16_t>(fu.shift);
            const int u = units_per_wave(c.vpu, 64 * words);
            n = n == 0 || u == 0 ? 0 : std::max(n, u);
            const uint32_t rows = std::min<uint32_t>(bn, pieces_per_wave(vpr, 64 * words));
            if (bo != bn) m = std::max(m, (rows + bo - 2) / bo + 1);
        }
        // By scalar loads: one or two old blocks of each of one or two new ones, or one of each of four of equal size.
        for (int64_t d0 = 0; d0 < n_desc; d0 += per_launch) {
            a.new_desc = desc + d0;
            a.n_new_desc = static_cast<uint32_t>(std::min<int64_t>(per_launch, n_desc - d0));
            const uint64_t wgs = (a.n_new_desc * max_vpu + threads * words - 1) / (threads * words);
            const dim3 grid(static_cast<uint32_t>(a.xcd ? xcd_grid(wgs) : wgs), static_cast<uint32_t>(cnt), 2);
            if (lookup) {
                hipLaunchKernelGGL(copy_local_rows, grid, dim3(threads), 0, stream, a);
                if (remp_status st = hip_check(hipGetLastError(), "copy_local_rows launch")) return st;
                continue;
            }
            switch (n) {
                case 1:
                    if (m == 1) launch_local_n<1, 1>(a, grid, threads, vec, words, stream);
                    else if (m == 2) launch_local_n<1, 2>(a, grid, threads, vec, words, stream);
                    else launch_local_n<1, 0>(a, grid, threads, vec, words, stream);
                    break;
                case 2:
                    if (m == 1) launch_local_n<2, 1>(a, grid, threads, vec, words, stream);
                    else if (m == 2) launch_local_n<2, 2>(a, grid, threads, vec, words, stream);
                    else launch_local_n<2, 0>(a, grid, threads, vec, words, stream);
                    break;
                case 4:
                    if (bo == bn) launch_local_n<4, 1>(a, grid, threads, vec, words, stream);
                    else launch_local_n<4, 0>(a, grid, threads, vec, words, stream);
                    break;
                default: launch_local_n<0, 1>(a, grid, threads, vec, words, stream); break;
            }
            if (remp_status st = hip_check(hipGetLastError(), "copy_local launch")) return st;
        }
    }
    if (g_trace_stop) {
        if (remp_status st = hip_check(hipEventRecord(g_trace_stop, stream), "trace stop event")) return st;
    }
    return REMP_OK;
}

static bool ranges_overlap(uint64_t a, uint64_t an, uint64_t b, uint64_t bn) { return a < b + bn && b < a + an; }

// Argument checks shared by the unpack entry points (everything but the workspace and the tables).
static remp_status check_unpack_args(const remp_kv_plan_t* plan, int32_t new_rank, int32_t layer_begin,
                                     int32_t layer_end, const remp_buffer* staging, const remp_kv_pool* dst,
                                     uint32_t flags) {
    if (flags & ~static_cast<uint32_t>(REMP_KV_SKIP_LOCAL | REMP_KV_REUSE_DESCRIPTORS))
        return fail(REMP_E_INVALID, "unknown flags");
    if (new_rank < 0 || new_rank >= plan->own_new.world())
        return fail(REMP_E_RANGE, "new_rank " + std::to_string(new_rank) + " outside [0, " +
                                      std::to_string(plan->own_new.world()) + ")");
    if (remp_status st = check_window(plan, layer_begin, layer_end)) return st;
    if (remp_status st = check_pool(plan, dst, plan->own_new.layers_of_rank(new_rank), plan->shape.new_block_size,
                                    "destination"))
        return st;
    if (!staging) return fail(REMP_E_INVALID, "staging array is NULL");
    return REMP_OK;
}

// Unpack with its scratch areas at `ws` (laid out by workspace_layout) and the status flag at `flag`.
static remp_status unpack_impl(const remp_kv_plan_t* plan, int32_t new_rank, int32_t layer_begin, int32_t layer_end,
                               const remp_buffer* staging, const remp_kv_pool* dst,
                               const remp_block_tables* new_tables, const remp_dev_tables* new_dev_tables, char* ws,
                               int32_t* flag, uint32_t flags, hipStream_t stream) {
    int64_t nnz = 0;
    uint64_t new_stamp = 0;
    if (remp_status st = check_new_tables(plan, new_tables, dst, &nnz, &new_stamp)) return st;
    if (remp_status st = check_dev_tables(plan, new_dev_tables, nnz, "new")) return st;

    std::vector<HostSlice> slices;
    if (remp_status st = collect_slices(*plan, false, new_rank, layer_begin, layer_end, *dst, staging,
                                        (flags & REMP_KV_SKIP_LOCAL) != 0, slices))
        return st;
    if (dst->layout != kLayoutNHD)
        if (remp_status st = check_tile_fits(plan, plan->shape.new_block_size, "unpack")) return st;
    if (layer_begin == layer_end || plan->new_live_blocks == 0) return REMP_OK;   // as in pack
    const remp_kv_shape& sh = plan->shape;
    const int64_t row_stride = static_cast<int64_t>(plan->own_new.heads_per_rank()) * sh.head_dim * sh.elem_bytes;
    const WorkspaceLayout L = workspace_layout(*plan);
    uint64_t* new_at = reinterpret_cast<uint64_t*>(ws + L.stamp_new);
    StampCheck check = no_check(flag);
    if (flags & REMP_KV_REUSE_DESCRIPTORS) {
        check.at[0] = new_at;
        check.want[0] = new_stamp;
    } else {
        if (remp_status st = launch_expand(*plan, *new_dev_tables, sh.new_block_size, nnz, new_tables->num_blocks,
                                           plan->new_live_blocks, ws, flag, L.scan_new, L.desc_new, true, stream,
                                           L.bucket_new, L.sorted_new, new_at, new_stamp))
            return st;
    }
    if (dst->layout != kLayoutNHD)
        return launch_tiles<false>(*plan, slices, plan->new_live_blocks, sh.new_block_size,
                                   row_stride * sh.new_block_size, dst->layout, ws, L.sorted_new, check, stream);
    bool done = false;
    if (remp_status st = launch_rows<false>(*plan, slices, plan->own_new.heads_per_rank(), plan->new_live_blocks,
                                            sh.new_block_size, row_stride * sh.new_block_size,
                                            static_cast<int32_t>(row_stride), ws, L.sorted_new, check, stream, &done))
        return st;
    if (done) return REMP_OK;
    return launch_copy<false>(*plan, slices, plan->new_live_blocks, sh.new_block_size, row_stride * sh.new_block_size,
                              static_cast<int32_t>(row_stride), ws, L.sorted_new, check, stream);
}

// ---------------------------------------------------------------------------
// static scratch of the allocation-free unpack
// ---------------------------------------------------------------------------
//
// remp_kv_unpack_noalloc keeps its workspace areas in this array instead of a
// caller buffer.  Each device that loads the library holds its own copy until
// the process ends; the host-side name below is only a stand-in, so kernels
// get the device address that hipGetSymbolAddress returns for the current
// device, resolved once per device on that device's first call.
constexpr int64_t kScratchBytes = REMP_KV_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[kScratchBytes];

constexpr int kMaxScratchDevices = 64;
static std::atomic<char*> g_scratch_ptr[kMaxScratchDevices];
static std::mutex g_scratch_mu;

static remp_status scratch_of_current_device(hipStream_t stream, char** out) {
    int dev = -1;
    if (remp_status st = hip_check(hipGetDevice(&dev), "hipGetDevice")) return st;
    if (stream) {   // the kernels run on the stream's device: its scratch must be that device's copy
        hipDevice_t sdev = -1;
        if (remp_status st = hip_check(hipStreamGetDevice(stream, &sdev), "hipStreamGetDevice")) return st;
        if (sdev != dev)
            return fail(REMP_E_INVALID, "the stream belongs to device " + std::to_string(sdev) +
                                            ", the current device is " + std::to_string(dev));
    }
    if (dev < 0 || dev >= kMaxScratchDevices)
        return fail(REMP_E_UNSUPPORTED, "device index " + std::to_string(dev) + " beyond the static scratch table");
    char* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
        if (!p) {
            void* addr = nullptr;
            if (remp_status st = hip_check(hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch)),
                                           "hipGetSymbolAddress(scratch)"))
                return st;
            if (!addr || !aligned(addr, 256)) return fail(REMP_E_HIP, "static scratch has no 256-byte aligned address");
            p = static_cast<char*>(addr);
            g_scratch_ptr[dev].store(p, std::memory_order_release);
        }
    }
    *out = p;
    return REMP_OK;
}

}  // namespace remp

using namespace remp;

extern "C" {

void remp_kv_set_trace_events(hipEvent_t start, hipEvent_t stop) {
    g_trace_start = start;
    g_trace_stop = stop;
}

remp_status remp_kv_pack(const remp_kv_plan_t* plan, int32_t old_rank, int32_t layer_begin, int32_t layer_end,
                         const remp_kv_pool* src, const remp_dev_tables* old_tables, const remp_buffer* staging,
                         void* workspace, int64_t workspace_bytes_, uint32_t flags, hipStream_t stream) {
    clear_error();
    if (!plan) return fail(REMP_E_INVALID, "plan is NULL");
    if (flags & ~static_cast<uint32_t>(REMP_KV_SKIP_LOCAL | REMP_KV_REUSE_DESCRIPTORS))
        return fail(REMP_E_INVALID, "unknown flags");
    if (old_rank < 0 || old_rank >= plan->own_old.world())
        return fail(REMP_E_RANGE, "old_rank " + std::to_string(old_rank) + " outside [0, " +
                                      std::to_string(plan->own_old.world()) + ")");
    if (remp_status st = check_window(plan, layer_begin, layer_end)) return st;
    if (remp_status st = check_pool(plan, src, plan->own_old.layers_of_rank(old_rank), plan->shape.old_block_size,
                                    "source"))
        return st;
    if (!staging) return fail(REMP_E_INVALID, "staging array is NULL");
    if (remp_status st = check_workspace(plan, workspace, workspace_bytes_)) return st;
    if (src->num_blocks < plan->old_num_blocks)
        return fail(REMP_E_SIZE, "source pool has fewer blocks than the old tables address");
    if (remp_status st = check_dev_tables(plan, old_tables, plan->old_nnz, "old")) return st;

    std::vector<HostSlice> slices;
    if (remp_status st = collect_slices(*plan, true, old_rank, layer_begin, layer_end, *src, staging,
                                        (flags & REMP_KV_SKIP_LOCAL) != 0, slices))
        return st;
    if (src->layout != kLayoutNHD && !hnd_single_heads(src->layout, slices))
        if (remp_status st = check_tile_fits(plan, plan->shape.old_block_size, "pack")) return st;
    // an empty window or cache does nothing; otherwise the tables are expanded (and their stamp
    // written) even when the rank has no slice in the window, so that later calls may reuse them
    if (layer_begin == layer_end || plan->old_live_blocks == 0) return REMP_OK;
    const remp_kv_shape& sh = plan->shape;
    const int64_t row_stride = static_cast<int64_t>(plan->own_old.heads_per_rank()) * sh.head_dim * sh.elem_bytes;
    const WorkspaceLayout L = workspace_layout(*plan);
    char* ws = static_cast<char*>(workspace);
    uint64_t* old_at = reinterpret_cast<uint64_t*>(ws + L.stamp_old);
    int32_t* flag = reinterpret_cast<int32_t*>(ws);
    StampCheck check = no_check(flag);
    if (flags & REMP_KV_REUSE_DESCRIPTORS) {
        check.at[0] = old_at;
        check.want[0] = old_stamp(*plan);
    } else if (remp_status st = launch_expand(*plan, *old_tables, sh.old_block_size, plan->old_nnz,
                                              plan->old_num_blocks, plan->old_live_blocks, ws, flag, L.scan_old,
                                              L.desc_old, true, stream, -1, -1, old_at, old_stamp(*plan))) {
        return st;
    }
    if (hnd_single_heads(src->layout, slices))
        return launch_copy<true>(*plan, slices, plan->old_live_blocks, sh.old_block_size,
                                 row_stride * sh.old_block_size,
                                 static_cast<int32_t>(row_stride / plan->own_old.heads_per_rank()), ws, L.desc_old,
                                 check, stream);
    if (src->layout != kLayoutNHD)
        return launch_tiles<true>(*plan, slices, plan->old_live_blocks, sh.old_block_size,
                                  row_stride * sh.old_block_size, src->layout, ws, L.desc_old, check, stream);
    bool done = false;
    if (remp_status st = launch_rows<true>(*plan, slices, plan->own_old.heads_per_rank(), plan->old_live_blocks,
                                           sh.old_block_size, row_stride * sh.old_block_size,
                                           static_cast<int32_t>(row_stride), ws, L.desc_old, check, stream, &done))
        return st;
    if (done) return REMP_OK;
    return launch_copy<true>(*plan, slices, plan->old_live_blocks, sh.old_block_size, row_stride * sh.old_block_size,
                             static_cast<int32_t>(row_stride), ws, L.desc_old, check, stream);
}

remp_status remp_kv_unpack(const remp_kv_plan_t* plan, int32_t new_rank, int32_t layer_begin, int32_t layer_end,
                           const remp_buffer* staging, const remp_kv_pool* dst, const remp_block_tables* new_tables,
                           const remp_dev_tables* new_dev_tables, void* workspace, int64_t workspace_bytes_,
                           uint32_t flags, hipStream_t stream) {
    clear_error();
    if (!plan) return fail(REMP_E_INVALID, "plan is NULL");
    if (remp_status st = check_unpack_args(plan, new_rank, layer_begin, layer_end, staging, dst, flags)) return st;
    if (remp_status st = check_workspace(plan, workspace, workspace_bytes_)) return st;
    char* ws = static_cast<char*>(workspace);
    return unpack_impl(plan, new_rank, layer_begin, layer_end, staging, dst, new_tables, new_dev_tables, ws,
                       reinterpret_cast<int32_t*>(ws), flags, stream);
}

remp_status remp_kv_unpack_noalloc(const remp_kv_plan_t* plan, int32_t new_rank, int32_t layer_begin,
                                   int32_t layer_end, const remp_buffer* staging, const remp_kv_pool* dst,
                                   const remp_block_tables* new_tables, const remp_dev_tables* new_dev_tables,
                                   int32_t* status, uint32_t flags, hipStream_t stream) {
    clear_error();
    if (!plan) return fail(REMP_E_INVALID, "plan is NULL");
    if (workspace_bytes(*plan) > kScratchBytes)
        return fail(REMP_E_SIZE, "the plan needs " + std::to_string(workspace_bytes(*plan)) +
                                     " bytes of scratch, the static scratch holds " + std::to_string(kScratchBytes));
    if (status && !aligned(status, 4)) return fail(REMP_E_ALIGN, "status is not 4-byte aligned");
    if (remp_status st = check_unpack_args(plan, new_rank, layer_begin, layer_end, staging, dst, flags)) return st;
    char* ws = nullptr;
    if (remp_status st = scratch_of_current_device(stream, &ws)) return st;
    return unpack_impl(plan, new_rank, layer_begin, layer_end, staging, dst, new_tables, new_dev_tables, ws,
                       status ? status : reinterpret_cast<int32_t*>(ws), flags, stream);
}

remp_status remp_kv_copy_local(const remp_kv_plan_t* plan, int32_t rank, int32_t layer_begin, int32_t layer_end,
                               const remp_kv_pool* src, const remp_dev_tables* old_tables, const remp_kv_pool* dst,
                               const remp_block_tables* new_tables, const remp_dev_tables* new_dev_tables,
                               void* workspace, int64_t workspace_bytes_, uint32_t flags, hipStream_t stream) {
    clear_error();
    if (!plan) return fail(REMP_E_INVALID, "plan is NULL");
    if (flags & ~static_cast<uint32_t>(REMP_KV_REUSE_DESCRIPTORS)) return fail(REMP_E_INVALID, "unknown flags");
    if (rank < 0 || rank >= plan->own_old.world() || rank >= plan->own_new.world())
        return fail(REMP_E_RANGE, "rank " + std::to_string(rank) + " is not a rank of both topologies");
    if (remp_status st = check_window(plan, layer_begin, layer_end)) return st;
    if (remp_status st = check_pool(plan, src, plan->own_old.layers_of_rank(rank), plan->shape.old_block_size,
                                    "source"))
        return st;
    if (remp_status st = check_pool(plan, dst, plan->own_new.layers_of_rank(rank), plan->shape.new_block_size,
                                    "destination"))
        return st;
    if (remp_status st = check_workspace(plan, workspace, workspace_bytes_)) return st;
    if (src->num_blocks < plan->old_num_blocks)
        return fail(REMP_E_SIZE, "source pool has fewer blocks than the old tables address");
    if (remp_status st = check_dev_tables(plan, old_tables, plan->old_nnz, "old")) return st;
    int64_t nnz = 0;
    uint64_t new_stamp = 0;
    if (remp_status st = check_new_tables(plan, new_tables, dst, &nnz, &new_stamp)) return st;
    if (remp_status st = check_dev_tables(plan, new_dev_tables, nnz, "new")) return st;

    const remp_kv_shape& sh = plan->shape;
    const int64_t hrow = static_cast<int64_t>(sh.head_dim) * sh.elem_bytes;
    const int64_t old_layer_bytes = plan->own_old.heads_per_rank() * hrow * sh.old_block_size * src->num_blocks;
    const int64_t new_layer_bytes = plan->own_new.heads_per_rank() * hrow * sh.new_block_size * dst->num_blocks;
    const int32_t eb = sh.elem_bytes;
    std::vector<HostLocal> items;
    for (const Item& it : plan->items) {
        if (it.src != rank || it.dst != rank || it.layer < layer_begin || it.layer >= layer_end) continue;
        const int32_t lo = it.layer - plan->own_old.first_layer(rank), ln = it.layer - plan->own_new.first_layer(rank);
        void* sk = src->k[lo];
        void* sv = src->v[lo];
        void* dk = dst->k[ln];
        void* dv = dst->v[ln];
        if (!sk || !sv || !dk || !dv)
            return fail(REMP_E_INVALID, "pool storage of layer " + std::to_string(it.layer) + " is NULL");
        if (!aligned(sk, eb) || !aligned(sv, eb) || !aligned(dk, eb) || !aligned(dv, eb))
            return fail(REMP_E_ALIGN, "pool storage not element aligned");
        const uint64_t s2[2] = {reinterpret_cast<uint64_t>(sk), reinterpret_cast<uint64_t>(sv)};
        const uint64_t d2[2] = {reinterpret_cast<uint64_t>(dk), reinterpret_cast<uint64_t>(dv)};
        for (uint64_t a : s2)
            for (uint64_t b : d2)
                if (ranges_overlap(a, old_layer_bytes, b, new_layer_bytes))
                    return fail(REMP_E_INVALID, "old and new storage of layer " + std::to_string(it.layer) + " overlap");
        // offset of the slice's first head: a row run in NHD, a whole head tile in the tile layouts
        const uint64_t ostep = src->layout == kLayoutNHD ? hrow : hrow * sh.old_block_size;
        const uint64_t nstep = dst->layout == kLayoutNHD ? hrow : hrow * sh.new_block_size;
        HostLocal h;
        h.src_k = s2[0] + static_cast<uint64_t>(it.head_begin - plan->own_old.first_head(rank)) * ostep;
        h.src_v = s2[1] + static_cast<uint64_t>(it.head_begin - plan->own_old.first_head(rank)) * ostep;
        h.dst_k = d2[0] + static_cast<uint64_t>(it.head_begin - plan->own_new.first_head(rank)) * nstep;
        h.dst_v = d2[1] + static_cast<uint64_t>(it.head_begin - plan->own_new.first_head(rank)) * nstep;
        h.row_bytes = static_cast<uint32_t>(it.head_count * hrow);
        items.push_back(h);
    }
    if (src->layout != kLayoutNHD || dst->layout != kLayoutNHD) {
        if (remp_status st = check_tile_fits(plan, sh.new_block_size, "local copy")) return st;
    }
    if (sh.new_block_size > kMaxLocalRows)
        return fail(REMP_E_UNSUPPORTED, "new block size above the local-copy row limit");
    if (layer_begin == layer_end || plan->new_live_blocks == 0) return REMP_OK;   // as in pack
    const WorkspaceLayout L = workspace_layout(*plan);
    char* ws = static_cast<char*>(workspace);
    uint64_t* old_at = reinterpret_cast<uint64_t*>(ws + L.stamp_old);
    uint64_t* new_at = reinterpret_cast<uint64_t*>(ws + L.stamp_new);
    int32_t* flag = reinterpret_cast<int32_t*>(ws);
    StampCheck check = no_check(flag);
    if (flags & REMP_KV_REUSE_DESCRIPTORS) {
        check.at[0] = old_at;
        check.want[0] = old_stamp(*plan);
        check.at[1] = new_at;
        check.want[1] = new_stamp;
    } else {
        if (remp_status st = launch_expand(*plan, *old_tables, sh.old_block_size, plan->old_nnz,
                                           plan->old_num_blocks, plan->old_live_blocks, ws, flag, L.scan_old,
                                           L.desc_old, true, stream, -1, -1, old_at, old_stamp(*plan)))
            return st;
        if (remp_status st = launch_expand(*plan, *new_dev_tables, sh.new_block_size, nnz, new_tables->num_blocks,
                                           plan->new_live_blocks, ws, flag, L.scan_new, L.desc_new, false, stream,
                                           L.bucket_new, L.sorted_new, new_at, new_stamp))
            return st;
    }
    if (src->layout != kLayoutNHD || dst->layout != kLayoutNHD)
        return launch_local_tiles(*plan, items, src->layout, dst->layout, ws, check, stream);
    return launch_local(*plan, items, ws, check, stream);
}

}  // extern "C"
