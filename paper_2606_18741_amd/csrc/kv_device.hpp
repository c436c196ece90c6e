// Device data structures and launch constants of the KV-migration kernels.
// Included by migrate.hip only (one translation unit holds every kernel).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_util.hpp"
#include "plan.hpp"

namespace remp {

// ---------------------------------------------------------------------------
// device data structures
// ---------------------------------------------------------------------------

// One live block of one sequence: physical block id, position of its first
// token on the sequence-major token axis, number of live tokens in it, and
// the sequence it belongs to.
struct BlockDesc {
    int32_t block;
    int32_t tok;
    int32_t n;
    int32_t seq;
};

// Values of the workspace status flag (int32 at byte 0 of the workspace).
constexpr int32_t kFlagTables = 1;   // the device tables would have indexed out of range
constexpr int32_t kFlagStale = 2;    // a reusing call found descriptors of other tables

// Check of reused descriptors.  A call that expands its own descriptors passes
// at[] = NULL; a call that reuses them names the stamps they must carry (one
// per side it reads: old and new).  On a mismatch every workgroup leaves
// before it writes anything outside LDS, and the first one sets the flag.
// Kernels whose prologue only reads the descriptor array itself test the
// result after that prologue (the stamp load then overlaps the descriptor
// loads); kernels that follow a descriptor to other arrays test it first.
struct StampCheck {
    const uint64_t* at[2];
    uint64_t want[2];
    int32_t* flag;
};

__device__ __forceinline__ bool stamps_differ(const StampCheck& c) {
    bool differ = false;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (c.at[i] && *c.at[i] != c.want[i]) differ = true;
    return differ;
}

__device__ __forceinline__ void report_stale(const StampCheck& c) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *c.flag = kFlagStale;
}

__device__ __forceinline__ bool stale_descriptors(const StampCheck& c) {
    if (!stamps_differ(c)) return false;
    report_stale(c);
    return true;
}

// Vectors of 16 bytes: what a lane of the copy kernels moves.  Loads are non-temporal and so are stores
// (the data is touched once).
constexpr uint32_t kVecBytes = 16;
typedef unsigned int Vec16 __attribute__((ext_vector_type(4)));
typedef Vec16 Vec16Any __attribute__((aligned(1)));   // the same at any address

// Global-memory view of an address: loads and stores through it are global instructions (a generic pointer
// compiles to flat ones, which also wait for LDS).
#define REMP_GLOBAL __attribute__((address_space(1)))
#define REMP_CONSTANT __attribute__((address_space(4)))

// Slices per copy launch.  Launches of a few slices beat one launch of all of them (A/B on MI355X, 70B
// GQA share: 96 per launch 5.71, 40: 5.73, 10: 5.79-5.83, 5: 5.80, 2: 5.76, 1: 5.66 TB/s), and the kernel
// arguments stay small.
constexpr int kMaxItems = 8;
// Calls of small slices take more to a launch, up to kLaunchBytes of payload: a launch takes 2.5 us beside its copy
// (MI355X, 70B GQA, 2304 tokens, pack and unpack of 80 slices each: 10 launches of 8 131 us, two of 40 86 us).
constexpr int kMaxSmallItems = 64;
constexpr uint64_t kLaunchBytes = uint64_t(64) << 20;
constexpr int kMaxUnitsPerWg = 128;   // head tiles per workgroup
// Threads of a pack / unpack workgroup: one wave that moves 1 KiB, one vector per lane.  Measured on MI355X
// (7 GiB, 4 KiB units gathered at random): one wave with one vector 6.29 TB/s, with two 5.99, with four 5.70;
// four waves with one vector each 6.24, sixteen 6.10.  Whole rows split among three or more destinations
// are packed by four waves, so that one compute unit reads a row's 4 KiB and writes all its pieces
// (four shares of 128 B to 2 KiB: 6.67-7.16 TB/s, against 6.33-6.53 with one wave).
constexpr int kRunThreads = 64;
constexpr int kRowsPackThreads = 256;
constexpr int kMaxRunThreads = 1024;   // the most the tuning override asks for
constexpr int kScanThreads = 1024;
// Rows that are not whole vectors go by 8-byte words up to these bytes, where they are aligned to that.
constexpr uint32_t kPackWordRow = 512, kUnpackWordRow = 256, kLocalWordRow = 512;
// Such words of a lane: 2 (1 KiB to a wave), and 4 in the local copy where a block has as many, so that its look-ups serve
// more bytes (MI355X, us, 2 / 4 words: 200-byte rows in blocks of 64 718 / 666, blocks of 64 to 20 706 / 672; but of 72
// bytes, blocks of 32 to 16, 897 / 1100).
constexpr int kLocalWords = 4;

struct CopyItem {
    uint64_t paged_k;     // K storage of the layer, offset to the slice's first head
    uint64_t paged_v;
    uint64_t stage;       // first byte of the slice in its staging buffer (K part)
    uint32_t row_bytes;   // head_count * head_dim * elem_bytes
    uint32_t vpr_magic;   // fast division by words per row
    uint32_t vpu;         // words (kRows: rows) per (block, K or V) unit
    uint32_t vpu_magic;   // fast division by vpu
    uint16_t vpr_shift;
    uint16_t vpu_shift;
    uint32_t rows;        // rows per wave (kRows)
};

// The unit (live block, K or V) that a lane works on.  The words of a slice's units (16-byte vectors, or words of 8 or 4
// bytes) are numbered unit after unit, `vpu` to a unit, and a wave takes 1 KiB of consecutive ones from w0 (the same
// for all its lanes), so it meets the few units unit(w0), unit(w0) + 1, ...: their descriptors come by scalar
// loads, and each lane keeps the one its word falls into.  N bounds the units a wave can meet
// (units_per_wave); N == 0 means any number, each lane loading its own descriptor.  Per-lane loads
// cost 15% of the copy (MI355X, 4 KiB units: 5.30 against 6.29 TB/s), so they are left to units of less than
// 128 bytes.
typedef int Int4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void choose(bool yes, const Int4& v, Int4* own) { *own = yes ? v : *own; }

// N values in registers.  Not an array: a lane's choice among an array's elements is compiled to an indexed access, for
// which the array goes to LDS or scratch.
template <typename T, int N>
struct Values {
    T v;
    Values<T, N - 1> next;

    template <typename F>
    __device__ __forceinline__ void fill(const F& f, uint32_t k = 0) {
        v = f(k);
        next.fill(f, k + 1);
    }
    // Moves *own on by one value for every `size` that fits into *x.
    __device__ __forceinline__ void advance(uint32_t size, uint32_t* x, uint32_t* passed, T* own) const {
        const bool past = *x >= size;
        const T mine = v;
        *x -= past ? size : 0;
        *passed += past;
        choose(past, mine, own);
        next.advance(size, x, passed, own);
    }
};

template <typename T>
struct Values<T, 0> {
    template <typename F>
    __device__ __forceinline__ void fill(const F&, uint32_t = 0) {}
    __device__ __forceinline__ void advance(uint32_t, uint32_t*, uint32_t*, T*) const {}
};

template <int N>
struct WaveUnits {
    Values<Int4, N> v;
    uint32_t w0, u0, r0;   // the wave's first word, its unit and its position there

    // False when the wave lies past the last unit.
    __device__ __forceinline__ bool load(const BlockDesc* desc, uint32_t n_desc, uint32_t first, uint32_t vpu,
                                         uint32_t magic, uint32_t shift) {
        w0 = first;
        if constexpr (N > 0) {
            u0 = fast_div(w0, magic, shift);
            if (u0 >= n_desc) return false;
            r0 = w0 - u0 * vpu;
            const REMP_CONSTANT Int4* table = (const REMP_CONSTANT Int4*)(reinterpret_cast<uint64_t>(desc));
            v.fill([&](uint32_t k) { return table[min(u0 + k, n_desc - 1)]; });
        }
        return true;
    }

    // Descriptor of the wave's i-th word and its position r in its unit; false past the last unit.
    __device__ __forceinline__ bool pick(const BlockDesc* desc, uint32_t n_desc, uint32_t i, uint32_t vpu,
                                         uint32_t magic, uint32_t shift, BlockDesc* d, uint32_t* r) const {
        if constexpr (N == 0) {
            const uint32_t u = fast_div(w0 + i, magic, shift);
            if (u >= n_desc) return false;
            *r = w0 + i - u * vpu;
            *d = desc[u];
            return true;
        } else {
            uint32_t u = u0;
            *r = r0 + i;
            Int4 own = v.v;
            v.next.advance(vpu, r, &u, &own);
            *d = BlockDesc{own.x, own.y, own.z, own.w};
            return u < n_desc;
        }
    }
};

template <int N>
__device__ __forceinline__ bool pick_unit(const BlockDesc* desc, uint32_t n_desc, uint32_t w0, uint32_t lane,
                                          uint32_t vpu, uint32_t magic, uint32_t shift, BlockDesc* d, uint32_t* r) {
    WaveUnits<N> units;
    return units.load(desc, n_desc, w0, vpu, magic, shift) &&
           units.pick(desc, n_desc, lane, vpu, magic, shift, d, r);
}

// Pieces of `size` words, one after another, that the `wave` consecutive words of a wave can touch; waves begin at multiples of
// `wave`, pieces at multiples of `size`.
inline uint32_t pieces_per_wave(uint32_t size, uint32_t wave) {
    return size % wave == 0 ? 1 : wave % size == 0 ? wave / size : (wave - 2) / size + 2;
}

// The same for units of vpu words, as the template argument of pick_unit: 1, 2, 4 or 8, and 0 beyond 8.
inline int units_per_wave(uint32_t vpu, uint32_t wave = 64) {
    const uint32_t most = pieces_per_wave(vpu, wave);
    return most <= 1 ? 1 : most <= 2 ? 2 : most <= 4 ? 4 : most <= 8 ? 8 : 0;
}

// The dispatcher deals consecutive workgroups to the 8 XCDs in turn.  The tile copies and those of rows that
// are not whole vectors are numbered so that an XCD gets kXcdRun consecutive positions: neighbours share lines
// where a head row, a strip or a run is not a multiple of 128 bytes, and those then meet in one L2.  The grid is a multiple of 8 * kXcdRun.  Measured on
// MI355X, runs of 1 / 4 / 16 / 64 (us, pack and unpack): HND heads of 160 bytes 2069 / 1847 / 1646 / 1596, 7B MHA
// HND 2428 / 2461 / 2392 / 2418, ROCm fp8 in 64-token blocks 2569 / 2564 / 2406 / 2446.
constexpr uint32_t kXcdRun = 16;

__device__ __forceinline__ uint32_t xcd_position(uint32_t wg) {
    const uint32_t l = wg % (8 * kXcdRun);
    return wg - l + (l & 7u) * kXcdRun + (l >> 3);
}

// First vector of the wave, in a grid whose x dimension numbers the vectors.
__device__ __forceinline__ uint32_t wave_first(uint32_t xcd) {
    const uint32_t wg = xcd ? xcd_position(blockIdx.x) : blockIdx.x;
    return static_cast<uint32_t>(
        __builtin_amdgcn_readfirstlane(static_cast<int>((wg * blockDim.x + threadIdx.x) & ~63u)));
}

// What one lane moves at a time, held in registers: a word of V (16, 8 or 4) bytes at an aligned address, or (V == 0) at
// most 16 bytes at any address (hardware takes unaligned global vectors): fewer, in parts of 8, 4, 2 and 1, where a
// run ends.  `left`: bytes of the run from here on.  Callers load all they move before they store any of it: a
// part that was stored before the next was loaded cost a wave a second trip to memory.
template <int V>
struct Moved {
    typedef typename VecT<V>::type Word;
    Word w;

    __device__ __forceinline__ void load(uint64_t src, uint32_t) {
        w = __builtin_nontemporal_load((const REMP_GLOBAL Word*)src);
    }
    __device__ __forceinline__ void store(uint64_t dst, uint32_t) const {
        __builtin_nontemporal_store(w, (REMP_GLOBAL Word*)dst);
    }
};

template <>
struct Moved<0> {
    typedef uint64_t Part8 __attribute__((aligned(1)));
    typedef uint32_t Part4 __attribute__((aligned(1)));
    typedef uint16_t Part2 __attribute__((aligned(1)));
    Vec16Any w;
    uint64_t p8;
    uint32_t p4;
    uint16_t p2;
    uint8_t p1;

    __device__ __forceinline__ void load(uint64_t src, uint32_t left) {
        if (left >= kVecBytes) {
            w = __builtin_nontemporal_load((const REMP_GLOBAL Vec16Any*)src);
            return;
        }
        const uint32_t at4 = left & 8u, at2 = at4 + (left & 4u), at1 = at2 + (left & 2u);
        if (left & 8u) p8 = *(const REMP_GLOBAL Part8*)src;
        if (left & 4u) p4 = *(const REMP_GLOBAL Part4*)(src + at4);
        if (left & 2u) p2 = *(const REMP_GLOBAL Part2*)(src + at2);
        if (left & 1u) p1 = *(const REMP_GLOBAL uint8_t*)(src + at1);
    }
    __device__ __forceinline__ void store(uint64_t dst, uint32_t left) const {
        if (left >= kVecBytes) {
            __builtin_nontemporal_store(w, (REMP_GLOBAL Vec16Any*)dst);
            return;
        }
        const uint32_t at4 = left & 8u, at2 = at4 + (left & 4u), at1 = at2 + (left & 2u);
        if (left & 8u) *(REMP_GLOBAL Part8*)dst = p8;
        if (left & 4u) *(REMP_GLOBAL Part4*)(dst + at4) = p4;
        if (left & 2u) *(REMP_GLOBAL Part2*)(dst + at2) = p2;
        if (left & 1u) *(REMP_GLOBAL uint8_t*)(dst + at1) = p1;
    }
};

// Bytes [off, off + 16) of a run of `len` bytes, or what the run still has of them.
template <bool ODD>
__device__ __forceinline__ void move_vector(uint64_t src, uint64_t dst, uint32_t off, uint32_t len) {
    Moved<ODD ? 0 : 16> m;
    m.load(src + off, len - off);
    m.store(dst + off, len - off);
}

template <int ITEMS>
struct CopyArgs {
    const BlockDesc* desc;
    int64_t block_stride;     // bytes per block on the paged side
    int64_t total_tokens;     // T: a slice's V part starts T * row_bytes after its K part
    uint32_t n_desc;
    uint32_t row_stride;      // bytes per token row on the paged side (all local heads)
    uint32_t xcd;             // number the workgroups by xcd_position (shares_lines)
    StampCheck check;
    CopyItem items[ITEMS];
};
static_assert(sizeof(CopyArgs<kMaxSmallItems>) < 4096, "copy kernel arguments must stay below 4 KiB");

}  // namespace remp
