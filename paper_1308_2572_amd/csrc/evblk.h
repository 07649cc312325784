// Event-ordered blocks: the prepared YET's second layout.
//
// The trials are cut into blocks of `et` <= 8128 consecutive trials.  A
// block's occurrences are stored by event: event e's occurrences are the
// entries [start, start + n) of the block, one 16-bit word each,
//     bits 0..12   the trial in the block
//     bits 13..15  the event's number in its group of eight (e % 8)
// in no particular order.  Where the lists lie is told by a header, in one
// of two forms chosen by the mean list length:
//   sparse  per group of eight events {the first entry of the group, the
//           eight list lengths in four bits each, 15 = fifteen or more}: 1
//           byte per event; a list behind a length of 15 in its group is
//           found by the numbers in its entries
//   dense   the first entry of every event (4 bytes per event): lists long
//           enough that the lengths would not fit four bits
// A YET prepared with positions holds, in the entries' order, each
// occurrence's position in its trial too.
// A kernel that needs only some events (those with a loss in a layer: a few
// per cent of the catalogue) reads only their lists.
#pragma once

#include "ara_internal.h"

namespace ara {

constexpr int kEvMaxTrials = 8192;     // that an entry can name
constexpr int kEvBlockTrials = 8128;   // of a block: the forward keeps other things in the last places of its LDS
constexpr int kEvTrialBits = 13;
constexpr uint32_t kEvTrialMask = (1u << kEvTrialBits) - 1u;
// Entries readable past the last one (lists are read in 16-byte pieces).
constexpr int kEvPad = 32;

// Words of the `misc` block of a prepared YET.
enum { kMiscErr = 0, kMiscMaxOcc = 1, kMiscLong = 3, kMiscCodes = 4, kMiscMaxLen = 5, kMiscBadOff = 6 };

struct EvBlocks {
    const uint16_t *ent;     // [nnz + kEvPad]
    const uint16_t *pos;     // [nnz + kEvPad] position in the trial of each entry, or null
    const uint2 *hdr;        // sparse form: [neb][ng], the last group of a block holds its end
    const uint32_t *start;   // dense form: [neb][catalog + 1]
    const int64_t *base;     // [neb + 1] first entry of each block
    const int64_t *misc;     // kMiscMaxLen: occurrences of the longest trial
    int64_t n_trials;
    int32_t et, neb, ng, dense, catalog, pad;
};

// The event-ordered blocks of a prepared YET (false: it has none).
bool ev_blocks(const ara_yet *yet, EvBlocks *out);
// The same, for the binary64 forward (false: it takes the code stream).
bool ev_forward_blocks(const ara_yet *yet, EvBlocks *out);
// A mark set by hand on a YET that has blocks: the one-row backward goes through
// them whatever its rule says (tests compare the ways at sizes where it would
// not; both give the same integers).
bool ev_always_backward(const ara_yet *yet);
// The same for secondary uncertainty, of the YET's rule and of the layers'.
bool ev_always_uncertain(const ara_yet *yet);

// Eight entries, from any place on.
struct __attribute__((packed, aligned(2))) EvEight {
    uint32_t a[4];
    __device__ __forceinline__ uint32_t operator[](uint32_t k) const { return (k & 1u) ? a[k >> 1] >> 16 : a[k >> 1] & 0xFFFFu; }
};

// Whether one of the eight lengths of a sparse header is 15.
__device__ __forceinline__ bool ev_long(uint32_t nib) {
    uint32_t t = nib & (nib >> 1);
    t &= t >> 2;
    return (t & 0x11111111u) != 0u;
}

// First of the entries [0, n) of a group whose event number is at least k.
__device__ __forceinline__ uint32_t ev_lower(const uint16_t *ent, uint32_t n, uint32_t k) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((static_cast<uint32_t>(ent[mid]) >> kEvTrialBits) < k) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Start of event number k's list from its group's header, and its length
// (exact unless ev_long(h.y)).
__device__ __forceinline__ void ev_short_list(uint2 h, uint32_t k, uint32_t &s, uint32_t &n) {
    const uint32_t m = h.y & ((1u << (4 * k)) - 1u);
    const uint32_t pairs = (m & 0x0F0F0F0Fu) + ((m >> 4) & 0x0F0F0F0Fu);
    s = h.x + __builtin_amdgcn_sad_u8(pairs, 0u, 0u);
    n = (h.y >> (4 * k)) & 15u;
}

// Event e's list in block b: entries [s, s + n) of the block.
__device__ __forceinline__ void ev_list(const EvBlocks &B, int b, int e, uint32_t &s, uint32_t &n) {
    if (B.dense) {
        const uint32_t *p = B.start + static_cast<size_t>(b) * (B.catalog + 1) + e;
        s = p[0];
        n = p[1] - s;
        return;
    }
    const uint2 *p = B.hdr + static_cast<size_t>(b) * B.ng + (e >> 3);
    const uint2 h = *p;
    const uint32_t k = static_cast<uint32_t>(e & 7);
    if (ev_long(h.y)) {
        const uint16_t *ent = B.ent + B.base[b] + h.x;
        const uint32_t all = p[1].x - h.x;
        const uint32_t a = ev_lower(ent, all, k), z = ev_lower(ent, all, k + 1);
        s = h.x + a;
        n = z - a;
    } else {
        ev_short_list(h, k, s, n);
    }
}

// ---- building (prepare.hip lays the pieces out and calls these) ----

constexpr int kEvChunk = 16384;   // occurrences sorted by tile at once
constexpr int kEvMark = 1024;     // one trial mark per this many occurrences

struct EvGeometry {
    int32_t et, neb, ng, dense;
    int32_t te_bits, n_tiles;     // events per tile (a power of two) and tiles
    int64_t n_chunks, n_marks;
};
EvGeometry ev_geometry(int64_t n_trials, int64_t nnz, int32_t catalog);

struct EvBuild {
    EvGeometry g;
    const int64_t *off;
    const int32_t *ids;
    int64_t n_trials, nnz;
    int32_t catalog;
    // the layout
    uint16_t *ent;
    uint16_t *pos;         // or null
    uint2 *hdr;
    uint32_t *start;
    int64_t *base;
    int64_t *misc;
    int32_t *t_ids;        // the copy of the IDs to write alongside, or null
    // scratch
    uint32_t *rec;         // [nnz]
    uint16_t *rpos;        // [nnz] with pos
    uint16_t *tstart;      // [n_chunks][n_tiles + 1]
    uint32_t *tbase;       // [neb][n_tiles + 1]
    uint32_t *mark;        // [n_marks]
};
// Enqueues the build; offsets and IDs are valid.  A block of 2^32 entries or
// more leaves ARA_E_LIMIT in misc[kMiscErr].
int32_t ev_build(const EvBuild &B, hipStream_t st);

// Occurrences of every event (counts, or null) and the largest of them
// (misc[kMiscMaxOcc]).
int32_t ev_count(const EvBlocks &B, int32_t *counts, hipStream_t st);

// The event-major copy (tr_off, tr_ent) from the blocks; ssum is scratch of
// ev_major_sums() words.  A (slice, catalogue range) of 2^32 occurrences or
// more leaves ARA_E_LIMIT in misc[kMiscErr].
size_t ev_major_sums(int32_t catalog);
int32_t ev_major(const EvBlocks &B, int64_t slice_trials, int64_t *tr_off, uint32_t *tr_ent, int64_t *ssum,
                 int64_t *misc, hipStream_t st);

}  // namespace ara
