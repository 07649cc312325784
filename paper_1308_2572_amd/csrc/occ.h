// Occurrence tables shared by the forward and the backward.
//
// Steps one to three of Algorithm 1 (look up each ELT's loss, apply that
// ELT's financial terms, sum over the layer's ELTs in listed order, apply the
// occurrence retention and limit) depend only on the event, not on the trial.
// They are therefore evaluated once per catalogue event and per call, and the
// result O(e) is stored compactly per "super-range" of 65,536 events:
//   br[s][w]   = {bits of word w (events 32w..32w+31 of super-range s),
//                 number of set bits in words 0..w-1}
//   vals[s][i] = O of the i-th set event of super-range s (binary64)
//   cnt[s][i]  = number of the layer's ELTs holding that event (hits mode)
// built in two steps: each chunk of 4096 events finds its set events, their
// bitmap words and count, and O in event order at the start of the chunk's
// slice of `dense`; then every chunk's ranks start after the earlier chunks'
// counts and its values move into `vals`.
// The set events are those with O != 0 ("hot"), or, when hit counts are
// requested, every event present in at least one of the layer's ELTs.
#pragma once

#include "wave.h"
#include "evblk.h"

namespace ara {

constexpr int kMaxJ = ARA_MAX_ELTS_PER_LAYER;
constexpr int kOccChunkWords = 128;                    // 4096 events per chunk
constexpr int kOccChunks = kSrWords / kOccChunkWords;   // 16 chunks per super-range

// What one chunk's events tell about its layer (phase one, for the
// event-ordered forward).
struct OccChunkStat {
    unsigned long long max_bits;   // largest O, as binary64 bits
    int32_t low;                   // smallest power of two that some O is an odd multiple of (INT32_MAX: no O)
    int32_t n_union;               // events held by any of the layer's ELTs
    int32_t count;                 // set events
    int32_t pad;
};

// How the event-ordered forward serves a layer.  Its totals are integers:
// O = (hi * 2^frac + lo) * 2^(gexp - frac) exactly, lo < 2^frac, with hi's sum
// over any trial below 2^64.  In the plain form lo's sum stays below 2^32 by
// itself (frac = 32 - b, where 2^b occurrences are no fewer than the longest
// trial's) and no O may have a bit 94 - 2b places or more below the largest
// O's power of two; for values of 53 bits a ratio of 2^21 with b = 10, 2^9 with
// b = 16.  With kEvCarry lo uses its 32 bits and what wraps goes to hi: 96 - b
// places, 2^33 and 2^27.  Of mode 0 is what neither holds, or an infinity: the
// code stream serves the layer.
constexpr int kEvLayout = 3;   // 1: records in event order over the whole catalogue;
                               // 2: the chunks' own places (the events held exceed half the table's room)
constexpr int kEvCarry = 4;
struct EvLayer {
    int32_t mode, n_set, gexp, frac;
};

// The binary64 value nearest to (hi 2^frac + lo) 2^(gexp - frac).
__device__ __forceinline__ double ev_total(unsigned long long hi, unsigned long long lo, const EvLayer &L) {
    const unsigned __int128 v = (static_cast<unsigned __int128>(hi) << L.frac) + lo;
    const unsigned long long top = static_cast<unsigned long long>(v >> 64), low = static_cast<unsigned long long>(v);
    const int bits = top ? 128 - __clzll(static_cast<long long>(top)) : (low ? 64 - __clzll(static_cast<long long>(low)) : 0);
    if (bits <= 53) return ldexp(static_cast<double>(low), L.gexp - L.frac);
    const int sh = bits - 53;
    unsigned long long q = static_cast<unsigned long long>(v >> sh);
    const unsigned __int128 rest = v - (static_cast<unsigned __int128>(q) << sh);
    const unsigned __int128 half = static_cast<unsigned __int128>(1) << (sh - 1);
    if (rest > half || (rest == half && (q & 1ull))) ++q;   // to nearest, ties to even
    return ldexp(static_cast<double>(q), sh + L.gexp - L.frac);
}

// A set event of an event-ordered layer, in event order (at vals).
struct __attribute__((aligned(16))) EvRec {
    unsigned long long hi;
    uint32_t lo, ev;
};

struct OccTables {
    uint2 *br;          // [n_sr][kSrWords]
    double *vals;       // [n_sr][kSr]
    uint8_t *cnt;       // [n_sr][kSr] or null
    int32_t *count;     // [n_sr]
    int32_t *pcount;    // [n_sr][kOccChunks]  set events per chunk (phase one)
    uint32_t *bits;     // [n_sr][kSrWords]  set-event bitmap (phase one)
    double *dense;      // [n_sr][kSr]       O of each chunk's set events, from the chunk's start (phase one)
    uint8_t *dense_nb;  // [n_sr][kSr]       their ELT counts (hits mode)
    OccChunkStat *stat; // [n_sr][kOccChunks]
    EvLayer *ev_space;  // room for ev
    EvLayer *ev;        // where the layer's form is left, or null: always the tables br, vals, cnt
    const int64_t *max_len;   // with ev: occurrences of the YET's longest trial
};

__device__ __forceinline__ OccTables load_tables(const OccTables *p) {
    OccTables t = *p;
    t.br = device_ptr(t.br);
    t.vals = device_ptr(t.vals);
    t.cnt = device_ptr(t.cnt);
    t.count = device_ptr(t.count);
    t.pcount = device_ptr(t.pcount);
    t.bits = device_ptr(t.bits);
    t.dense = device_ptr(t.dense);
    t.dense_nb = device_ptr(t.dense_nb);
    t.stat = device_ptr(t.stat);
    t.ev = device_ptr(t.ev);
    t.max_len = device_ptr(t.max_len);
    return t;
}

// min(max(v - R, 0), L), evaluated exactly as the oracle does: a separately
// rounded subtraction and two selects (no fused operations; the build uses
// -ffp-contract=off).
__device__ __forceinline__ double xl(double v, double r, double lim) {
    const double y = v - r;
    const double a = (y > 0.0) ? y : 0.0;
    return (a < lim) ? a : lim;
}

struct OccLayoutSizes {
    int n_sr;
    size_t per_layer;
    size_t br, vals, cnt, count, pcount, bits, dense, dense_nb, stat, ev;
};

inline OccLayoutSizes occ_sizes(int32_t catalog, bool with_cnt) {
    OccLayoutSizes z{};
    z.n_sr = (catalog + kSr - 1) / kSr;
    z.br = align256(static_cast<size_t>(z.n_sr) * kSrWords * sizeof(uint2));
    z.vals = align256(static_cast<size_t>(z.n_sr) * kSr * sizeof(double));
    z.cnt = with_cnt ? align256(static_cast<size_t>(z.n_sr) * kSr) : 0;
    z.count = align256(static_cast<size_t>(z.n_sr) * sizeof(int32_t));
    z.pcount = align256(static_cast<size_t>(z.n_sr) * kOccChunks * sizeof(int32_t));
    z.bits = align256(static_cast<size_t>(z.n_sr) * kSrWords * sizeof(uint32_t));
    z.dense = align256(static_cast<size_t>(z.n_sr) * kSr * sizeof(double));
    z.dense_nb = with_cnt ? align256(static_cast<size_t>(z.n_sr) * kSr) : 0;
    z.stat = align256(static_cast<size_t>(z.n_sr) * kOccChunks * sizeof(OccChunkStat));
    z.ev = align256(sizeof(EvLayer));
    z.per_layer = z.stat + z.ev + z.br + z.vals + z.cnt + z.count + z.pcount + z.bits + z.dense + z.dense_nb;
    return z;
}

inline OccTables occ_carve(Carver &c, const OccLayoutSizes &z, bool with_cnt) {
    OccTables t{};
    t.br = c.take<uint2>(static_cast<size_t>(z.n_sr) * kSrWords);
    t.vals = c.take<double>(static_cast<size_t>(z.n_sr) * kSr);
    t.cnt = with_cnt ? c.take<uint8_t>(static_cast<size_t>(z.n_sr) * kSr) : nullptr;
    t.count = c.take<int32_t>(static_cast<size_t>(z.n_sr));
    t.pcount = c.take<int32_t>(static_cast<size_t>(z.n_sr) * kOccChunks);
    t.bits = c.take<uint32_t>(static_cast<size_t>(z.n_sr) * kSrWords);
    t.dense = c.take<double>(static_cast<size_t>(z.n_sr) * kSr);
    t.dense_nb = with_cnt ? c.take<uint8_t>(static_cast<size_t>(z.n_sr) * kSr) : nullptr;
    t.stat = c.take<OccChunkStat>(static_cast<size_t>(z.n_sr) * kOccChunks);
    t.ev_space = c.take<EvLayer>(1);
    return t;
}

// One unit of forward work: one layer over one block of trials, with the
// trial range [t0, t1) whose outputs are written (row bases indexed t - t0).
struct FwdItem {
    const OccTables *tab;      // device pointer to the layer's occurrence tables
    const double *lterm;       // device pointer to the layer's (OccR, OccL, AggR, AggL)
    int32_t block;
    int32_t pad;
    int64_t t0, t1;
    double *ylt;
    double *s_pre;             // or null
    int32_t *hits;             // or null
};

__device__ __forceinline__ FwdItem load_item(const FwdItem *p) {
    FwdItem it = *p;
    it.tab = device_ptr(it.tab);
    it.lterm = device_ptr(it.lterm);
    it.ylt = device_ptr(it.ylt);
    it.s_pre = device_ptr(it.s_pre);
    it.hits = device_ptr(it.hits);
    return it;
}

// Enqueue the forward streaming kernel over a device array of items.
// The regular set of forward items: every layer over the blocks b0 ..
// b0 + nb - 1 of one trial range [t0, t1), rows of ylt / s_pre / hits
// indexed t - t0 (formed on the device, so nothing is copied per call).
struct FwdRegular {
    const OccTables *tabs;     // device, [n_layers]
    const double *lterm;       // device, [n_layers][4]
    double *ylt, *s_pre;
    int32_t *hits;
    int64_t t0, t1;
    int32_t b0, nb;
    int32_t nl;                // layers
    // the event-ordered forward: its blocks, the workgroups each (layer, block)
    // is split over, and the partial totals' room (parts > 1)
    unsigned char *partial;
    int32_t parts, ev_b0, ev_nb;
    // ... or, with sweep > 0 and uneven layers, the workgroups of each block, and
    // room for the table that deals them to the layers ([sweep + nl + 2])
    int32_t sweep;
    uint32_t *share;
};

// Bytes of one workgroup's partial totals: hi, lo and (with hits) the counts
// of every trial of a block.
__host__ __device__ inline size_t ev_slot_bytes(int et, bool hits) {
    return align256(static_cast<size_t>(et) * (hits ? 16 : 12));
}

// The event-ordered forward over the regular set: every layer over blocks
// ev_b0 .. ev_b0 + ev_nb - 1, each (layer, block) split over reg.parts
// workgroups by its set events.
int32_t launch_ev_forward(const EvBlocks &B, const ara_yet *yet, bool hits, const FwdRegular &reg, hipStream_t st);

// The same over a list of items in launch order (slot 8k + x is the k-th on
// XCD x; block -1: empty), each split over `parts` workgroups; partial:
// n_items * parts slots of ev_slot_bytes when parts > 1.
int32_t launch_ev_list(const EvBlocks &B, const ara_yet *yet, const FwdItem *d_items, int n_items, int parts,
                       unsigned char *partial, hipStream_t st);

// Workgroups each (layer, block) is split over: as few rounds of one
// workgroup per CU as possible, and at most `slots` partial totals.
int ev_parts(int64_t n_items, int64_t slots);

// Workgroups of a regular launch: one per block with one layer; with L
// layers, L per block over whole groups of kXcds blocks (the XCD-aware
// mapping of the forward kernel; workgroups past the last block exit).
inline int fwd_regular_items(int n_layers, int nb) {
    if (n_layers <= 1) return nb;
    return n_layers * kXcds * ((nb + kXcds - 1) / kXcds);
}

// LDS plan of a forward workgroup (bytes of the table-slice buffer, values
// it holds); ARA_E_LIMIT when the layout leaves no room for a slice.
int32_t fwd_lds_plan(int tb, int n_ranges, bool hits, bool f32, int32_t *buf_bytes, int32_t *capv);

// f32: binary32 occurrence values (tables built with f32_vals) and totals.
// Items come from d_items, or (d_items null) from `reg`.
// shared: workgroups of the same block are adjacent on one XCD, so the codes
// are loaded through L2 (a regular set decides this from its layer count).
int32_t launch_forward(const ara_yet *yet, int n_sr, bool hits, bool f32, const FwdItem *d_items, int n_items,
                       hipStream_t st, const FwdRegular *reg = nullptr, bool shared = false);

// Checks the arguments of a forward call (those of ara_ylt_forward but the
// workspace); *need receives the workspace bytes the call takes, *least what
// it can do with (without room for partial totals).
int32_t forward_args(const ara_tables *tables, const ara_yet *yet, const ara_layers *layers, const double *elt_terms,
                     const double *layer_terms, int64_t trial_begin, int64_t trial_end, uint32_t flags,
                     const double *ylt, const int32_t *hits, size_t *need, size_t *least);
// Enqueues a checked forward call with at least one layer and one trial on
// `st`, over a workspace of ws_bytes, at least forward_args' *least (its first
// int32 receives the device-side status).
int32_t forward_run(const ara_tables *tables, const ara_yet *yet, const ara_layers *layers, const double *elt_terms,
                    const double *layer_terms, int64_t trial_begin, int64_t trial_end, uint32_t flags, double *ylt,
                    double *s_pre, int32_t *hits, void *ws, size_t ws_bytes, hipStream_t st);

// A layer's set-event bitmap folded onto 2^20 bits by OR (128 KB, staged in
// LDS by the kernels that stream the trial-major YET): one filter per layer.
constexpr int kFilterWords = 1 << 15;
int32_t launch_set_filter(const OccTables *d_tabs, int n_words, uint32_t *filter, int n_layers, hipStream_t st);

// Validates the layer list on the host; returns ARA_OK or an error.
int32_t check_layers(const ara_layers *layers, int32_t n_elts);

// Enqueue the occurrence-table kernel for every layer.  `tabs` has one entry
// per layer; the layer CSR must already be on the device.  f32_vals stores
// each O rounded to binary32 (vals then holds floats at the same indices).
// max_j: at least the ELTs of any of the layers (layers_max_j).  with_ev: some
// table has ev set.
int32_t layers_max_j(const ara_layers *layers);
int32_t launch_occ(const ara_tables *tables, const int32_t *d_elt_off, const int32_t *d_elt_ids,
                   const double *elt_terms, const double *layer_terms, int32_t n_layers, bool union_mode,
                   bool f32_vals, OccTables *d_tabs, int n_sr, int32_t *d_err, int32_t max_j, hipStream_t st, bool with_ev = false);

}  // namespace ara
