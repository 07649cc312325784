// Forward: stream the prepared YET (16-bit codes), gather each occurrence's
// O(e) from the occurrence table held in LDS, accumulate per trial, apply
// the aggregate terms (Algorithm 1, steps three and four).
//
// One workgroup per block of trials; wavefront g owns trial group g of the
// block.  The per-trial totals live in LDS for the whole pass over the
// catalogue, so each trial's total is accumulated by a single wavefront in a
// fixed order: deterministic.  The catalogue is walked one range (2^15
// events) at a time; the range's slice of the occurrence table (bitmap words
// with ranks, then the values) is copied into LDS by LDS DMA
// (global_load_lds_dwordx4).  A workgroup takes 80 KB of LDS and at most 64
// registers per lane, so two workgroups share a CU (8 wavefronts per SIMD):
// while one waits for its next table slice the other streams.
#include "fwd_block.h"

#include <algorithm>
#include <string>

namespace ara {

template <bool HITS, bool F32, bool SHARED, bool FEW>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_fwd(FwdParams P) {
    __shared__ __align__(16) unsigned char smem[kLdsBytes];
    const FwdItem I = fwd_item(P, blockIdx.x);
    if (I.block < 0) return;   // uniform over the workgroup, before any barrier
    fwd_block<HITS, F32, SHARED, FEW>(P, I, smem);
}

// LDS of one forward workgroup: the per-trial totals (and hit counts), the
// range table and segment windows, and what is left for one range's table
// slice: its 8 KB of bitmap words with ranks, then capv values (and capv
// ELT counts with hits; values and counts past capv are read from global
// memory).  Signed arithmetic: with the largest blocks, hit counts and the
// largest catalogue the fixed parts leave no room, which is a limit of this
// layout (ARA_E_LIMIT), not a wrap-around.
int32_t fwd_lds_plan(int tb, int n_ranges, bool hits, bool f32, int32_t *buf_bytes, int32_t *capv_out) {
    const int64_t vb = f32 ? 4 : 8;
    const int64_t fixed = static_cast<int64_t>(fwd_acc_lds(tb, hits, static_cast<size_t>(vb))) +
                          static_cast<int64_t>(fwd_meta_lds(n_ranges));
    const int64_t per_buf = (static_cast<int64_t>(kLdsBytes) - fixed) / 256 * 256;
    const int64_t room = per_buf - kBrBytes - (hits ? 16 : 0);
    int64_t capv = room > 0 ? (hits ? room / (vb + 1) : room / vb) : 0;
    capv = capv / 16 * 16;
    if (capv < 16)
        return fail(ARA_E_LIMIT, "forward: " + std::to_string(tb) + " trials per block and " + std::to_string(n_ranges) +
                                     " catalogue ranges leave no LDS for the table slice" +
                                     (hits ? " with hit counts" : ""));
    *buf_bytes = static_cast<int32_t>(per_buf);
    *capv_out = static_cast<int32_t>(capv);
    return ARA_OK;
}

int32_t fwd_params(const ara_yet *yet, bool hits, bool f32, FwdParams &P) {
    P.code = yet->code;
    P.pad = yet->code + yet->n_codes;
    P.seg_base = yet->seg_base;
    P.seg_run = yet->seg_run;
    P.lane_start = yet->lane_start;
    P.n_trials = yet->n_trials;
    P.tg = yet->trials_per_group;
    P.tb = yet->trials_per_block;
    P.n_ranges = yet->n_ranges;
    // the range's table slice: [bitmap words with ranks][values][counts (hits mode)]
    return fwd_lds_plan(P.tb, P.n_ranges, hits, f32, &P.buf_bytes, &P.capv);
}

// Whether binary32 totals are streamed four codes a lane and chunk instead of
// eight.  A wavefront's run in one range is padded to four codes a lane, so
// that of a run of four or of twelve a chunk of eight is half skip codes; one
// of eight is a chunk of eight.  A whole call over 2M events, 15 ELTs of 20k, us
// of four codes and of eight by the mean run: 4.0 (100,000 x 1000) 200, 233;
// 7.5 (3M x 20) 345, 324; 7.9 (3M x 50) 355, 333; 9.6 (250,000 x 1000) 304,
// 324; 11.9 329, 359; 20 508, 529; 32 767, 778.
static bool fwd_few(const ara_yet *yet) {
    const double lanes = static_cast<double>(yet->n_blocks) * yet->n_ranges * kGroups * 64;
    const double run = static_cast<double>(yet->n_codes) / lanes;
    return run < 7.0 || run > 8.0;
}

int32_t launch_forward(const ara_yet *yet, int n_sr, bool hits, bool f32, const FwdItem *d_items, int n_items,
                       hipStream_t st, const FwdRegular *reg, bool shared) {
    (void)n_sr;
    if (n_items <= 0) return ARA_OK;
    FwdParams P{};
    const int32_t rc = fwd_params(yet, hits, f32, P);
    if (rc) return rc;
    P.items = d_items;
    if (reg) {
        P.reg_tabs = reg->tabs;
        P.reg_lterm = reg->lterm;
        P.reg_ylt = reg->ylt;
        P.reg_s_pre = reg->s_pre;
        P.reg_hits = reg->hits;
        P.reg_t0 = reg->t0;
        P.reg_t1 = reg->t1;
        P.reg_b0 = reg->b0;
        P.reg_nb = reg->nb;
        P.reg_nl = reg->nl;
        shared = reg->nl > 1;
    }
#define ARA_FWD_LAUNCH(H, F, FEW)                                              \
    do {                                                                     \
        if (shared) k_fwd<H, F, true, FEW><<<n_items, 1024, 0, st>>>(P);     \
        else k_fwd<H, F, false, FEW><<<n_items, 1024, 0, st>>>(P);           \
    } while (0)
    if (f32) {
        if (hits) ARA_FWD_LAUNCH(true, true, false);
        else if (fwd_few(yet)) ARA_FWD_LAUNCH(false, true, true);
        else ARA_FWD_LAUNCH(false, true, false);
    } else {
        if (hits) ARA_FWD_LAUNCH(true, false, false);
        else ARA_FWD_LAUNCH(false, false, false);
    }
#undef ARA_FWD_LAUNCH
    ARA_HIP(hipGetLastError());
    return ARA_OK;
}

// The workgroups of a block that may walk it together (k_ev_share), or 0.
// Four layers or more: two share too little for the parts' totals they write
// (400,000 x 1000, 10 and 15 ELTs: 253 us, dealt 299; three layers 347 and
// 353).  Blocks of 6M occurrences, 12 MB of lists beside 16 parts' 1.5 MB of
// totals (1M x 250, four layers: 402 and 486).  And at least eight blocks per
// XCD, since a block stays on one (150,000 x 1000, 19 blocks: 202 and 237;
// 1M x 1000, some 120 blocks: 1161 and 783).
constexpr int kSweep = 16;
constexpr int kSweepLeast = 4, kSweepMost = 16;   // layers
constexpr int64_t kSweepEntries = 6'000'000;
constexpr int kShareWords = kSweep + kSweepMost + 2;

static int ev_sweep(int n_layers, const EvBlocks &B, const ara_yet *yet, int64_t blocks) {
    const bool yes = n_layers >= kSweepLeast && n_layers <= kSweepMost && blocks >= 8 * kXcds &&
                     yet->nnz / std::max(B.neb, 1) >= kSweepEntries;
    return yes ? kSweep : 0;
}

static size_t fwd_workspace(const ara_tables *tables, const ara_layers *layers, bool hits) {
    const OccLayoutSizes z = occ_sizes(tables->catalog, hits);
    const int L = layers->n_layers;
    const int nJ = L > 0 ? layers->elt_off[L] : 0;
    size_t b = kWsHeaderBytes;
    b += align256(static_cast<size_t>(L + 1) * sizeof(int32_t));
    b += align256(static_cast<size_t>(std::max(nJ, 1)) * sizeof(int32_t));
    b += align256(static_cast<size_t>(std::max(L, 1)) * sizeof(OccTables));
    b += align256(kShareWords * sizeof(uint32_t));
    b += static_cast<size_t>(L) * z.per_layer;
    return b;
}

// Partial totals a forward workspace has room for: those of two rounds of
// one workgroup per CU, and of every block's where its workgroups walk it
// together.
static size_t partial_bytes(const ara_yet *yet, int n_layers, bool hits, bool f32) {
    EvBlocks B{};
    if (f32 || !ev_forward_blocks(yet, &B)) return 0;
    const size_t slots = std::max(static_cast<size_t>(2 * device_cu_count()),
                                  static_cast<size_t>(ev_sweep(n_layers, B, yet, B.neb)) * static_cast<size_t>(B.neb));
    return slots * ev_slot_bytes(B.et, hits);
}

static int32_t check_pair(const ara_tables *tables, const ara_yet *yet) {
    if (!tables || !yet) return fail(ARA_E_INVAL, "null tables or yet");
    if (tables->catalog != yet->catalog) return fail(ARA_E_INVAL, "tables and YET use different catalogues");
    if (yet->range_bits != kRangeBits || yet->groups != kGroups) return fail(ARA_E_INVAL, "YET not prepared by this library");
    return ARA_OK;
}

}  // namespace ara

using namespace ara;

extern "C" int32_t ara_ylt_workspace_bytes(const ara_tables *tables, const ara_yet *yet, const ara_layers *layers,
                                           uint32_t flags, size_t *bytes) {
    if (!bytes) return fail(ARA_E_INVAL, "null output");
    int32_t rc = check_pair(tables, yet);
    if (rc) return rc;
    if ((rc = check_layers(layers, tables->n_elts))) return rc;
    if (flags & ~(ARA_F_EMIT_HITS | ARA_F_FP32_ACCUM)) return fail(ARA_E_INVAL, "unknown flag");
    int32_t bb = 0, cv = 0;
    if ((rc = fwd_lds_plan(yet->trials_per_block, yet->n_ranges, (flags & ARA_F_EMIT_HITS) != 0,
                           (flags & ARA_F_FP32_ACCUM) != 0, &bb, &cv)))
        return rc;
    *bytes = fwd_workspace(tables, layers, (flags & ARA_F_EMIT_HITS) != 0) +
             partial_bytes(yet, layers->n_layers, (flags & ARA_F_EMIT_HITS) != 0, (flags & ARA_F_FP32_ACCUM) != 0);
    return ARA_OK;
}

namespace ara {

// Checks the arguments of a forward call; on success *need holds the
// workspace bytes it takes and *least those it can do with.
int32_t forward_args(const ara_tables *tables, const ara_yet *yet, const ara_layers *layers, const double *elt_terms,
                     const double *layer_terms, int64_t trial_begin, int64_t trial_end, uint32_t flags,
                     const double *ylt, const int32_t *hits, size_t *need, size_t *least) {
    int32_t rc = check_pair(tables, yet);
    if (rc) return rc;
    if ((rc = check_layers(layers, tables->n_elts))) return rc;
    if (flags & ~(ARA_F_EMIT_HITS | ARA_F_FP32_ACCUM)) return fail(ARA_E_INVAL, "unknown flag");
    const bool want_hits = (flags & ARA_F_EMIT_HITS) != 0;
    if (hits && !want_hits) return fail(ARA_E_INVAL, "hits output requires ARA_F_EMIT_HITS");
    if (trial_begin < 0 || trial_end < trial_begin || trial_end > yet->n_trials)
        return fail(ARA_E_RANGE, "trial range outside the YET");
    if (layers->n_layers > 0 && trial_end > trial_begin && (!ylt || !elt_terms || !layer_terms))
        return fail(ARA_E_INVAL, "null output or terms");
    int32_t bb = 0, cv = 0;
    if ((rc = fwd_lds_plan(yet->trials_per_block, yet->n_ranges, want_hits, (flags & ARA_F_FP32_ACCUM) != 0, &bb, &cv)))
        return rc;
    *least = fwd_workspace(tables, layers, want_hits);
    *need = *least + partial_bytes(yet, layers->n_layers, want_hits, (flags & ARA_F_FP32_ACCUM) != 0);
    return ARA_OK;
}

// The forward proper, once the arguments are checked, over a workspace of
// at least the bytes forward_args gave.
int32_t forward_run(const ara_tables *tables, const ara_yet *yet, const ara_layers *layers, const double *elt_terms,
                    const double *layer_terms, int64_t trial_begin, int64_t trial_end, uint32_t flags, double *ylt,
                    double *s_pre, int32_t *hits, void *ws, size_t ws_bytes, hipStream_t st) {
    int32_t rc = ARA_OK;
    const bool want_hits = (flags & ARA_F_EMIT_HITS) != 0;
    const bool f32 = (flags & ARA_F_FP32_ACCUM) != 0;
    const int L = layers->n_layers;
    const OccLayoutSizes z = occ_sizes(tables->catalog, want_hits);
    const int nJ = layers->elt_off[L];
    Carver c(ws);
    int32_t *d_err = c.take<int32_t>(kWsHeaderBytes / sizeof(int32_t));
    int32_t *d_off = c.take<int32_t>(static_cast<size_t>(L + 1));
    int32_t *d_ids = c.take<int32_t>(static_cast<size_t>(std::max(nJ, 1)));
    OccTables *d_tabs = c.take<OccTables>(static_cast<size_t>(L));
    uint32_t *d_share = c.take<uint32_t>(kShareWords);
    const int64_t b_lo = trial_begin / yet->trials_per_block;
    const int64_t b_hi = (trial_end + yet->trials_per_block - 1) / yet->trials_per_block;
    const int nb = static_cast<int>(b_hi - b_lo);
    const int64_t n = trial_end - trial_begin;
    std::vector<OccTables> tabs(static_cast<size_t>(L));
    for (int j = 0; j < L; ++j) tabs[j] = occ_carve(c, z, want_hits);
    EvBlocks B{};
    // binary32 totals stay with the code stream although it is slower (100,000
    // trials of 1000: 212 us where exact sums of the rounded O took 109): they
    // round at every addition in the trial's order, and those are the results
    const bool ev = !f32 && ev_forward_blocks(yet, &B);
    if (ev)
        for (OccTables &t : tabs) {
            t.ev = t.ev_space;
            t.max_len = B.misc + kMiscMaxLen;
        }
    FwdRegular reg{};
    reg.tabs = d_tabs;
    reg.lterm = layer_terms;
    reg.ylt = ylt;
    reg.s_pre = s_pre;
    reg.hits = hits;
    reg.t0 = trial_begin;
    reg.t1 = trial_end;
    reg.b0 = static_cast<int32_t>(b_lo);
    reg.nb = nb;
    reg.nl = L;
    HeadImage img(ws);
    img.cover(d_err + kWsHeaderBytes / sizeof(int32_t));
    img.put(d_off, layers->elt_off, static_cast<size_t>(L + 1));
    img.put(d_ids, layers->elt_ids, static_cast<size_t>(nJ));
    img.put(d_tabs, tabs.data(), tabs.size());
    if ((rc = img.send(st))) return rc;

    {
        ProfScope prof(ARA_PROF_OCC, st);
        if ((rc = launch_occ(tables, d_off, d_ids, elt_terms, layer_terms, L, want_hits, f32, d_tabs, z.n_sr, d_err,
                             layers_max_j(layers), st, ev)))
            return rc;
    }
    ProfScope prof(ARA_PROF_FWD, st);
    if (ev) {
        reg.ev_b0 = static_cast<int32_t>(trial_begin / B.et);
        reg.ev_nb = static_cast<int32_t>((trial_end + B.et - 1) / B.et) - reg.ev_b0;
        const size_t slot = ev_slot_bytes(B.et, want_hits);
        const size_t used = c.bytes();
        const int64_t slots = ws_bytes > used ? static_cast<int64_t>((ws_bytes - used) / slot) : 0;
        reg.parts = ev_parts(static_cast<int64_t>(L) * reg.ev_nb, slots);
        reg.sweep = ev_sweep(L, B, yet, reg.ev_nb);
        if (static_cast<int64_t>(reg.sweep) * reg.ev_nb > slots) reg.sweep = 0;
        reg.share = d_share;
        reg.partial = reinterpret_cast<unsigned char *>(ws) + used;
        return launch_ev_forward(B, yet, want_hits, reg, st);
    }
    return launch_forward(yet, z.n_sr, want_hits, f32, nullptr, fwd_regular_items(L, nb), st, &reg);
}

}  // namespace ara

extern "C" int32_t ara_ylt_forward(const ara_tables *tables, const ara_yet *yet, const ara_layers *layers,
                                   const double *elt_terms, const double *layer_terms, int64_t trial_begin,
                                   int64_t trial_end, uint32_t flags, double *ylt, double *s_pre, int32_t *hits,
                                   void *ws, size_t ws_bytes, void *stream) {
    size_t need = 0, least = 0;
    int32_t rc = forward_args(tables, yet, layers, elt_terms, layer_terms, trial_begin, trial_end, flags, ylt, hits,
                              &need, &least);
    if (rc) return rc;
    if (!ws) return fail(ARA_E_INVAL, "null workspace");
    if (ws_bytes < need) return fail(ARA_E_NOSPACE, "forward workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (layers->n_layers == 0 || trial_end == trial_begin) {
        ARA_HIP(hipMemsetAsync(ws, 0, kWsHeaderBytes, st));
        return ARA_OK;
    }
    return forward_run(tables, yet, layers, elt_terms, layer_terms, trial_begin, trial_end, flags, ylt, s_pre, hits,
                       ws, ws_bytes, st);
}
