// The event-ordered forward: a layer's set events (O != 0), each with the
// list of the trials of a block that it occurs in, scatter their O into the
// trials' totals in LDS.
//
// What bounds it is memory: it reads the lists of the layer's events and the
// headers that tell where they are, 1.8 GB of the 2.25 GB that a 1M x 1000
// YET's blocks take with 7.6% of the catalogue set (152,000 of 2,000,000
// events; lists of four 16-bit entries, so most 128-byte lines hold some set
// event's list), in 304 us (124 blocks of 8065 trials in two parts).  The code
// stream reads 2.1 GB and spends some 27 instructions on every occurrence: 560
// us.  One workgroup per (layer, block, part): a block's totals take 96 KB of
// LDS, so a workgroup has a CU for itself; its 16 wavefronts take 64 set
// events at a time, one per lane, with the next 64 events' headers and the
// ones' after lists in flight.  Larger blocks make longer lists and fewer
// bytes: a prototype took 302 us with 7872 trials, 390 with 3936 and 510 with
// 1968.  Layers of one block run together on one XCD and share its lists in
// L2: four uneven layers 722 us and 47 of adding the parts up (the code stream
// grouped by four 1750 us).
//
// The totals are integers (EvLayer): O in fixed point, two words, exact, so
// the sum does not depend on the order in which wavefronts add, on the parts
// or on the trial range, and the one rounding to binary64 comes at the end.
#include "fwd_block.h"

#include <algorithm>

namespace ara {

constexpr int kEvfThreads = 1024;
constexpr int kEvfWaves = kEvfThreads / kWave;
constexpr int kRunUnits = 4;
// Lists of more than kLong entries, or kLonger, or kLongest, are added by a whole
// wavefront instead of their lanes (long_lists).
constexpr uint32_t kLong = 48, kLonger = 128, kLongest = 1024;
constexpr uint32_t kTaskList = 2048;  // beyond this many, by the workgroup's wavefronts together
constexpr int kTasks = 60;            // pieces of those that wait for them
static_assert(kEvMaxTrials - kEvBlockTrials >= kTasks + 1, "the last trials' places hold the pieces");
static_assert(kEvfWaves % kRunUnits == 0, "runs to wavefronts");

struct EvfParams {
    EvBlocks B;
    const FwdItem *items;      // one (layer, block) per `parts` workgroups, or null: the regular set below
    int32_t n_items;
    const OccTables *tabs;
    const double *lterm;
    double *ylt, *s_pre;
    int32_t *hits;
    int64_t t0, t1;
    int32_t b0, nb, nl, parts;
    unsigned char *partial;
    const uint32_t *share;     // k_ev_share's table, when sweep > 0
    int32_t sweep;             // workgroups of a block that may walk it together, or 0
    int32_t spread;            // the parts take runs of units in turn
    FwdParams fwd;             // for the layers of mode 0 (k_ev_rest)
};

// Sixteen bytes of a list, from an even entry on.  (A vector: of a struct the
// compiler copies the words one by one behind each conditional load, and so
// waits for it there.)
typedef uint32_t EvPiece __attribute__((ext_vector_type(4), aligned(4)));

// Waits for this wavefront's loads: behind a loop that loads one step too far,
// so that the compiler does not wait for those, and with them for all others,
// where it next uses their registers, on the path that had no such loop too.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// The lanes whose lists of c entries the wavefront adds together.  The lanes by
// themselves take as many steps of 16 entries as the longest list needs, the
// wavefront the time of some four for each list: so the few above a length, if
// one of them is longer by 64 entries for each of them, and any of many entries.
__device__ __forceinline__ uint64_t long_lists(uint32_t c) {
    uint64_t m = __ballot(c > kLong);
    if (!m) return m;
    uint32_t n = static_cast<uint32_t>(__popcll(m));
    if (n <= 12u && __any(c > kLong + 64u * n)) return m;
    m = __ballot(c > kLonger);
    n = static_cast<uint32_t>(__popcll(m));
    if (n <= 24u && __any(c > kLonger + 64u * n)) return m;
    return __ballot(c > kLongest);
}

// Several layers of a block read most of its lines each (a line of 128 bytes
// holds the lists of some 16 events, and a layer with a tenth of the catalogue
// set touches four lines in five), from HBM unless one of them has just brought
// them to the XCD's L2.  Layers of one size walk a block side by side by
// themselves; of uneven ones the smaller run ahead and every layer reads for
// itself: 6.4 GB at 5.5 TB/s, 1161 us, for four layers of 8 to 20 ELTs over a
// 1M x 1000 YET's 2.3 GB.  So a block's `sweep` workgroups are dealt to its
// layers in proportion to their set events, and each walks every parts-th unit
// of its layer's, from the block's first event to its last: all of them go
// through the block at one speed.  726 us and 52 for adding 16 parts a block
// up (8 workgroups 827 + 31, 32 workgroups 785 + 89; 12, 20 and 24 do not
// divide an XCD's 32 CUs: 819 to 888).
//
// It pays where the layers are uneven and read much: this kernel says so
// (`uneven`) where the largest layer has half as many set events again as the
// smallest and they hold a fifth of the catalogue or more together (eight
// equal layers 598 us, so dealt 645; four layers of 3 to 6 ELTs 230 and 263),
// and the host asks it only for what kSweepLeast and its like describe.
//
// share[r]: workgroup r's layer, its part and the layer's parts (8, 8 and 16
// bits); share[sweep + j]: layer j's first workgroup; share[sweep + nl + 1]:
// uneven.
__global__ __launch_bounds__(kWave) void k_ev_share(const OccTables *__restrict__ tabs, int nl, int sweep,
                                                    int32_t catalog, uint32_t *__restrict__ share) {
    const int l = threadIdx.x;
    const bool in = l < nl;
    float w = 0.0f;
    bool ok = true;
    if (in) {
        const EvLayer L = *device_ptr(tabs[l].ev);
        w = static_cast<float>(max(L.n_set, 1));
        ok = (L.mode & kEvLayout) == 1;
    }
    float sum = w, most = in ? w : 0.0f, least = in ? w : 3e38f;
    for (int o = 32; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o);
        most = fmaxf(most, __shfl_xor(most, o));
        least = fminf(least, __shfl_xor(least, o));
    }
    const bool uneven = __all(ok) && most >= 1.5f * least && 5.0f * sum >= static_cast<float>(catalog);
    // one workgroup each and the proportional share of the others rounded
    // down; those left over (fewer than the layers) to the layers with the
    // most events per workgroup
    int p = in ? 1 + static_cast<int>(static_cast<float>(sweep - nl) * (w / sum)) : 0;
    int left = p;
    for (int o = 32; o > 0; o >>= 1) left += __shfl_xor(left, o);
    for (left = sweep - left; left > 0; --left) {
        const float load = in ? w / static_cast<float>(p) : -1.0f;
        float top = load;
        for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
        if (l == __builtin_ctzll(__ballot(load == top))) ++p;
    }
    int first = p;
    for (int o = 1; o < kWave; o <<= 1) {
        const int v = __shfl_up(first, o);
        if (l >= o) first += v;
    }
    first -= p;
    if (l <= nl) share[sweep + l] = static_cast<uint32_t>(first);
    if (l == 0) share[sweep + nl + 1] = uneven ? 1u : 0u;
    for (int q = 0; q < p && first + q < sweep; ++q)
        share[first + q] = static_cast<uint32_t>(l) | static_cast<uint32_t>(q) << 8 | static_cast<uint32_t>(p) << 16;
}

template <bool HITS, bool DENSE>
__global__ __launch_bounds__(kEvfThreads) void k_ev_fwd(EvfParams P) {
    __shared__ __align__(16) unsigned char smem[kEvMaxTrials * (HITS ? 16 : 12)];
    unsigned long long *hi = reinterpret_cast<unsigned long long *>(smem);
    uint32_t *lo = reinterpret_cast<uint32_t *>(smem + kEvMaxTrials * 8);
    int32_t *hc = reinterpret_cast<int32_t *>(smem + kEvMaxTrials * 12);   // with hits
    // in the places of the trials from kEvBlockTrials on, which no block has
    uint2 *task_range = reinterpret_cast<uint2 *>(hi + kEvBlockTrials);    // [kTasks] entries of ent2
    uint32_t *n_task = lo + kEvBlockTrials;
    uint32_t *task_rec = n_task + 1;                                       // [kTasks] of set event
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup 8k + x is the k-th on XCD x
    const int x = blockIdx.x & (kXcds - 1), k = blockIdx.x / kXcds;
    const OccTables *tab;
    const double *lterm;
    double *ylt, *s_pre;
    int32_t *hits = nullptr;
    int64_t t0, t1;
    int b, part, parts = P.parts;
    size_t slot;              // of the partial totals
    const bool together = P.sweep > 0 && P.share[P.sweep + P.nl + 1] != 0u;   // uniform over the launch
    if (P.items) {            // the item's parts one after another on its XCD
        const int i = (k / P.parts) * kXcds + x;
        part = k % P.parts;
        if (i >= P.n_items) return;   // uniform, before any barrier
        const FwdItem I = load_item(P.items + i);
        b = I.block;
        if (b < 0) return;    // uniform
        tab = I.tab;
        lterm = I.lterm;
        ylt = I.ylt;
        s_pre = I.s_pre;
        t0 = I.t0;
        t1 = I.t1;
        slot = static_cast<size_t>(i) * P.parts + part;
    } else {
        int j, bi;
        if (together) {       // a block's workgroups one after another
            const int r = k % P.sweep;
            bi = (k / P.sweep) * kXcds + x;
            if (bi >= P.nb) return;   // uniform
            const uint32_t s = P.share[r];
            j = static_cast<int>(s & 255u);
            part = static_cast<int>((s >> 8) & 255u);
            parts = static_cast<int>(s >> 16);
            slot = static_cast<size_t>(bi) * P.sweep + r;
        } else {              // the layers of one (block, part) one after another
            j = k % P.nl;
            const int item = (k / P.nl) * kXcds + x;
            bi = item / P.parts;
            part = item - bi * P.parts;
            if (bi >= P.nb) return;   // uniform
            slot = static_cast<size_t>(j) * P.nb * P.parts + static_cast<size_t>(item);
        }
        b = P.b0 + bi;
        t0 = P.t0;
        t1 = P.t1;
        const size_t n = static_cast<size_t>(t1 - t0);
        tab = P.tabs + j;
        lterm = P.lterm + 4 * j;
        ylt = P.ylt + static_cast<size_t>(j) * n;
        s_pre = P.s_pre ? P.s_pre + static_cast<size_t>(j) * n : nullptr;
        if (HITS && P.hits) hits = P.hits + static_cast<size_t>(j) * n;
    }
    const OccTables T = load_tables(tab);
    const EvLayer L = *T.ev;
    const int64_t bt0 = static_cast<int64_t>(b) * P.B.et;
    const int nt = static_cast<int>(min<int64_t>(P.B.et, P.B.n_trials - bt0));
    if (!L.mode) return;   // uniform: the stream's (k_ev_rest)
    for (int i = tid; i < nt; i += kEvfThreads) {
        hi[i] = 0ull;
        lo[i] = 0u;
        if (HITS) hc[i] = 0;
    }
    if (tid == 0) *n_task = 0u;
    __syncthreads();

    const EvRec *rec = reinterpret_cast<const EvRec *>(T.vals);
    // the block's entries: base may be odd, and pieces are read from an even place on
    const int64_t base = P.B.base[b];
    const uint32_t skew = static_cast<uint32_t>(base & 1);
    const uint16_t *ent2 = device_ptr(P.B.ent) + (base - skew);
    const uint16_t *ent = ent2 + skew;
    const uint2 *hdr = DENSE ? nullptr : P.B.hdr + static_cast<size_t>(b) * P.B.ng;
    const uint32_t *start = DENSE ? P.B.start + static_cast<size_t>(b) * (P.B.catalog + 1) : nullptr;
    // A part is a range of the units; where some events are far more frequent
    // than most (P.spread), every parts-th run of kRunUnits units, since the
    // range with those would have most of the work; or, where the block's
    // workgroups walk it together, every parts-th unit.
    const int n_units = (L.n_set + kWave - 1) / kWave;
    const int run = together ? 1 : (P.spread ? kRunUnits : 0);   // uniform
    const int u1 = run ? n_units : static_cast<int>(static_cast<int64_t>(n_units) * (part + 1) / parts);
    const int first_u = run ? ((w / run) * parts + part) * run + w % run : static_cast<int>(static_cast<int64_t>(n_units) * part / parts) + w;
    const int step_u = run ? kEvfWaves * parts : kEvfWaves;
    const int n_set = min(L.n_set, u1 * kWave);   // set events before the part's end

    // set event i, its header, its list [s, s + c) of entries
    auto load_rec = [&](int i, EvRec &r, int &nb) {
        r = EvRec{0, 0, ~0u};
        nb = 0;
        if ((L.mode & kEvLayout) == 2) {   // uniform
            constexpr int kChunk = kOccChunkWords * 32;
            if (i < n_set && i % kChunk < T.pcount[i / kChunk]) {
                const uint2 v = reinterpret_cast<const uint2 *>(T.dense)[i];
                r.hi = reinterpret_cast<const unsigned long long *>(T.vals)[i];
                r.lo = v.x;
                r.ev = v.y;
                if (HITS) nb = T.cnt[i];
            }
        } else if (i < n_set) {
            const uint4 v = *reinterpret_cast<const uint4 *>(rec + i);
            r.hi = static_cast<unsigned long long>(v.x) | (static_cast<unsigned long long>(v.y) << 32);
            r.lo = v.z;
            r.ev = v.w;
            if (HITS) nb = T.cnt[i];
        }
    };
    auto load_hdr = [&](uint32_t ev) -> uint2 {
        const uint32_t e = ev == ~0u ? 0u : ev;   // event 0's header (always there) for lanes without one
        if (DENSE) return make_uint2(start[e], start[e + 1]);
        return hdr[e >> 3];
    };
    auto find = [&](uint32_t ev, uint2 h, uint32_t &s, uint32_t &c) {
        if (DENSE) {
            s = h.x;
            c = h.y - h.x;
        } else {
            ev_short_list(h, ev & 7u, s, c);
            if (ev != ~0u && ev_long(h.y)) {
                const uint32_t all = hdr[(ev >> 3) + 1].x - h.x;
                const uint32_t a = ev_lower(ent + h.x, all, ev & 7u), z = ev_lower(ent + h.x, all, (ev & 7u) + 1u);
                s = h.x + a;
                c = z - a;
            }
        }
        if (ev == ~0u) c = 0;
        s += skew;
    };
    // piece p of the list: entries of ent2 from the even place at or before
    // its first, eight at a time (the entries are padded past the last one)
    auto load_piece = [&](uint32_t s, uint32_t c, uint32_t p, EvPiece &d) {
        if (8u * p < (s & 1u) + c) d = *reinterpret_cast<const EvPiece *>(ent2 + (s & ~1u) + static_cast<size_t>(8u * p));
    };
    // r added to the trials of the entries i of piece d that in(i) names.  With
    // carry lo takes all of its 32 bits, and an addition that wraps it adds one
    // to hi.
    const bool carry = (L.mode & kEvCarry) != 0;   // uniform
    auto add = [&](const EvPiece &d, auto in, const EvRec &r, int nb) {
        auto trial = [&](uint32_t i) { return ((i & 1u) ? d[i >> 1] >> 16 : d[i >> 1]) & kEvTrialMask; };
        if (!carry) {
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i)
                if (in(i)) {
                    const uint32_t t = trial(i);
                    atomicAdd(&hi[t], r.hi);
                    atomicAdd(&lo[t], r.lo);
                    if (HITS) atomicAdd(&hc[t], nb);
                }
        } else {
            uint32_t old[8];
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i)
                if (in(i)) old[i] = atomicAdd(&lo[trial(i)], r.lo);
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i)
                if (in(i)) {
                    const uint32_t t = trial(i);
                    atomicAdd(&hi[t], r.hi + (old[i] + r.lo < old[i] ? 1ull : 0ull));
                    if (HITS) atomicAdd(&hc[t], nb);
                }
        }
    };
    auto add_piece = [&](uint32_t s, uint32_t c, uint32_t p, const EvPiece &d, const EvRec &r, int nb) {
        const uint32_t first = 8u * p - (s & 1u);   // entry 0 of the piece in the list (wraps below 0)
        add(d, [&](uint32_t i) { return first + i < c; }, r, nb);
    };
    // the entries [a, z) of ent2, none before place s, added by a wavefront,
    // eight a lane and two loads in flight
    auto add_wide = [&](uint32_t s, uint32_t a, uint32_t z, const EvRec &r, int nb) {
        a &= ~1u;
        EvPiece d, d2;
        const uint32_t a0 = a;
        auto load = [&](uint32_t at, EvPiece &to) {
            const uint32_t k = at + 8u * lane;
            to = *reinterpret_cast<const EvPiece *>(ent2 + (k < z ? k : a0));
        };
        auto put = [&](uint32_t at, const EvPiece &from) {
            const uint32_t k = at + 8u * lane;
            add(from, [&](uint32_t i) { return k + i >= s && k + i < z; }, r, nb);
        };
        load(a, d);
        for (; a < z; a += 1024u) {   // uniform
            load(a + 512u, d2);
            put(a, d);
            load(a + 1024u, d);
            put(a + 512u, d2);
        }
        wait_loads();
    };

    EvRec r0, r1, r2;
    int n0, n1, n2;
    uint32_t s0, c0, s1, c1;
    EvPiece a1{}, e1{};   // the first two pieces of the next lists to be added
    load_rec(first_u * kWave + lane, r0, n0);
    load_rec((first_u + step_u) * kWave + lane, r1, n1);
    {
        const uint2 h = load_hdr(r0.ev);
        find(r0.ev, h, s0, c0);
    }
    load_piece(s0, c0, 0, a1);
    load_piece(s0, c0, 1, e1);
    uint2 h1 = load_hdr(r1.ev);
    for (int u = first_u; u < u1; u += step_u) {
        load_rec((u + 2 * step_u) * kWave + lane, r2, n2);
        find(r1.ev, h1, s1, c1);
        // the pieces have come with the headers, which were loaded after them;
        // taken over any earlier they would be waited for by themselves (left
        // to itself the compiler may do so right behind their loads)
        EvPiece a0 = a1;
        const EvPiece e0 = e1;
        load_piece(s1, c1, 0, a1);
        load_piece(s1, c1, 1, e1);
        h1 = load_hdr(r2.ev);
        // a list of many entries: the wavefront's lanes take them together, and
        // one of very many is left, in up to as many pieces as there are
        // wavefronts, to all of them after the others (where there is room)
        uint64_t big = long_lists(c0);
        for (; big; big &= big - 1) {
            const int l = __builtin_ctzll(big);
            const uint32_t s = __builtin_amdgcn_readlane(s0, l), c = __builtin_amdgcn_readlane(c0, l);
            if (lane == l) c0 = 0;
            if (c > kTaskList) {
                const uint32_t per = max((c / kEvfWaves + 1024u) & ~1023u, kTaskList);   // entries of a piece
                const uint32_t n = (c + per - 1u) / per;
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(n_task, n);
                at = __builtin_amdgcn_readfirstlane(at);
                if (at + n <= static_cast<uint32_t>(kTasks)) {
                    if (static_cast<uint32_t>(lane) < n) {
                        task_range[at + lane] = make_uint2(s + lane * per, s + min(c, (lane + 1u) * per));
                        task_rec[at + lane] = static_cast<uint32_t>(u * kWave + l);
                    }
                    continue;
                }
                if (static_cast<uint32_t>(lane) < n && at + lane < static_cast<uint32_t>(kTasks))
                    task_range[at + lane] = make_uint2(0u, 0u);   // reserved, but not for this list
            }
            EvRec r;
            r.hi = __shfl(r0.hi, l);
            r.lo = __builtin_amdgcn_readlane(r0.lo, l);
            add_wide(s, s, s + c, r, HITS ? __builtin_amdgcn_readlane(n0, l) : 0);
        }
        add_piece(s0, c0, 0, a0, r0, n0);
        if (__any((s0 & 1u) + c0 > 8u)) {
            add_piece(s0, c0, 1, e0, r0, n0);
            if (!__any((s0 & 1u) + c0 > 32u)) {
                for (uint32_t p = 2; __any((s0 & 1u) + c0 > 8u * p); ++p) {
                    load_piece(s0, c0, p, a0);
                    add_piece(s0, c0, p, a0, r0, n0);
                }
            } else {   // two more pieces in flight while two are added
                // (from the block's first entries for the lanes without: a
                // branch around a load makes the compiler wait for all of them)
                EvPiece x, y, x2, y2;
                auto load_any = [&](uint32_t p, EvPiece &d) {
                    const uint32_t at = 8u * p < (s0 & 1u) + c0 ? (s0 & ~1u) + 8u * p : 0u;
                    d = *reinterpret_cast<const EvPiece *>(ent2 + at);
                };
                load_any(2, x);
                load_any(3, y);
                for (uint32_t p = 2; __any((s0 & 1u) + c0 > 8u * p); p += 4) {
                    load_any(p + 2, x2);
                    load_any(p + 3, y2);
                    add_piece(s0, c0, p, x, r0, n0);
                    add_piece(s0, c0, p + 1, y, r0, n0);
                    load_any(p + 4, x);
                    load_any(p + 5, y);
                    add_piece(s0, c0, p + 2, x2, r0, n0);
                    add_piece(s0, c0, p + 3, y2, r0, n0);
                }
                wait_loads();
            }
        }
        r0 = r1;
        n0 = n1;
        s0 = s1;
        c0 = c1;
        r1 = r2;
        n1 = n2;
    }
    __syncthreads();
    // the pieces left over
    const int nt_left = min(static_cast<int>(*n_task), kTasks);   // uniform
    for (int q = w; q < nt_left; q += kEvfWaves) {
        const uint2 range = task_range[q];
        const uint32_t a = __builtin_amdgcn_readfirstlane(range.x), z = __builtin_amdgcn_readfirstlane(range.y);
        if (a >= z) continue;
        EvRec r;
        int nb;
        load_rec(static_cast<int>(__builtin_amdgcn_readfirstlane(task_rec[q])), r, nb);
        add_wide(a, a, z, r, nb);
    }
    if (nt_left > 0) __syncthreads();

    if (parts > 1) {
        unsigned char *p = P.partial + slot * ev_slot_bytes(P.B.et, HITS);
        unsigned long long *ph = reinterpret_cast<unsigned long long *>(p);
        uint32_t *pl = reinterpret_cast<uint32_t *>(p + static_cast<size_t>(P.B.et) * 8);
        int32_t *pc = reinterpret_cast<int32_t *>(p + static_cast<size_t>(P.B.et) * 12);
        for (int i = tid; i < nt; i += kEvfThreads) {
            ph[i] = hi[i];
            pl[i] = lo[i];
            if (HITS) pc[i] = hc[i];
        }
        return;
    }
    const double aggR = lterm[2], aggL = lterm[3];
    const int i0 = static_cast<int>(max<int64_t>(t0 - bt0, 0)), i1 = static_cast<int>(min<int64_t>(t1 - bt0, nt));
    for (int i = i0 + tid; i < i1; i += kEvfThreads) {
        const double S = ev_total(hi[i], lo[i], L);
        const size_t o = static_cast<size_t>(bt0 + i - t0);
        ylt[o] = xl(S, aggR, aggL);
        if (s_pre) s_pre[o] = S;
        if (HITS && hits) hits[o] = hc[i];
    }
}

// The results of a split launch's trials from the parts' totals (integers: in
// any order).  Regular set: one run of NT / G trials of a (layer, block) per
// workgroup, by its first NT threads, G lanes per trial where there are few, so that its parts' loads
// overlap.  List: the same of an item.
constexpr int kRestThreads = 1024;
constexpr int kAddThreads = 256;

template <bool HITS, int NT>
__device__ __forceinline__ void ev_add(const EvfParams &P, int G, int per) {
    if (threadIdx.x >= NT) return;
    const int u = blockIdx.x / per, c = blockIdx.x - u * per;
    if (u >= (P.items ? P.n_items : P.nl * P.nb)) return;
    int b;
    int64_t t0, t1;
    const OccTables *tab;
    const double *lterm;
    double *ylt, *s_pre;
    int32_t *hits = nullptr;
    if (P.items) {
        const FwdItem I = load_item(P.items + u);
        b = I.block;
        if (b < 0) return;
        t0 = I.t0;
        t1 = I.t1;
        tab = I.tab;
        lterm = I.lterm;
        ylt = I.ylt;
        s_pre = I.s_pre;
    } else {
        const int j = u / P.nb;
        b = P.b0 + (u - j * P.nb);
        t0 = P.t0;
        t1 = P.t1;
        const size_t n = static_cast<size_t>(t1 - t0);
        tab = P.tabs + j;
        lterm = P.lterm + 4 * j;
        ylt = P.ylt + static_cast<size_t>(j) * n;
        s_pre = P.s_pre ? P.s_pre + static_cast<size_t>(j) * n : nullptr;
        if (HITS && P.hits) hits = P.hits + static_cast<size_t>(j) * n;
    }
    const EvLayer L = *device_ptr(tab->ev);
    if (!L.mode) return;   // uniform
    const int i = (c * NT + static_cast<int>(threadIdx.x)) / G, sub = threadIdx.x & (G - 1);
    const int64_t t = static_cast<int64_t>(b) * P.B.et + i;
    if (i >= P.B.et || t < t0 || t >= t1) return;   // all lanes of a trial together
    const size_t slot = ev_slot_bytes(P.B.et, HITS);
    int parts = P.parts;
    size_t slot0 = static_cast<size_t>(u) * P.parts;
    if (P.sweep > 0 && P.share[P.sweep + P.nl + 1] != 0u) {   // (G is 1: many blocks)
        const int j = u / P.nb, bi = u - j * P.nb;
        const uint32_t f = P.share[P.sweep + j];
        parts = static_cast<int>(P.share[P.sweep + j + 1] - f);
        slot0 = static_cast<size_t>(bi) * P.sweep + f;
    }
    if (parts == 1) return;   // uniform: the results are there
    const unsigned char *p = P.partial + (slot0 + sub) * slot;
    unsigned long long h = 0, l = 0;
    int32_t k = 0;
#pragma unroll 4
    for (int q = sub; q < parts; q += G, p += static_cast<size_t>(G) * slot) {
        h += reinterpret_cast<const unsigned long long *>(p)[i];
        l += reinterpret_cast<const uint32_t *>(p + static_cast<size_t>(P.B.et) * 8)[i];
        if (HITS) k += reinterpret_cast<const int32_t *>(p + static_cast<size_t>(P.B.et) * 12)[i];
    }
    for (int d = G / 2; d > 0; d >>= 1) {
        h += __shfl_xor(h, d, G);
        l += __shfl_xor(l, d, G);
        if (HITS) k += __shfl_xor(k, d, G);
    }
    if (sub != 0) return;
    const double S = ev_total(h, l, L);
    const size_t o = static_cast<size_t>(t - t0);
    ylt[o] = xl(S, lterm[2], lterm[3]);
    if (s_pre) s_pre[o] = S;
    if (HITS && hits) hits[o] = k;
}

// By itself, of a block's workgroups that walked it together: 16 parts of every
// trial, four layers over 1M trials 51 us, as a part of k_ev_rest 65.
template <bool HITS>
__global__ __launch_bounds__(kAddThreads) void k_ev_add(EvfParams P, int per) {
    ev_add<HITS, kAddThreads>(P, 1, per);
}

// What is left behind k_ev_fwd: the first n_add workgroups add the parts up,
// the others stream the layers that its integers do not fit, as k_fwd would
// (two workgroups on a CU, where k_ev_fwd has one).  In one launch, since such
// layers are rare and only the device knows of them: the workgroups find none
// and end.
template <bool HITS, bool SHARED, bool LIST>
__global__ __launch_bounds__(kRestThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_ev_rest(EvfParams P, int G, int per,
                                                                                                  int nt, int n_add) {
    __shared__ __align__(16) unsigned char smem[kLdsBytes];
    if (static_cast<int>(blockIdx.x) < n_add) {
        if (nt == kAddThreads) ev_add<HITS, kAddThreads>(P, G, per);
        else ev_add<HITS, kRestThreads>(P, G, per);
        return;
    }
    const int first = static_cast<int>(blockIdx.x) - n_add, step = static_cast<int>(gridDim.x) - n_add;
    int n = P.n_items;
    if (!LIST) {
        bool any = false;
        for (int j = threadIdx.x & 63; j < P.nl; j += kWave) any = any || device_ptr(P.tabs[j].ev)->mode == 0;
        if (!__any(any)) return;   // uniform
        n = P.nl <= 1 ? P.fwd.reg_nb : P.nl * kXcds * ((P.fwd.reg_nb + kXcds - 1) / kXcds);   // fwd_regular_items
    }
    for (int i = first; i < n; i += step) {
        FwdItem I = fwd_item(P.fwd, i);
        if (I.block < 0 || device_ptr(I.tab->ev)->mode) continue;   // uniform
        int k = I.block, k1 = k + 1;
        if (LIST) {   // the stream's blocks that meet the item's
            const int64_t bt0 = static_cast<int64_t>(I.block) * P.B.et;
            const int64_t a = max(I.t0, bt0), z = min(I.t1, min(bt0 + P.B.et, P.B.n_trials));
            I.ylt += a - I.t0;
            if (I.s_pre) I.s_pre += a - I.t0;
            I.t0 = a;
            I.t1 = z;
            k = static_cast<int>(a / P.fwd.tb);
            k1 = static_cast<int>((z + P.fwd.tb - 1) / P.fwd.tb);
        }
        for (; k < k1; ++k) {
            I.block = k;
            __syncthreads();   // the previous block's totals have been read
            fwd_block<HITS, false, SHARED, true>(P.fwd, I, smem);
        }
    }
}

static int32_t launch_ev(const EvfParams &P, bool hits, unsigned grid, int n_sets, hipStream_t st) {
    if (hits) {
        if (P.B.dense) k_ev_fwd<true, true><<<grid, kEvfThreads, 0, st>>>(P);
        else k_ev_fwd<true, false><<<grid, kEvfThreads, 0, st>>>(P);
    } else {
        if (P.B.dense) k_ev_fwd<false, true><<<grid, kEvfThreads, 0, st>>>(P);
        else k_ev_fwd<false, false><<<grid, kEvfThreads, 0, st>>>(P);
    }
    int G = 1, per = 0, nt = kRestThreads;
    if (P.sweep > 0) {
        const int pa = (P.B.et + kAddThreads - 1) / kAddThreads;
        const unsigned g = static_cast<unsigned>(n_sets) * static_cast<unsigned>(pa);
        if (hits) k_ev_add<true><<<g, kAddThreads, 0, st>>>(P, pa);
        else k_ev_add<false><<<g, kAddThreads, 0, st>>>(P, pa);
    } else if (P.parts > 1) {   // lanes per trial: while that leaves the device room
        while (2 * G <= std::min(P.parts, kWave) && static_cast<int64_t>(2 * G) * n_sets * P.B.et <= 65536) G *= 2;
        // and few threads of a workgroup while that leaves each CU one: the loads
        // come from more CUs (2000 trials 4.7 us, with all of the threads 5.7;
        // 23,000 trials with hits 9.1, 10.2)
        if (static_cast<int64_t>(n_sets) * P.B.et * G <= static_cast<int64_t>(kAddThreads) * device_cu_count()) nt = kAddThreads;
        per = (P.B.et * G + nt - 1) / nt;
    }
    // (a multiple of the XCDs, so that what follows goes to them in turn)
    const int n_add = (n_sets * per + kXcds - 1) / kXcds * kXcds;
    // the stream's two workgroups on each CU, a multiple of the XCDs
    const int n_rest = std::min(P.items ? P.n_items : fwd_regular_items(P.nl, P.fwd.reg_nb), 2 * device_cu_count());
    const unsigned ga = static_cast<unsigned>(n_add + (n_rest + kXcds - 1) / kXcds * kXcds);
    per = std::max(per, 1);
#define ARA_REST_LAUNCH(H, S, L) k_ev_rest<H, S, L><<<ga, kRestThreads, 0, st>>>(P, G, per, nt, n_add)
    if (P.items) ARA_REST_LAUNCH(false, true, true);
    else if (hits && P.nl > 1) ARA_REST_LAUNCH(true, true, false);
    else if (hits) ARA_REST_LAUNCH(true, false, false);
    else if (P.nl > 1) ARA_REST_LAUNCH(false, true, false);
    else ARA_REST_LAUNCH(false, false, false);
#undef ARA_REST_LAUNCH
    ARA_HIP(hipGetLastError());
    return ARA_OK;
}

int ev_parts(int64_t n_items, int64_t slots) {
    const int cu = device_cu_count();
    // rounds of one workgroup per CU over the parts a block is cut into, with
    // a little for each part's share of the adding up; at most 64 (a block's
    // 64 parts add up about as long as they run where the YET is that small)
    int best = 1;
    double cost = 1e300;
    for (int p = 1; p <= 64; ++p) {
        if (p > 1 && n_items * p > slots) break;
        const double c = static_cast<double>((n_items * p + cu - 1) / cu) / p + 0.002 * p;
        if (c < cost) {
            cost = c;
            best = p;
        }
    }
    return best;
}

static int32_t ev_params(const EvBlocks &B, const ara_yet *yet, bool hits, int parts, EvfParams &P) {
    if (B.et < 1 || B.et > kEvBlockTrials || parts < 1)
        return fail(ARA_E_INVAL, "event-ordered forward: blocks not prepared by this library");
    P.B = B;
    P.parts = parts;
    const double blocks = std::max(B.neb, 1);   // entries of the longest list, and of one on average
    P.spread = yet->max_occ / blocks > 64.0 + 8.0 * static_cast<double>(yet->nnz) / (blocks * std::max(B.catalog, 1));
    return fwd_params(yet, hits, false, P.fwd);
}

int32_t launch_ev_forward(const EvBlocks &B, const ara_yet *yet, bool hits, const FwdRegular &reg, hipStream_t st) {
    if (reg.nl <= 0 || reg.ev_nb <= 0) return ARA_OK;
    EvfParams P{};
    const int32_t rc = ev_params(B, yet, hits, reg.parts, P);
    if (rc) return rc;
    P.tabs = reg.tabs;
    P.lterm = reg.lterm;
    P.ylt = reg.ylt;
    P.s_pre = reg.s_pre;
    P.hits = reg.hits;
    P.t0 = reg.t0;
    P.t1 = reg.t1;
    P.b0 = reg.ev_b0;
    P.nb = reg.ev_nb;
    P.nl = reg.nl;
    P.partial = reg.partial;
    P.fwd.reg_tabs = reg.tabs;
    P.fwd.reg_lterm = reg.lterm;
    P.fwd.reg_ylt = reg.ylt;
    P.fwd.reg_s_pre = reg.s_pre;
    P.fwd.reg_hits = reg.hits;
    P.fwd.reg_t0 = reg.t0;
    P.fwd.reg_t1 = reg.t1;
    P.fwd.reg_b0 = reg.b0;
    P.fwd.reg_nb = reg.nb;
    P.fwd.reg_nl = reg.nl;
    if (reg.sweep > 0) {
        P.sweep = reg.sweep;
        P.share = reg.share;
        k_ev_share<<<1, kWave, 0, st>>>(P.tabs, P.nl, P.sweep, B.catalog, reg.share);
    }
    const int64_t items = (static_cast<int64_t>(reg.ev_nb) * reg.parts + kXcds - 1) / kXcds * kXcds;
    const int64_t blocks = (static_cast<int64_t>(reg.ev_nb) + kXcds - 1) / kXcds * kXcds;
    return launch_ev(P, hits, static_cast<unsigned>(std::max(items * reg.nl, blocks * reg.sweep)), reg.nl * reg.ev_nb, st);
}

int32_t launch_ev_list(const EvBlocks &B, const ara_yet *yet, const FwdItem *d_items, int n_items, int parts,
                       unsigned char *partial, hipStream_t st) {
    if (n_items <= 0) return ARA_OK;
    EvfParams P{};
    const int32_t rc = ev_params(B, yet, false, parts, P);
    if (rc) return rc;
    P.items = P.fwd.items = d_items;
    P.n_items = n_items;
    P.nl = 1;
    P.partial = partial;
    return launch_ev(P, false, static_cast<unsigned>((n_items + kXcds - 1) / kXcds * kXcds * parts), n_items, st);
}

}  // namespace ara
