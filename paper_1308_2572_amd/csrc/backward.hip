// Backward: gradients of sum_t c_t * Y_t with respect to every ELT term
// (scale, retention, limit) and every layer term (OccR, OccL, AggR, AggL),
// for up to ARA_MAX_COTANGENTS cotangent rows c at once -- the reverse sweep
// of Algorithm 1.
//
// Chain rule through the forward (branch-following subgradients):
//   Y_t = f_agg(S_t),  S_t = sum over occurrences d of O(e_d),
//   O(e) = f_occ(x_e),  x_e = sum over the layer's ELTs k of g_k(l_k(e)).
//   dY_t/dS_t = a_t (aggregate clamp in its linear branch), so with
//   v_t = c_t * a_t and W(e) = sum_t v_t * (occurrences of e in trial t):
//     dAggR = -sum_t c_t a_t,  dAggL = sum_t c_t [aggregate limit binds]
//     dOccR = -sum_e W(e) b_e, dOccL = sum_e W(e) [occurrence limit binds]
//     ds_k  =  sum_e W(e) b_e lin_k(e) l_k(e)
//     dR_k  = -sum_e W(e) b_e lin_k(e),  dL_k = sum_e W(e) b_e [ELT limit binds]
//   (b_e: occurrence clamp linear; lin_k: ELT clamp linear).  Only events
//   with O(e) != 0 can have b_e or a binding occurrence limit, so W is kept
//   for those "hot" events only, indexed by the occurrence table's rank.
//
// The forward gathers O(e) per trial; its adjoint scatters v_t per event.
// Read through the event-major copy of the YET the scatter is a gather
// again, and only the hot events' occurrence lists are read at all.
//
// Kernels: (1) the hot occurrence tables (shared with the forward);
// (2) v_t per cotangent row, its largest magnitude and the aggregate-term
// sums; (3) v_t in 64-bit fixed point, scaled so that no partial sum of W
// can overflow (|W| <= max|v| * largest occurrence count of one event);
// (4) the list of hot events; (5) W(e) per hot event, gathered per trial
// slice over the event-major YET and combined with integer atomics, so the
// result does not depend on the order; (6) over the hot events, W times
// the per-event derivatives, reduced in a fixed order; (7) a fixed-order sum
// of the chunk partials into the outputs.
//
// Step (5) has a second form for cotangents that take one value on most
// trials, as the metrics' do (AAL: the same weight wherever the aggregate
// clamp is linear; PML, TVaR: zero outside the tied or top trials).  With c
// that common fixed-point value and D the trials whose value differs,
//   W(e) = c * (occurrences of e in the call's trials)
//          + sum over t in D of (v_t - c) * (occurrences of e in t),
// integer arithmetic that gives the gather's result bit for bit.  The
// occurrence counts come from the event-major offsets: over all trials the
// per-event totals, over part of them the list lengths of the trial slices
// the range covers whole, plus a count of the in-range entries of the (at
// most two) slices it cuts; the second term comes from the trial-major copy
// of the deviating trials' events.  It is used when the trials to walk are
// at most a sixteenth of all (each walked trial costs about sixteen times
// its share of the gather's time).
//
// A third form serves cotangents of two values, as the metrics' are where
// many years exceed the aggregate limit (zero there, the AAL's weight on the
// others): with a the second value,
//   W(e) = c * (occurrences) + (a - c) * (occurrences in trials of value a)
//          + sum over t of neither value of (v_t - c) * (occurrences in t),
// the second count from one bit per trial.
//
// The decision is taken on the device from the counts, so all forms are
// enqueued and those not chosen return at once.
#include "occ.h"
#include "wave.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace ara {

constexpr int kBwdThreads = 1024;
constexpr int kMaxCot = ARA_MAX_COTANGENTS;

struct VScale {
    unsigned long long maxabs_bits;   // max |v| as binary64 bits (non-negative: order-preserving)
    int32_t sigma;                    // v is stored as round(v * 2^sigma)
    int32_t pad;
};

__device__ __forceinline__ bool agg_linear(double S, double aggR, double aggL) {
    const double y = S - aggR;
    const double a = (y > 0.0) ? y : 0.0;
    return (y > 0.0) && (a < aggL);
}

__device__ __forceinline__ bool agg_capped(double S, double aggR, double aggL) {
    const double y = S - aggR;
    const double a = (y > 0.0) ? y : 0.0;
    return a >= aggL;
}

__device__ __forceinline__ void chunk_range(int64_t n, int nwg, int wg, int64_t &lo, int64_t &hi) {
    const int64_t c = (n + nwg - 1) / nwg;
    lo = std::min<int64_t>(n, static_cast<int64_t>(wg) * c);
    hi = std::min<int64_t>(n, lo + c);
}

// (2) largest |c_t a_t| per (layer, row); aggregate-term partial sums.  One
// pass over the trials of the workgroup's chunk reads S once for every row;
// the sums meet in fixed order (each thread's trials, DPP across the
// wavefront, the wavefronts in index order).
__global__ __launch_bounds__(kBwdThreads) void k_bwd_vmax(const double *__restrict__ cot, const double *__restrict__ s_pre,
                                                         const double *__restrict__ layer_terms, int64_t n, int n_layers,
                                                         int n_cot, int nwg, VScale *__restrict__ vs,
                                                         double *__restrict__ aggpart) {
    __shared__ double red[kBwdThreads / 64][kMaxCot][3];
    const int wg = blockIdx.x, j = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const double aggR = layer_terms[4 * j + 2], aggL = layer_terms[4 * j + 3];
    int64_t lo, hi;
    chunk_range(n, nwg, wg, lo, hi);
    const double *S = s_pre + static_cast<size_t>(j) * n;
    double m[kMaxCot], sr[kMaxCot], sl[kMaxCot];
#pragma unroll
    for (int c = 0; c < kMaxCot; ++c) m[c] = sr[c] = sl[c] = 0.0;
    for (int64_t t = lo + tid; t < hi; t += blockDim.x) {
        const double st = S[t];
        const bool lin = agg_linear(st, aggR, aggL), cap = agg_capped(st, aggR, aggL);
#pragma unroll
        for (int c = 0; c < kMaxCot; ++c)
            if (c < n_cot) {
                const double g = cot[(static_cast<size_t>(c) * n_layers + j) * n + t];
                if (lin) {
                    sr[c] += g;
                    m[c] = fmax(m[c], fabs(g));
                }
                if (cap) sl[c] += g;
            }
    }
#pragma unroll
    for (int c = 0; c < kMaxCot; ++c)
        if (c < n_cot) {
            double mc = m[c];
            for (int o = 32; o > 0; o >>= 1) mc = fmax(mc, __shfl_down(mc, o));
            const double tr = wave_inclusive_sum(sr[c]), tl = wave_inclusive_sum(sl[c]);
            if (lane == 0) red[w][c][2] = mc;
            if (lane == 63) {
                red[w][c][0] = tr;
                red[w][c][1] = tl;
            }
        }
    __syncthreads();
    if (tid < n_cot * 2) {
        const int c = tid >> 1, h = tid & 1;
        double t = 0.0;
        for (int i = 0; i < static_cast<int>(blockDim.x >> 6); ++i) t += red[i][c][h];
        aggpart[((static_cast<size_t>(j) * n_cot + c) * nwg + wg) * 2 + h] = h ? t : -t;
    } else if (tid >= 64 && tid < 64 + n_cot) {   // one atomic per (workgroup, row)
        const int c = tid - 64;
        double mc = 0.0;
        for (int i = 0; i < static_cast<int>(blockDim.x >> 6); ++i) mc = fmax(mc, red[i][c][2]);
        if (mc > 0.0)
            atomicMax(&vs[j * n_cot + c].maxabs_bits, static_cast<unsigned long long>(__double_as_longlong(mc)));
    }
}

__device__ __forceinline__ int sigma_of(const VScale &v, int max_occ) {
    const double m = __longlong_as_double(static_cast<long long>(v.maxabs_bits));
    if (!(m > 0.0)) return 0;
    int e;
    frexp(m * static_cast<double>(max_occ > 0 ? max_occ : 1), &e);   // m*max_occ < 2^e
    return 62 - e;
}

// (3) fixed-point weights vq[j][t][c] = round(c_t a_t 2^sigma), the rows of
// one trial side by side (cs >= n_cot slots, the spare ones zero) so that one
// gather fetches every row.
__global__ void k_bwd_vq(const double *__restrict__ cot, const double *__restrict__ s_pre,
                         const double *__restrict__ layer_terms, int64_t n, int n_layers, int n_cot, int cs,
                         int max_occ, VScale *__restrict__ vs, int64_t *__restrict__ vq) {
    const int j = blockIdx.y;
    const double aggR = layer_terms[4 * j + 2], aggL = layer_terms[4 * j + 3];
    const double *S = s_pre + static_cast<size_t>(j) * n;
    int sg[kMaxCot];
    for (int c = 0; c < n_cot; ++c) {
        sg[c] = sigma_of(vs[j * n_cot + c], max_occ);
        if (blockIdx.x == 0 && threadIdx.x == 0) vs[j * n_cot + c].sigma = sg[c];
    }
    int64_t *q = vq + static_cast<size_t>(j) * n * cs;
    for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < n;
         t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const bool lin = agg_linear(S[t], aggR, aggL);
        for (int c = 0; c < cs; ++c) {
            int64_t r = 0;
            if (c < n_cot && lin) {
                const double v = cot[(static_cast<size_t>(c) * n_layers + j) * n + t];
                r = (v == 0.0) ? 0 : static_cast<int64_t>(__double2ll_rn(ldexp(v, sg[c])));
            }
            q[static_cast<size_t>(t) * cs + c] = r;
        }
    }
}

// (4) the layer's hot events (O(e) != 0) as one list, in (super-range,
// rank) order: hot_ev[g] is the event of hot index g = hot_base[s] + rank;
// the weight accumulators of every hot index start at zero.
__global__ __launch_bounds__(256) void k_bwd_hot(const OccTables *__restrict__ tabs, int n_sr, int n_cot,
                                                 int32_t catalog, int32_t *__restrict__ hot_ev,
                                                 int32_t *__restrict__ hot_base, int64_t *__restrict__ W) {
    __shared__ int32_t red[4];
    const int s = blockIdx.x, j = blockIdx.y, tid = threadIdx.x;
    const OccTables T = load_tables(tabs + j);
    int32_t part = 0;
    for (int i = tid; i < s; i += blockDim.x) part += T.count[i];
    for (int o = 32; o > 0; o >>= 1) part += __shfl_down(part, o);
    if ((tid & 63) == 0) red[tid >> 6] = part;
    __syncthreads();
    const int32_t base = red[0] + red[1] + red[2] + red[3];
    int32_t *hb = hot_base + static_cast<size_t>(j) * (n_sr + 1);
    if (tid == 0) {
        hb[s] = base;
        if (s == n_sr - 1) hb[n_sr] = base + T.count[s];
    }
    int32_t *hev = hot_ev + static_cast<size_t>(j) * catalog;
    int64_t *Wj = W + static_cast<size_t>(j) * n_cot * catalog;
    for (int i = tid; i < kSrWords; i += blockDim.x) {
        const uint2 q = T.br[static_cast<size_t>(s) * kSrWords + i];
        uint32_t m = q.x;
        int32_t g = base + static_cast<int32_t>(q.y);
        while (m) {
            const int bit = __builtin_ctz(m);
            hev[g] = s * kSr + 32 * i + bit;
            for (int c = 0; c < n_cot; ++c) Wj[static_cast<size_t>(c) * catalog + g] = 0;
            ++g;
            m &= m - 1;
        }
    }
}

__device__ __forceinline__ uint32_t lanes_under(uint64_t m) {   // bits of m below this lane
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

constexpr int kCand = 8;   // candidates for the common value of a row: 0 and seven sampled trials
constexpr int kDevChunk = 4096;   // trials per workgroup when counting and listing them

struct BwdSparse {
    const int64_t *vq;                 // [n_layers][n][cs]
    int64_t n, t0, n_trials;
    int32_t cs, n_cot, catalog, n_sr;
    int64_t slice_trials;              // trials of one slice of the event-major copy
    const int64_t *tr_off;             // event-major copy: list offsets per (slice, event)
    const uint32_t *tr_ent;            //   and the lists' slice-local trial indices
    unsigned long long *ndev, *nalt;   // [n_layers] trials of neither value, trials of the second value
    int64_t *common;                   // [n_layers][kMaxCot] the chosen common value
    int64_t *alt;                      // [n_layers][kMaxCot] the chosen second value (the common one: none)
    int32_t *dev;                      // [n_layers][n] trials (call-relative) of neither value from the front,
                                       //   of the second from the back
    uint2 *abits;                      // [n_layers][aw] bit t: trial t has the second value
    int64_t aw;                        // 64-bit words of a layer's bits
    int32_t two, two_bytes;            // whether the third form is available, and its LDS
    int32_t segs;                      // wavefronts for each trial that is walked
    const int32_t *t_cnt;              // occurrences of each event
    const int64_t *t_off;              // trial-major copy
    const int32_t *t_ids;
    const OccTables *tabs;
    const int32_t *hot_ev, *hot_base;
    int64_t *W;                        // [n_layers][n_cot][catalog], by hot index
};

__device__ __forceinline__ int64_t cand_value(const BwdSparse &P, int j, int c, int k) {
    if (k == 0 || P.n == 0) return 0;
    const int64_t t = (static_cast<int64_t>(k) * P.n) / kCand;
    return P.vq[(static_cast<size_t>(j) * P.n + t) * P.cs + c];
}

// Whether some row's common value is non-zero (W then starts from c times
// the occurrence counts).
__device__ __forceinline__ bool common_nonzero(const BwdSparse &P, int j) {
    for (int c = 0; c < P.n_cot; ++c)
        if (P.common[static_cast<size_t>(j) * kMaxCot + c] != 0) return true;
    return false;
}

// Trial slice x of the event-major copy holds trials [x S, min((x + 1) S, N)).
__device__ __forceinline__ bool slice_inside(const BwdSparse &P, int x) {
    const int64_t lo = static_cast<int64_t>(x) * P.slice_trials;
    const int64_t hi = min(lo + P.slice_trials, P.n_trials);
    return lo >= P.t0 && hi <= P.t0 + P.n;
}

__device__ __forceinline__ bool slice_cut(const BwdSparse &P, int x) {
    const int64_t lo = static_cast<int64_t>(x) * P.slice_trials;
    const int64_t hi = min(lo + P.slice_trials, P.n_trials);
    return max(lo, P.t0) < min(hi, P.t0 + P.n) && !slice_inside(P, x);
}

// Which form serves layer j, the same in every kernel that asks: the second
// where the trials to walk are at most a sixteenth of all, the third where
// those of neither value are a thirty-second (counting the second value takes a
// third of the gather's time by itself), the first otherwise.
constexpr int kWalkShare = 16;
enum { kDense = 1, kOneValue = 2, kTwoValues = 3 };
__device__ __forceinline__ int form_of(const BwdSparse &P, int j) {
    const int64_t dev = static_cast<int64_t>(P.ndev[j]), alt = static_cast<int64_t>(P.nalt[j]);
    if ((dev + alt) * kWalkShare <= P.n_trials) return kOneValue;
    return P.two && 2 * dev * kWalkShare <= P.n_trials ? kTwoValues : kDense;
}

struct BwdGather {
    const int64_t *tr_off;        // event-major YET
    const uint32_t *tr_ent;
    int32_t catalog, n_sr, n_cot, pad;
    int64_t slice_trials;
    int64_t t0, t1, n;            // trial range of the call
    const int32_t *hot_ev;        // [n_layers][catalog]
    const int32_t *hot_base;      // [n_layers][n_sr + 1]
    const int64_t *vq;            // [n_layers][n][CS]
    int64_t *W;                   // [n_layers][n_cot][catalog], by hot index
    BwdSparse sp;                 // the second form's state
    int32_t use_sp;               // 0 when the second form is not available (no trial-major copy)
    int32_t n_layers;
    EvBlocks B;                   // event-ordered blocks
    int64_t ev_least;             // hot events, of all layers, from which one row goes through them
};

// (5) W(e) = sum of v_t over the occurrences (t, e), per hot event, as a
// gather over the event-major YET.  Workgroup i works on trial slice i mod 8
// only, which keeps its gathers of v in the L2 of one XCD; a group of G
// lanes owns one hot event at a time, reads its list coalesced (G
// consecutive entries per step, streamed past the cache) and sums the
// trials' fixed-point weights; the group's sums meet in a lane reduction and
// the eight slice sums in one integer atomic add per (event, row) -- exact
// in any order.
// Workgroup wi of nw on slice x, `threads` threads; kU entries per lane in
// flight.
template <int CS, int G, int kU>
__device__ __forceinline__ void gather_w(const BwdGather &P, int x, int wi, int nw, int j, int threads) {
    const int tid = static_cast<int>(threadIdx.x);
    const int64_t tx0 = static_cast<int64_t>(x) * P.slice_trials;
    const int64_t ulo = max<int64_t>(P.t0 - tx0, 0), uhi = min<int64_t>(P.t1 - tx0, P.slice_trials);
    if (uhi <= ulo) return;   // the slice lies outside the call's trials
    const uint32_t u0 = static_cast<uint32_t>(ulo), span = static_cast<uint32_t>(uhi - ulo);
    const int64_t *vq = P.vq + (static_cast<size_t>(j) * P.n + static_cast<size_t>(tx0 + ulo - P.t0)) * CS;
    const int H = P.hot_base[static_cast<size_t>(j) * (P.n_sr + 1) + P.n_sr];
    const int32_t *hev = P.hot_ev + static_cast<size_t>(j) * P.catalog;
    const int64_t *off = P.tr_off + static_cast<int64_t>(x) * P.catalog;
    int64_t *Wj = P.W + static_cast<size_t>(j) * P.n_cot * P.catalog;
    const int sub = tid & (G - 1);
    const int ngrp = nw * threads / G;
    // wavefronts to the workgroups in turn: a few hundred events, of long lists,
    // are then walked on all CUs (1000 events, 400,000 x 1000: 1561 us in
    // workgroups of 256 threads, in these 2516 when the first ones took them all)
    for (int g = ((tid / kWave * nw + wi) * kWave + tid % kWave) / G; g < H; g += ngrp) {
        const int e = hev[g];
        const int64_t o0 = off[e], o1 = off[e + 1];
        int64_t acc[CS];
#pragma unroll
        for (int c = 0; c < CS; ++c) acc[c] = 0;
        for (int64_t i = o0 + sub; i < o1; i += G * kU) {
            uint32_t d[kU];
#pragma unroll
            for (int v = 0; v < kU; ++v)
                d[v] = (i + v * G < o1) ? __builtin_nontemporal_load(P.tr_ent + i + v * G) - u0 : span;   // span = skip
#pragma unroll
            for (int v = 0; v < kU; ++v) {
                if (d[v] < span) {
                    const int64_t *q = vq + static_cast<size_t>(d[v]) * CS;
                    if constexpr (CS == 1) {
                        acc[0] += q[0];
                    } else {
#pragma unroll
                        for (int h = 0; h < CS; h += 2) {
                            const longlong2 t = *reinterpret_cast<const longlong2 *>(q + h);
                            acc[h] += t.x;
                            acc[h + 1] += t.y;
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CS; ++c)
            for (int s = G / 2; s > 0; s >>= 1) acc[c] += __shfl_xor(acc[c], s, G);
        if (sub == 0) {
#pragma unroll
            for (int c = 0; c < CS; ++c)
                if (c < P.n_cot && acc[c] != 0)
                    atomicAdd(reinterpret_cast<unsigned long long *>(&Wj[static_cast<size_t>(c) * P.catalog + g]),
                              static_cast<unsigned long long>(acc[c]));
        }
    }
}

template <int CS, int G>
__global__ __launch_bounds__(256) void k_bwd_w(BwdGather P) {
    const int j = blockIdx.y;
    if (P.use_sp && form_of(P.sp, j) != kDense) return;   // W comes from the other forms
    gather_w<CS, G, 2>(P, blockIdx.x % kSlices, blockIdx.x / kSlices, gridDim.x / kSlices, j, 256);
}

// One row over the event-ordered blocks.  The gather fetches 8 bytes of v per
// occurrence from L2, a line each, and is bound by the lines (131e9 a second).
// Here a workgroup keeps its share of the hot events, up to two per thread, and
// goes through the blocks of trials with a block's v, 64 KB, in LDS: the lists
// are read once, two bytes an occurrence, W stays in a register and is stored
// once.  The next block's v, headers and first eight entries are loaded while
// the present one's are added.  Every workgroup stages all of v, which costs
// about as much as the lists, so there is one per CU and no more (two, of one
// event per thread, 209 us where this takes 187; the gather 262: 300,000 x
// 800, two layers of 10 and 15 ELTs).  The layers' workgroups over one part of
// the catalogue run on one XCD, block by block together, and share the lists
// in L2.  Which of the two serves a layer: ev_least.
constexpr int kBwdEvThreads = 1024;
constexpr int kEvPer = 2;                // hot events per thread
constexpr uint32_t kBwdLongList = 256;   // lists beyond this many entries are added by the whole wavefront

// A barrier for LDS alone: the loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int G>
__global__ __launch_bounds__(kBwdEvThreads) void k_bwd_w1(BwdGather P) {
    __shared__ int64_t v[2][kEvMaxTrials];
    const int i = blockIdx.x, x = i & (kXcds - 1);
    int64_t hot = 0;   // of all layers
    for (int l = threadIdx.x & 63; l < P.n_layers; l += kWave) hot += P.hot_base[static_cast<size_t>(l) * (P.n_sr + 1) + P.n_sr];
    for (int o = 32; o > 0; o >>= 1) hot += __shfl_xor(hot, o);
    if (hot < P.ev_least) {   // uniform, and the same in every workgroup
        // the gather, one layer after another over all the workgroups, so that
        // an XCD's L2 holds one slice of one layer's v (of three layers at once
        // some 1240 us where this order took 810 to 855)
        static_assert(kXcds == kSlices, "a slice per XCD");
        for (int l = 0; l < P.n_layers; ++l)
            if (!P.use_sp || form_of(P.sp, l) == kDense)
                gather_w<1, G, 4>(P, x, i / kSlices, static_cast<int>(gridDim.x) / kSlices, l, kBwdEvThreads);
        return;
    }
    const int j = (i / kXcds) % P.n_layers;
    const int wg = (i / kXcds) / P.n_layers * kXcds + x, n_wg = static_cast<int>(gridDim.x) / P.n_layers;
    if (P.use_sp && form_of(P.sp, j) != kDense) return;   // uniform: W comes from the other forms
    const int H = P.hot_base[static_cast<size_t>(j) * (P.n_sr + 1) + P.n_sr];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t *vq = P.vq + static_cast<size_t>(j) * P.n;
    const int32_t *hev = P.hot_ev + static_cast<size_t>(j) * P.catalog;
    const EvBlocks &B = P.B;
    const int b0 = static_cast<int>(P.t0 / B.et), b1 = static_cast<int>((P.t1 + B.et - 1) / B.et);
    const int g1 = static_cast<int>(static_cast<int64_t>(H) * (wg + 1) / n_wg);
    // v of the trials k 1024 + tid of block b, 0 outside the call's
    constexpr int kPer = kEvMaxTrials / kBwdEvThreads;
    int64_t nv[kPer];
    auto load_v = [&](int b) {
        const int64_t base = static_cast<int64_t>(b) * B.et - P.t0;   // the block's trial 0 in the call
        const int lo = static_cast<int>(max<int64_t>(-base, 0)), hi = static_cast<int>(min<int64_t>(P.n - base, B.et));
        const char *vb = reinterpret_cast<const char *>(vq + base);
        uint32_t at = static_cast<uint32_t>(tid) * 8u;
        asm("" : "+v"(at));   // formed here: eight addresses kept from the loop's start would be spilled
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int t = k * kBwdEvThreads + tid;
            nv[k] = 0;
            if (t >= lo && t < hi) nv[k] = *reinterpret_cast<const int64_t *>(vb + k * kBwdEvThreads * 8 + at);
        }
    };
    auto put_v = [&](int b) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) v[b & 1][k * kBwdEvThreads + tid] = nv[k];
    };
    for (int gb = static_cast<int>(static_cast<int64_t>(H) * wg / n_wg); gb < g1; gb += kEvPer * kBwdEvThreads) {   // uniform
        int e[kEvPer];   // the thread's events, -1: none
        int64_t acc[kEvPer];
        uint32_t s[kEvPer], c[kEvPer];   // their lists in the present block
        EvEight d[kEvPer] = {};          // and the first entries
        uint2 h[kEvPer];                 // the next block's headers
#pragma unroll
        for (int q = 0; q < kEvPer; ++q) {
            const int g = gb + q * kBwdEvThreads + tid;
            e[q] = g < g1 ? hev[g] : -1;
            acc[q] = 0;
        }
        auto load_hdr = [&](int b, int q) -> uint2 {
            const int ev = max(e[q], 0);   // event 0's lists (always there) for threads without one
            if (b >= b1) return make_uint2(0u, 0u);
            if (B.dense) {
                const uint32_t *p = B.start + static_cast<size_t>(b) * (B.catalog + 1) + ev;
                return make_uint2(p[0], p[1]);
            }
            return B.hdr[static_cast<size_t>(b) * B.ng + (ev >> 3)];
        };
        auto find = [&](int b, int q, uint32_t &s1, uint32_t &c1) {
            if (B.dense) {
                s1 = h[q].x;
                c1 = h[q].y - h[q].x;
            } else {
                ev_short_list(h[q], static_cast<uint32_t>(e[q]) & 7u, s1, c1);
                if (e[q] >= 0 && ev_long(h[q].y)) ev_list(B, b, e[q], s1, c1);
            }
            if (e[q] < 0 || b >= b1) c1 = 0;
        };
        auto load8 = [&](int b, uint32_t at, EvEight &to) { to = *reinterpret_cast<const EvEight *>(B.ent + B.base[b] + at); };
        auto add8 = [&](const int64_t *vb, const EvEight &en, uint32_t n, int64_t &to) {
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k)
                if (k < n) to += vb[((k & 1u) ? en.a[k >> 1] >> 16 : en.a[k >> 1]) & kEvTrialMask];
        };
        load_v(b0);
#pragma unroll
        for (int q = 0; q < kEvPer; ++q) h[q] = load_hdr(b0, q);
#pragma unroll
        for (int q = 0; q < kEvPer; ++q) {
            find(b0, q, s[q], c[q]);
            if (c[q] > 0) load8(b0, s[q], d[q]);
            h[q] = load_hdr(b0 + 1, q);
        }
        __syncthreads();   // the last batch's v has been read
        put_v(b0);
        __syncthreads();
        for (int b = b0; b < b1; ++b) {
            const int64_t *vb = v[b & 1];
            if (b + 1 < b1) load_v(b + 1);
            uint32_t s1[kEvPer], c1[kEvPer];
            EvEight d1[kEvPer] = {};
#pragma unroll
            for (int q = 0; q < kEvPer; ++q) {
                find(b + 1, q, s1[q], c1[q]);
                if (c1[q] > 0) load8(b + 1, s1[q], d1[q]);
                h[q] = load_hdr(b + 2, q);
            }
#pragma unroll
            for (int q = 0; q < kEvPer; ++q) {
                for (uint64_t big = __ballot(c[q] > kBwdLongList); big; big &= big - 1) {
                    const int l = __builtin_ctzll(big);
                    const uint32_t sl = __shfl(s[q], l), cl = __shfl(c[q], l);
                    const uint16_t *ent = B.ent + B.base[b] + sl;
                    unsigned long long sum = 0;
                    for (uint32_t k = lane; k < cl; k += kWave) sum += static_cast<unsigned long long>(vb[ent[k] & kEvTrialMask]);
                    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
                    if (lane == l) {
                        acc[q] = static_cast<int64_t>(static_cast<unsigned long long>(acc[q]) + sum);
                        c[q] = 0;
                    }
                }
                add8(vb, d[q], c[q], acc[q]);
                for (uint32_t k = 8; __any(k < c[q]); k += 8)
                    if (k < c[q]) {
                        load8(b, s[q] + k, d[q]);
                        add8(vb, d[q], c[q] - k, acc[q]);
                    }
                s[q] = s1[q];
                c[q] = c1[q];
                d[q] = d1[q];
            }
            // block b + 1's buffer was last read before the barrier that ended block b - 1
            if (b + 1 < b1) put_v(b + 1);
            lds_barrier();
        }
#pragma unroll
        for (int q = 0; q < kEvPer; ++q)
            if (e[q] >= 0) P.W[static_cast<size_t>(j) * P.catalog + gb + q * kBwdEvThreads + tid] = acc[q];
    }
}

template <int G>
static void launch_bwd_w(int cs, dim3 grid, hipStream_t st, const BwdGather &S, double mean_list) {
    if (cs == 1 && S.ev_least == INT64_MAX && mean_list >= 4096.0) {
        // lists so long that a wavefront takes each: of a few events, a group of
        // 16 lanes walks its list alone (20 events of 62,500 a list 0.9 to 1.8 ms)
        k_bwd_w<1, kWave><<<grid, 256, 0, st>>>(S);
    } else if (cs == 1 && S.ev_least == INT64_MAX) {
        // the gather for sure: in workgroups of 256 (frequencies as u^6, one event
        // in a tenth of the occurrences, 7.6 ms; in those of k_bwd_w1 9.1; 20
        // events 0.93 and 1.6)
        k_bwd_w<1, G><<<grid, 256, 0, st>>>(S);
    } else if (cs == 1) {
        // a workgroup per CU over the layers, a multiple of the slices for each
        const int per = std::max(1, device_cu_count() / (S.n_layers * kXcds));
        k_bwd_w1<G><<<static_cast<unsigned>(per * kXcds) * static_cast<unsigned>(S.n_layers), kBwdEvThreads, 0, st>>>(S);
    } else if (cs == 2) k_bwd_w<2, G><<<grid, 256, 0, st>>>(S);
    else k_bwd_w<4, G><<<grid, 256, 0, st>>>(S);
}

// (5a) the common value of every row: of 0 and the values at seven sampled
// trials, the one held by most of 1024 evenly spaced trials (the first on
// ties); and the second value, of all rows together: of the same eight, the
// one held by most of those trials that do not have the common one in every
// row.  Any choice gives the same W; a good one keeps the list of deviating
// trials short.  One workgroup per layer.
constexpr int kPickSamples = 1024;

__global__ __launch_bounds__(kPickSamples) void k_bwd_pick(BwdSparse P) {
    __shared__ uint32_t cnt[kMaxCot * kCand], cnt2[kCand];
    __shared__ int64_t cm[kMaxCot];
    const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    if (tid < kMaxCot * kCand) cnt[tid] = 0;
    if (tid < kCand) cnt2[tid] = 0;
    __syncthreads();
    const int64_t t = (static_cast<int64_t>(tid) * P.n) / kPickSamples;
    const int64_t *q = P.vq + (static_cast<size_t>(j) * P.n + t) * P.cs;
    uint32_t same = (1u << kCand) - 1u;   // candidates that the trial equals in every row
    for (int c = 0; c < P.n_cot; ++c) {
        const int64_t v = q[c];
        for (int k = 0; k < kCand; ++k) {
            const bool is = v == cand_value(P, j, c, k);
            const uint64_t m = __ballot(is);
            if (lane == 0 && m) atomicAdd(&cnt[c * kCand + k], static_cast<uint32_t>(__popcll(m)));
            if (!is) same &= ~(1u << k);
        }
    }
    __syncthreads();
    if (tid < kMaxCot) {
        int64_t v = 0;
        if (tid < P.n_cot) {
            int best = 0;
            for (int k = 1; k < kCand; ++k)
                if (cnt[tid * kCand + k] > cnt[tid * kCand + best]) best = k;
            v = cand_value(P, j, tid, best);
        }
        cm[tid] = v;
        P.common[static_cast<size_t>(j) * kMaxCot + tid] = v;
    }
    __syncthreads();
    bool dev = false;
    for (int c = 0; c < P.n_cot; ++c) dev = dev || q[c] != cm[c];
    for (int k = 0; k < kCand; ++k) {
        const uint64_t m = __ballot(dev && ((same >> k) & 1u));
        if (lane == 0 && m) atomicAdd(&cnt2[k], static_cast<uint32_t>(__popcll(m)));
    }
    __syncthreads();
    if (tid < kMaxCot) {
        int best = 0;
        for (int k = 1; k < kCand; ++k)
            if (cnt2[k] > cnt2[best]) best = k;
        P.alt[static_cast<size_t>(j) * kMaxCot + tid] =
            cnt2[best] == 0 ? cm[tid] : (tid < P.n_cot ? cand_value(P, j, tid, best) : 0);
    }
}

// (5b) the trials that do not have the common value in every row: those of
// the second value, as a list and as bits, and the others, as a list.  A
// workgroup gathers those of its chunk of kDevChunk trials in LDS and reserves
// their place in each list with one atomic.
__global__ __launch_bounds__(1024) void k_bwd_dev(BwdSparse P) {
    __shared__ int32_t buf[kDevChunk];   // of neither value from the front, of the second from the back
    __shared__ uint32_t nbuf, nab;
    __shared__ unsigned long long base, abase;
    const int j = blockIdx.y, lane = threadIdx.x & 63;
    int64_t cm[kMaxCot], am[kMaxCot];
#pragma unroll
    for (int c = 0; c < kMaxCot; ++c) {
        cm[c] = P.common[static_cast<size_t>(j) * kMaxCot + c];
        am[c] = P.alt[static_cast<size_t>(j) * kMaxCot + c];
    }
    if (threadIdx.x == 0) nbuf = nab = 0;
    __syncthreads();
    const int64_t *q = P.vq + static_cast<size_t>(j) * P.n * P.cs;
    uint2 *ab = P.abits + static_cast<size_t>(j) * P.aw;
    const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kDevChunk;
    const int64_t c1 = min<int64_t>(c0 + kDevChunk, P.n);
    for (int64_t t0 = c0; t0 < c1; t0 += blockDim.x) {   // uniform
        const int64_t t = t0 + threadIdx.x;
        bool d = false, a = true;
        if (t < c1)
#pragma unroll
            for (int c = 0; c < kMaxCot; ++c)
                if (c < P.n_cot) {
                    const int64_t v = q[static_cast<size_t>(t) * P.cs + c];
                    d = d || v != cm[c];
                    a = a && v == am[c];
                }
        a = a && d;
        d = d && !a;
        const uint64_t m = __ballot(d), ma = __ballot(a);
        if (lane == 0 && t < c1) ab[t >> 6] = make_uint2(static_cast<uint32_t>(ma), static_cast<uint32_t>(ma >> 32));
        if (m) {
            uint32_t wb = 0;
            if (lane == 0) wb = atomicAdd(&nbuf, static_cast<uint32_t>(__popcll(m)));
            wb = __shfl(wb, 0);
            if (d) buf[wb + lanes_under(m)] = static_cast<int32_t>(t);
        }
        if (ma) {
            uint32_t wb = 0;
            if (lane == 0) wb = atomicAdd(&nab, static_cast<uint32_t>(__popcll(ma)));
            wb = __shfl(wb, 0);
            if (a) buf[kDevChunk - 1 - (wb + lanes_under(ma))] = static_cast<int32_t>(t);
        }
    }
    __syncthreads();
    const uint32_t nb = nbuf, na = nab;
    if (threadIdx.x == 0 && nb) base = atomicAdd(&P.ndev[j], static_cast<unsigned long long>(nb));
    if (threadIdx.x == 0 && na) abase = atomicAdd(&P.nalt[j], static_cast<unsigned long long>(na));
    __syncthreads();
    int32_t *dv = P.dev + static_cast<size_t>(j) * P.n;
    for (uint32_t i = threadIdx.x; i < nb; i += blockDim.x) dv[base + i] = buf[i];
    for (uint32_t i = threadIdx.x; i < na; i += blockDim.x) dv[P.n - 1 - static_cast<int64_t>(abase + i)] = buf[kDevChunk - 1 - i];
}

// (5c) the counted part of W(e) for every hot event: c times the occurrences
// of e in the call's trials and, in the third form, (a - c) times those in
// trials of the second value a.  (The accumulators are zero from step 4.)
//
// The first comes from the event-major offsets: over all trials the
// per-event totals, over part of them the list lengths of the slices inside
// the range and, of the slices it cuts (at most two), the list entries in
// range, counted.  The second counts the entries of every slice whose trial's
// bit is set, the slice's bits in LDS: a bit from LDS per entry, where the
// first form gathers each trial's rows from L2 (32 bytes each with three
// rows, 620 us for half of 1M trials of 1000 and 15 ELTs).  Behind the quote
// server, three rows over parts of 1M trials of 1000, years above the
// aggregate limit in a third of the layers: 136 us a quote, where the gather,
// the counts and the cut slices in kernels of their own took 250.
//
// Workgroup i works on slice i mod 8 (second form: on a cut slice, so that all
// of them have work); G lanes per hot event read its list coalesced; the
// counts meet W in one integer atomic per row.
template <int G>
__global__ __launch_bounds__(256) void k_bwd_count(BwdSparse P, int2 cut, int ncut) {
    extern __shared__ uint32_t bits[];
    constexpr int kU = 4;
    const int j = blockIdx.y, tid = threadIdx.x;
    const int form = form_of(P, j);
    if (form == kDense) return;   // uniform
    int64_t cm[kMaxCot], da[kMaxCot];
#pragma unroll
    for (int c = 0; c < kMaxCot; ++c) {
        cm[c] = P.common[static_cast<size_t>(j) * kMaxCot + c];
        da[c] = static_cast<int64_t>(static_cast<unsigned long long>(P.alt[static_cast<size_t>(j) * kMaxCot + c]) -
                                     static_cast<unsigned long long>(cm[c]));
    }
    const bool any_c = common_nonzero(P, j);
    const int H = P.hot_base[static_cast<size_t>(j) * (P.n_sr + 1) + P.n_sr];
    const int32_t *hev = P.hot_ev + static_cast<size_t>(j) * P.catalog;
    int64_t *Wj = P.W + static_cast<size_t>(j) * P.n_cot * P.catalog;
    auto add = [&](int g, uint64_t n_c, uint64_t n_a) {   // exact modulo 2^64, like every sum below
#pragma unroll
        for (int c = 0; c < kMaxCot; ++c)
            if (c < P.n_cot) {
                const unsigned long long v = static_cast<unsigned long long>(cm[c]) * n_c + static_cast<unsigned long long>(da[c]) * n_a;
                if (v != 0) atomicAdd(reinterpret_cast<unsigned long long *>(&Wj[static_cast<size_t>(c) * P.catalog + g]), v);
            }
    };
    if (any_c) {
        const bool all = P.t0 == 0 && P.n == P.n_trials;   // uniform
        for (int g = blockIdx.x * 256 + tid; g < H; g += gridDim.x * 256) {
            const int e = hev[g];
            int64_t cnt = 0;
            if (all) {
                cnt = P.t_cnt[e];
            } else {
#pragma unroll
                for (int x = 0; x < kSlices; ++x)
                    if (slice_inside(P, x)) {
                        const int64_t *off = P.tr_off + static_cast<int64_t>(x) * P.catalog;
                        cnt += off[e + 1] - off[e];
                    }
            }
            add(g, static_cast<uint64_t>(cnt), 0);
        }
    }
    const bool two = form == kTwoValues;
    if (!two && (ncut == 0 || !any_c)) return;   // uniform
    const int ns = two ? kSlices : ncut;
    const int k = blockIdx.x % ns, wi = blockIdx.x / ns, nw = gridDim.x / ns;
    if (wi >= nw) return;   // uniform
    const int x = two ? k : (k == 0 ? cut.x : cut.y);
    const bool is_cut = any_c && slice_cut(P, x);
    const int64_t tx0 = static_cast<int64_t>(x) * P.slice_trials;
    const int64_t ulo = max<int64_t>(P.t0 - tx0, 0), uhi = min<int64_t>(P.t0 + P.n - tx0, P.slice_trials);
    if (uhi <= ulo || (!two && !is_cut)) return;   // uniform: nothing of the slice is asked for
    const uint32_t u0 = static_cast<uint32_t>(ulo), span = static_cast<uint32_t>(uhi - ulo);
    uint32_t first = 0;   // bit of the slice's first trial in range
    if (two) {
        const int64_t b0 = tx0 + ulo - P.t0;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(P.abits + static_cast<size_t>(j) * P.aw);
        first = static_cast<uint32_t>(b0 & 31);
        const int nwords = static_cast<int>((first + span + 31) / 32);
        for (int i = tid; i < nwords; i += 256) bits[i] = src[(b0 >> 5) + i];
        __syncthreads();
    }
    const int64_t *off = P.tr_off + static_cast<int64_t>(x) * P.catalog;
    const int sub = tid & (G - 1);
    const int ngrp = nw * 256 / G;
    for (int g = (wi * 256 + tid) / G; g < H; g += ngrp) {
        const int e = hev[g];
        const int64_t o0 = off[e], o1 = off[e + 1];
        uint32_t cnt = 0, na = 0;
        for (int64_t i = o0 + sub; i < o1; i += G * kU) {
            uint32_t d[kU];
#pragma unroll
            for (int v = 0; v < kU; ++v)
                d[v] = (i + v * G < o1) ? __builtin_nontemporal_load(P.tr_ent + i + v * G) - u0 : span;   // span = skip
#pragma unroll
            for (int v = 0; v < kU; ++v) {
                const bool in = d[v] < span;
                cnt += in ? 1u : 0u;
                if (two) {
                    const uint32_t b = first + (in ? d[v] : 0u);
                    na += in ? (bits[b >> 5] >> (b & 31u)) & 1u : 0u;
                }
            }
        }
        for (int s2 = G / 2; s2 > 0; s2 >>= 1) {
            cnt += static_cast<uint32_t>(__shfl_xor(static_cast<int>(cnt), s2, G));
            na += static_cast<uint32_t>(__shfl_xor(static_cast<int>(na), s2, G));
        }
        if (sub == 0) add(g, is_cut ? cnt : 0u, na);
    }
}

// (5d) the deviating trials of the range: a wavefront per trial, or P.segs of
// them where trials have more events than a wavefront takes in one round, adds
// v_t - c to W of each hot event of the trial, one integer atomic per
// (occurrence, row).  Whether an event is hot is asked of its bit in LDS
// first, the hot events' bitmap folded onto 2^19 bits by OR: a table word per
// occurrence is a line from L2 each, 43 of the 70 us that 10,000 trials of
// 1000 took (2M events, 7% hot); with the filter 51 us.
constexpr int kHotFilter = 1 << 14;   // words, 64 KB: two workgroups on a CU
constexpr int kSparseThreads = 1024;
constexpr int kSparseRound = 1024;      // events of a trial in flight

__global__ __launch_bounds__(kSparseThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_bwd_wsparse(BwdSparse P) {
    __shared__ uint32_t filt[kHotFilter];
    const int j = blockIdx.y, lane = threadIdx.x & 63;
    const int form = form_of(P, j);
    if (form == kDense) return;   // uniform over the workgroup
    const int64_t ndev = static_cast<int64_t>(P.ndev[j]);
    const int64_t nwalk = ndev + (form == kOneValue ? static_cast<int64_t>(P.nalt[j]) : 0);
    if (static_cast<int64_t>(blockIdx.x) * (kSparseThreads >> 6) >= nwalk * P.segs) return;   // uniform: no trial for it
    const OccTables T = load_tables(P.tabs + j);
    const uint4 *bits = reinterpret_cast<const uint4 *>(T.bits);
    const int n4 = P.n_sr * (kSrWords / 4);
#pragma unroll
    for (int k = 0; k < kHotFilter / 4 / kSparseThreads; ++k) {
        const int f = k * kSparseThreads + static_cast<int>(threadIdx.x);
        uint4 m = make_uint4(0u, 0u, 0u, 0u);
        for (int i = f; i < n4; i += 4 * (kHotFilter / 4)) {   // four pieces in flight
            uint4 b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) b[u] = bits[min(i + u * (kHotFilter / 4), n4 - 1 - (n4 - 1 - f) % (kHotFilter / 4))];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                m.x |= b[u].x;
                m.y |= b[u].y;
                m.z |= b[u].z;
                m.w |= b[u].w;
            }
        }
        reinterpret_cast<uint4 *>(filt)[f] = m;
    }
    __syncthreads();
    const int32_t *hb = P.hot_base + static_cast<size_t>(j) * (P.n_sr + 1);
    const int64_t *q = P.vq + static_cast<size_t>(j) * P.n * P.cs;
    int64_t *Wj = P.W + static_cast<size_t>(j) * P.n_cot * P.catalog;
    const int waves = gridDim.x * (blockDim.x >> 6);
    for (int64_t is = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); is < nwalk * P.segs; is += waves) {
        unsigned long long dl[kMaxCot];
        const int64_t i = is / P.segs;
        const int seg = static_cast<int>(is - i * P.segs);
        const int32_t u = P.dev[static_cast<size_t>(j) * P.n + (i < ndev ? i : P.n - 1 - (i - ndev))];
#pragma unroll
        for (int c = 0; c < kMaxCot; ++c)
            dl[c] = c < P.n_cot ? static_cast<unsigned long long>(q[static_cast<size_t>(u) * P.cs + c]) -
                                      static_cast<unsigned long long>(P.common[static_cast<size_t>(j) * kMaxCot + c])
                                : 0ull;
        const int64_t t = P.t0 + u;
        const int64_t a = P.t_off[t], b = P.t_off[t + 1];
        constexpr int kU = kSparseRound / kWave;   // events per lane in flight
        for (int64_t k0 = a + static_cast<int64_t>(seg) * kSparseRound; k0 < b; k0 += static_cast<int64_t>(P.segs) * kSparseRound) {
            int e[kU];
#pragma unroll
            for (int v = 0; v < kU; ++v) {
                const int64_t k = k0 + v * 64 + lane;
                e[v] = k < b ? P.t_ids[k] : -1;
            }
#pragma unroll
            for (int v = 0; v < kU; ++v)
                if (e[v] >= 0 && !((filt[(e[v] >> 5) & (kHotFilter - 1)] >> (e[v] & 31)) & 1u)) e[v] = -1;
            uint2 w[kU];
#pragma unroll
            for (int v = 0; v < kU; ++v) {
                w[v] = make_uint2(0u, 0u);
                if (e[v] >= 0) w[v] = T.br[e[v] >> 5];   // word e / 32 of the table
            }
#pragma unroll
            for (int v = 0; v < kU; ++v) {
                if (e[v] < 0) continue;
                const int s = e[v] >> kSrBits;
                const uint32_t bit = static_cast<uint32_t>(e[v] & 31);
                if ((w[v].x >> bit) & 1u) {
                    const int g = hb[s] + static_cast<int>(w[v].y + __popc(w[v].x & ((1u << bit) - 1u)));
#pragma unroll
                    for (int c = 0; c < kMaxCot; ++c)
                        if (dl[c])
                            atomicAdd(reinterpret_cast<unsigned long long *>(&Wj[static_cast<size_t>(c) * P.catalog + g]), dl[c]);
                }
            }
        }
    }
}

struct BwdGrad {
    const float *loss;
    const uint32_t *present;
    int32_t catalog, words;
    const int32_t *elt_off, *elt_ids;
    const double *elt_terms, *layer_terms;
    const OccTables *tabs;
    const int64_t *W;              // [n_layers][n_cot][catalog] by hot index
    const int32_t *hot_base;       // [n_layers][n_sr + 1]
    const int32_t *hot_ev;         // [n_layers][catalog]
    int32_t n_sr, n_cot, n_cw, n_elt_slots;   // cw = (workgroup, wavefront); slots = ELT positions of all layers
    const VScale *vs;
    double *part_elt;    // [n_cw / kGradWaves][n_elt_slots][n_cot][3]
    double *part_occ;    // [n_layers][n_cw][n_cot][2]
};

constexpr int kGradThreads = 256;                  // hot events per workgroup
constexpr int kGradWaves = kGradThreads / kWave;   // 4
constexpr int kGradBatch = 16;                     // ELTs whose presence words are loaded together
constexpr int kGradLoss = 4;                       // losses of one event loaded together

// LDS of k_bwd_grad for layers of up to J ELTs: the ELTs' terms, and every
// wavefront's sums.
static size_t grad_lds(int J, int n_cot) {
    return static_cast<size_t>(J) * (3 * sizeof(double) + sizeof(int64_t) + kGradWaves * n_cot * 3 * sizeof(double));
}

// (6) W(e) times the derivatives of O(e), over the layer's hot events
// (the only ones with W), one per thread: workgroup i takes hot indices
// 256 i .. 256 i + 255.  A thread asks only the ELTs that hold its event and
// adds each one's terms to its wavefront's sums in LDS: additions of one
// wavefront to one address apply in lane order and one instruction after
// another, so a wavefront's sums have a fixed order; the workgroup's are its
// wavefronts' in order, and the final sums (a fixed order over workgroups)
// are deterministic.  Forming every ELT's sums over a wavefront's lanes
// instead, nine reductions per ELT for three rows, took some 3900
// instructions per wavefront and 37 us (15 ELTs, 146,000 hot events, one
// row); 6.7 us.  Three rows among other work on the device 72 and 24 us.
__global__ __launch_bounds__(kGradThreads) void k_bwd_grad(BwdGrad P) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int hb = blockIdx.x, j = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int32_t *hbase = P.hot_base + static_cast<size_t>(j) * (P.n_sr + 1);
    const int H = hbase[P.n_sr];
    const int g0 = hb * kGradThreads;
    if (g0 >= H) return;   // uniform; the final sums read only the slots of workgroups with hot events
    const int a = P.elt_off[j];
    const int J = P.elt_off[j + 1] - a;
    const int vals = P.n_cot * 3;                          // sums per ELT
    double *ls = reinterpret_cast<double *>(smem);         // [J]
    double *lr = ls + J, *ll = lr + J;
    int64_t *lk = reinterpret_cast<int64_t *>(ll + J);     // [J] the ELT's index
    double *sums = reinterpret_cast<double *>(lk + J);     // [waves][J][n_cot][3]
    for (int q = tid; q < J; q += kGradThreads) {
        const int k = P.elt_ids[a + q];
        lk[q] = k;
        ls[q] = P.elt_terms[3 * k + 0];
        lr[q] = P.elt_terms[3 * k + 1];
        ll[q] = P.elt_terms[3 * k + 2];
    }
    for (int i = tid; i < kGradWaves * J * vals; i += kGradThreads) sums[i] = 0.0;
    __syncthreads();
    const double occL = P.layer_terms[4 * j + 1];
    const OccTables T = load_tables(P.tabs + j);

    // the thread's hot event: weight per row and occurrence-clamp branch.  O =
    // min(max(x - OccR, 0), OccL) is non-zero for these events, and it is
    // below OccL exactly when the occurrence clamp is linear.
    const int g = g0 + tid;
    const bool valid = g < H;
    const int e = valid ? P.hot_ev[static_cast<size_t>(j) * P.catalog + g] : 0;
    const int sr = e >> kSrBits;
    const double O = valid ? T.vals[static_cast<size_t>(sr) * kSr + (g - hbase[sr])] : 0.0;
    const bool lin_occ = valid && (O < occL);
    double W[kMaxCot], po[kMaxCot][2];
#pragma unroll
    for (int c = 0; c < kMaxCot; ++c) {
        W[c] = 0.0;
        if (valid && c < P.n_cot) {
            const int64_t acc = P.W[(static_cast<size_t>(j) * P.n_cot + c) * P.catalog + g];
            W[c] = ldexp(static_cast<double>(acc), -P.vs[j * P.n_cot + c].sigma);
        }
        po[c][0] = lin_occ ? 0.0 - W[c] : 0.0;
        po[c][1] = lin_occ ? 0.0 : W[c];
    }
    double *my = sums + static_cast<size_t>(w) * J * vals;
    if (lin_occ)
        for (int q0 = 0; q0 < J; q0 += kGradBatch) {
            uint32_t pw[kGradBatch];
#pragma unroll
            for (int u = 0; u < kGradBatch; ++u)
                pw[u] = P.present[static_cast<size_t>(lk[min(q0 + u, J - 1)]) * P.words + (e >> 5)];
            uint32_t held = 0;
#pragma unroll
            for (int u = 0; u < kGradBatch; ++u) held |= ((pw[u] >> (e & 31)) & 1u) << u;
            held &= J - q0 < kGradBatch ? (1u << (J - q0)) - 1u : ~0u;
            while (held) {
                float lv[kGradLoss];
                int q[kGradLoss];
#pragma unroll
                for (int u = 0; u < kGradLoss; ++u) {
                    q[u] = held ? q0 + __builtin_ctz(held) : -1;
                    held &= held - 1;
                    // element 0 (always valid) for lanes with fewer ELTs
                    lv[u] = P.loss[q[u] >= 0 ? lk[q[u]] * P.catalog + e : 0];
                }
#pragma unroll
                for (int u = 0; u < kGradLoss; ++u) {
                    if (q[u] < 0) continue;
                    const double l = static_cast<double>(lv[u]);
                    const double pre = ls[q[u]] * l - lr[q[u]];
                    const double av = (pre > 0.0) ? pre : 0.0;
                    double *to = my + q[u] * vals;
                    if (pre > 0.0 && av < ll[q[u]]) {
#pragma unroll
                        for (int c = 0; c < kMaxCot; ++c)
                            if (c < P.n_cot) {
                                atomicAdd(to + 3 * c, W[c] * l);
                                atomicAdd(to + 3 * c + 1, 0.0 - W[c]);
                            }
                    }
                    if (av >= ll[q[u]]) {
#pragma unroll
                        for (int c = 0; c < kMaxCot; ++c)
                            if (c < P.n_cot) atomicAdd(to + 3 * c + 2, W[c]);
                    }
                }
            }
        }
    // occurrence-term partials of this wavefront
    // (wavefront sums by DPP: lane 63 holds the total, in a fixed order)
    const size_t cw = static_cast<size_t>(hb) * kGradWaves + w;
#pragma unroll
    for (int c = 0; c < kMaxCot; ++c)
        if (c < P.n_cot) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const double v = wave_inclusive_sum(po[c][m]);
                if (lane == 63)
                    P.part_occ[((static_cast<size_t>(j) * P.n_cw + cw) * P.n_cot + c) * 2 + m] = v;
            }
        }
    __syncthreads();
    double *dst = P.part_elt + (static_cast<size_t>(hb) * P.n_elt_slots + a) * vals;
    for (int i = tid; i < J * vals; i += kGradThreads) {
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < kGradWaves; ++k) v += sums[k * J * vals + i];
        dst[i] = v;
    }
}

// Workgroups of k_bwd_grad that wrote partials for layer j: those with hot events.
__device__ __forceinline__ int grad_groups(const int32_t *hot_base, int n_sr, int j) {
    return (hot_base[static_cast<size_t>(j) * (n_sr + 1) + n_sr] + kGradThreads - 1) / kGradThreads;
}

// (7) fixed-order sums into the outputs: one workgroup per output value,
// each thread a fixed stride of the (chunk, wavefront) partials, eight of them
// in flight, then a fixed-order tree.
__global__ __launch_bounds__(256) void k_bwd_final(const int32_t *__restrict__ elt_off, const int32_t *__restrict__ elt_ids,
                                                  int n_layers, int n_elts, int n_cot, int n_cw,
                                                  const int32_t *__restrict__ hot_base, int n_sr, int n_elt_slots,
                                                  int nwg_v, const double *__restrict__ part_elt,
                                                  const double *__restrict__ part_occ,
                                                  const double *__restrict__ aggpart, double *__restrict__ grad_elt,
                                                  double *__restrict__ grad_layer) {
    __shared__ double red[256];
    const int o = blockIdx.x, tid = threadIdx.x;
    const int n_e = n_cot * n_elts * 3;
    double v = 0.0;
    if (o < n_e) {
        const int c = o / (n_elts * 3), k = (o / 3) % n_elts, m = o % 3;
        for (int j = 0; j < n_layers; ++j)
            for (int q = elt_off[j]; q < elt_off[j + 1]; ++q) {
                if (elt_ids[q] != k) continue;
                const int used = grad_groups(hot_base, n_sr, j);
#pragma unroll 8
                for (int i = tid; i < used; i += 256)
                    v += part_elt[((static_cast<size_t>(i) * n_elt_slots + q) * n_cot + c) * 3 + m];
            }
    } else {
        const int i = o - n_e;
        const int c = i / (n_layers * 4), j = (i / 4) % n_layers, m = i % 4;
        if (m < 2) {
            const int used = grad_groups(hot_base, n_sr, j) * kGradWaves;
#pragma unroll 8
            for (int cw = tid; cw < used; cw += 256)
                v += part_occ[((static_cast<size_t>(j) * n_cw + cw) * n_cot + c) * 2 + m];
        } else {
            for (int wg = tid; wg < nwg_v; wg += blockDim.x)
                v += aggpart[((static_cast<size_t>(j) * n_cot + c) * nwg_v + wg) * 2 + (m - 2)];
        }
    }
    red[tid] = v;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h) red[tid] += red[tid + h];
        __syncthreads();
    }
    if (tid == 0) {
        if (o < n_e) grad_elt[o] = red[0];
        else {
            const int i = o - n_e;
            const int c = i / (n_layers * 4), j = (i / 4) % n_layers, m = i % 4;
            grad_layer[(static_cast<size_t>(c) * n_layers + j) * 4 + m] = red[0];
        }
    }
}

struct BwdLayout {
    OccLayoutSizes z;
    int nwg_v, n_cw, cs;
    size_t bytes;
};

static int bwd_nwg_v(int64_t n) {   // about two trials per thread, at most 512 workgroups
    return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((n + 2047) / 2048, 512)));
}

// Hot events, of all layers, from which k_bwd_w1 goes through the event-ordered
// blocks.  A block costs every workgroup 2.6 us (its v from L2, latency) and 80
// ns for each entry of the longest list past the eighth, which all wait for, and
// the device 10 ps per hot event and 2.5 ps for each occurrence of its list past
// the fourth; the gather 280 ps per hot event and 6.5 per occurrence.  Where an
// event's lists have more than kBwdLongList entries on average the gather serves
// (400,000 x 1000 over 10,000 events 340 us, blocks 1430).  From these calls (us:
// gather, blocks): 1M x 1000 over 2M events, 15 ELTs 574, 608, 6 ELTs 279, 501;
// 300,000 x 800, two layers 407, 279, with few hot events 157, 205; 400,000 x
// 1000 over 3M, 1M, 400,000, 200,000, 120,000 and 50,000 events, a sixth of them
// hot, 646, 389; 493, 353; 462, 406; 446, 512; 430, 658; 397, 1097; a fortieth of
// 1M 155, 253; two layers over 200,000 799, 580; 100,000 x 1000 over 3M, 400,000
// and 120,000 290, 183; 196, 160; 166, 217; 100,000 x 200 over 1M 138, 134;
// frequencies as u^1.3, longest list 333, 626, 1063.  The blocks have to be a
// tenth the faster.
static int64_t ev_least(double blocks, double per_event, double longest) {
    if (longest > kBwdLongList) return INT64_MAX;
    const double list = per_event / blocks;
    const double fixed = blocks * (2.6e6 + 8e4 * std::max(longest - 8.0, 0.0));                                   // ps
    const double saved = 280.0 + 6.5 * per_event - blocks * (10.0 + 2.5 * std::max(list - 4.0, 0.0));   // per hot event
    return saved > 0.0 ? static_cast<int64_t>(std::min(1.1 * fixed / saved + 1.0, 1e15)) : INT64_MAX;
}

static int64_t dev_blocks(int64_t n) { return std::max<int64_t>(1, (n + kDevChunk - 1) / kDevChunk); }

static int64_t bit_words(int64_t n) { return (std::max<int64_t>(n, 1) + 63) / 64 + 1; }   // one past the last

static int bwd_cs(int n_cot) { return n_cot <= 1 ? 1 : (n_cot <= 2 ? 2 : 4); }

static BwdLayout bwd_layout(const ara_tables *tables, const ara_layers *layers, int n_cot, int64_t n) {
    BwdLayout B{};
    B.z = occ_sizes(tables->catalog, false);
    const int L = layers->n_layers;
    const int nJ = L > 0 ? layers->elt_off[L] : 0;
    B.nwg_v = bwd_nwg_v(n);
    B.n_cw = static_cast<int>((static_cast<int64_t>(tables->catalog) + kGradThreads - 1) / kGradThreads) * kGradWaves;
    B.cs = bwd_cs(n_cot);
    const size_t cat = static_cast<size_t>(tables->catalog);
    Carver c(nullptr);
    c.take<int32_t>(kWsHeaderBytes / 4);
    c.take<int32_t>(static_cast<size_t>(L + 1));
    c.take<int32_t>(static_cast<size_t>(std::max(nJ, 1)));
    c.take<OccTables>(static_cast<size_t>(std::max(L, 1)));
    size_t b = c.bytes() + static_cast<size_t>(L) * B.z.per_layer;
    Carver d(nullptr);
    d.take<VScale>(static_cast<size_t>(std::max(L * n_cot, 1)));
    d.take<unsigned long long>(static_cast<size_t>(std::max(L, 1)) * 2);
    d.take<int64_t>(static_cast<size_t>(std::max(L, 1)) * kMaxCot * 2);
    d.take<uint2>(static_cast<size_t>(L) * bit_words(n));
    d.take<int32_t>(static_cast<size_t>(L) * std::max<int64_t>(n, 1));
    d.take<double>(static_cast<size_t>(L) * n_cot * B.nwg_v * 2);
    d.take<int64_t>(static_cast<size_t>(L) * std::max<int64_t>(n, 1) * B.cs);
    d.take<int32_t>(static_cast<size_t>(L) * cat);
    d.take<int32_t>(static_cast<size_t>(L) * (B.z.n_sr + 1));
    d.take<int64_t>(static_cast<size_t>(L) * n_cot * cat);
    d.take<double>(static_cast<size_t>(B.n_cw / kGradWaves) * std::max(nJ, 1) * n_cot * 3);
    d.take<double>(static_cast<size_t>(L) * B.n_cw * n_cot * 2);
    B.bytes = b + d.bytes();
    return B;
}

static int32_t check_pair_b(const ara_tables *tables, const ara_yet *yet) {
    if (!tables || !yet) return fail(ARA_E_INVAL, "null tables or yet");
    if (tables->catalog != yet->catalog) return fail(ARA_E_INVAL, "tables and YET use different catalogues");
    if (yet->range_bits != kRangeBits || yet->groups != kGroups) return fail(ARA_E_INVAL, "YET not prepared by this library");
    if (yet->n_slices != kSlices || !yet->tr_off || (yet->nnz > 0 && !yet->tr_ent))
        return fail(ARA_E_INVAL, "the backward needs a YET prepared with ARA_PREP_TRANSPOSED");
    return ARA_OK;
}

}  // namespace ara

using namespace ara;

extern "C" int32_t ara_ylt_backward_workspace_bytes(const ara_tables *tables, const ara_yet *yet,
                                                    const ara_layers *layers, int32_t n_cot, size_t *bytes) {
    if (!bytes) return fail(ARA_E_INVAL, "null output");
    int32_t rc = check_pair_b(tables, yet);
    if (rc) return rc;
    if ((rc = check_layers(layers, tables->n_elts))) return rc;
    if (n_cot < 1 || n_cot > kMaxCot) return fail(ARA_E_LIMIT, "cotangent rows must be 1..ARA_MAX_COTANGENTS");
    *bytes = bwd_layout(tables, layers, n_cot, yet->n_trials).bytes;
    return ARA_OK;
}

extern "C" int32_t ara_ylt_backward(const ara_tables *tables, const ara_yet *yet, const ara_layers *layers,
                                    const double *elt_terms, const double *layer_terms, int64_t trial_begin,
                                    int64_t trial_end, const double *s_pre, int32_t n_cot, const double *grad_ylt,
                                    double *grad_elt, double *grad_layer, void *ws, size_t ws_bytes, void *stream) {
    int32_t rc = check_pair_b(tables, yet);
    if (rc) return rc;
    if ((rc = check_layers(layers, tables->n_elts))) return rc;
    if (n_cot < 1 || n_cot > kMaxCot) return fail(ARA_E_LIMIT, "cotangent rows must be 1..ARA_MAX_COTANGENTS");
    if (trial_begin < 0 || trial_end < trial_begin || trial_end > yet->n_trials)
        return fail(ARA_E_RANGE, "trial range outside the YET");
    if (!ws || !grad_elt || !grad_layer) return fail(ARA_E_INVAL, "null workspace or output");
    const int L = layers->n_layers;
    const int64_t n = trial_end - trial_begin;
    if (L > 0 && n > 0 && (!s_pre || !grad_ylt || !elt_terms || !layer_terms))
        return fail(ARA_E_INVAL, "null input");
    // workspace sized for the full trial range is valid for any sub-range
    const BwdLayout B = bwd_layout(tables, layers, n_cot, yet->n_trials);
    if (ws_bytes < B.bytes) return fail(ARA_E_NOSPACE, "backward workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (L == 0 || n == 0) {
        ARA_HIP(hipMemsetAsync(ws, 0, kWsHeaderBytes, st));
        ARA_HIP(hipMemsetAsync(grad_elt, 0, static_cast<size_t>(n_cot) * tables->n_elts * 3 * sizeof(double), st));
        if (L > 0) ARA_HIP(hipMemsetAsync(grad_layer, 0, static_cast<size_t>(n_cot) * L * 4 * sizeof(double), st));
        return ARA_OK;
    }
    // otherwise every output value is written by the final reduction

    const int nJ = layers->elt_off[L];
    Carver c(ws);
    int32_t *d_err = c.take<int32_t>(kWsHeaderBytes / 4);
    int32_t *d_off = c.take<int32_t>(static_cast<size_t>(L + 1));
    int32_t *d_ids = c.take<int32_t>(static_cast<size_t>(std::max(nJ, 1)));
    OccTables *d_tabs = c.take<OccTables>(static_cast<size_t>(L));
    VScale *vs = c.take<VScale>(static_cast<size_t>(L * n_cot));
    unsigned long long *ndev = c.take<unsigned long long>(static_cast<size_t>(L) * 2);
    int64_t *common = c.take<int64_t>(static_cast<size_t>(L) * kMaxCot * 2);
    std::vector<OccTables> tabs(static_cast<size_t>(L));
    for (int j = 0; j < L; ++j) tabs[j] = occ_carve(c, B.z, false);
    double *aggpart = c.take<double>(static_cast<size_t>(L) * n_cot * bwd_nwg_v(n) * 2);
    int64_t *vq = c.take<int64_t>(static_cast<size_t>(L) * n * B.cs);
    int32_t *hot_ev = c.take<int32_t>(static_cast<size_t>(L) * tables->catalog);
    int32_t *hot_base = c.take<int32_t>(static_cast<size_t>(L) * (B.z.n_sr + 1));
    int64_t *W = c.take<int64_t>(static_cast<size_t>(L) * n_cot * tables->catalog);
    double *part_elt = c.take<double>(static_cast<size_t>(B.n_cw / kGradWaves) * std::max(nJ, 1) * n_cot * 3);
    double *part_occ = c.take<double>(static_cast<size_t>(L) * B.n_cw * n_cot * 2);
    int32_t *dev = c.take<int32_t>(static_cast<size_t>(L) * std::max<int64_t>(n, 1));
    const int64_t aw = bit_words(n);
    uint2 *abits = c.take<uint2>(static_cast<size_t>(L) * aw);
    HeadImage img(ws);   // clears the error header, the weight scales and the deviating-trial counts
    img.put(d_off, layers->elt_off, static_cast<size_t>(L + 1));
    img.put(d_ids, layers->elt_ids, static_cast<size_t>(nJ));
    img.put(d_tabs, tabs.data(), tabs.size());
    img.cover(ndev + 2 * L);
    if ((rc = img.send(st))) return rc;

    {
        ProfScope prof(ARA_PROF_OCC, st);
        if ((rc = launch_occ(tables, d_off, d_ids, elt_terms, layer_terms, L, false, false, d_tabs, B.z.n_sr, d_err,
                             layers_max_j(layers), st)))
            return rc;
    }
    const int nwg_v = bwd_nwg_v(n);
    {
        ProfScope prof(ARA_PROF_BWD_RED, st);
        k_bwd_vmax<<<dim3(nwg_v, L), kBwdThreads, 0, st>>>(grad_ylt, s_pre, layer_terms, n, L, n_cot, nwg_v, vs, aggpart);
        const unsigned gx = static_cast<unsigned>(std::min<int64_t>((n + 255) / 256, 2048));
        k_bwd_vq<<<dim3(gx, L), 256, 0, st>>>(grad_ylt, s_pre, layer_terms, n, L, n_cot, B.cs, yet->max_occ, vs, vq);
        k_bwd_hot<<<dim3(B.z.n_sr, L), 256, 0, st>>>(d_tabs, B.z.n_sr, n_cot, tables->catalog, hot_ev, hot_base, W);
        ARA_HIP(hipGetLastError());
    }
    BwdGather S{};
    S.tr_off = yet->tr_off;
    S.tr_ent = yet->tr_ent;
    S.catalog = tables->catalog;
    S.n_sr = B.z.n_sr;
    S.n_cot = n_cot;
    S.n_layers = L;
    S.ev_least = INT64_MAX;
    if (ev_blocks(yet, &S.B) && S.B.et <= kEvMaxTrials && yet->nnz > 0) {
        const double blocks = static_cast<double>((trial_end + S.B.et - 1) / S.B.et - trial_begin / S.B.et);
        const double per_event = static_cast<double>(yet->nnz) / tables->catalog * static_cast<double>(n) / yet->n_trials;
        const double longest = static_cast<double>(yet->max_occ) / S.B.neb;   // mean list of the most frequent event
        S.ev_least = ev_always_backward(yet) ? 0 : ev_least(blocks, per_event, longest);
    }
    S.slice_trials = yet->slice_trials;
    S.t0 = trial_begin;
    S.t1 = trial_end;
    S.n = n;
    S.hot_ev = hot_ev;
    S.hot_base = hot_base;
    S.vq = vq;
    S.W = W;
    // the second form of step (5) needs the trial-major copy
    BwdSparse &Q = S.sp;
    // (the list of deviating trials holds call-relative int32 indices)
    S.use_sp = yet->t_off != nullptr && yet->t_ids != nullptr && yet->t_cnt != nullptr && n < (int64_t(1) << 31);
    Q.vq = vq;
    Q.n = n;
    Q.t0 = trial_begin;
    Q.n_trials = yet->n_trials;
    Q.cs = B.cs;
    Q.n_cot = n_cot;
    Q.catalog = tables->catalog;
    Q.n_sr = B.z.n_sr;
    Q.slice_trials = yet->slice_trials;
    Q.tr_off = yet->tr_off;
    Q.tr_ent = yet->tr_ent;
    Q.ndev = ndev;
    Q.nalt = ndev + L;
    Q.common = common;
    Q.alt = common + static_cast<size_t>(L) * kMaxCot;
    Q.abits = abits;
    Q.aw = aw;
    // the third form holds a slice's bits in LDS, a workgroup of four per CU
    // each: slices of up to 262,144 trials, 2M trials in all
    Q.two = yet->slice_trials <= 8 * 32 * 1024;
    Q.two_bytes = Q.two ? static_cast<int32_t>((yet->slice_trials + 31) / 32 + 1) * 4 : 4;
    // (2000 x 60,000, three rows, 20 trials walked: 1023 us with one)
    Q.segs = static_cast<int32_t>(std::min<int64_t>(std::max<int64_t>(yet->nnz / yet->n_trials / kSparseRound, 1), 1024));
    Q.dev = dev;
    Q.t_cnt = yet->t_cnt;
    Q.t_off = yet->t_off;
    Q.t_ids = yet->t_ids;
    Q.tabs = d_tabs;
    Q.hot_ev = hot_ev;
    Q.hot_base = hot_base;
    Q.W = W;
    {
        ProfScope prof(ARA_PROF_BWD, st);
        // four 256-thread workgroups per CU, a multiple of the slice count
        const int cu = device_cu_count();
        const unsigned gx = static_cast<unsigned>(kSlices * std::max(1, (4 * cu) / kSlices));
        const dim3 grid(gx, L);
        // lanes per hot event: about a third of the mean list length, 4 or 16
        const double mean_list = static_cast<double>(yet->nnz) / (static_cast<double>(kSlices) * tables->catalog);
        const bool wide = mean_list >= 24.0;
        if (S.use_sp) {
            const unsigned gt = static_cast<unsigned>(dev_blocks(n));
            k_bwd_pick<<<L, kPickSamples, 0, st>>>(Q);
            k_bwd_dev<<<dim3(gt, L), 1024, 0, st>>>(Q);
            // the slices the range cuts: at most its first and its last
            int cut[2], ncut = 0;
            for (int64_t t : {trial_begin, trial_end - 1}) {
                const int x = static_cast<int>(t / yet->slice_trials);
                const int64_t lo = static_cast<int64_t>(x) * yet->slice_trials;
                const int64_t hi = std::min(lo + yet->slice_trials, yet->n_trials);
                const bool inside = lo >= trial_begin && hi <= trial_end;
                if (n > 0 && !inside && (ncut == 0 || cut[0] != x)) cut[ncut++] = x;
            }
            const int2 cx = make_int2(ncut > 0 ? cut[0] : 0, ncut > 1 ? cut[1] : (ncut > 0 ? cut[0] : 0));
            const size_t lds = static_cast<size_t>(Q.two_bytes);
            if (wide) k_bwd_count<16><<<grid, 256, lds, st>>>(Q, cx, ncut);
            else k_bwd_count<4><<<grid, 256, lds, st>>>(Q, cx, ncut);
            // two workgroups a CU, of many layers four rounds: each lays out its
            // layer's filter before it walks a trial (64 layers 76 us, two a CU and
            // layer 117)
            const unsigned gs = static_cast<unsigned>(std::max(16, std::min(2 * cu, 8 * cu / L)));
            k_bwd_wsparse<<<dim3(gs, L), kSparseThreads, 0, st>>>(Q);
        }
        if (wide) launch_bwd_w<16>(B.cs, grid, st, S, mean_list);
        else launch_bwd_w<4>(B.cs, grid, st, S, mean_list);
        ARA_HIP(hipGetLastError());
    }
    BwdGrad Gp{};
    Gp.loss = tables->loss;
    Gp.present = tables->present;
    Gp.catalog = tables->catalog;
    Gp.words = tables->words;
    Gp.elt_off = d_off;
    Gp.elt_ids = d_ids;
    Gp.elt_terms = elt_terms;
    Gp.layer_terms = layer_terms;
    Gp.tabs = d_tabs;
    Gp.W = W;
    Gp.hot_base = hot_base;
    Gp.n_sr = B.z.n_sr;
    Gp.n_cot = n_cot;
    Gp.n_cw = B.n_cw;
    Gp.hot_ev = hot_ev;
    Gp.n_elt_slots = std::max(nJ, 1);
    Gp.vs = vs;
    Gp.part_elt = part_elt;
    Gp.part_occ = part_occ;
    {
        ProfScope prof(ARA_PROF_BWD_RED, st);
        const size_t lds = grad_lds(layers_max_j(layers), n_cot);
        if (lds > 64 * 1024)
            ARA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_bwd_grad),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
        k_bwd_grad<<<dim3(B.n_cw / kGradWaves, L), kGradThreads, lds, st>>>(Gp);
        const int outs = n_cot * tables->n_elts * 3 + n_cot * L * 4;
        k_bwd_final<<<outs, 256, 0, st>>>(d_off, d_ids, L, tables->n_elts, n_cot, B.n_cw, hot_base, B.z.n_sr,
                                          std::max(nJ, 1), nwg_v, part_elt, part_occ, aggpart, grad_elt, grad_layer);
        ARA_HIP(hipGetLastError());
    }
    return ARA_OK;
}
