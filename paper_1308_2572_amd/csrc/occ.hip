// Occurrence-table kernels: evaluate the per-event steps of Algorithm 1
// (lookup, financial terms, sum over the layer's ELTs, occurrence terms) once
// per catalogue event, then store the set events compactly in rank order.
#include "occ.h"

#include <algorithm>
#include <cmath>
#include <string>

namespace ara {

constexpr int kPassWords = kOccChunkWords;      // 4096 events per chunk
constexpr int kPasses = kOccChunks;             // 16 chunks per super-range
constexpr int kLossBatch = 4;                   // ELT losses of one event loaded together

__device__ __forceinline__ bool bad_scale(double s) { return !(s > 0.0) || !(s < INFINITY); }
__device__ __forceinline__ bool bad_retention(double r) { return !(r >= 0.0) || !(r < INFINITY); }
__device__ __forceinline__ bool bad_limit(double l) { return !(l > 0.0); }

// Exclusive prefix sum of v over the first 128 threads (two wavefronts);
// *total receives the sum.  Every thread of the block must call it.
__device__ __forceinline__ uint32_t scan128(uint32_t v, uint32_t *wtot, uint32_t *total) {
    const int tid = threadIdx.x, lane = tid & 63;
    uint32_t incl = v;
    if (tid < 128) {
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t x = __shfl_up(incl, o);
            if (lane >= o) incl += x;
        }
        if (lane == 63) wtot[tid >> 6] = incl;
    }
    __syncthreads();
    const uint32_t before = (tid >= 64 && tid < 128) ? wtot[0] : 0u;
    if (tid == 0) *total = wtot[0] + wtot[1];
    __syncthreads();
    return before + incl - v;
}

// Phase one: one workgroup per (4096-event chunk, layer).  The events held
// by at least one of the layer's ELTs are listed in event order; each is
// evaluated once: g_k summed over the ELTs that hold it, in listed order
// (four losses loaded together), then the occurrence terms.  The set events
// are compacted in event order: the chunk's bitmap words, its count, and O
// (and the ELT count) at the start of the chunk's slice of the staging arrays.
//
// A workgroup is a chain of dependent steps (the layer's list, 5 us with its
// presence words; the losses, 5 us; the compaction and stores, 3 us), so what
// counts is how many run at once.  512 threads for the chunk's some 600
// candidates (15 ELTs of 1% each) and LDS sized by the largest layer let four
// share a CU: four layers over 2M events, 1984 workgroups, 45 us, where 1024
// threads with room for 128 ELTs took 71 us in four rounds; two layers 36 and
// 22 us, one layer 18 and 15; 256 threads 47, 24 and 18.  With fewer
// workgroups than CUs there is nothing to share, and 1024 threads are the
// faster: 200,000 events 14.4 us, 512 threads 17.6.
//
// Asking every ELT for every candidate instead of those that hold it (a
// twelfth of them) took a third more of a small catalogue's 17 us.
struct __attribute__((aligned(16))) EltTerms {
    double scale, ret, lim;
    int64_t row;   // of the loss table
};

// LDS of k_occ_eval for layers of up to J ELTs: presence words, terms.
static size_t eval_lds(int J) { return static_cast<size_t>(std::max(J, 1)) * (kPassWords * sizeof(uint32_t) + sizeof(EltTerms)); }

template <bool UNION, int NT>
__global__ __launch_bounds__(NT) void k_occ_eval(const float *__restrict__ loss, const uint32_t *__restrict__ present,
                                                   int32_t catalog, int32_t words, const int32_t *__restrict__ elt_off,
                                                   const int32_t *__restrict__ elt_ids,
                                                   const double *__restrict__ elt_terms,
                                                   const double *__restrict__ layer_terms,
                                                   const OccTables *__restrict__ tabs, int32_t *__restrict__ err,
                                                 int32_t max_j) {
    constexpr int kWaves = NT / kWave;
    extern __shared__ __align__(16) unsigned char smem[];
    EltTerms *lt = reinterpret_cast<EltTerms *>(smem);               // [max_j]
    uint32_t *stage = reinterpret_cast<uint32_t *>(lt + max_j);      // [max_j][kPassWords]
    __shared__ double lterm[4];
    __shared__ uint32_t anyw[kPassWords], cbase[kPassWords], fbits[kPassWords];
    __shared__ uint16_t cand[kPassWords * 32];
    __shared__ uint32_t wtot[kWaves], wtot2[2], n_cand;
    __shared__ unsigned long long smax;
    __shared__ int slow;

    const int s = blockIdx.x / kPasses, p = blockIdx.x % kPasses, j = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const OccTables T = load_tables(tabs + j);
    const int a = elt_off[j];
    const int J = elt_off[j + 1] - a;
    const bool checker = blockIdx.x == 0;
    for (int q = tid; q < J; q += NT) {
        const int k = elt_ids[a + q];
        const EltTerms t{elt_terms[3 * k + 0], elt_terms[3 * k + 1], elt_terms[3 * k + 2], static_cast<int64_t>(k) * catalog};
        lt[q] = t;
        if (checker && (bad_scale(t.scale) || bad_retention(t.ret) || bad_limit(t.lim))) atomicCAS(err, 0, ARA_E_INVAL);
    }
    if (tid == 0) {
        smax = 0;
        slow = INT32_MAX;
    }
    if (tid < 4) {
        lterm[tid] = layer_terms[4 * j + tid];
        const bool bad = (tid & 1) ? bad_limit(lterm[tid]) : bad_retention(lterm[tid]);
        if (checker && bad) atomicCAS(err, 0, ARA_E_INVAL);
    }
    {
        // a thread's words are of one place in the rows of ELTs NT / 128 apart;
        // four loads in flight
        constexpr int kRows = NT / kPassWords;
        const int ww = tid % kPassWords;
        const int64_t gw = static_cast<int64_t>(s) * kSrWords + p * kPassWords + ww;
        const bool in = gw < words;
        for (int q0 = tid / kPassWords; q0 < J; q0 += 4 * kRows) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = min(q0 + u * kRows, J - 1);
                v[u] = in ? present[static_cast<size_t>(elt_ids[a + q]) * words + gw] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (q0 + u * kRows < J) stage[(q0 + u * kRows) * kPassWords + ww] = v[u];
        }
    }
    __syncthreads();
    // events held by any of the layer's ELTs, word by word, and where each
    // word's events start in the candidate list
    uint32_t any = 0;
    if (tid < kPassWords) {
        for (int q = 0; q < J; ++q) any |= stage[q * kPassWords + tid];
        anyw[tid] = any;
        fbits[tid] = 0u;
    }
    const uint32_t cb = scan128(__popc(any), wtot2, &n_cand);
    if (tid < kPassWords) cbase[tid] = cb;
    __syncthreads();
#pragma unroll 4
    for (int local = tid; local < kPassWords * 32; local += NT) {
        const uint32_t m = anyw[local >> 5];
        const uint32_t bit = static_cast<uint32_t>(local & 31);
        if ((m >> bit) & 1u) cand[cbase[local >> 5] + __popc(m & ((1u << bit) - 1u))] = static_cast<uint16_t>(local);
    }
    __syncthreads();
    const int nc = static_cast<int>(n_cand);
    const double occR = lterm[0], occL = lterm[1];
    const int64_t ev0 = static_cast<int64_t>(s) * kSr + p * (kPassWords * 32);
    double *ov = T.dense + ev0;                           // the chunk's compacted O
    uint8_t *onb = UNION ? T.dense_nb + ev0 : nullptr;    // and ELT counts
    uint32_t run = 0;                                     // set events before this pass
    unsigned long long mx = 0;                            // this thread's part of the chunk's stat
    int low = INT32_MAX;
    for (int i0 = 0; i0 < nc; i0 += NT) {   // uniform trip count: every thread reaches the barriers
        const int i = i0 + tid;
        const int local = i < nc ? cand[i] : 0;
        const int wip = local >> 5, bit = local & 31;
        const int64_t ev = ev0 + local;
        double x = 0.0;
        int nb = 0;
        if (i < nc) {
            for (int q0 = 0; q0 < J; q0 += 32) {
                // the ELTs among q0 .. q0 + 31 that hold the event
                uint32_t held = 0;
                const int nq = min(32, J - q0);
#pragma unroll 4
                for (int u = 0; u < nq; ++u) held |= ((stage[(q0 + u) * kPassWords + wip] >> bit) & 1u) << u;
                nb += __popc(held);
                while (held) {
                    float v[kLossBatch];
                    int q[kLossBatch];
#pragma unroll
                    for (int u = 0; u < kLossBatch; ++u) {
                        q[u] = held ? q0 + __builtin_ctz(held) : -1;
                        held &= held - 1;
                        // lanes with fewer read element 0 (always valid) and ignore it,
                        // so the loads are issued back to back
                        v[u] = loss[q[u] >= 0 ? lt[q[u]].row + ev : 0];
                    }
#pragma unroll
                    for (int u = 0; u < kLossBatch; ++u)
                        if (q[u] >= 0) {
                            const EltTerms t = lt[q[u]];
                            x = x + xl(t.scale * static_cast<double>(v[u]), t.ret, t.lim);
                        }
                }
            }
        }
        const double O = xl(x, occR, occL);
        const bool flag = i < nc && (UNION ? (nb > 0) : (O != 0.0));
        // rank among this pass's set events: lanes below, then wavefronts below
        const uint64_t m = __ballot(flag);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                         __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
        if (lane == 0) wtot[w] = static_cast<uint32_t>(__popcll(m));
        __syncthreads();
        uint32_t wb = 0, tot = 0;
        for (int k = 0; k < kWaves; ++k) {
            const uint32_t c = wtot[k];
            wb += (k < w) ? c : 0u;
            tot += c;
        }
        if (flag) {
            const uint32_t r = run + wb + below;
            ov[r] = O;
            if (UNION) onb[r] = static_cast<uint8_t>(nb > 255 ? 255 : nb);
            atomicOr(&fbits[wip], 1u << bit);
            const unsigned long long ob = static_cast<unsigned long long>(__double_as_longlong(O));
            if (ob != 0) {
                mx = max(mx, ob);
                const int ex = static_cast<int>(ob >> 52);
                const unsigned long long man = ob & 0xFFFFFFFFFFFFFull;
                low = min(low, ex ? ex - 1075 + __ffsll(static_cast<long long>(man | (1ull << 52))) - 1
                                  : __ffsll(static_cast<long long>(man)) - 1 - 1074);
            }
        }
        run += tot;
        __syncthreads();   // wtot is rewritten by the next pass
    }
    if (tid < kPassWords) T.bits[static_cast<size_t>(s) * kSrWords + p * kPassWords + tid] = fbits[tid];
    if (tid == 0) T.pcount[static_cast<size_t>(s) * kPasses + p] = static_cast<int32_t>(run);
    if (!T.ev) return;   // uniform
    // (zeroed before the first barrier; a wavefront without set events adds nothing)
    if (__any(mx != 0)) {
        for (int o = 32; o > 0; o >>= 1) {
            mx = max(mx, __shfl_xor(mx, o));
            low = min(low, __shfl_xor(low, o));
        }
        if (lane == 0) {
            atomicMax(&smax, mx);
            atomicMin(&slow, low);
        }
    }
    __syncthreads();
    if (tid == 0)
        T.stat[static_cast<size_t>(s) * kPasses + p] = OccChunkStat{smax, slow, nc, static_cast<int32_t>(run), 0};
}

// The chunks' stats of one layer together: its form for the event-ordered
// forward, and the set events of the chunks before `before`.  All threads of
// the workgroup (at most 1024) call it.
__device__ EvLayer occ_layer_form(const OccTables &T, int n_chunks, int before, uint32_t *base) {
    __shared__ unsigned long long smx[16], ssum[16];
    __shared__ int slow[16];
    __shared__ uint32_t sbef[16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, nw = blockDim.x >> 6;
    unsigned long long mx = 0, sum = 0;   // sum: events held << 32 | set events
    int low = INT32_MAX;
    uint32_t bef = 0;
    for (int c = tid; c < n_chunks; c += blockDim.x) {
        const OccChunkStat s = T.stat[c];
        mx = max(mx, s.max_bits);
        low = min(low, s.low);
        sum += (static_cast<unsigned long long>(static_cast<uint32_t>(s.n_union)) << 32) + static_cast<uint32_t>(s.count);
        bef += c < before ? static_cast<uint32_t>(s.count) : 0u;
    }
    for (int o = 32; o > 0; o >>= 1) {
        mx = max(mx, __shfl_xor(mx, o));
        low = min(low, __shfl_xor(low, o));
        sum += __shfl_xor(sum, o);
        bef += __shfl_xor(bef, o);
    }
    if (lane == 0) {
        smx[w] = mx;
        slow[w] = low;
        ssum[w] = sum;
        sbef[w] = bef;
    }
    __syncthreads();
    mx = sum = 0;
    low = INT32_MAX;
    bef = 0;
    for (int k = 0; k < nw; ++k) {
        mx = max(mx, smx[k]);
        low = min(low, slow[k]);
        sum += ssum[k];
        bef += sbef[k];
    }
    const uint32_t un = static_cast<uint32_t>(sum >> 32), cnt = static_cast<uint32_t>(sum);
    *base = bef;
    EvLayer L{0, static_cast<int32_t>(cnt), 0, 0};
    // bits of the longest trial's length: its total is below 2^(exponent of
    // the largest O + lbits)
    const int64_t len = max<int64_t>(*T.max_len, 1);
    const int lbits = len > 1 ? 64 - __clzll(len - 1) : 0;
    const int ex = static_cast<int>(mx >> 52);
    if (lbits > 32 || ex >= 0x7FF) return L;   // an infinity (or, with invalid terms, no number or a negative one)
    const int top = (ex ? ex - 1022 : -1021) + lbits;   // every total < 2^top
    L.gexp = top - 62;
    L.frac = 32 - lbits;
    int carry = 0;
    if (low < L.gexp - L.frac) {
        carry = kEvCarry;
        L.gexp = top - 64;
        L.frac = 32;
        if (low < L.gexp - L.frac) return L;
    }
    const int slots = n_chunks * (kOccChunkWords * 32);
    const int layout = 2ull * un <= static_cast<unsigned long long>(slots) ? 1 : 2;
    L.mode = layout | carry;
    if (layout == 2) L.n_set = slots;
    return L;
}

// Phase two: one workgroup per (chunk, layer): the chunk's rank base (set
// events of the super-range's earlier chunks), the rank of every bitmap word,
// and the chunk's compacted values moved to their place in rank order.
// Catalogues of more than kFormChunks chunks: the layer's form and the set
// events before every chunk (left in stat.pad), once per layer instead of
// once per chunk.
constexpr int kFormChunks = 2048;

__global__ __launch_bounds__(1024) void k_occ_form(const OccTables *__restrict__ tabs, int n_chunks) {
    __shared__ uint32_t wsum[16];
    const OccTables T = load_tables(tabs + blockIdx.x);
    if (!T.ev) return;   // uniform
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t run = 0;
    for (int c0 = 0; c0 < n_chunks; c0 += 1024) {
        const uint32_t v = c0 + tid < n_chunks ? static_cast<uint32_t>(T.stat[c0 + tid].count) : 0u;
        uint32_t incl = v;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t x = __shfl_up(incl, o);
            if (lane >= o) incl += x;
        }
        if (lane == 63) wsum[w] = incl;
        __syncthreads();
        uint32_t at = run + incl - v, all = 0;
        for (int k = 0; k < 16; ++k) {
            at += k < w ? wsum[k] : 0u;
            all += wsum[k];
        }
        if (c0 + tid < n_chunks) T.stat[c0 + tid].pad = static_cast<int32_t>(at);
        run += all;
        __syncthreads();
    }
    uint32_t none;
    const EvLayer L = occ_layer_form(T, n_chunks, 0, &none);
    if (tid == 0) *T.ev = L;
}

// With T.ev, the layer's form comes from every chunk's stat, and in its
// event-ordered form the chunk's set events become records (value in fixed
// point, event) in event order over the whole catalogue, instead.
constexpr int kRankThreads = 256;

template <bool UNION, bool F32>
__global__ __launch_bounds__(kRankThreads) void k_occ_rank(const OccTables *__restrict__ tabs) {
    __shared__ uint32_t wtot2[2], tot;
    const int s = blockIdx.x / kPasses, p = blockIdx.x % kPasses, j = blockIdx.y;
    const int tid = threadIdx.x;
    const OccTables T = load_tables(tabs + j);
    const int32_t *pc = T.pcount + static_cast<size_t>(s) * kPasses;
    const uint32_t cnt = static_cast<uint32_t>(pc[p]);
    const size_t w0 = static_cast<size_t>(s) * kSrWords + p * kPassWords;
    const size_t src = static_cast<size_t>(s) * kSr + static_cast<size_t>(p) * (kPassWords * 32);
    const uint32_t b = tid < kPassWords ? T.bits[w0 + tid] : 0u;
    const uint32_t r = scan128(__popc(b), wtot2, &tot);
    if (!F32 && T.ev) {   // uniform
        uint32_t gbase;
        EvLayer L;
        if (static_cast<int>(gridDim.x) > kFormChunks) {
            L = *T.ev;
            gbase = static_cast<uint32_t>(T.stat[blockIdx.x].pad);
        } else {
            L = occ_layer_form(T, gridDim.x, blockIdx.x, &gbase);
            if (blockIdx.x == 0 && tid == 0) *T.ev = L;
        }
        if (L.mode) {
            // the chunk's set events in order, then a thread per event
            __shared__ uint16_t list[kPassWords * 32];
            if (tid < kPassWords) {
                uint32_t m = b, at = r;
                for (; m; m &= m - 1) list[at++] = static_cast<uint16_t>(32 * tid + __builtin_ctz(m));
            }
            __syncthreads();
            EvRec *rec = reinterpret_cast<EvRec *>(T.vals) + gbase;
            const bool compact = (L.mode & kEvLayout) == 1;
            const size_t cdst = compact ? gbase : src;
            for (uint32_t i = tid; i < cnt; i += kRankThreads) {
                const unsigned long long ob = static_cast<unsigned long long>(__double_as_longlong(T.dense[src + i]));
                EvRec v{0, 0, static_cast<uint32_t>(src) + list[i]};
                if (ob != 0) {
                    const int ex = static_cast<int>(ob >> 52);
                    unsigned long long m = (ob & 0xFFFFFFFFFFFFFull) | (ex ? 1ull << 52 : 0ull);
                    int sh = (ex ? ex - 1075 : -1074) - (L.gexp - L.frac);   // O = m 2^sh units of 2^(gexp - frac)
                    if (sh < 0) {   // trailing zeros only: O is a multiple of the unit
                        m >>= -sh;
                        sh = 0;
                    }
                    // sh <= 43: the value is below 2^(64 + frac), m at least 2^52 (or, of a subnormal, the
                    // exponent at its lowest)
                    v.hi = sh >= L.frac ? m << (sh - L.frac) : m >> (L.frac - sh);
                    v.lo = static_cast<uint32_t>((m << sh) & ((1ull << L.frac) - 1ull));
                }
                if (compact) {
                    rec[i] = v;
                } else {   // dense[src + i] has just been read by this thread, and by no other
                    reinterpret_cast<unsigned long long *>(T.vals)[src + i] = v.hi;
                    reinterpret_cast<uint2 *>(T.dense)[src + i] = make_uint2(v.lo, v.ev);
                }
                if (UNION) T.cnt[cdst + i] = T.dense_nb[src + i];
            }
            return;
        }
    }
    uint32_t base = 0;
    for (int k = 0; k < p; ++k) base += static_cast<uint32_t>(pc[k]);
    if (tid < kPassWords) T.br[w0 + tid] = make_uint2(b, base + r);
    if (p == kPasses - 1 && tid == 0) T.count[s] = static_cast<int32_t>(base + cnt);
    const size_t dst = static_cast<size_t>(s) * kSr + base;
    // four events a thread in flight: 200,000 events, all of them in the union,
    // 6.2 us, one at a time 12
    constexpr uint32_t kU = 4;
    for (uint32_t i0 = tid; i0 < cnt; i0 += kU * kRankThreads) {
        double v[kU];
        uint8_t nb[kU];
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            const size_t i = src + min(i0 + u * kRankThreads, cnt - 1);
            v[u] = T.dense[i];
            nb[u] = UNION ? T.dense_nb[i] : 0;
        }
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            const uint32_t i = i0 + u * kRankThreads;
            if (i >= cnt) break;
            if (F32) reinterpret_cast<float *>(T.vals)[dst + i] = static_cast<float>(v[u]);
            else T.vals[dst + i] = v[u];
            if (UNION) T.cnt[dst + i] = nb[u];
        }
    }
}

int32_t check_layers(const ara_layers *layers, int32_t n_elts) {
    if (!layers) return fail(ARA_E_INVAL, "null layers");
    if (layers->n_layers < 0) return fail(ARA_E_INVAL, "negative layer count");
    if (layers->n_layers > ARA_MAX_LAYERS) return fail(ARA_E_LIMIT, "more than ARA_MAX_LAYERS layers in one call");
    if (layers->n_layers == 0) return ARA_OK;
    if (!layers->elt_off || !layers->elt_ids) return fail(ARA_E_INVAL, "null layer arrays");
    if (layers->elt_off[0] != 0) return fail(ARA_E_RANGE, "elt_off[0] must be 0");
    for (int32_t j = 0; j < layers->n_layers; ++j) {
        const int32_t J = layers->elt_off[j + 1] - layers->elt_off[j];
        if (J < 0) return fail(ARA_E_RANGE, "elt_off must be non-decreasing");
        if (J > kMaxJ) return fail(ARA_E_LIMIT, "layer covers more than ARA_MAX_ELTS_PER_LAYER ELTs");
        for (int32_t q = layers->elt_off[j]; q < layers->elt_off[j + 1]; ++q)
            if (layers->elt_ids[q] < 0 || layers->elt_ids[q] >= n_elts)
                return fail(ARA_E_RANGE, "layer refers to an ELT index out of range");
    }
    return ARA_OK;
}

template <bool UNION, int NT>
static void eval(dim3 grid, const ara_tables *tables, const int32_t *d_elt_off, const int32_t *d_elt_ids,
                 const double *elt_terms, const double *layer_terms, const OccTables *d_tabs, int32_t *d_err, int32_t max_j,
                 hipStream_t st) {
    const size_t lds = eval_lds(max_j);
    if (lds > 48 * 1024)   // beside the fixed 11 KB
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k_occ_eval<UNION, NT>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    k_occ_eval<UNION, NT><<<grid, NT, lds, st>>>(tables->loss, tables->present, tables->catalog, tables->words, d_elt_off,
                                                 d_elt_ids, elt_terms, layer_terms, d_tabs, d_err, max_j);
}

int32_t layers_max_j(const ara_layers *layers) {
    int32_t m = 1;
    for (int32_t j = 0; j < layers->n_layers; ++j) m = std::max(m, layers->elt_off[j + 1] - layers->elt_off[j]);
    return m;
}

int32_t launch_occ(const ara_tables *tables, const int32_t *d_elt_off, const int32_t *d_elt_ids,
                   const double *elt_terms, const double *layer_terms, int32_t n_layers, bool union_mode,
                   bool f32_vals, OccTables *d_tabs, int n_sr, int32_t *d_err, int32_t max_j, hipStream_t st, bool with_ev) {
    if (n_layers == 0 || n_sr == 0) return ARA_OK;
    const dim3 grid(static_cast<unsigned>(n_sr * kPasses), static_cast<unsigned>(n_layers));
    const bool form = with_ev && n_sr * kPasses > kFormChunks;
    const bool few = static_cast<int64_t>(n_sr) * kPasses * n_layers <= device_cu_count();
    if (union_mode) {
        if (few) eval<true, 1024>(grid, tables, d_elt_off, d_elt_ids, elt_terms, layer_terms, d_tabs, d_err, max_j, st);
        else eval<true, 512>(grid, tables, d_elt_off, d_elt_ids, elt_terms, layer_terms, d_tabs, d_err, max_j, st);
        if (form) k_occ_form<<<n_layers, 1024, 0, st>>>(d_tabs, n_sr * kPasses);
        if (f32_vals) k_occ_rank<true, true><<<grid, kRankThreads, 0, st>>>(d_tabs);
        else k_occ_rank<true, false><<<grid, kRankThreads, 0, st>>>(d_tabs);
    } else {
        if (few) eval<false, 1024>(grid, tables, d_elt_off, d_elt_ids, elt_terms, layer_terms, d_tabs, d_err, max_j, st);
        else eval<false, 512>(grid, tables, d_elt_off, d_elt_ids, elt_terms, layer_terms, d_tabs, d_err, max_j, st);
        if (form) k_occ_form<<<n_layers, 1024, 0, st>>>(d_tabs, n_sr * kPasses);
        if (f32_vals) k_occ_rank<false, true><<<grid, kRankThreads, 0, st>>>(d_tabs);
        else k_occ_rank<false, false><<<grid, kRankThreads, 0, st>>>(d_tabs);
    }
    ARA_HIP(hipGetLastError());
    return ARA_OK;
}

}  // namespace ara
