// YET preparation: validate the trials and lay them out by (block of trials,
// catalogue range, trial group) so that the forward kernel can keep one
// range's occurrence table in LDS while streaming, in 16-bit codes; and, on
// request, the event-major copy that the backward reads.
//
// Code stream of one segment (block b, range r, group g): the occurrences of
// the group's trials whose event lies in range r, in trial order (storage
// order inside a trial), one 16-bit code each:
//     bit 15      advance to the next trial of the group before this code
//     bits 0..14  the event's offset in the range
// 0xFFFF means "advance, no event": it stands for each trial of the group
// with no event in the range between two that have some, for the advance of
// an event at offset 0x7FFF that opens a trial (which then follows as plain
// 0x7FFF), and for padding.  The padded stream is dealt to the 64 lanes as
// runs of `run` consecutive codes (run a multiple of 4), lane j starting from
// trial lane_start[j] of the group; code s of lane j sits at
//     base + (s / 4) * 256 + 4 * j + s % 4,
// so a wavefront reads four steps of all its lanes as one 512-byte block.
//
// With positions, a second array of the same shape holds, at each code's
// slot, the occurrence's position in its trial (its index less the trial's
// first index; 0xFFFF for gap codes and padding), so that a walk of the code
// stream can name each occurrence by its trial-major index.  Trials then hold
// at most 65536 occurrences.
#include "evblk.h"

#include <algorithm>
#include <string>

namespace ara {

constexpr uint16_t kAdvance = 0x8000;
constexpr uint16_t kSkip = 0xFFFF;
constexpr int kChunk = 8192;         // occurrences of a trial group sorted by range at once
constexpr int kScanPer = 4;          // segments per thread of the scan of their sizes
constexpr int kScanBlock = 1024 * kScanPer;

struct Geometry {
    int tg, tb, n_blocks, n_ranges;
    int slice_blocks;   // blocks per trial slice of the event-major copy
    size_t nseg;
};

static Geometry geometry(int64_t n_trials, int32_t catalog) {
    Geometry g{};
    const int64_t cu = device_cu_count();
    // two blocks per CU: the forward runs two workgroups on every CU
    int64_t tg = (n_trials + 2 * kGroups * cu - 1) / (2 * kGroups * cu);
    tg = std::max<int64_t>(1, std::min<int64_t>(tg, kMaxTrialsPerGroup));
    g.tg = static_cast<int>(tg);
    g.tb = kGroups * g.tg;
    g.n_blocks = static_cast<int>((n_trials + g.tb - 1) / g.tb);
    g.n_ranges = (catalog + kRange - 1) / kRange;
    g.nseg = static_cast<size_t>(g.n_blocks) * g.n_ranges * kGroups;
    g.slice_blocks = std::max(1, (g.n_blocks + kSlices - 1) / kSlices);
    return g;
}

// Upper bound of the codes: a segment holds its events, at most tg - 1 gap
// codes, at most tg - 1 advances for events at offset 0x7FFF, and fewer than
// 4 * 64 padding codes.
static int64_t max_codes(const Geometry &g, int64_t nnz) {
    return nnz + static_cast<int64_t>(g.nseg) * (2 * g.tg + 4 * kWave);
}

// The pieces of the caller's buffer.
struct Prepared {
    uint16_t *code;
    int64_t *seg_base;
    int32_t *seg_run;
    uint8_t *lane_start;
    int64_t *misc;
    int64_t *tr_off, *ssum;
    uint32_t *tr_ent;
    int64_t *t_off;
    int32_t *t_ids, *t_cnt;
    uint16_t *pos;
    // event-ordered blocks
    uint16_t *ent, *ev_pos;
    uint2 *hdr;
    uint32_t *start;
    int64_t *ev_base;
    // scratch of the preparation
    uint32_t *rec, *rsum;
    uint16_t *rpos, *rstart, *ev_rpos;
    int64_t *bsum;
    uint16_t *tstart;
    uint32_t *tbase, *mark;
};

static int64_t n_groups_of(const Geometry &g, int64_t n_trials) { return (n_trials + g.tg - 1) / g.tg; }

// What stays with the prepared YET.
static Prepared carve(Carver &c, const Geometry &g, int64_t n_trials, int64_t nnz, int32_t catalog, uint32_t flags) {
    Prepared p{};
    const size_t occ = static_cast<size_t>(std::max<int64_t>(nnz, 1));
    p.code = c.take<uint16_t>(static_cast<size_t>(max_codes(g, nnz)) + kPadCodes);
    p.seg_base = c.take<int64_t>(g.nseg);
    p.seg_run = c.take<int32_t>(g.nseg);
    p.lane_start = c.take<uint8_t>(g.nseg * kWave);
    p.misc = c.take<int64_t>(32);
    if (flags & ARA_PREP_TRANSPOSED) {
        p.tr_off = c.take<int64_t>(static_cast<size_t>(kSlices) * catalog + 1);
        p.tr_ent = c.take<uint32_t>(occ);
    }
    if (flags & ARA_PREP_TRIAL_MAJOR) {
        p.t_off = c.take<int64_t>(static_cast<size_t>(n_trials) + 1);
        p.t_ids = c.take<int32_t>(occ);
        p.t_cnt = c.take<int32_t>(static_cast<size_t>(catalog));
    }
    if (flags & ARA_PREP_POSITIONS) {
        p.pos = c.take<uint16_t>(static_cast<size_t>(max_codes(g, nnz)) + kPadCodes);
        if (!p.t_off) p.t_off = c.take<int64_t>(static_cast<size_t>(n_trials) + 1);
    }
    const EvGeometry eg = ev_geometry(n_trials, nnz, catalog);
    const size_t neb = static_cast<size_t>(eg.neb);
    p.ent = c.take<uint16_t>(occ + kEvPad);
    if (eg.dense) p.start = c.take<uint32_t>(neb * (static_cast<size_t>(catalog) + 1));
    else p.hdr = c.take<uint2>(neb * static_cast<size_t>(eg.ng));
    p.ev_base = c.take<int64_t>(neb + 1);
    if (flags & ARA_PREP_POSITIONS) p.ev_pos = c.take<uint16_t>(occ + kEvPad);
    return p;
}

// What only the preparation needs: 4 bytes per occurrence for the sorted
// records (in the event-major lists' place, written last, where the caller
// gives the scratch by itself: lend), two more with positions, and the runs'
// bounds.  The records' positions of the first sort lie in the place of the
// blocks' entries, which are written after the codes.
static void carve_scratch(Carver &c, Prepared &p, const Geometry &g, int64_t n_trials, int64_t nnz, int32_t catalog,
                          uint32_t flags, bool lend) {
    const size_t occ = static_cast<size_t>(std::max<int64_t>(nnz, 1));
    const EvGeometry eg = ev_geometry(n_trials, nnz, catalog);
    const size_t neb = static_cast<size_t>(eg.neb);
    p.rec = lend && (flags & ARA_PREP_TRANSPOSED) ? p.tr_ent : c.take<uint32_t>(occ);
    if (flags & ARA_PREP_TRANSPOSED) p.ssum = c.take<int64_t>(ev_major_sums(catalog));
    if (flags & ARA_PREP_POSITIONS) {
        p.rpos = p.ent;
        p.ev_rpos = c.take<uint16_t>(occ);
    }
    const size_t chunks = static_cast<size_t>(nnz / kChunk + 2 * n_groups_of(g, n_trials) + 2);
    p.rstart = c.take<uint16_t>(chunks * static_cast<size_t>(g.n_ranges + 1));
    p.rsum = c.take<uint32_t>(chunks * static_cast<size_t>(g.n_ranges));
    p.bsum = c.take<int64_t>(g.nseg / kScanBlock + 1);
    p.tstart = c.take<uint16_t>(static_cast<size_t>(eg.n_chunks) * static_cast<size_t>(eg.n_tiles + 1));
    p.tbase = c.take<uint32_t>(neb * static_cast<size_t>(eg.n_tiles + 1));
    p.mark = c.take<uint32_t>(static_cast<size_t>(eg.n_marks));
}

struct PrepareBytes {
    size_t keep, scratch;
};

static PrepareBytes prepare_bytes(const Geometry &g, int64_t n_trials, int64_t nnz, int32_t catalog, uint32_t flags, bool lend) {
    Carver c(nullptr), s(nullptr);
    Prepared p = carve(c, g, n_trials, nnz, catalog, flags);
    carve_scratch(s, p, g, n_trials, nnz, catalog, flags, lend);
    return {c.bytes(), s.bytes()};
}

// How the codes are made: a scattered store per code leaves every segment's
// lines open from the first trial of a group to its last (2 GB of lines at
// 1M x 1000: each 2-byte store became its own memory write), so nothing is
// scattered to memory here.  k_prep_part sorts chunks of kChunk occurrences
// of one trial group by range inside LDS (stably) and writes them back as
// (trial, offset) records in runs; k_prep_sizes counts each segment's codes
// from the runs' summaries; a scan gives the segments' bases; k_prep_emit
// gathers one segment's runs, forms its codes in LDS in their final places
// and writes the segment as whole lines.  Bound by the bytes moved (IDs,
// records written and read, codes) and by the ballots of the sort; at 1M x
// 1000 the two passes that scattered took 4.2 + 20.4 ms, these take 5.1 + 2.8.
constexpr int kPartThreads = 512;
constexpr int kPartWaves = kPartThreads / kWave;
constexpr int kPartItems = kChunk / kPartThreads;   // slices of 64 occurrences per wavefront, at most
constexpr int kPartWin = 256;                       // ranges sorted at once
constexpr int kEmitThreads = 256;
constexpr int kEmitWaves = kEmitThreads / kWave;

// The chunks of trial group g, whose occurrences start at o0: chunk c of the
// group holds occurrences [o0 + c kChunk, ...) and has index
// chunk_base(g, o0) + c: a closed form that leaves every group room.
__device__ __forceinline__ int64_t chunk_base(int64_t g, int64_t o0) { return o0 / kChunk + 2 * g; }

// Offsets never decrease (with offsets[0] = 0 and offsets[n] = the number of
// IDs, checked on the host, every trial then lies inside the IDs: the
// kernels after this one read nothing when the check failed).  Also the
// longest trial.
__global__ __launch_bounds__(256) void k_prep_check(const int64_t *__restrict__ off, int64_t n_trials,
                                                    int64_t *__restrict__ misc, int64_t max_len) {
    int64_t longest = 0;
    bool bad = false;
    for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < n_trials;
         t += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t len = off[t + 1] - off[t];
        bad = bad || len < 0;
        longest = max(longest, len);
    }
    __shared__ int64_t red[4];
    for (int o = 32; o > 0; o >>= 1) longest = max(longest, static_cast<int64_t>(__shfl_xor(longest, o)));
    const bool any_bad = __any(bad);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = any_bad ? -1 : longest;
    __syncthreads();
    if (threadIdx.x != 0) return;   // one set of atomics per workgroup
    longest = max(max(red[0], red[1]), max(red[2], red[3]));
    if (min(min(red[0], red[1]), min(red[2], red[3])) < 0) {
        atomicCAS(reinterpret_cast<int32_t *>(misc + kMiscErr), 0, ARA_E_RANGE);
        atomicOr(reinterpret_cast<int32_t *>(misc + kMiscBadOff), 1);
    }
    if (longest > 0) atomicMax(reinterpret_cast<unsigned long long *>(misc + kMiscMaxLen), static_cast<unsigned long long>(longest));
    if (longest > max_len) atomicOr(reinterpret_cast<int32_t *>(misc + kMiscLong), 1);
}

struct PartParams {
    const int64_t *off;
    const int32_t *ids;
    int64_t n_trials;
    int32_t catalog, tg, n_ranges;
    uint32_t *rec;      // [nnz] trial in the group << 15 | offset in the range, sorted by range within each chunk
    uint16_t *rpos;     // [nnz] their positions in the trial, or null
    uint16_t *rstart;   // [chunk][n_ranges + 1] where each range's records start in the chunk
    uint32_t *rsum;     // [chunk][n_ranges] extra codes | first trial << 8 | last trial << 16 | first offset is 0x7FFF << 24
    int64_t *misc;
};

__device__ __forceinline__ uint32_t uni32(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// One workgroup per trial group, chunk by chunk.  Each wavefront takes an
// eighth of the chunk's occurrences, in order, in 64-wide slices held in
// registers; an occurrence's rank among its range's in the wavefront comes
// from ballots over the range's bits (lane order = storage order) and a
// counter per range in LDS.
template <bool POS>
__global__ __launch_bounds__(kPartThreads) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_prep_part(PartParams P) {
    __shared__ uint32_t srec[kChunk];
    __shared__ uint16_t spos[POS ? kChunk : 1];
    __shared__ uint32_t cnt[kPartWaves][kPartWin];
    __shared__ uint32_t ext[kPartWin];
    __shared__ uint32_t wsum[kPartWaves];
    __shared__ int32_t soff[kMaxTrialsPerGroup + 1];   // trial starts, relative to the chunk
    if (P.misc[kMiscBadOff] != 0) return;   // uniform: only k_prep_check writes it
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = static_cast<int>(uni32(tid >> 6));
    const int64_t g = blockIdx.x;
    const int64_t t0 = g * P.tg;
    if (t0 >= P.n_trials) return;
    const int nt = static_cast<int>(min<int64_t>(P.tg, P.n_trials - t0));
    const int64_t o0 = P.off[t0], o1 = P.off[t0 + nt];
    const int64_t cb = chunk_base(g, o0);
    for (int64_t ks = o0, ch = cb; ks < o1; ks += kChunk, ++ch) {
        const int nin = static_cast<int>(min<int64_t>(kChunk, o1 - ks));
        const int32_t far = 1 << 30;
        __syncthreads();   // the previous chunk's LDS is free
        for (int i = tid; i <= nt; i += kPartThreads)
            soff[i] = static_cast<int32_t>(max<int64_t>(-far, min<int64_t>(far, P.off[t0 + i] - ks)));
        int32_t id[kPartItems];
        const int ns = (nin + kPartThreads - 1) / kPartThreads;   // slices per wavefront
        const int kw = w * ns * kWave;
        const int32_t *src = P.ids + ks;
#pragma unroll
        for (int s = 0; s < kPartItems; ++s) {
            const uint32_t k = static_cast<uint32_t>(kw + s * kWave + lane);
            id[s] = s < ns && k < static_cast<uint32_t>(nin) ? src[k] : 0;
        }
        __syncthreads();
        // each occurrence's trial in the group, by way of its place in srec
        uint32_t tr[kPartItems];   // trial << 16 | rank in the wavefront
        {
            int lo = 0, hi = nt;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (static_cast<int32_t>(uni32(static_cast<uint32_t>(soff[mid]))) <= kw) lo = mid;
                else hi = mid;
            }
            int tcur = lo;
#pragma unroll 1
            for (int s = 0; s < ns; ++s) {
                const int k = kw + s * kWave + lane, last = kw + s * kWave + (kWave - 1);
                uint32_t tl = static_cast<uint32_t>(tcur);
                while (tcur + 1 < nt) {
                    const int b = static_cast<int32_t>(uni32(static_cast<uint32_t>(soff[tcur + 1])));
                    if (b > last) break;
                    tl += k >= b ? 1u : 0u;
                    ++tcur;
                }
                srec[k] = tl << 16;
            }
#pragma unroll
            for (int s = 0; s < kPartItems; ++s) tr[s] = s < ns ? srec[kw + s * kWave + lane] : 0u;
        }
        uint32_t woff = 0;   // records of the ranges before this window
        for (int w0 = 0; w0 < P.n_ranges; w0 += kPartWin) {
            const int wn = min(kPartWin, P.n_ranges - w0);
            int gb = 0;
            while ((1 << gb) < wn) ++gb;
            for (int i = tid; i < kPartWaves * kPartWin; i += kPartThreads) (&cnt[0][0])[i] = 0u;
            if (tid < kPartWin) ext[tid] = 0u;
            __syncthreads();
            volatile uint32_t *mycnt = cnt[w];
#pragma unroll
            for (int s = 0; s < kPartItems; ++s) {
                if (s >= ns) break;
                const int k = kw + s * kWave + lane;
                const bool in = k < nin;
                const bool bad = in && (id[s] < 0 || id[s] >= P.catalog);
                if (bad && w0 == 0) atomicCAS(reinterpret_cast<int32_t *>(P.misc + kMiscErr), 0, ARA_E_RANGE);
                const int r = (id[s] >> kRangeBits) - w0;
                const bool active = in && !bad && r >= 0 && r < wn;
                uint64_t peers = __ballot(active);
                for (int bit = 0; bit < gb; ++bit) {
                    const bool on = (r >> bit) & 1;
                    const uint64_t m = __ballot(on);
                    peers &= on ? m : ~m;
                }
                const uint32_t rank = lanes_below(peers);
                uint32_t before = 0;
                if (active) before = mycnt[r];
                wave_fence();
                if (active && rank == 0) mycnt[r] = before + static_cast<uint32_t>(__popcll(peers));
                wave_fence();
                tr[s] = (tr[s] & 0xFFFF0000u) | (before + rank);
            }
            __syncthreads();
            // where each (range, wavefront) starts (thread i < 256: range i)
            uint32_t c[kPartWaves], tot = 0;
#pragma unroll
            for (int v = 0; v < kPartWaves; ++v) {
                c[v] = tid < kPartWin ? cnt[v][tid] : 0u;
                tot += c[v];
            }
            uint32_t incl = tot;
            for (int o = 1; o < kWave; o <<= 1) {
                const uint32_t x = __shfl_up(incl, o);
                if (lane >= o) incl += x;
            }
            if (lane == kWave - 1) wsum[w] = incl;
            __syncthreads();
            uint32_t start = woff + incl - tot, all = 0;
            for (int v = 0; v < kPartWaves; ++v) {
                start += v < w ? wsum[v] : 0u;
                all += wsum[v];
            }
            uint32_t at = start;
            if (tid < kPartWin) {
#pragma unroll
                for (int v = 0; v < kPartWaves; ++v) {
                    cnt[v][tid] = at;
                    at += c[v];
                }
            }
            if (tid < wn) P.rstart[ch * (P.n_ranges + 1) + w0 + tid] = static_cast<uint16_t>(start);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < kPartItems; ++s) {
                if (s >= ns) break;
                const int k = kw + s * kWave + lane;
                const int r = (id[s] >> kRangeBits) - w0;
                if (k < nin && id[s] >= 0 && id[s] < P.catalog && r >= 0 && r < wn) {
                    const uint32_t p = cnt[w][r] + (tr[s] & 0xFFFFu);
                    const uint32_t tl = tr[s] >> 16;
                    srec[p] = (static_cast<uint32_t>(r) << 23) | (tl << kRangeBits) | static_cast<uint32_t>(id[s] & (kRange - 1));
                    if (POS) spos[p] = static_cast<uint16_t>(k - soff[tl]);
                }
            }
            __syncthreads();
            // the records out, and the codes a change of trial needs beside the event's own
            for (uint32_t i = woff + tid; i < woff + all; i += kPartThreads) {
                const uint32_t e = srec[i];
                if (i > woff) {
                    const uint32_t q = srec[i - 1];
                    const uint32_t te = (e >> kRangeBits) & 255u, tq = (q >> kRangeBits) & 255u;
                    if ((e >> 23) == (q >> 23) && te != tq) {
                        const uint32_t x = te - tq - 1u + ((e & (kRange - 1)) == kRange - 1 ? 1u : 0u);
                        if (x) atomicAdd(&ext[e >> 23], x);
                    }
                }
                P.rec[ks + i] = e & 0x7FFFFFu;
                if (POS) P.rpos[ks + i] = spos[i];
            }
            __syncthreads();
            if (tid < wn) {
                uint32_t sum = 0;
                if (tot) {
                    const uint32_t f = srec[start], l = srec[start + tot - 1];
                    sum = ext[tid] | (((f >> kRangeBits) & 255u) << 8) | (((l >> kRangeBits) & 255u) << 16) |
                          ((f & (kRange - 1)) == kRange - 1 ? 1u << 24 : 0u);
                }
                P.rsum[ch * P.n_ranges + w0 + tid] = sum;
            }
            woff += all;
            __syncthreads();
        }
        if (tid == 0) P.rstart[ch * (P.n_ranges + 1) + P.n_ranges] = static_cast<uint16_t>(woff);
    }
}

// Codes per lane of every segment: its events, the gap codes inside its runs
// and those between one run's last trial and the next run's first.
__global__ __launch_bounds__(256) void k_prep_sizes(PartParams P, int n_groups, int32_t *__restrict__ seg_run) {
    if (P.misc[kMiscBadOff] != 0) return;
    const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (i >= static_cast<int64_t>(n_groups) * P.n_ranges) return;
    const int64_t g = i / P.n_ranges;
    const int r = static_cast<int>(i - g * P.n_ranges);
    int64_t codes = 0;
    const int64_t t0 = g * P.tg;
    if (t0 < P.n_trials) {
        const int64_t o0 = P.off[t0], o1 = P.off[min<int64_t>(t0 + P.tg, P.n_trials)];
        int last = -1;
        for (int64_t ks = o0, ch = chunk_base(g, o0); ks < o1; ks += kChunk, ++ch) {
            const uint16_t *rs = P.rstart + ch * (P.n_ranges + 1) + r;
            const int n = static_cast<int>(rs[1]) - static_cast<int>(rs[0]);
            if (n <= 0) continue;
            const uint32_t m = P.rsum[ch * P.n_ranges + r];
            const int first = static_cast<int>((m >> 8) & 255u);
            codes += n + static_cast<int>(m & 255u);
            if (last >= 0 && first != last) codes += first - last - 1 + static_cast<int>((m >> 24) & 1u);
            last = static_cast<int>((m >> 16) & 255u);
        }
    }
    if (codes > (int64_t(1) << 31) - 512) {   // codes of a segment are counted in 32 bits
        atomicCAS(reinterpret_cast<int32_t *>(P.misc + kMiscErr), 0, ARA_E_LIMIT);
        codes = 0;
    }
    const int64_t b = g / kGroups;
    seg_run[(b * P.n_ranges + r) * kGroups + g % kGroups] = static_cast<int32_t>(((codes + kWave - 1) / kWave + 3) & ~int64_t(3));
}

// Exclusive scan of 64 * seg_run into seg_base: workgroup sums, the scan of
// the sums by one workgroup (which also leaves the total), then each
// workgroup's own scan on top.
__device__ __forceinline__ int64_t scan1024_i64(int64_t v, int64_t *wsum, int64_t *total) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int64_t incl = v;
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t x = __shfl_up(incl, o);
        if (lane >= o) incl += x;
    }
    if (lane == kWave - 1) wsum[w] = incl;
    __syncthreads();
    int64_t before = 0, tot = 0;
    for (int i = 0; i < 16; ++i) {
        const int64_t c = wsum[i];
        before += i < w ? c : 0;
        tot += c;
    }
    *total = tot;
    __syncthreads();
    return before + incl - v;
}

__global__ __launch_bounds__(1024) void k_scan_sums(const int32_t *__restrict__ seg_run, int64_t n, int64_t *__restrict__ bsum) {
    __shared__ int64_t wsum[16];
    int64_t v = 0, tot = 0;
    for (int q = 0; q < kScanPer; ++q) {
        const int64_t i = blockIdx.x * static_cast<int64_t>(kScanBlock) + threadIdx.x * kScanPer + q;
        if (i < n) v += seg_run[i];
    }
    scan1024_i64(v, wsum, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot * kWave;
}

// bsum[0..n) becomes its exclusive scan; *total gets the sum.
__global__ __launch_bounds__(1024) void k_scan_top(int64_t *__restrict__ bsum, int64_t n, int64_t *__restrict__ total) {
    __shared__ int64_t wsum[16];
    int64_t run = 0;
    for (int64_t i0 = 0; i0 < n; i0 += 1024) {
        const int64_t i = i0 + threadIdx.x;
        const int64_t v = i < n ? bsum[i] : 0;
        int64_t tot = 0;
        const int64_t ex = scan1024_i64(v, wsum, &tot);
        if (i < n) bsum[i] = run + ex;
        run += tot;
    }
    if (threadIdx.x == 0) *total = run;
}

// bsum null: one block alone, and *total gets the sum.
__global__ __launch_bounds__(1024) void k_scan_bases(const int32_t *__restrict__ seg_run, int64_t n,
                                                     const int64_t *__restrict__ bsum, int64_t *__restrict__ seg_base,
                                                     int64_t *__restrict__ total) {
    __shared__ int64_t wsum[16];
    int64_t c[kScanPer], v = 0, tot = 0;
    const int64_t i0 = blockIdx.x * static_cast<int64_t>(kScanBlock) + threadIdx.x * kScanPer;
    for (int q = 0; q < kScanPer; ++q) {
        c[q] = i0 + q < n ? static_cast<int64_t>(seg_run[i0 + q]) * kWave : 0;
        v += c[q];
    }
    int64_t at = scan1024_i64(v, wsum, &tot);
    if (bsum) at += bsum[blockIdx.x];
    else if (threadIdx.x == 0) *total = tot;
    for (int q = 0; q < kScanPer; ++q) {
        if (i0 + q < n) seg_base[i0 + q] = at;
        at += c[q];
    }
}

struct EmitParams {
    PartParams part;
    int32_t n_groups;
    const int64_t *seg_base;
    const int32_t *seg_run;
    uint16_t *code, *pos;
    uint8_t *lane_start;
};

// One wavefront per segment: the segment's runs in chunk order, each record
// preceded by its gap codes, into LDS at the codes' final places, then out as
// whole lines (padding included).  A segment of more than CAP codes per lane
// is written to memory directly (CAP is chosen above the mean, so these are
// segments of crowded ranges).  The last workgroup writes the skip codes
// after the last code.
template <int CAP, bool POS>
__global__ __launch_bounds__(kEmitThreads) void k_prep_emit(EmitParams P) {
    __shared__ __align__(16) uint16_t scode_all[kEmitWaves][CAP * kWave];
    __shared__ __align__(16) uint16_t spos_all[POS ? kEmitWaves : 1][POS ? CAP * kWave : 8];
    __shared__ __align__(16) uint8_t sstart_all[kEmitWaves][kWave];
    const int32_t *err = reinterpret_cast<const int32_t *>(P.part.misc + kMiscErr);
    if (*err != 0) return;
    const int lane = threadIdx.x & 63;
    const int w = static_cast<int>(uni32(threadIdx.x >> 6));
    const int nr = P.part.n_ranges;
    const int64_t wg = grid_index(), last_wg = (static_cast<int64_t>(P.n_groups) * nr + kEmitWaves - 1) / kEmitWaves;
    if (wg > last_wg) return;
    if (wg == last_wg) {
        const int64_t total = P.part.misc[kMiscCodes];
        for (int i = threadIdx.x; i < kPadCodes; i += kEmitThreads) {
            P.code[total + i] = kSkip;
            if (POS) P.pos[total + i] = kSkip;
        }
        return;
    }
    const int64_t idx = wg * kEmitWaves + w;
    if (idx >= static_cast<int64_t>(P.n_groups) * nr) return;   // no barriers below
    const int64_t g = idx / nr;
    const int r = static_cast<int>(idx - g * nr);
    const size_t si = (static_cast<size_t>(g / kGroups) * nr + r) * kGroups + static_cast<size_t>(g % kGroups);
    const int R = static_cast<int>(uni32(static_cast<uint32_t>(P.seg_run[si])));
    const int64_t base = P.seg_base[si];
    uint8_t *ls = P.lane_start + si * kWave;
    if (R == 0) {
        ls[lane] = 0;
        return;
    }
    const bool staged = R <= CAP;
    uint16_t *sc = scode_all[w], *sp = spos_all[POS ? w : 0];
    uint8_t *ss = sstart_all[w];
    const uint4 ff = make_uint4(~0u, ~0u, ~0u, ~0u);
    uint4 *gcode = reinterpret_cast<uint4 *>(P.code + base), *gpos = reinterpret_cast<uint4 *>(POS ? P.pos + base : nullptr);
    if (staged) {
        ss[lane] = 0;
        for (int i = lane; i < 8 * R; i += kWave) {
            reinterpret_cast<uint4 *>(sc)[i] = ff;
            if (POS) reinterpret_cast<uint4 *>(sp)[i] = ff;
        }
        wave_fence();
    } else {
        ls[lane] = 0;
        for (int i = lane; i < 8 * R; i += kWave) {
            gcode[i] = ff;
            if (POS) gpos[i] = ff;
        }
        __threadfence();   // before this wavefront's own stores to the same lines
    }
    const float inv = 1.0f / static_cast<float>(R);
    // place q of the segment's stream: lane q / R, step q % R
    auto put = [&](int64_t q, bool event, uint16_t c, uint32_t start, uint16_t at) {
        int lj, s;
        if (staged) {   // q < 64 CAP: the binary32 quotient is within one of the true one
            lj = static_cast<int>(static_cast<float>(static_cast<int>(q)) * inv);
            s = static_cast<int>(q) - lj * R;
            if (s < 0) {
                --lj;
                s += R;
            } else if (s >= R) {
                ++lj;
                s -= R;
            }
        } else {
            lj = static_cast<int>(q / R);
            s = static_cast<int>(q - static_cast<int64_t>(lj) * R);
        }
        const int slot = (s >> 2) * (4 * kWave) + 4 * lj + (s & 3);
        if (staged) {
            if (event) {
                sc[slot] = c;
                if (POS) sp[slot] = at;
            }
            if (s == 0) ss[lj] = static_cast<uint8_t>(start);
        } else {
            if (event) {
                P.code[base + slot] = c;
                if (POS) P.pos[base + slot] = at;
            }
            if (s == 0) ls[lj] = static_cast<uint8_t>(start);
        }
    };
    const int64_t t0 = g * P.part.tg;
    const int64_t o0 = P.part.off[t0], o1 = P.part.off[min<int64_t>(t0 + P.part.tg, P.part.n_trials)];
    const int64_t cb = chunk_base(g, o0);
    const int64_t nch = (o1 - o0 + kChunk - 1) / kChunk;
    int64_t p = 0;        // codes placed (uniform)
    int prev = -1;        // trial of the last record (uniform)
    for (int64_t c0 = 0; c0 < nch; c0 += kWave) {
        // the run bounds of up to 64 chunks, one per lane
        uint32_t ra = 0, rb = 0;
        if (c0 + lane < nch) {
            const uint16_t *rs = P.part.rstart + (cb + c0 + lane) * (nr + 1) + r;
            ra = rs[0];
            rb = rs[1];
        }
        const int nc = static_cast<int>(min<int64_t>(kWave, nch - c0));
        // the runs in steps of up to 64 records, the next step's loads in
        // flight while one is placed
        int c = -1, i = 0, end = 0;   // uniform: the run being read
        uint32_t e = 0, e_nxt = 0;
        uint16_t at = 0, at_nxt = 0;
        auto fetch = [&]() -> int {   // records of the next step (0: none left)
            while (i >= end) {
                if (++c >= nc) return 0;
                i = static_cast<int>(__builtin_amdgcn_readlane(ra, c));
                end = static_cast<int>(__builtin_amdgcn_readlane(rb, c));
            }
            const int n = min(kWave, end - i);
            const int64_t k = o0 + (c0 + c) * kChunk + i;
            if (lane < n) {
                e_nxt = P.part.rec[k + lane];
                if (POS) at_nxt = P.part.rpos[k + lane];
            }
            i += n;
            return n;
        };
        int n_nxt = fetch();
        while (n_nxt > 0) {
            const int n_in = n_nxt;
            e = e_nxt;
            at = at_nxt;
            n_nxt = fetch();
            const bool in = lane < n_in;
            const int t = static_cast<int>(e >> kRangeBits);
            const uint32_t local = e & (kRange - 1);
            int tp = __shfl_up(t, 1);
            if (lane == 0) tp = prev;
            const bool opens = in && tp >= 0 && t != tp;
            int gap = opens ? t - tp - 1 : 0;
            bool adv = opens;
            if (opens && local == kRange - 1) {   // offset 0x7FFF cannot carry the flag
                ++gap;
                adv = false;
            }
            int64_t q = p + lane;
            int total = n_in;
            if (__ballot(gap > 0) != 0) {
                int incl = in ? 1 + gap : 0;
                for (int o = 1; o < kWave; o <<= 1) {
                    const int x = __shfl_up(incl, o);
                    if (lane >= o) incl += x;
                }
                total = __shfl(incl, kWave - 1);
                q = p + incl - 1;
                for (int z = 0; z < gap; ++z) put(q - gap + z, false, kSkip, static_cast<uint32_t>(tp + z), kSkip);
            }
            if (in)
                put(q, true, static_cast<uint16_t>((adv ? kAdvance : 0) | local), static_cast<uint32_t>(t - (adv ? 1 : 0)), at);
            p += total;
            prev = __builtin_amdgcn_readlane(t, n_in - 1);
        }
    }
    if (staged) {
        wave_fence();
        ls[lane] = ss[lane];
        for (int i = lane; i < 8 * R; i += kWave) {
            gcode[i] = reinterpret_cast<const uint4 *>(sc)[i];
            if (POS) gpos[i] = reinterpret_cast<const uint4 *>(sp)[i];
        }
    }
}

// Marks a prepared YET whose buffer holds event-ordered blocks, with the
// flags it was prepared with: the pieces' places follow from the sizes and
// those flags.
constexpr int32_t kHasEvBlocks = 0x100;
// ... and one whose binary64 forward takes them.
constexpr int32_t kEvForward = 0x200;
constexpr int32_t kEvAlwaysBackward = 0x400;   // (ev_always_backward)
constexpr int32_t kEvAlwaysUncertain = 0x800;  // (ev_always_uncertain)
constexpr int32_t kEvMarks = kEvForward | kEvAlwaysBackward | kEvAlwaysUncertain;

// Whether the forward of a YET takes its event-ordered blocks.  It depends on
// the YET alone, so that a layer's results are the same in every call.  The
// blocks are the faster of the two but for (us of one layer's call over
// uniform event frequencies: blocks, stream):
//   * events in most years, whose lists a few workgroups have to themselves:
//     on average 3200 entries a list 274, 255 (400,000 x 1000), 2670 entries
//     236, 255; one event's 11,000, all of the 64 most frequent held by the
//     layer 146, 139 (100,000 x 1000), 3400 entries 118, 140;
//   * few ranges and few occurrences, where the stream is as short as the
//     blocks' chain of launches: 20,000 x 1000 over 10,000 events 80, 53,
//     30,000 61, 55, 60,000 62, 57, 100,000 57, 62; over 10,000 events 50,000 x
//     1000 88, 71 and 100,000 x 1000 90, 94;
//   * many short years, whose blocks are walked for a few entries: 3M x 60 over
//     2M events (0.24 a list) 458, 352, 3M x 150 (0.61) 496, 491, 10M x 10 over
//     300,000 (0.27) 257, 213, x 60 (1.6) 380, 432; with no more blocks than
//     workgroups run at once the blocks win (1M x 10 over 2M 161, 242).
static bool ev_pays(const EvGeometry &g, int64_t nnz, int32_t catalog, int32_t max_occ) {
    const double mean = static_cast<double>(nnz) / (static_cast<double>(catalog) * g.neb);
    if (mean > 3000.0 || static_cast<double>(max_occ) > 10000.0 * g.neb) return false;
    if (catalog <= 3 * kRange && static_cast<double>(nnz) * catalog < 1.3e12) return false;
    return g.neb <= 150 || mean >= 0.85;
}

bool ev_forward_blocks(const ara_yet *yet, EvBlocks *out) { return (yet->reserved & kEvForward) != 0 && ev_blocks(yet, out); }

bool ev_always_backward(const ara_yet *yet) { return (yet->reserved & kEvAlwaysBackward) != 0; }

bool ev_always_uncertain(const ara_yet *yet) { return (yet->reserved & kEvAlwaysUncertain) != 0; }

bool ev_blocks(const ara_yet *yet, EvBlocks *out) {
    if ((yet->reserved & ~(static_cast<int32_t>(kPrepFlags) | kEvMarks)) != kHasEvBlocks || yet->n_blocks == 0) return false;
    const uint32_t flags = static_cast<uint32_t>(yet->reserved) & kPrepFlags;
    Geometry g{};
    g.tg = yet->trials_per_group;
    g.tb = yet->trials_per_block;
    g.n_blocks = yet->n_blocks;
    g.n_ranges = yet->n_ranges;
    g.nseg = static_cast<size_t>(g.n_blocks) * g.n_ranges * kGroups;
    Carver c(yet->code);
    const Prepared p = carve(c, g, yet->n_trials, yet->nnz, yet->catalog, flags);
    const EvGeometry eg = ev_geometry(yet->n_trials, yet->nnz, yet->catalog);
    out->ent = p.ent;
    out->pos = p.ev_pos;
    out->hdr = p.hdr;
    out->start = p.start;
    out->base = p.ev_base;
    out->misc = p.misc;
    out->n_trials = yet->n_trials;
    out->et = eg.et;
    out->neb = eg.neb;
    out->ng = eg.ng;
    out->dense = eg.dense;
    out->catalog = yet->catalog;
    return true;
}

}  // namespace ara

using namespace ara;

static int32_t check_sizes(const char *what, int64_t n_trials, int64_t nnz, int32_t catalog, uint32_t flags) {
    const std::string at = std::string(what) + ": ";
    if (n_trials < 0 || nnz < 0 || catalog <= 0) return fail(ARA_E_INVAL, at + "negative size");
    if (catalog > ARA_MAX_CATALOG) return fail(ARA_E_LIMIT, "catalog exceeds ARA_MAX_CATALOG");
    if (flags & ~kPrepFlags) return fail(ARA_E_INVAL, at + "unknown flag");
    return ARA_OK;
}

extern "C" int32_t ara_yet_prepare_bytes(int64_t n_trials, int64_t nnz, int32_t catalog, uint32_t flags,
                                         size_t *bytes) {
    if (!bytes) return fail(ARA_E_INVAL, "ara_yet_prepare_bytes: null output");
    const int32_t rc = check_sizes("ara_yet_prepare_bytes", n_trials, nnz, catalog, flags);
    if (rc) return rc;
    const PrepareBytes b = prepare_bytes(geometry(n_trials, catalog), n_trials, nnz, catalog, flags, false);
    *bytes = b.keep + b.scratch;
    return ARA_OK;
}

extern "C" int32_t ara_yet_prepare_split_bytes(int64_t n_trials, int64_t nnz, int32_t catalog, uint32_t flags,
                                               size_t *keep, size_t *scratch) {
    if (!keep || !scratch) return fail(ARA_E_INVAL, "ara_yet_prepare_split_bytes: null output");
    const int32_t rc = check_sizes("ara_yet_prepare_split_bytes", n_trials, nnz, catalog, flags);
    if (rc) return rc;
    const PrepareBytes b = prepare_bytes(geometry(n_trials, catalog), n_trials, nnz, catalog, flags, true);
    *keep = b.keep;
    *scratch = b.scratch;
    return ARA_OK;
}

// scratch null: it follows what stays in buf, without lent places.
static int32_t prepare(const char *what, const int64_t *offsets, const int32_t *ids, int64_t n_trials, int32_t catalog,
                       uint32_t flags, void *buf, size_t buf_bytes, void *scratch, size_t scratch_bytes, void *stream,
                       ara_yet *out) {
    const std::string at = std::string(what) + ": ";
    if (!offsets || !buf || !out) return fail(ARA_E_INVAL, at + "null pointer");
    if (n_trials < 0 || catalog <= 0) return fail(ARA_E_INVAL, at + "bad size");
    if (catalog > ARA_MAX_CATALOG) return fail(ARA_E_LIMIT, "catalog exceeds ARA_MAX_CATALOG");
    if (flags & ~kPrepFlags) return fail(ARA_E_INVAL, at + "unknown flag");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Geometry g = geometry(n_trials, catalog);
    int64_t ends[2] = {0, 0};
    ARA_HIP(hipMemcpyAsync(&ends[0], offsets, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    ARA_HIP(hipMemcpyAsync(&ends[1], offsets + n_trials, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    ARA_HIP(hipStreamSynchronize(st));
    if (ends[0] != 0 || ends[1] < 0) return fail(ARA_E_RANGE, "offsets[0] must be 0 and offsets[n] >= 0");
    const int64_t nnz = ends[1];
    if (nnz > 0 && !ids) return fail(ARA_E_INVAL, at + "null ids");
    const PrepareBytes need = prepare_bytes(g, n_trials, nnz, catalog, flags, scratch != nullptr);
    if (buf_bytes < need.keep + (scratch ? 0 : need.scratch)) return fail(ARA_E_NOSPACE, at + "buffer too small");
    if (scratch && scratch_bytes < need.scratch) return fail(ARA_E_NOSPACE, at + "scratch too small");

    Carver c(buf);
    Prepared p = carve(c, g, n_trials, nnz, catalog, flags);
    Carver s(scratch ? scratch : static_cast<char *>(buf) + need.keep);
    carve_scratch(s, p, g, n_trials, nnz, catalog, flags, scratch != nullptr);
    const bool transposed = (flags & ARA_PREP_TRANSPOSED) != 0, positions = (flags & ARA_PREP_POSITIONS) != 0;
    if (flags & ARA_PREP_TRIAL_MAJOR) {
        ARA_HIP(hipMemsetAsync(p.t_cnt, 0, static_cast<size_t>(catalog) * sizeof(int32_t), st));
    }
    if (p.t_off)
        ARA_HIP(hipMemcpyAsync(p.t_off, offsets, (static_cast<size_t>(n_trials) + 1) * sizeof(int64_t),
                               hipMemcpyDeviceToDevice, st));
    ARA_HIP(hipMemsetAsync(p.misc, 0, 32 * sizeof(int64_t), st));

    ara_yet y{};
    y.n_trials = n_trials;
    y.nnz = nnz;
    y.catalog = catalog;
    y.range_bits = kRangeBits;
    y.n_ranges = g.n_ranges;
    y.groups = kGroups;
    y.trials_per_group = g.tg;
    y.trials_per_block = g.tb;
    y.n_blocks = g.n_blocks;
    y.code = p.code;
    y.seg_base = p.seg_base;
    y.seg_run = p.seg_run;
    y.lane_start = p.lane_start;
    y.t_off = p.t_off;
    y.t_ids = p.t_ids;
    y.t_cnt = p.t_cnt;
    y.pos = p.pos;
    if (transposed) {
        y.n_slices = kSlices;
        y.slice_trials = static_cast<int64_t>(g.slice_blocks) * g.tb;
        y.tr_off = p.tr_off;
        y.tr_ent = p.tr_ent;
    }
    if (g.n_blocks == 0) {
        if (transposed)   // every list is empty
            ARA_HIP(hipMemsetAsync(p.tr_off, 0, (static_cast<size_t>(kSlices) * catalog + 1) * sizeof(int64_t), st));
        ARA_HIP(hipStreamSynchronize(st));
        *out = y;
        return ARA_OK;
    }
    // the codes: sort by range, count, place
    PartParams P{};
    P.off = offsets;
    P.ids = ids;
    P.n_trials = n_trials;
    P.catalog = catalog;
    P.tg = g.tg;
    P.n_ranges = g.n_ranges;
    P.rec = p.rec;
    P.rpos = p.rpos;
    P.rstart = p.rstart;
    P.rsum = p.rsum;
    P.misc = p.misc;
    const int64_t ng = n_groups_of(g, n_trials);
    const int n_groups = g.n_blocks * kGroups;   // the last block's empty groups have segments too
    k_prep_check<<<static_cast<unsigned>(std::min<int64_t>((n_trials + 255) / 256, 512)), 256, 0, st>>>(
        offsets, n_trials, p.misc, positions ? kMaxPositions : INT64_MAX);
    if (positions) k_prep_part<true><<<static_cast<unsigned>(ng), kPartThreads, 0, st>>>(P);
    else k_prep_part<false><<<static_cast<unsigned>(ng), kPartThreads, 0, st>>>(P);
    const int64_t n_segs = static_cast<int64_t>(g.nseg);
    k_prep_sizes<<<static_cast<unsigned>((n_segs + 255) / 256), 256, 0, st>>>(P, n_groups, p.seg_run);
    const int64_t n_scan = (n_segs + kScanBlock - 1) / kScanBlock;
    if (n_scan > 1) {
        k_scan_sums<<<static_cast<unsigned>(n_scan), 1024, 0, st>>>(p.seg_run, n_segs, p.bsum);
        k_scan_top<<<1, 1024, 0, st>>>(p.bsum, n_scan, p.misc + kMiscCodes);
    }
    k_scan_bases<<<static_cast<unsigned>(n_scan), 1024, 0, st>>>(p.seg_run, n_segs, n_scan > 1 ? p.bsum : nullptr, p.seg_base,
                                                                p.misc + kMiscCodes);
    ARA_HIP(hipGetLastError());
    int64_t head[8] = {};
    ARA_HIP(hipMemcpyAsync(head, p.misc, sizeof(head), hipMemcpyDeviceToHost, st));
    ARA_HIP(hipStreamSynchronize(st));
    const int32_t err_h = static_cast<int32_t>(head[kMiscErr] & 0xffffffff);
    if (err_h == ARA_E_LIMIT) return fail(err_h, "ara_yet_prepare: 2^31 or more codes in one segment");
    if (err_h) return fail(err_h, "ara_yet_prepare: an event ID lies outside [0, catalog) or offsets decrease");
    if (head[kMiscLong] != 0)
        return fail(ARA_E_LIMIT, "ara_yet_prepare: a trial holds more than 65536 occurrences (positions)");
    const int64_t total = head[kMiscCodes];
    if (total > max_codes(g, nnz)) return fail(ARA_E_LIMIT, "ara_yet_prepare: code bound exceeded");
    EmitParams M{};
    M.part = P;
    M.n_groups = n_groups;
    M.seg_base = p.seg_base;
    M.seg_run = p.seg_run;
    M.code = p.code;
    M.pos = p.pos;
    M.lane_start = p.lane_start;
    // codes per lane staged in LDS: 48 leaves room for five workgroups on a
    // CU and holds the segments of up to 40 codes per lane on average; 128
    // (16 KB a wavefront) those of the densest groups
    const bool small = static_cast<double>(nnz) <= 40.0 * kWave * static_cast<double>(ng) * g.n_ranges;
    const dim3 ge = grid_of((n_segs + kEmitWaves - 1) / kEmitWaves + 1);
    if (positions) {
        if (small) k_prep_emit<48, true><<<ge, kEmitThreads, 0, st>>>(M);
        else k_prep_emit<128, true><<<ge, kEmitThreads, 0, st>>>(M);
    } else {
        if (small) k_prep_emit<48, false><<<ge, kEmitThreads, 0, st>>>(M);
        else k_prep_emit<128, false><<<ge, kEmitThreads, 0, st>>>(M);
    }
    ARA_HIP(hipGetLastError());
    EvBuild E{};
    E.g = ev_geometry(n_trials, nnz, catalog);
    E.off = offsets;
    E.ids = ids;
    E.n_trials = n_trials;
    E.nnz = nnz;
    E.catalog = catalog;
    E.ent = p.ent;
    E.pos = p.ev_pos;
    E.rpos = p.ev_rpos;
    E.hdr = p.hdr;
    E.start = p.start;
    E.base = p.ev_base;
    E.misc = p.misc;
    E.t_ids = p.t_ids;
    E.rec = p.rec;
    E.tstart = p.tstart;
    E.tbase = p.tbase;
    E.mark = p.mark;
    int32_t rc = ev_build(E, st);
    if (rc) return rc;
    y.reserved = kHasEvBlocks | static_cast<int32_t>(flags);
    y.n_codes = total;
    EvBlocks B{};
    ev_blocks(&y, &B);
    if ((rc = ev_count(B, p.t_cnt, st))) return rc;
    if (transposed && (rc = ev_major(B, y.slice_trials, p.tr_off, p.tr_ent, p.ssum, p.misc, st))) return rc;
    ARA_HIP(hipMemcpyAsync(head, p.misc, sizeof(head), hipMemcpyDeviceToHost, st));
    ARA_HIP(hipStreamSynchronize(st));
    if ((head[kMiscErr] & 0xffffffff) != 0)
        return fail(ARA_E_LIMIT, "ara_yet_prepare: 2^32 or more occurrences in one (slice, range) or one block of 8128 trials");
    y.max_occ = static_cast<int32_t>(head[kMiscMaxOcc] & 0xffffffff);
    if (ev_pays(E.g, nnz, catalog, y.max_occ)) y.reserved |= kEvForward;
    *out = y;
    return ARA_OK;
}

extern "C" int32_t ara_yet_prepare(const int64_t *offsets, const int32_t *ids, int64_t n_trials, int32_t catalog,
                                   uint32_t flags, void *buf, size_t buf_bytes, void *stream, ara_yet *out) {
    return prepare("ara_yet_prepare", offsets, ids, n_trials, catalog, flags, buf, buf_bytes, nullptr, 0, stream, out);
}

extern "C" int32_t ara_yet_prepare_split(const int64_t *offsets, const int32_t *ids, int64_t n_trials, int32_t catalog,
                                         uint32_t flags, void *buf, size_t buf_bytes, void *scratch,
                                         size_t scratch_bytes, void *stream, ara_yet *out) {
    if (!scratch) return fail(ARA_E_INVAL, "ara_yet_prepare_split: null pointer");
    return prepare("ara_yet_prepare_split", offsets, ids, n_trials, catalog, flags, buf, buf_bytes, scratch,
                   scratch_bytes, stream, out);
}
