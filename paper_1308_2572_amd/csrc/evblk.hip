// Building the event-ordered blocks (evblk.h) and what is derived from them:
// the events' occurrence counts and the event-major copy of the backward.
//
// A block's 8 million occurrences (8065 trials x 1000) are sorted by event in
// two levels, each inside LDS and written as runs: chunks of 16384
// occurrences by tile of 2^te_bits events (k_ev_part), then each tile's
// 16,600 records by event (k_ev_sort).  Each level reads and writes every
// occurrence once and is bound by that and by keeping enough loads in flight
// (2.7-3.1 and 2.7 ms at 1M x 1000: 8 and 6.3 GB).  The event-major lists are
// then gathered from the blocks (3.1 ms; scattering each entry to its place
// cost one memory write per entry: 26.7 ms), and the events' counts from the
// headers (0.24 ms; from the code stream, one workgroup per range, 8.7 ms).
// With positions each record carries its occurrence's position through both
// levels beside it, in half the workgroups per CU (250,000 x 1000: 0.88 and
// 1.2 ms).
#include "evblk.h"

#include <algorithm>

namespace ara {

constexpr int kEvThreads = 1024;
constexpr int kEvWaves = kEvThreads / kWave;
constexpr int kEvItems = kEvChunk / kEvThreads;      // slices of 64 occurrences per wavefront
constexpr int kEvWin = 1024;                         // tiles counted at once
// Records per thread of a tile sorted in registers, and of the tile: 20480, and
// one per thread less with positions, whose entries take twice the LDS.
constexpr int sort_items(bool pos) { return pos ? 19 : 20; }
constexpr int sort_cap(bool pos) { return sort_items(pos) * kEvThreads; }
constexpr int kSortRuns = 2048;                      // runs of a tile listed at once
constexpr int kEvSlotBits = 14;                      // event in the tile, in a record
constexpr int kEvTileBits = 12;                      // largest tile of a catalogue of up to kEvTileMany of them
constexpr int64_t kEvTileMany = 4096;

// LDS of k_ev_sort for tiles of 2^te_bits events.
constexpr size_t sort_lds(int te_bits, bool pos) {
    return ((size_t(1) << te_bits) + 2 * kSortRuns + 1 + kEvWaves) * sizeof(uint32_t) +
           (pos ? 2 : 1) * static_cast<size_t>(sort_cap(pos)) * sizeof(uint16_t);
}
static_assert(sort_lds(kEvSlotBits, true) <= 160 * 1024 && sort_lds(kEvSlotBits, false) <= 160 * 1024,
              "the largest tile's workgroup fits a CU's LDS");
static_assert((int64_t(ARA_MAX_CATALOG) >> kEvSlotBits) <= kEvTileMany, "tiles of the largest catalogue");
static_assert(kEvWin == kEvThreads, "one counter per thread");
static_assert(kEvItems * kWave == kEvMark, "a wavefront's share of a chunk starts at a mark");

EvGeometry ev_geometry(int64_t n_trials, int64_t nnz, int32_t catalog) {
    EvGeometry g{};
    // blocks of equal size, as few as 8128 trials allow (longer lists per
    // event: at 1M x 1000 and 7% of the events read, a prototype took 302 us
    // over blocks of 7872 trials, 390 over 3936 and 510 over 1968), and of less than
    // 2^31 entries on average
    const int64_t neb = std::max<int64_t>({1, (n_trials + kEvBlockTrials - 1) / kEvBlockTrials, nnz >> 31});
    g.et = static_cast<int32_t>(std::max<int64_t>(1, (n_trials + neb - 1) / neb));
    g.neb = static_cast<int32_t>((n_trials + g.et - 1) / g.et);
    g.ng = (catalog + 7) / 8 + 1;
    const double mean = static_cast<double>(nnz) / (static_cast<double>(catalog) * std::max(g.neb, 1));
    // from about six per list on, lengths of fifteen and more get common (of
    // a Poisson count of mean 6, one in 1400; of mean 8, one in 120)
    g.dense = mean > 6.0;
    // the largest tile of at most 18,000 records on average, at most 4096
    // events (16 KB of counters) while that gives at most 4096 tiles
    const int most = static_cast<int64_t>(catalog) > kEvTileMany << kEvTileBits ? kEvSlotBits : kEvTileBits;
    g.te_bits = 3;
    while (g.te_bits < most && mean * (2 << g.te_bits) <= 18000.0) ++g.te_bits;
    if (g.te_bits < most)   // crowded small catalogues: no more tiles than a chunk can count in few windows
        while ((static_cast<int64_t>(catalog) >> g.te_bits) > kEvTileMany) ++g.te_bits;
    g.n_tiles = static_cast<int32_t>((static_cast<int64_t>(catalog) + (int64_t(1) << g.te_bits) - 1) >> g.te_bits);
    g.n_chunks = nnz / kEvChunk + g.neb + 1;
    g.n_marks = nnz / kEvMark + 1;
    return g;
}

// Set by a kernel before the caller's, if at all: the same for all its threads.
__device__ __forceinline__ bool ev_failed(const int64_t *misc) { return *reinterpret_cast<const int32_t *>(misc + kMiscErr) != 0; }

// A value the compiler does not know: what is computed from it is computed
// again instead of being kept in registers from an earlier loop over the same
// array (in k_ev_part without positions 117 registers, and with this 64, 18
// of them spilled: 76 bytes a lane).
__device__ __forceinline__ void keep_apart(int &v) { asm("" : "+v"(v)); }

__device__ __forceinline__ uint32_t uni32(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// First entry of every block, and the trial holding every kEvMark-th
// occurrence.
__global__ __launch_bounds__(256) void k_ev_marks(EvBuild B) {
    const int64_t i0 = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t t = i0; t < B.n_trials; t += step) {
        const int64_t a = B.off[t], z = B.off[t + 1];
        for (int64_t j = (a + kEvMark - 1) / kEvMark; j * kEvMark < z; ++j) B.mark[j] = static_cast<uint32_t>(t);
    }
    for (int64_t b = i0; b <= B.g.neb; b += step) {
        const int64_t t0 = min<int64_t>(b * B.g.et, B.n_trials);
        B.base[b] = B.off[t0];
        if (b < B.g.neb && B.off[min<int64_t>(t0 + B.g.et, B.n_trials)] - B.off[t0] >= (int64_t(1) << 32) - kEvPad)
            atomicCAS(reinterpret_cast<int32_t *>(B.misc + kMiscErr), 0, ARA_E_LIMIT);
    }
}

// The occurrences [q kEvChunk, (q + 1) kEvChunk) of block b are its chunk q,
// with index q + b (a block's first and last chunks may be partial; the next
// block's first chunk has the next index).
__device__ __forceinline__ int64_t ev_chunk0(const int64_t *base, int b) { return base[b] / kEvChunk + b; }

// One workgroup per chunk: records (trial in the block << 14 | event in the
// tile) sorted by tile inside LDS, each tile's start in the chunk, and the
// copy of the IDs.
template <bool POS>
__global__ __launch_bounds__(kEvThreads) __attribute__((amdgpu_waves_per_eu(POS ? 4 : 8, 8))) void k_ev_part(EvBuild B) {
    __shared__ uint32_t srec[kEvChunk];
    __shared__ uint16_t spos[POS ? kEvChunk : 1];
    __shared__ uint32_t cnt[kEvWin];
    __shared__ uint32_t wsum[kEvWaves];
    __shared__ int32_t s_b;
    if (ev_failed(B.misc)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = static_cast<int>(uni32(tid >> 6));
    const int64_t ch = blockIdx.x;
    if (tid == 0) s_b = -1;
    __syncthreads();
    for (int b = tid; b < B.g.neb; b += kEvThreads)
        if (ch >= ev_chunk0(B.base, b) && ch < ev_chunk0(B.base, b + 1)) s_b = b;
    __syncthreads();
    const int b = static_cast<int>(uni32(static_cast<uint32_t>(s_b)));
    if (b < 0) return;   // uniform
    const int64_t q = ch - b;
    const int64_t o0 = B.base[b], o1 = B.base[b + 1];
    const int64_t ks = q * kEvChunk;                     // element 0 of the chunk's frame
    const int lo = static_cast<int>(max<int64_t>(o0 - ks, 0));
    const int hi = static_cast<int>(min<int64_t>(o1 - ks, kEvChunk));
    uint16_t *ts = B.tstart + ch * (B.g.n_tiles + 1);
    if (hi <= lo) {   // uniform
        for (int i = tid; i <= B.g.n_tiles; i += kEvThreads) ts[i] = 0;
        return;
    }
    const int kw = w * kEvMark;
    int32_t id[kEvItems];
    const int32_t *src = B.ids + ks;
    int32_t *tcopy = B.t_ids ? B.t_ids + ks : nullptr;
#pragma unroll
    for (int s = 0; s < kEvItems; ++s) {
        const int k = kw + s * kWave + lane;
        id[s] = k >= lo && k < hi ? src[static_cast<uint32_t>(k)] : -1;
    }
    // each occurrence's trial in the block, left in the place of srec with
    // its number: from the mark (or the block's first trial) on, 64 trial
    // ends at a time
    if (kw < hi) {   // uniform over the wavefront
        const int64_t T0 = static_cast<int64_t>(b) * B.g.et;
        const int nt = static_cast<int>(min<int64_t>(B.g.et, B.n_trials - T0));
        int t = 0;
        if (ks + kw > o0) t = static_cast<int>(uni32(static_cast<uint32_t>(B.mark[(ks + kw) / kEvMark] - T0)));
        int ends = 0, tw = t - kWave;   // lane l of `ends`: where trial tw + 1 + l starts
        const int far = 1 << 30;
#pragma unroll 1
        for (int s = 0; s < kEvItems; ++s) {
            const int k = kw + s * kWave + lane, last = kw + s * kWave + (kWave - 1);
            uint32_t tl = static_cast<uint32_t>(t);
            while (t + 1 < nt) {
                if (t - tw >= kWave) {
                    tw = t;
                    const int i = t + 1 + lane;
                    ends = i < nt ? static_cast<int>(max<int64_t>(-1, min<int64_t>(far, B.off[T0 + i] - ks))) : far;
                }
                const int e = __builtin_amdgcn_readlane(ends, t - tw);
                if (e > last) break;
                tl += k >= e ? 1u : 0u;
                ++t;
            }
            srec[k] = tl;
        }
    }
    uint32_t tr[kEvItems];
#pragma unroll
    for (int s = 0; s < kEvItems; ++s) tr[s] = srec[kw + s * kWave + lane];
    uint32_t at[POS ? kEvItems : 1];   // positions in the trial
    if (POS) {
        const int64_t *first = B.off + static_cast<int64_t>(b) * B.g.et;
#pragma unroll
        for (int s = 0; s < kEvItems; ++s) {
            const int k = kw + s * kWave + lane;
            at[s] = id[s] >= 0 ? static_cast<uint32_t>(ks + k - first[tr[s]]) : 0u;
        }
    }
    if (tcopy)
#pragma unroll
        for (int s = 0; s < kEvItems; ++s)
        {
            int v = id[s];
            keep_apart(v);
            if (v >= 0) tcopy[static_cast<uint32_t>(kw + s * kWave + lane)] = v;
        }
    const uint32_t emask = (1u << B.g.te_bits) - 1u;
    uint32_t woff = 0;
    for (int w0 = 0; w0 < B.g.n_tiles; w0 += kEvWin) {
        const int wn = min(kEvWin, B.g.n_tiles - w0);
        for (int i = tid; i < kEvWin; i += kEvThreads) cnt[i] = 0u;
        __syncthreads();   // (also: the trials have been read from srec)
#pragma unroll
        for (int s = 0; s < kEvItems; ++s) {
            int v = id[s];
            keep_apart(v);
            const int r = (v >> B.g.te_bits) - w0;
            if (v >= 0 && r >= 0 && r < wn) atomicAdd(&cnt[r], 1u);
        }
        __syncthreads();
        // exclusive scan of the window's counts, one per thread
        const uint32_t c = cnt[tid];
        uint32_t incl = c;
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t x = __shfl_up(incl, o);
            if (lane >= o) incl += x;
        }
        if (lane == kWave - 1) wsum[w] = incl;
        __syncthreads();
        uint32_t to = woff + incl - c, all = 0;
        for (int v = 0; v < kEvWaves; ++v) {
            to += v < w ? wsum[v] : 0u;
            all += wsum[v];
        }
        cnt[tid] = to;
        if (tid < wn) ts[w0 + tid] = static_cast<uint16_t>(to);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kEvItems; ++s) {
            int v = id[s];
            keep_apart(v);
            const int r = (v >> B.g.te_bits) - w0;
            if (v >= 0 && r >= 0 && r < wn) {
                const uint32_t to = atomicAdd(&cnt[r], 1u);
                srec[to] = (tr[s] << kEvSlotBits) | (static_cast<uint32_t>(v) & emask);
                if (POS) spos[to] = static_cast<uint16_t>(at[s]);
            }
        }
        woff += all;
        __syncthreads();
    }
    if (tid == 0) ts[B.g.n_tiles] = static_cast<uint16_t>(woff);
    uint32_t *dst = B.rec + ks + lo;
    for (uint32_t i = tid; i < woff; i += kEvThreads) dst[i] = srec[i];
    if (POS) {
        uint16_t *pdst = B.rpos + ks + lo;
        for (uint32_t i = tid; i < woff; i += kEvThreads) pdst[i] = spos[i];
    }
}

// Where a block has many chunks and tiles (few blocks, long trials): their sums
// beforehand, over shares of the block's chunks, into tbase, which is zero.
constexpr int kTileShare = 256;   // chunks of a workgroup

__global__ __launch_bounds__(256) void k_ev_tile_zero(EvBuild B) {
    const size_t n = static_cast<size_t>(B.g.neb) * (B.g.n_tiles + 1);
    for (size_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += static_cast<size_t>(gridDim.x) * 256) B.tbase[i] = 0u;
}

__global__ __launch_bounds__(256) void k_ev_tile_sums(EvBuild B) {
    if (ev_failed(B.misc)) return;
    const int b = blockIdx.z, t = blockIdx.x * 256 + threadIdx.x, nt = B.g.n_tiles;
    const int64_t end = ev_chunk0(B.base, b + 1);
    if (t >= nt) return;
    uint32_t v = 0;
    for (int64_t c0 = ev_chunk0(B.base, b) + static_cast<int64_t>(blockIdx.y) * kTileShare; c0 < end;
         c0 += static_cast<int64_t>(gridDim.y) * kTileShare) {
        const uint16_t *p = B.tstart + c0 * (nt + 1) + t;
        const int64_t c1 = min(end, c0 + kTileShare);
#pragma unroll 8
        for (int64_t c = c0; c < c1; ++c, p += nt + 1) v += static_cast<uint32_t>(p[1]) - static_cast<uint32_t>(p[0]);
    }
    if (v) atomicAdd(&B.tbase[static_cast<size_t>(b) * (nt + 1) + t], v);
}

// Each block's first entry of every tile (relative to the block).
template <bool SUMS>
__global__ __launch_bounds__(1024) void k_ev_tiles(EvBuild B) {
    __shared__ uint32_t wsum[16];
    if (ev_failed(B.misc)) return;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t c0 = ev_chunk0(B.base, b), c1 = ev_chunk0(B.base, b + 1);
    const int nt = B.g.n_tiles;
    uint32_t run = 0;
    for (int t0 = 0; t0 < nt; t0 += 1024) {
        const int t = t0 + tid;
        uint32_t v = 0;
        if (SUMS) {
            if (t < nt) v = B.tbase[static_cast<size_t>(b) * (nt + 1) + t];
        } else if (t < nt) {
            const uint16_t *p = B.tstart + c0 * (nt + 1) + t;
#pragma unroll 8
            for (int64_t c = c0; c < c1; ++c, p += nt + 1) v += static_cast<uint32_t>(p[1]) - static_cast<uint32_t>(p[0]);
        }
        uint32_t incl = v;
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t x = __shfl_up(incl, o);
            if (lane >= o) incl += x;
        }
        if (lane == kWave - 1) wsum[w] = incl;
        __syncthreads();
        uint32_t at = run + incl - v, all = 0;
        for (int i = 0; i < 16; ++i) {
            at += i < w ? wsum[i] : 0u;
            all += wsum[i];
        }
        if (t < nt) B.tbase[static_cast<size_t>(b) * (nt + 1) + t] = at;
        run += all;
        __syncthreads();
    }
    if (tid == 0) B.tbase[static_cast<size_t>(b) * (nt + 1) + nt] = run;
}

// One workgroup per (block, tile): the tile's records from the block's runs,
// ranked by event with LDS counters, the header from the counters' scan, the
// entries placed in LDS and written out in order.  A tile of at most sort_cap
// records is read once (held in registers between counting and placing); a
// larger one is read twice and its entries are stored directly.
template <bool POS>
__global__ __launch_bounds__(kEvThreads) __attribute__((amdgpu_waves_per_eu(POS ? 4 : 8, 8))) void k_ev_sort(EvBuild B) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int kSortItems = sort_items(POS), kSortCap = sort_cap(POS);
    const int te = 1 << B.g.te_bits;
    uint32_t *cnt = reinterpret_cast<uint32_t *>(smem);                       // [te]
    uint32_t *rcum = cnt + te;                                                // [kSortRuns + 1] records before each run
    uint32_t *rsrc = rcum + kSortRuns + 1;                                    // [kSortRuns] each run's first record in the block
    uint32_t *wsum = rsrc + kSortRuns;                                        // [kEvWaves]
    uint16_t *out = reinterpret_cast<uint16_t *>(wsum + kEvWaves);            // [kSortCap]
    uint16_t *outp = out + kSortCap;                                          // [kSortCap] with positions
    if (ev_failed(B.misc)) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = static_cast<int>(uni32(tid >> 6));
    const int nt = B.g.n_tiles;
    const int64_t item = grid_index();
    if (item >= static_cast<int64_t>(B.g.neb) * nt) return;   // uniform, before any barrier
    const int b = static_cast<int>(item / nt), tile = static_cast<int>(item - static_cast<int64_t>(b) * nt);
    const int64_t c0 = ev_chunk0(B.base, b), c1 = ev_chunk0(B.base, b + 1);
    const int64_t o0 = B.base[b];
    const uint32_t t0 = B.tbase[static_cast<size_t>(b) * (nt + 1) + tile];
    const uint32_t total = B.tbase[static_cast<size_t>(b) * (nt + 1) + tile + 1] - t0;
    for (int i = tid; i < te; i += kEvThreads) cnt[i] = 0u;

    // lists up to kSortRuns runs from chunk c on; returns the records in them
    auto list_runs = [&](int64_t c, int n) -> uint32_t {
        __syncthreads();
        uint32_t run = 0;
        for (int i0 = 0; i0 < n; i0 += kEvThreads) {
            const int i = i0 + tid;
            uint32_t v = 0;
            if (i < n) {
                const uint16_t *p = B.tstart + (c + i) * (nt + 1) + tile;
                v = static_cast<uint32_t>(p[1]) - static_cast<uint32_t>(p[0]);
                // the chunk's records start at its first occurrence
                const int64_t k = max<int64_t>((c + i - b) * kEvChunk, o0);
                rsrc[i] = static_cast<uint32_t>(k - o0) + p[0];
            }
            uint32_t incl = v;
            for (int o = 1; o < kWave; o <<= 1) {
                const uint32_t x = __shfl_up(incl, o);
                if (lane >= o) incl += x;
            }
            if (lane == kWave - 1) wsum[w] = incl;
            __syncthreads();
            uint32_t at = run + incl - v, all = 0;
            for (int q = 0; q < kEvWaves; ++q) {
                at += q < w ? wsum[q] : 0u;
                all += wsum[q];
            }
            if (i < n) rcum[i] = at;
            run += all;
            __syncthreads();
        }
        if (tid == 0) rcum[n] = run;
        __syncthreads();
        return run;
    };
    // the run holding record i (uniform argument)
    auto run_of = [&](uint32_t i, int n) -> int {
        int lo = 0, hi = n;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (uni32(rcum[mid]) <= i) lo = mid;
            else hi = mid;
        }
        return lo;
    };
    const uint32_t *rec = B.rec + o0;
    const uint16_t *rpos = POS ? B.rpos + o0 : nullptr;
    uint16_t *ent = B.ent + o0 + t0;
    uint16_t *pos = POS ? B.pos + o0 + t0 : nullptr;
    const bool in_regs = total <= static_cast<uint32_t>(kSortCap) && c1 - c0 <= kSortRuns;   // uniform
    uint32_t rv[kSortItems];
    uint16_t pv[POS ? kSortItems : 1];
    if (in_regs) {
        const int n = static_cast<int>(c1 - c0);
        list_runs(c0, n);
        const int ns = static_cast<int>((total + kEvThreads - 1) / kEvThreads);   // slices per wavefront
        const uint32_t kw = static_cast<uint32_t>(w * ns * kWave);
        int r = kw < total ? run_of(kw, n) : n - 1;
#pragma unroll
        for (int s = 0; s < kSortItems; ++s) {
            rv[s] = ~0u;
            if (s < ns) {
                const uint32_t i = kw + s * kWave + lane, last = kw + s * kWave + (kWave - 1);
                int my = r;
                while (r + 1 < n) {
                    const uint32_t next = uni32(rcum[r + 1]);
                    if (next > last) break;
                    ++r;
                    my += i >= next ? 1 : 0;
                }
                if (i < total) {
                    const uint32_t from = rsrc[my] + (i - rcum[my]);
                    rv[s] = rec[from];
                    if (POS) pv[s] = rpos[from];
                }
            }
        }
#pragma unroll
        for (int s = 0; s < kSortItems; ++s)
            if (rv[s] != ~0u) atomicAdd(&cnt[rv[s] & ((1u << kEvSlotBits) - 1u)], 1u);
    } else {
        for (int64_t c = c0; c < c1; c += kSortRuns) {
            const int n = static_cast<int>(min<int64_t>(kSortRuns, c1 - c));
            const uint32_t have = list_runs(c, n);
            for (uint32_t i = tid; i < have; i += kEvThreads) {
                int lo = 0, hi = n;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (rcum[mid] <= i) lo = mid;
                    else hi = mid;
                }
                atomicAdd(&cnt[rec[rsrc[lo] + (i - rcum[lo])] & ((1u << kEvSlotBits) - 1u)], 1u);
            }
        }
    }
    __syncthreads();
    // counts become first places (relative to the tile)
    const int per = (te + kEvThreads - 1) / kEvThreads;
    uint32_t sum = 0;
    for (int j = 0; j < per; ++j)
        if (tid * per + j < te) sum += cnt[tid * per + j];
    uint32_t incl = sum;
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t x = __shfl_up(incl, o);
        if (lane >= o) incl += x;
    }
    if (lane == kWave - 1) wsum[w] = incl;
    __syncthreads();
    uint32_t at = incl - sum;
    for (int q = 0; q < w; ++q) at += wsum[q];
    for (int j = 0; j < per; ++j)
        if (tid * per + j < te) {
            const uint32_t c = cnt[tid * per + j];
            cnt[tid * per + j] = at;
            at += c;
        }
    __syncthreads();
    // the header
    const int64_t e0 = static_cast<int64_t>(tile) << B.g.te_bits;
    const int nev = static_cast<int>(min<int64_t>(te, B.catalog - e0));
    if (B.g.dense) {
        uint32_t *st = B.start + static_cast<size_t>(b) * (B.catalog + 1) + e0;
        for (int i = tid; i < nev; i += kEvThreads) st[i] = t0 + cnt[i];
        if (tile == nt - 1 && tid == 0) st[nev] = t0 + total;
    } else {
        uint2 *h = B.hdr + static_cast<size_t>(b) * B.g.ng + (e0 >> 3);
        for (int i = tid; i < (nev + 7) / 8; i += kEvThreads) {
            uint32_t nib = 0, prev = cnt[8 * i];
            const uint32_t first = prev;
            for (int k = 0; k < 8; ++k) {
                const uint32_t next = 8 * i + k + 1 < te ? cnt[8 * i + k + 1] : total;
                nib |= min(next - prev, 15u) << (4 * k);
                prev = next;
            }
            h[i] = make_uint2(t0 + first, nib);
        }
        if (tile == nt - 1 && tid == 0) h[(nev + 7) / 8] = make_uint2(t0 + total, 0u);
    }
    __syncthreads();   // the header is read from the counters before they become cursors
    if (in_regs) {
#pragma unroll
        for (int s = 0; s < kSortItems; ++s) {
            if (rv[s] != ~0u) {
                const uint32_t e = rv[s] & ((1u << kEvSlotBits) - 1u);
                const uint32_t to = atomicAdd(&cnt[e], 1u);
                out[to] = static_cast<uint16_t>(((e & 7u) << kEvTrialBits) | (rv[s] >> kEvSlotBits));
                if (POS) outp[to] = pv[s];
            }
        }
        __syncthreads();
        if (POS)
            for (uint32_t i = tid; i < total; i += kEvThreads) pos[i] = outp[i];
        // two entries per store once the place is even
        const uint32_t odd = static_cast<uint32_t>((o0 + t0) & 1);
        if (odd && tid == 0 && total > 0) ent[0] = out[0];
        const uint32_t np = total > odd ? (total - odd) / 2 : 0;
        uint32_t *dst = reinterpret_cast<uint32_t *>(ent + odd);
        for (uint32_t i = tid; i < np; i += kEvThreads)
            dst[i] = static_cast<uint32_t>(out[odd + 2 * i]) | (static_cast<uint32_t>(out[odd + 2 * i + 1]) << 16);
        if (tid == 0 && odd + 2 * np < total) ent[total - 1] = out[total - 1];
    } else {
        for (int64_t c = c0; c < c1; c += kSortRuns) {
            const int n = static_cast<int>(min<int64_t>(kSortRuns, c1 - c));
            const uint32_t have = list_runs(c, n);
            for (uint32_t i = tid; i < have; i += kEvThreads) {
                int lo = 0, hi = n;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (rcum[mid] <= i) lo = mid;
                    else hi = mid;
                }
                const uint32_t from = rsrc[lo] + (i - rcum[lo]);
                const uint32_t v = rec[from];
                const uint32_t e = v & ((1u << kEvSlotBits) - 1u);
                const uint32_t to = atomicAdd(&cnt[e], 1u);
                ent[to] = static_cast<uint16_t>(((e & 7u) << kEvTrialBits) | (v >> kEvSlotBits));
                if (POS) pos[to] = rpos[from];
            }
        }
    }
}

int32_t ev_build(const EvBuild &B, hipStream_t st) {
    if (B.g.neb <= 0) return ARA_OK;
    const unsigned gm = static_cast<unsigned>(std::min<int64_t>((std::max<int64_t>(B.n_trials, B.g.neb + 1) + 255) / 256, 4096));
    k_ev_marks<<<gm, 256, 0, st>>>(B);
    if (B.pos) k_ev_part<true><<<static_cast<unsigned>(B.g.n_chunks), kEvThreads, 0, st>>>(B);
    else k_ev_part<false><<<static_cast<unsigned>(B.g.n_chunks), kEvThreads, 0, st>>>(B);
    // (2000 x 60,000, one block of 7324 chunks and 7813 tiles: 4.6 ms by itself)
    const int64_t per_block = B.nnz / kEvChunk / B.g.neb + 2;   // chunks
    const int64_t steps = per_block * ((B.g.n_tiles + 1023) / 1024);   // of one workgroup in k_ev_tiles, 0.6 us for eight
    if (steps > 2048 && B.g.neb <= 65535) {
        const unsigned shares = static_cast<unsigned>(std::min<int64_t>((per_block + kTileShare - 1) / kTileShare, 1024));
        k_ev_tile_zero<<<1024, 256, 0, st>>>(B);
        k_ev_tile_sums<<<dim3(static_cast<unsigned>((B.g.n_tiles + 255) / 256), shares, static_cast<unsigned>(B.g.neb)), 256, 0, st>>>(B);
        k_ev_tiles<true><<<static_cast<unsigned>(B.g.neb), 1024, 0, st>>>(B);
    } else {
        k_ev_tiles<false><<<static_cast<unsigned>(B.g.neb), 1024, 0, st>>>(B);
    }
    const size_t lds = sort_lds(B.g.te_bits, B.pos != nullptr);
    const auto sort = B.pos ? k_ev_sort<true> : k_ev_sort<false>;
    ARA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(sort), hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(lds)));
    sort<<<grid_of(static_cast<int64_t>(B.g.neb) * B.g.n_tiles), kEvThreads, lds, st>>>(B);
    ARA_HIP(hipGetLastError());
    return ARA_OK;
}

// ---------------------------------------------------------------------------

// The occurrences of the eight events of group `gr` in block b, added to c[].
__device__ __forceinline__ void ev_group_counts(const EvBlocks &B, int b, int gr, uint64_t (&c)[8]) {
    if (!B.dense) {
        const uint2 h = B.hdr[static_cast<size_t>(b) * B.ng + gr];
        if (!ev_long(h.y)) {
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] += (h.y >> (4 * k)) & 15u;
            return;
        }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (8 * gr + k < B.catalog) {
            uint32_t s, n;
            ev_list(B, b, 8 * gr + k, s, n);
            c[k] += n;
        }
}

// Occurrences of each event over all blocks: one thread per group of eight
// events, whose headers lie side by side with its neighbours'.
__global__ __launch_bounds__(256) void k_ev_count(EvBlocks B, int32_t *__restrict__ counts, int32_t *__restrict__ max_occ) {
    __shared__ uint32_t red[4];
    if (ev_failed(B.misc)) return;
    const int gr = blockIdx.x * 256 + threadIdx.x;
    uint64_t c[8] = {};
    if (gr < B.ng - 1)
#pragma unroll 4
        for (int b = 0; b < B.neb; ++b) ev_group_counts(B, b, gr, c);
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t v = static_cast<uint32_t>(min<uint64_t>(c[k], 0x7FFFFFFFu));
        if (counts && gr < B.ng - 1 && 8 * gr + k < B.catalog) counts[8 * gr + k] = static_cast<int32_t>(v);
        m = max(m, v);
    }
    for (int o = 32; o > 0; o >>= 1) m = max(m, static_cast<uint32_t>(__shfl_xor(static_cast<int>(m), o)));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        m = max(max(red[0], red[1]), max(red[2], red[3]));
        if (m) atomicMax(max_occ, static_cast<int32_t>(m));
    }
}

int32_t ev_count(const EvBlocks &B, int32_t *counts, hipStream_t st) {
    if (B.neb <= 0) return ARA_OK;
    k_ev_count<<<static_cast<unsigned>((B.ng - 1 + 255) / 256), 256, 0, st>>>(
        B, counts, reinterpret_cast<int32_t *>(const_cast<int64_t *>(B.misc) + kMiscMaxOcc));
    ARA_HIP(hipGetLastError());
    return ARA_OK;
}

// ---------------------------------------------------------------------------
// The event-major copy: thread = event, over the blocks that meet the slice.

constexpr int kMajorEvents = 256;
constexpr int kMajorCap = 18432;   // entries of a (slice, 256 events) staged in LDS: 72 KB, two workgroups per CU
constexpr int kMajorParts = 4;     // threads per event
constexpr int kMajorBatch = 2;     // blocks whose lists a thread has in flight
constexpr uint32_t kMajorFar = 24;     // entries from which a list is left to the second loop
constexpr uint32_t kMajorWide = 256;   // ... and a wavefront takes a list, or a group's, together

struct EvMajor {
    EvBlocks B;
    int64_t slice_trials;
    int64_t *tr_off, *ssum, *misc;
    uint32_t *tr_ent;
    int32_t n_sub;
};

struct SliceBlocks {
    int64_t lo, hi;   // the slice's trials
    int b0, b1;       // the blocks that meet it
};

__device__ __forceinline__ SliceBlocks slice_blocks_of(const EvMajor &M, int x) {
    SliceBlocks s;
    s.lo = min<int64_t>(static_cast<int64_t>(x) * M.slice_trials, M.B.n_trials);
    s.hi = min<int64_t>(s.lo + M.slice_trials, M.B.n_trials);
    s.b0 = static_cast<int>(s.lo / M.B.et);
    s.b1 = s.hi > s.lo ? static_cast<int>((s.hi + M.B.et - 1) / M.B.et) : s.b0;
    return s;
}

__device__ __forceinline__ bool block_inside(const EvMajor &M, const SliceBlocks &s, int b) {
    const int64_t t0 = static_cast<int64_t>(b) * M.B.et;
    return t0 >= s.lo && min<int64_t>(t0 + M.B.et, M.B.n_trials) <= s.hi;
}

// Occurrences of each event in the slice, and of every 256 events together:
// one thread per group of eight events, 32 threads per 256.
__global__ __launch_bounds__(256) void k_ev_major_count(EvMajor M) {
    if (ev_failed(M.misc)) return;
    const int x = blockIdx.y;
    const int gr = blockIdx.x * 256 + threadIdx.x;
    const SliceBlocks S = slice_blocks_of(M, x);
    uint64_t c[8] = {}, all = 0;
    if (gr < M.B.ng - 1) {
#pragma unroll 4
        for (int b = S.b0; b < S.b1; ++b) {
            if (block_inside(M, S, b)) ev_group_counts(M.B, b, gr, c);
        }
    }
    // the blocks that the slice cuts: the group's entries inside it, counted by
    // the lane, or by the wavefront where there are many (frequent events:
    // 185 ms when lanes counted them, frequencies as u^6 over 2M events, 400,000
    // x 1000)
    for (int b = S.b0; b < S.b1; ++b) {   // uniform
        if (block_inside(M, S, b)) continue;
        uint32_t s0 = 0, s1 = 0;
        if (gr < M.B.ng - 1) {
            if (M.B.dense) {
                const uint32_t *p = M.B.start + static_cast<size_t>(b) * (M.B.catalog + 1);
                s0 = p[8 * gr];
                s1 = p[min(8 * gr + 8, M.B.catalog)];
            } else {
                const uint2 *p = M.B.hdr + static_cast<size_t>(b) * M.B.ng + gr;
                s0 = p[0].x;
                s1 = p[1].x;
            }
        }
        const int64_t base = M.B.base[b];
        const uint16_t *p = M.B.ent + base;
        const uint32_t shift = static_cast<uint32_t>(static_cast<int64_t>(b) * M.B.et - S.lo);
        const uint32_t span = static_cast<uint32_t>(S.hi - S.lo);
        uint64_t some = 0;   // eight counts of one byte
        uint32_t n = 0;
        auto flush = [&](uint64_t (&to)[8]) {
#pragma unroll
            for (int k = 0; k < 8; ++k) to[k] += (some >> (8 * k)) & 255u;
            some = 0;
            n = 0;
        };
        auto count = [&](uint32_t v) {
            if (shift + (v & kEvTrialMask) < span) some += 1ull << (8 * (v >> kEvTrialBits));
        };
        for (uint64_t big = __ballot(s1 - s0 > kMajorWide); big; big &= big - 1) {
            const int l = __builtin_ctzll(big);
            const uint32_t a = __builtin_amdgcn_readlane(s0, l), z = __builtin_amdgcn_readlane(s1, l);
            uint64_t part[8] = {};
            const int64_t step = 8 * kWave;
            int64_t i = static_cast<int64_t>(a) + 8 * (threadIdx.x & 63);
            EvEight d{}, next{};
            if (i < z) d = *reinterpret_cast<const EvEight *>(p + i);
            for (; i < z; i += step) {
                if (i + step < z) next = *reinterpret_cast<const EvEight *>(p + i + step);
#pragma unroll
                for (uint32_t k = 0; k < 8; ++k)
                    if (i + k < z) count(d[k]);
                if ((n += 8u) > 240u) flush(part);
                d = next;
            }
            flush(part);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                for (int o = 32; o > 0; o >>= 1) part[k] += __shfl_xor(part[k], o);
                if (static_cast<int>(threadIdx.x & 63) == l) c[k] += part[k];
            }
            if (static_cast<int>(threadIdx.x & 63) == l) s1 = s0;
        }
#pragma unroll 4
        for (uint32_t i = s0; i < s1; ++i) {
            count(p[i]);
            if (++n == 255u) flush(c);
        }
        flush(c);
    }
    if (gr < M.B.ng - 1) {
        int64_t *off = M.tr_off + static_cast<int64_t>(x) * M.B.catalog + 8 * static_cast<int64_t>(gr);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (8 * gr + k < M.B.catalog) off[k] = static_cast<int64_t>(c[k]);
            all += c[k];
        }
    }
    constexpr int kLanes = kMajorEvents / 8;
    for (int o = kLanes / 2; o > 0; o >>= 1) all += __shfl_xor(all, o, kLanes);
    const int sub = gr / kLanes;
    if (gr % kLanes == 0 && sub < M.n_sub) M.ssum[static_cast<int64_t>(x) * M.n_sub + sub] = static_cast<int64_t>(all);
}

// ssum[0..n) becomes its exclusive scan, ssum[n] the total: one workgroup,
// eight sums per thread at a time.
__global__ __launch_bounds__(1024) void k_ev_major_scan(int64_t *__restrict__ ssum, int64_t n, int64_t *__restrict__ end) {
    __shared__ int64_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int64_t run = 0;
    for (int64_t i0 = 0; i0 < n; i0 += 8192) {
        int64_t c[8], v = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t i = i0 + tid * 8 + q;
            c[q] = i < n ? ssum[i] : 0;
            v += c[q];
        }
        int64_t incl = v;
        for (int o = 1; o < kWave; o <<= 1) {
            const int64_t x = __shfl_up(incl, o);
            if (lane >= o) incl += x;
        }
        if (lane == kWave - 1) wsum[w] = incl;
        __syncthreads();
        int64_t at = run + incl - v, all = 0;
        for (int q = 0; q < 16; ++q) {
            at += q < w ? wsum[q] : 0;
            all += wsum[q];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t i = i0 + tid * 8 + q;
            if (i < n) ssum[i] = at;
            at += c[q];
        }
        run += all;
        __syncthreads();
    }
    if (tid == 0) {
        ssum[n] = run;
        *end = run;
    }
}

// No (slice, catalogue range) may hold 2^32 occurrences.
__global__ __launch_bounds__(256) void k_ev_major_check(EvMajor M, int n_ranges) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kSlices * n_ranges) return;
    constexpr int kPer = kRange / kMajorEvents;
    const int x = i / n_ranges, r = i % n_ranges;
    const int64_t a = static_cast<int64_t>(x) * M.n_sub + static_cast<int64_t>(r) * kPer;
    const int64_t z = static_cast<int64_t>(x) * M.n_sub + min<int64_t>(static_cast<int64_t>(r + 1) * kPer, M.n_sub);
    if (M.ssum[z] - M.ssum[a] >= (int64_t(1) << 32)) atomicCAS(reinterpret_cast<int32_t *>(M.misc + kMiscErr), 0, ARA_E_LIMIT);
}

// List starts, then the entries: kMajorParts threads per event share the
// slice's blocks, each reserving its entries' places in the event's list with
// an LDS cursor (the order inside a list is free), so that the lists of all
// blocks are in flight together; the 256 lists are staged in LDS and written
// as one run (longer ones straight to memory).
__global__ __launch_bounds__(kMajorEvents * kMajorParts) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_ev_major_fill(EvMajor M) {
    __shared__ uint32_t stage[kMajorCap];
    __shared__ unsigned long long cur[kMajorEvents];
    __shared__ int64_t wsum[kMajorEvents / kWave];
    if (ev_failed(M.misc)) return;
    const int x = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int le = tid % kMajorEvents, part = tid / kMajorEvents;
    const int64_t e = blockIdx.x * static_cast<int64_t>(kMajorEvents) + le;
    const bool in = e < M.B.catalog;
    const SliceBlocks S = slice_blocks_of(M, x);
    const int64_t si = static_cast<int64_t>(x) * M.n_sub + blockIdx.x;
    const int64_t s0 = M.ssum[si], total = M.ssum[si + 1] - s0;
    if (part == 0) {
        int64_t *off = M.tr_off + static_cast<int64_t>(x) * M.B.catalog + e;
        const int64_t c = in ? *off : 0;
        int64_t incl = c;
        for (int o = 1; o < kWave; o <<= 1) {
            const int64_t v = __shfl_up(incl, o);
            if (lane >= o) incl += v;
        }
        if (lane == kWave - 1) wsum[w] = incl;
        cur[le] = static_cast<unsigned long long>(incl - c);
    }
    __syncthreads();
    if (part == 0) {
        int64_t at = static_cast<int64_t>(cur[le]);
        for (int q = 0; q < w; ++q) at += wsum[q];
        cur[le] = static_cast<unsigned long long>(at);
        if (in) M.tr_off[static_cast<int64_t>(x) * M.B.catalog + e] = s0 + at;
    }
    __syncthreads();
    if (total == 0) return;   // uniform
    const bool staged = total <= kMajorCap;   // uniform
    uint32_t *dst = M.tr_ent + s0;
    bool far = false;   // one of the thread's lists is long
    if (in) {
        for (int b0 = S.b0 + part * kMajorBatch; b0 < S.b1; b0 += kMajorBatch * kMajorParts) {
            uint32_t s[kMajorBatch], n[kMajorBatch];
            uint4 v[kMajorBatch];
#pragma unroll
            for (int u = 0; u < kMajorBatch; ++u) {
                s[u] = n[u] = 0;
                if (b0 + u < S.b1) ev_list(M.B, b0 + u, static_cast<int>(e), s[u], n[u]);
            }
#pragma unroll
            for (int u = 0; u < kMajorBatch; ++u) {
                v[u] = make_uint4(0, 0, 0, 0);
                if (n[u]) {   // entries from the even place at or before the list's first
                    const uint32_t *p = reinterpret_cast<const uint32_t *>(
                        M.B.ent + ((M.B.base[b0 + u] + s[u]) & ~int64_t(1)));
                    v[u] = make_uint4(p[0], p[1], p[2], p[3]);
                }
            }
#pragma unroll
            for (int u = 0; u < kMajorBatch; ++u) {
                if (!n[u]) continue;
                const int b = b0 + u;
                const int64_t first = M.B.base[b] + s[u];
                const int64_t shift = static_cast<int64_t>(b) * M.B.et - S.lo;   // block trial to slice trial
                const uint32_t span = static_cast<uint32_t>(S.hi - S.lo);
                const int odd = static_cast<int>(first & 1);
                const uint32_t a[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                uint32_t t[7], ok = 0;   // slice trials; those outside the slice (of a block it cuts) wrap or exceed it
#pragma unroll
                for (int i = 0; i < 7; ++i) {
                    const uint32_t even = (i & 1) ? a[i >> 1] >> 16 : a[i >> 1];
                    const uint32_t oddw = (i & 1) ? a[(i + 1) >> 1] : a[i >> 1] >> 16;
                    t[i] = static_cast<uint32_t>(shift) + ((odd ? oddw : even) & kEvTrialMask);
                    ok |= (i < static_cast<int>(n[u]) && t[i] < span) ? 1u << i : 0u;
                }
                unsigned long long at = atomicAdd(&cur[le], static_cast<unsigned long long>(__popc(ok)));
#pragma unroll
                for (int i = 0; i < 7; ++i)
                    if ((ok >> i) & 1u) {
                        if (staged) stage[at] = t[i];
                        else dst[at] = t[i];
                        ++at;
                    }
                if (n[u] > kMajorFar) {
                    far = true;
                    continue;
                }
                for (uint32_t i = 7; i < n[u]; ++i) {
                    const uint32_t tt = static_cast<uint32_t>(shift) + (M.B.ent[first + i] & kEvTrialMask);
                    if (tt >= span) continue;
                    at = atomicAdd(&cur[le], 1ull);
                    if (staged) stage[at] = tt;
                    else dst[at] = tt;
                }
            }
        }
    }
    // The long lists' entries from the eighth on, eight at a time, and by the
    // wavefront together where there are many (frequent events: 279 ms when each
    // lane took its own entry by entry, frequencies as u^6 over 2M events, 400,000
    // x 1000; 10 ms).  The lists are found again, so that the loop above has
    // nothing more to hold.
    if (__any(far)) {
        for (int b0 = S.b0 + part * kMajorBatch; b0 < S.b1; b0 += kMajorBatch * kMajorParts)   // uniform over the wavefront
            for (int b = b0; b < min(b0 + kMajorBatch, S.b1); ++b) {
                uint32_t s = 0, n = 0;
                if (in) ev_list(M.B, b, static_cast<int>(e), s, n);
                const uint32_t shift = static_cast<uint32_t>(static_cast<int64_t>(b) * M.B.et - S.lo);
                const uint32_t span = static_cast<uint32_t>(S.hi - S.lo);
                const uint16_t *ent = M.B.ent + M.B.base[b];
                // of the entries i .. i + 7 of a list of nl, those in the slice
                auto inside = [&](const EvEight &d, int64_t i, int64_t nl) {
                    uint32_t ok = 0;
#pragma unroll
                    for (uint32_t k = 0; k < 8; ++k) ok |= i + k < nl && shift + (d[k] & kEvTrialMask) < span ? 1u << k : 0u;
                    return ok;
                };
                auto put = [&](const EvEight &d, uint32_t ok, unsigned long long at) {
#pragma unroll
                    for (uint32_t k = 0; k < 8; ++k)
                        if ((ok >> k) & 1u) {
                            const uint32_t t = shift + (d[k] & kEvTrialMask);
                            if (staged) stage[at] = t;
                            else dst[at] = t;
                            ++at;
                        }
                };
                for (uint64_t big = __ballot(n > kMajorWide); big; big &= big - 1) {
                    const int l = __builtin_ctzll(big);
                    const int64_t nl = __builtin_amdgcn_readlane(n, l);
                    const uint16_t *p = ent + __builtin_amdgcn_readlane(s, l);
                    unsigned long long *c = &cur[le - lane + l];
                    constexpr int64_t kStep = 8 * kWave;
                    int64_t i = 7 + 8 * lane;
                    EvEight d{}, next{};
                    if (i < nl) d = *reinterpret_cast<const EvEight *>(p + i);
                    for (int64_t i0 = 7; i0 < nl; i0 += kStep, i += kStep) {   // uniform
                        if (i + kStep < nl) next = *reinterpret_cast<const EvEight *>(p + i + kStep);
                        const uint32_t ok = inside(d, i, nl);
                        uint32_t incl = static_cast<uint32_t>(__popc(ok));
                        for (int o = 1; o < kWave; o <<= 1) {
                            const uint32_t x2 = __shfl_up(incl, o);
                            if (lane >= o) incl += x2;
                        }
                        const uint32_t all = __builtin_amdgcn_readlane(incl, kWave - 1);
                        unsigned long long at = 0;
                        if (lane == 0 && all) at = atomicAdd(c, static_cast<unsigned long long>(all));
                        put(d, ok, __shfl(at, 0) + incl - static_cast<uint32_t>(__popc(ok)));
                        d = next;
                    }
                    if (lane == l) n = 0;
                }
                if (n > kMajorFar) {
                    const uint16_t *p = ent + s;
                    EvEight d = *reinterpret_cast<const EvEight *>(p + 7), next{};
                    for (uint32_t i = 7; i < n; i += 8) {
                        if (i + 8 < n) next = *reinterpret_cast<const EvEight *>(p + i + 8);
                        const uint32_t ok = inside(d, i, n);
                        if (ok) put(d, ok, atomicAdd(&cur[le], static_cast<unsigned long long>(__popc(ok))));
                        d = next;
                    }
                }
            }
    }
    if (!staged) return;
    __syncthreads();
    for (int64_t i = tid; i < total; i += kMajorEvents * kMajorParts) dst[i] = stage[i];
}

static int32_t major_subs(int32_t catalog) { return (catalog + kMajorEvents - 1) / kMajorEvents; }

size_t ev_major_sums(int32_t catalog) { return static_cast<size_t>(kSlices) * major_subs(catalog) + 1; }

int32_t ev_major(const EvBlocks &B, int64_t slice_trials, int64_t *tr_off, uint32_t *tr_ent, int64_t *ssum,
                 int64_t *misc, hipStream_t st) {
    EvMajor M{};
    M.B = B;
    M.slice_trials = slice_trials;
    M.tr_off = tr_off;
    M.tr_ent = tr_ent;
    M.ssum = ssum;
    M.misc = misc;
    M.n_sub = major_subs(B.catalog);
    const int n_ranges = (B.catalog + kRange - 1) / kRange;
    const dim3 grid(static_cast<unsigned>(M.n_sub), kSlices);
    k_ev_major_count<<<dim3(static_cast<unsigned>((B.ng - 1 + 255) / 256), kSlices), 256, 0, st>>>(M);
    k_ev_major_scan<<<1, 1024, 0, st>>>(ssum, static_cast<int64_t>(kSlices) * M.n_sub,
                                        tr_off + static_cast<int64_t>(kSlices) * B.catalog);
    k_ev_major_check<<<static_cast<unsigned>((kSlices * n_ranges + 255) / 256), 256, 0, st>>>(M, n_ranges);
    k_ev_major_fill<<<grid, kMajorEvents * kMajorParts, 0, st>>>(M);
    ARA_HIP(hipGetLastError());
    return ARA_OK;
}

}  // namespace ara
