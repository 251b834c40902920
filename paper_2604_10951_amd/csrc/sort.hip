// sort.hip -- per-tile depth ordering of the (tile << 32 | depth-key, record)
// pairs and per-tile ranges (surfels are blended depth-sorted, Sec. 3.1; the
// pipeline is tile based, Sec. 3.2).
//
// The required order is (tile, depth key, record): the order a stable sort on
// the 64-bit key gives, since a record is emitted at most once per tile and
// records are emitted in increasing order.  It is produced in two steps that
// suit a list split into many short per-tile runs:
//   1. a counting sort by tile: per-tile counts (LDS histograms over the tile
//      window of each 8192-pair chunk), one exclusive scan that also yields
//      every tile's [start, end)
//      range, and a scatter that places each pair at its tile's start plus a
//      cursor (any order inside the tile);
//   2. a sort of every tile's run by (depth key, record), as 64-bit composite
//      keys: runs of up to kWaveCap entries by one wave each (bitonic network
//      in the wave's registers), up to kLargeCap by a workgroup (distributed
//      in 64 KB of LDS over parts cut by samples of the run), longer runs by a stable
//      one-workgroup LSD radix sort through global memory.  The scan that writes the ranges
//      also lists the long runs.
// Every launch is sized from the capacity, not from the device-side pair
// count, so the sequence can be captured in a graph.
#include "fs_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaveCap = 256;     // entries per run sorted by one wave (4 per lane, in registers): short +
                                  // long kernels 26.2 us on the 1M-surfel 1280x720 frame, 30.0 with 512,
                                  // 26.5 with 128; sixteen views 163, 162 and 169
constexpr int kMidCap = 512;      // entries per run sorted by a quarter of a long-run workgroup
constexpr int kLargeCap = 8192;   // entries per run sorted in LDS by a workgroup (64 KB)
constexpr int kLdsTiles = 16384;  // tile counts kept in LDS by the count and scatter kernels
constexpr int kChunk = 8192;      // pairs per workgroup in the count and scatter kernels
constexpr int kChunkThreads = 1024;
constexpr int kPerThread = kChunk / kChunkThreads;   // pairs per thread and chunk
constexpr int kLongGrid = 512;    // workgroups working through the long-run list
constexpr int kLongThreads = 1024;
constexpr int kScanItems = 4;
constexpr int kScanPart = kThreads * kScanItems;
constexpr uint64_t kFlagAgg = 1ull << 62;
constexpr uint64_t kFlagPre = 2ull << 62;
constexpr uint64_t kValMask = (1ull << 62) - 1;
constexpr int kLongShift = 31;   // scan values: pairs (fewer than 2^30), long runs above
constexpr uint64_t kPairMask = (1ull << kLongShift) - 1;

FS_DEV int64_t load_count(const int64_t* num_pairs, int64_t capacity) {
    const int64_t p = *num_pairs;
    return p < capacity ? p : capacity;
}

__global__ void sort_clear_kernel(uint32_t* __restrict__ cnt, uint32_t* __restrict__ fill, int64_t tiles,
                                  uint64_t* __restrict__ status, int64_t parts, uint32_t* __restrict__ ticket) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < tiles; i += stride) {
        cnt[i] = 0;
        fill[i] = 0;
    }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < parts; i += stride) status[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x < 2) ticket[threadIdx.x] = 0;   // scan ticket, long-run count
}

// Tile window of a chunk of pairs: [lo, hi] over its valid tile ids (lo >
// hi when it has none), reduced over the workgroup.  Pairs are emitted
// record by record and records view by view, so a chunk's tiles lie within
// one view (two where it straddles a boundary): the window of a view with at
// most kLdsTiles tiles fits the LDS histograms below whatever the total.
FS_DEV void chunk_window(const uint64_t* __restrict__ keys, int64_t c0, int64_t c1, int64_t tiles, uint32_t& lo,
                         uint32_t& hi, uint32_t* s_red) {
    uint32_t a = 0xffffffffu, b = 0u;
    for (int64_t i = c0 + threadIdx.x; i < c1; i += kChunkThreads) {
        const uint64_t t = keys[i] >> 32;
        if (t < (uint64_t)tiles) {
            a = (uint32_t)t < a ? (uint32_t)t : a;
            b = (uint32_t)t > b ? (uint32_t)t : b;
        }
    }
    a = __ockl_wfred_min_u32(a);
    b = __ockl_wfred_max_u32(b);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        s_red[2 * wave] = a;
        s_red[2 * wave + 1] = b;
    }
    __syncthreads();
    lo = 0xffffffffu;
    hi = 0u;
    for (int w = 0; w < kChunkThreads / 64; ++w) {
        lo = s_red[2 * w] < lo ? s_red[2 * w] : lo;
        hi = s_red[2 * w + 1] > hi ? s_red[2 * w + 1] : hi;
    }
}

// Per-tile counts.  Every workgroup counts a chunk of kChunk pairs: in an LDS
// histogram over the chunk's tile window when it spans at most kLdsTiles
// tiles, adding its non-zero bins to the global counts (a tile with many
// pairs costs one global atomic per workgroup, not one per pair); with global
// atomics per pair otherwise.
__global__ void __launch_bounds__(kChunkThreads)
sort_count_kernel(const uint64_t* __restrict__ keys, const int64_t* __restrict__ num_pairs, int64_t capacity,
                  int64_t tiles, uint32_t* __restrict__ cnt) {
    __shared__ uint32_t h[kLdsTiles];
    __shared__ uint32_t s_red[2 * (kChunkThreads / 64)];
    const int64_t P = load_count(num_pairs, capacity);
    const int64_t c0 = (int64_t)blockIdx.x * kChunk;
    if (c0 >= P) return;   // uniform across the workgroup
    const int64_t c1 = c0 + kChunk < P ? c0 + kChunk : P;
    uint32_t lo = 0u, hi = (uint32_t)(tiles - 1);   // all tiles fit: no window needed
    if (tiles > kLdsTiles) {
        chunk_window(keys, c0, c1, tiles, lo, hi, s_red);
        if (hi < lo) return;
    }
    const uint32_t W = hi - lo + 1u;
    if (W > (uint32_t)kLdsTiles) {
        for (int64_t i = c0 + threadIdx.x; i < c1; i += kChunkThreads) {
            const uint64_t t = keys[i] >> 32;
            if (t < (uint64_t)tiles) atomicAdd(&cnt[t], 1u);
        }
        return;
    }
    // the thread's keys of the chunk, all loads in flight together
    uint64_t kk[kPerThread];
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
        const int64_t i = c0 + threadIdx.x + (int64_t)u * kChunkThreads;
        kk[u] = i < c1 ? keys[i] : ~0ull;
    }
    for (uint32_t i = threadIdx.x; i < W; i += kChunkThreads) h[i] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
        const uint64_t t = kk[u] >> 32;
        if (t < (uint64_t)tiles) atomicAdd(&h[(uint32_t)t - lo], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < W; i += kChunkThreads)
        if (h[i]) atomicAdd(&cnt[lo + i], h[i]);
}

FS_DEV uint32_t wave_inclusive_scan(uint32_t x) { return __ockl_wfscan_add_u32(x, true); }

// Exclusive scan of the tile counts into ranges (single pass: partitions by
// atomic ticket, decoupled look-back with one wave reading 64 predecessors
// per round trip).  The same scan numbers the runs longer than kWaveCap (in
// the upper half of the status words' values) and lists their tiles, their
// count going to ticket[1] (appended one by one through an atomic counter,
// which the memory side serialises at about 50 ns each, they held up the
// short-run kernel: 90 -> 50 us on the sixteen-view frame).
__global__ void __launch_bounds__(kThreads)
sort_scan_kernel(const uint32_t* __restrict__ cnt, int64_t tiles, uint32_t* __restrict__ ranges,
                 uint64_t* __restrict__ status, uint32_t* __restrict__ ticket, int64_t parts,
                 uint32_t* __restrict__ long_list) {
    __shared__ uint32_t s_part;
    __shared__ uint64_t s_wave[kThreads / 64];
    __shared__ uint64_t s_prefix;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) s_part = atomicAdd(ticket, 1u);
    __syncthreads();
    const int64_t part = s_part;
    if (part >= parts) return;
    const int64_t base = part * kScanPart + (int64_t)tid * kScanItems;
    uint32_t c[kScanItems];
    uint32_t sum = 0, longs = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        c[j] = base + j < tiles ? cnt[base + j] : 0u;
        sum += c[j];
        longs += c[j] > (uint32_t)kWaveCap ? 1u : 0u;
    }
    const uint32_t incl = wave_inclusive_scan(sum), lincl = wave_inclusive_scan(longs);
    if (lane == 63) s_wave[wave] = incl | (uint64_t)lincl << kLongShift;
    __syncthreads();
    uint64_t wave_excl = 0, total = 0;
    for (int w = 0; w < kThreads / 64; ++w) {
        if (w < wave) wave_excl += s_wave[w];
        total += s_wave[w];
    }
    if (wave == 0) {
        uint64_t prefix = 0;
        if (part == 0) {
            if (lane == 0)
                __hip_atomic_store(status + part, kFlagPre | total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            if (lane == 0)
                __hip_atomic_store(status + part, kFlagAgg | total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int64_t j = part - 1;
            while (true) {
                const int64_t idx = j - lane;
                const uint64_t st = idx >= 0 ? __hip_atomic_load(status + idx, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_AGENT)
                                             : kFlagPre;   // before partition 0: an empty inclusive prefix
                const uint64_t flag = st & ~kValMask;
                const uint64_t notready = __ballot(flag == 0);
                const uint64_t pre = __ballot(flag == kFlagPre);
                const int limit = notready ? __builtin_ctzll(notready) : 64;
                const int first_pre = pre ? __builtin_ctzll(pre) : 64;
                const bool found = first_pre < limit;
                const int take = found ? first_pre + 1 : limit;
                uint64_t v = lane < take ? (st & kValMask) : 0ull;
                prefix += __ockl_wfred_add_u64(v);
                if (found) break;
                j -= take;
                if (take == 0) __builtin_amdgcn_s_sleep(1);
            }
            if (lane == 0)
                __hip_atomic_store(status + part, kFlagPre | (prefix + total), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        if (lane == 0) s_prefix = prefix;
    }
    __syncthreads();
    const uint64_t before = s_prefix + wave_excl;
    uint32_t off = (uint32_t)(before & kPairMask) + (incl - sum);
    uint32_t slot = (uint32_t)(before >> kLongShift) + (lincl - longs);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        if (base + j < tiles) {
            ranges[2 * (base + j)] = off;
            ranges[2 * (base + j) + 1] = off + c[j];
            if (c[j] > (uint32_t)kWaveCap) long_list[slot++] = (uint32_t)(base + j);
        }
        off += c[j];
    }
    if (part == parts - 1 && tid == 0) ticket[1] = (uint32_t)((s_prefix + total) >> kLongShift);
}

// Pair i goes to its tile's start plus a cursor, as (depth key, record).
// Per chunk, as in the count: over an LDS window of at most kLdsTiles tiles
// the workgroup reserves, per tile, one run of positions for its whole chunk
// (one global atomic per tile it touches) and hands them out with LDS
// cursors; otherwise every pair takes a global atomic.
__global__ void __launch_bounds__(kChunkThreads)
sort_scatter_kernel(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                    const int64_t* __restrict__ num_pairs, int64_t capacity, int64_t tiles,
                    const uint32_t* __restrict__ ranges, uint32_t* __restrict__ fill, uint2* __restrict__ out) {
    __shared__ uint32_t h[kLdsTiles];
    __shared__ uint32_t s_red[2 * (kChunkThreads / 64)];
    const int64_t P = load_count(num_pairs, capacity);
    const int64_t c0 = (int64_t)blockIdx.x * kChunk;
    if (c0 >= P) return;   // uniform across the workgroup
    const int64_t c1 = c0 + kChunk < P ? c0 + kChunk : P;
    uint32_t lo = 0u, hi = (uint32_t)(tiles - 1);   // all tiles fit: no window needed
    if (tiles > kLdsTiles) {
        chunk_window(keys, c0, c1, tiles, lo, hi, s_red);
        if (hi < lo) return;
    }
    const uint32_t W = hi - lo + 1u;
    if (W > (uint32_t)kLdsTiles) {
        for (int64_t i = c0 + threadIdx.x; i < c1; i += kChunkThreads) {
            const uint64_t k = keys[i];
            const uint64_t t = k >> 32;
            if (t < (uint64_t)tiles) {
                const uint32_t pos = ranges[2 * t] + atomicAdd(&fill[t], 1u);
                if ((int64_t)pos < P) out[pos] = make_uint2((uint32_t)k, vals[i]);
            }
        }
        return;
    }
    // the thread's pairs of the chunk, all loads in flight together; kept in
    // registers for the scatter below
    uint64_t kk[kPerThread];
    uint32_t vv[kPerThread];
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
        const int64_t i = c0 + threadIdx.x + (int64_t)u * kChunkThreads;
        kk[u] = i < c1 ? keys[i] : ~0ull;
        vv[u] = i < c1 ? vals[i] : 0u;
    }
    for (uint32_t i = threadIdx.x; i < W; i += kChunkThreads) h[i] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
        const uint64_t t = kk[u] >> 32;
        if (t < (uint64_t)tiles) atomicAdd(&h[(uint32_t)t - lo], 1u);
    }
    __syncthreads();
    // first position of this chunk's run in every tile it touches: the
    // (memory-side) reservations of a thread are independent, so all are
    // issued before the first result is waited for
    static_assert(kLdsTiles % kChunkThreads == 0, "whole rounds of bins");
    constexpr int kRounds = kLdsTiles / kChunkThreads;
    uint32_t cnt[kRounds], got[kRounds], first[kRounds];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
        const uint32_t i = threadIdx.x + (uint32_t)k * kChunkThreads;
        cnt[k] = i < W ? h[i] : 0u;
        got[k] = 0u;
        first[k] = 0u;
        if (cnt[k] != 0u) {
            got[k] = atomicAdd(&fill[lo + i], cnt[k]);
            first[k] = ranges[2 * (lo + i)];
        }
    }
#pragma unroll
    for (int k = 0; k < kRounds; ++k)
        if (cnt[k] != 0u) h[threadIdx.x + k * kChunkThreads] = first[k] + got[k];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPerThread; ++u) {
        const uint64_t t = kk[u] >> 32;
        if (t < (uint64_t)tiles) {
            const uint32_t pos = atomicAdd(&h[(uint32_t)t - lo], 1u);
            if ((int64_t)pos < P) out[pos] = make_uint2((uint32_t)kk[u], vv[u]);
        }
    }
}

FS_DEV uint64_t composite(uint2 e) { return ((uint64_t)e.x << 32) | e.y; }

// Bitonic sort of one run of 1 <= n <= 64 E entries by one wave, in
// registers: element i = lane * E + e of the padded run (padding = ~0) is
// x[e] of its lane.  Compare-exchange partners i ^ j with j < E sit in the
// same lane; with j >= E they are the same register of lane ^ (j / E),
// fetched by a shuffle.  The network is the textbook one (stage k, distance
// j, ascending where i & k == 0), so the result is the sorted run.
template <int LOGE>
FS_DEV void sort_run_wave(const uint2* __restrict__ in, uint64_t tile, uint32_t start, int n,
                          uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    constexpr int E = 1 << LOGE;
    const int lane = (int)threadIdx.x & 63;
    uint64_t x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = lane * E + e;
        x[e] = i < n ? composite(in[start + i]) : ~0ull;
    }
    wave_network<LOGE>(x);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = lane * E + e;
        if (i < n) {
            keys[start + i] = (tile << 32) | (x[e] >> 32);
            vals[start + i] = (uint32_t)x[e];
        }
    }
}

// The thread's index, opaque to the compiler: a workgroup sorts its long runs in a
// loop with a form for each length, and the addresses and masks of all forms would
// be hoisted out of that loop and spilled.
FS_DEV int own_thread() {
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

// Sort of one run of n <= G E entries by a group of G threads in one distribution
// step: entries go to LDS grouped by part, the parts in order, and an entry's
// place inside its part is the number of the part's entries before it, counted
// directly.  64 samples (128 for the longest runs) tell how to cut: equal parts of
// the depth range where the samples spread over it; where they crowd, the
// intervals between the sorted samples, each cut into equal parts of its range of
// (depth, record).  A part then holds a few entries however the depths are spread
// (equal parts alone put a camera-facing wall in front of a far background into one
// part; sorting 3,600 runs of 1,000 such entries, with the 20 us that restore the
// pairs, took 237 us with a network for such runs, 222 with chunks sorted by waves
// and merged, 146 this way; normally distributed depths 127, 221 and 120, and 900
// runs of 8,000 such entries 280, 373 and 177).
// Returns false, having written nothing, if a part holds more than kPartMax
// entries (a pair repeated that often): uniform over the group.
// All threads of the workgroup call it together (barriers); n = 0: nothing to do.
constexpr uint32_t kPartMax = 1024;
template <int G, int P>
struct PartShared {
    uint64_t split[129];           // crowded: interval k is [split[k], split[k + 1]); entries outside go to its ends
    uint32_t part[P];              // entries, then next place, in the end the end of every part
    uint32_t red[2 * (G / 64)];
    uint32_t cell[512];            // samples in each 512th of the range
    uint32_t lo, even;
    float scale;
};
// E = 0: runs of up to kLargeCap entries, read again in every phase (held in
// registers, 8 per thread, they spill).
template <int G, int E, int P>
FS_DEV bool sort_run_parts(uint64_t* s, PartShared<G, P>& b, const uint2* __restrict__ in, uint64_t tile, uint32_t start,
                           int n, uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    constexpr int kWaves = G / 64, kLogS = E > 0 ? 0 : 1, kS = 64 << kLogS, kParts = E == 1 ? P / 2 : P, kSub = kParts / kS;
    // samples in one 512th of the range beyond which they crowd: normal, uniform
    // and exponential depths give 2 to 5, forty equal planes 5 to 8
    constexpr uint32_t kCrowd = E > 0 ? 4u : 6u;
    constexpr int kPer = kParts / G;   // parts per thread
    static_assert(kPer * G == kParts, "whole parts per thread");
    const int tid = own_thread() & (G - 1), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto fence = [] {   // one wave's LDS accesses complete in order
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    uint64_t v[E > 0 ? E : 1];   // this thread's entries, and their parts
    uint32_t at[E > 0 ? E : 1];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = tid + e * G < n ? composite(in[start + tid + e * G]) : 0ull;
    if (wave == kWaves - 1 && n > 0) {   // entries arrive in no particular order: evenly spaced ones are the samples
        uint64_t x[1 << kLogS];
        uint32_t lo = ~0u, hi = 0u;
#pragma unroll
        for (int j = 0; j < 1 << kLogS; ++j) {
            x[j] = composite(in[start + (uint32_t)(((lane << kLogS) + j) * n / kS)]);
            lo = min(lo, (uint32_t)(x[j] >> 32));
            hi = max(hi, (uint32_t)(x[j] >> 32));
        }
        lo = __ockl_wfred_min_u32(lo);
        hi = __ockl_wfred_max_u32(hi);
        const uint32_t margin = (hi - lo) >> 2;   // for the entries beyond the outermost samples
        lo = lo > margin ? lo - margin : 0u;
        const float scale = (float)kParts / ((float)(hi - lo) + (float)margin + 1.f);
#pragma unroll
        for (int j = 0; j < 8; ++j) b.cell[lane + 64 * j] = 0u;
        fence();
        const float cells = scale * (512.f / (float)kParts);
#pragma unroll
        for (int j = 0; j < 1 << kLogS; ++j)
            atomicAdd(&b.cell[min(511, (int)((float)((uint32_t)(x[j] >> 32) - lo) * cells))], 1u);
        fence();
        uint32_t crowd = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j) crowd = max(crowd, b.cell[lane + 64 * j]);
        const bool even = __ockl_wfred_max_u32(crowd) <= kCrowd;
        if (!even) {
            wave_network<kLogS>(x);
#pragma unroll
            for (int j = 0; j < 1 << kLogS; ++j) b.split[(lane << kLogS) + j] = x[j];
            fence();
            if (lane == 0) {
                const uint64_t s0 = b.split[0], s1 = b.split[kS - 1];
                const uint64_t below = 2u * (b.split[2] - s0), above = 2u * (s1 - b.split[kS - 3]) + 1u;
                b.split[0] = s0 > below ? s0 - below : 0ull;
                b.split[kS] = ~0ull - s1 > above ? s1 + above : ~0ull;
            }
        }
        if (lane == 0) {
            b.lo = lo;
            b.scale = scale;
            b.even = even ? 1u : 0u;
        }
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) b.part[tid + j * G] = 0u;
    __syncthreads();
    const bool even = b.even != 0u;
    const uint32_t lo = b.lo;
    const float scale = b.scale;
    auto part_of = [&](uint64_t x) {   // monotone in x
        if (even) {
            const uint32_t d = (uint32_t)(x >> 32);
            return (uint32_t)fminf((float)(d > lo ? d - lo : 0u) * scale, (float)(kParts - 1));
        }
        int k = 0;
#pragma unroll
        for (int h = kS / 2; h > 0; h >>= 1) k += b.split[k + h] <= x ? h : 0;
        const uint64_t from = b.split[k], to = b.split[k + 1];
        const float f = (float)(x > from ? x - from : 0ull) *
                        ((float)kSub * __builtin_amdgcn_rcpf((float)(to - from) + 1.f));
        return (uint32_t)(k * kSub + (int)fminf(f, (float)(kSub - 1)));
    };
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (tid + e * G < n) {
            at[e] = part_of(v[e]);
            atomicAdd(&b.part[at[e]], 1u);
        }
    if constexpr (E == 0)
        for (int i = tid; i < n; i += G) atomicAdd(&b.part[part_of(composite(in[start + i]))], 1u);
    __syncthreads();
    uint32_t c[kPer], sum = 0u, cmax = 0u;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        c[j] = b.part[tid * kPer + j];
        sum += c[j];
        cmax = max(cmax, c[j]);
    }
    const uint32_t incl = wave_inclusive_scan(sum);
    cmax = __ockl_wfred_max_u32(cmax);
    if (lane == 63) {
        b.red[wave] = incl;
        b.red[kWaves + wave] = cmax;
    }
    __syncthreads();
    uint32_t first = incl - sum, largest = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        first += w < wave ? b.red[w] : 0u;
        largest = b.red[kWaves + w] > largest ? b.red[kWaves + w] : largest;
    }
    if (largest > kPartMax) return false;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        b.part[tid * kPer + j] = first;
        first += c[j];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (tid + e * G < n) s[atomicAdd(&b.part[at[e]], 1u)] = v[e];
    if constexpr (E == 0)
        for (int i = tid; i < n; i += G) {
            const uint64_t x = composite(in[start + i]);
            s[atomicAdd(&b.part[part_of(x)], 1u)] = x;
        }
    __syncthreads();
    // by slots, not by this thread's own entries: a wave's lanes then count in the
    // same few parts, and their places, close to their slots, fill whole lines
    // (by own entries a wave waits for the largest part any of them is in: 900 runs
    // of 8,000 entries of a wall and its background 485 us, 235 by slots)
#pragma unroll 1
    for (int i = tid; i < n; i += G) {
        const uint64_t x = s[i];
        const uint32_t q = part_of(x), p1 = b.part[q];
        uint32_t r = q > 0u ? b.part[q - 1u] : 0u;
        for (uint32_t p = r; p < p1; ++p) {
            const uint64_t y = s[p];
            // equal entries (the caller's own lists may repeat a pair) by their
            // slots, so that no two share a place
            r += y < x || (y == x && p < (uint32_t)i) ? 1u : 0u;
        }
        keys[start + r] = (tile << 32) | (x >> 32);
        vals[start + r] = (uint32_t)x;
    }
    return true;
}

// One wave per tile: runs of up to kWaveCap entries are sorted in the wave's
// registers (1, 2 or 4 entries per lane by run length); longer ones are on
// the list the long-run kernel works through.
__global__ void __launch_bounds__(kThreads)
sort_short_runs_kernel(const uint2* __restrict__ in, const uint32_t* __restrict__ ranges, int64_t tiles,
                       uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    static_assert(kWaveCap == 256, "runs up to 4 entries per lane");
    const int wave = threadIdx.x >> 6;
    const int64_t t = (int64_t)blockIdx.x * (kThreads / 64) + wave;
    if (t >= tiles) return;   // uniform per wave
    const uint32_t start = ranges[2 * t], end = ranges[2 * t + 1];
    const int n = (int)(end - start);
    if (n == 0 || n > kWaveCap) return;
    if (n <= 64)
        sort_run_wave<0>(in, (uint64_t)t, start, n, keys, vals);
    else if (n <= 128)
        sort_run_wave<1>(in, (uint64_t)t, start, n, keys, vals);
    else
        sort_run_wave<2>(in, (uint64_t)t, start, n, keys, vals);
}

// Stable LSD radix sort of one run through global memory, 8-bit digits of the
// 64-bit composite key, ping-ponging between a[start, start + n) (input) and
// b[start, start + n); passes whose digit is the same for the whole run are
// skipped.  Ends with the sorted run written as final keys and values (b may
// alias the keys: each thread reads its element before writing it).
template <int NT>
FS_DEV void sort_run_global(uint2* a, uint2* b, uint64_t tile, uint32_t start, uint32_t n,
                            uint64_t* keys, uint32_t* __restrict__ vals, uint32_t* hist, uint32_t* wcnt,
                            uint32_t* flag) {
    constexpr int kWaves = NT / 64;
    const int tid = own_thread(), lane = tid & 63, wave = tid >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    uint2* src = a + start;
    uint2* dst = b + start;
    for (int pass = 0; pass < 8; ++pass) {
        const int shift = 8 * pass;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < n; i += NT) atomicAdd(&hist[(composite(src[i]) >> shift) & 0xff], 1u);
        __syncthreads();
        if (tid == 0) {
            uint32_t acc = 0;
            uint32_t single = 0;
            for (int d = 0; d < 256; ++d) {
                const uint32_t c = hist[d];
                if (c == n) single = 1;   // one digit value: identity permutation
                hist[d] = acc;
                acc += c;
            }
            *flag = single;
        }
        __syncthreads();
        if (*flag) continue;   // uniform
        for (uint32_t c0 = 0; c0 < n; c0 += NT) {
            const uint32_t i = c0 + tid;
            const bool valid = i < n;
            const uint2 e = valid ? src[i] : make_uint2(0u, 0u);
            const uint32_t d = (uint32_t)(composite(e) >> shift) & 0xffu;
            // rank among equal digits of this chunk: inside the wave by ballot
            // matching, across waves from per-wave digit counts
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool x = (d >> bit) & 1u;
                const uint64_t bb = __ballot(x);
                peers &= x ? bb : ~bb;
            }
            for (int i = tid; i < kWaves * 256; i += NT) wcnt[i] = 0;
            __syncthreads();
            if (valid && ((peers >> lane) >> 1) == 0ull) wcnt[wave * 256 + d] = (uint32_t)__popcll(peers);
            __syncthreads();
            if (valid) {
                uint32_t before = 0;
                for (int w = 0; w < wave; ++w) before += wcnt[w * 256 + d];
                dst[hist[d] + before + (uint32_t)__popcll(peers & lt)] = e;
            }
            __syncthreads();
            if (tid < 256) {
                uint32_t tot = 0;
                for (int w = 0; w < kWaves; ++w) tot += wcnt[w * 256 + tid];
                hist[tid] += tot;
            }
            __syncthreads();
        }
        uint2* tmp = src;
        src = dst;
        dst = tmp;
    }
    for (uint32_t i = tid; i < n; i += NT) {
        const uint2 e = src[i];
        keys[start + i] = (tile << 32) | e.x;
        vals[start + i] = e.y;
    }
}

// Runs longer than kWaveCap, from the list: up to kMidCap entries four at a time,
// by a quarter of the workgroup each (3,600 runs of 300 entries, depths spread and
// bunched: 52 and 59 us, 73 and 138 by whole workgroups with equal parts, 58 and 58 by
// a wave each, which for a list as short as the 1M-surfel 1280x720 frame's is 4 us
// slower), up to kLargeCap by the workgroup, longer ones by the global radix sort.
// Two workgroups per CU (64 VGPRs at most) keep every long run of a frame
// in flight at once.
__global__ void __launch_bounds__(kLongThreads) __attribute__((amdgpu_waves_per_eu(8)))
sort_long_runs_kernel(uint2* __restrict__ in, const uint32_t* __restrict__ ranges,
                      const uint32_t* __restrict__ long_list, const uint32_t* __restrict__ long_count,
                      uint64_t* keys, uint32_t* __restrict__ vals) {
    constexpr int kMid = 256, kMids = kLongThreads / kMid;   // threads per run of at most kMidCap entries
    static_assert(kMidCap == 2 * kMid, "two entries per thread");
    __shared__ union {
        struct {
            uint64_t s[kLargeCap];
            PartShared<kLongThreads, 2048> parts;
        } all;
        struct {
            uint64_t s[kMidCap];
            PartShared<kMid, 512> parts;
        } mid[kMids];
    } sm;
    uint64_t* s = sm.all.s;
    __shared__ uint32_t s_todo[kLongThreads];   // this workgroup's runs: short ones from the front, others from the back
    __shared__ uint32_t s_num[2];
    const int tid = (int)threadIdx.x;
    const uint32_t count = *long_count, grid = gridDim.x;
    for (uint32_t base = blockIdx.x; base < count; base += grid * kLongThreads) {
        // every grid-th run of the list, looked up in one round trip
        if (tid < 2) s_num[tid] = 0u;
        __syncthreads();
        const uint32_t mine = (count - base + grid - 1) / grid;
        if ((uint32_t)tid < mine) {
            const uint32_t t = long_list[base + (uint32_t)tid * grid];
            const bool mid = ranges[2 * (int64_t)t + 1] - ranges[2 * (int64_t)t] <= (uint32_t)kMidCap;
            const uint32_t i = atomicAdd(&s_num[mid ? 0 : 1], 1u);
            s_todo[mid ? i : kLongThreads - 1 - i] = t;
        }
        __syncthreads();
        const uint32_t mids = __builtin_amdgcn_readfirstlane(s_num[0]), longs = __builtin_amdgcn_readfirstlane(s_num[1]);
        for (uint32_t i = 0; i < mids; i += kMids) {
            const uint32_t g = __builtin_amdgcn_readfirstlane((uint32_t)tid / kMid);
            const uint32_t t = __builtin_amdgcn_readfirstlane(i + g < mids ? s_todo[i + g] : 0u);   // (uniform in a wave)
            const uint32_t start = ranges[2 * (int64_t)t];
            const uint32_t n = i + g < mids ? ranges[2 * (int64_t)t + 1] - start : 0u;
            sort_run_parts<kMid, 2>(sm.mid[g].s, sm.mid[g].parts, in, t, start, (int)n, keys, vals);
            __syncthreads();   // LDS is reused by the next runs
        }
        for (uint32_t i = 0; i < longs; ++i) {
            const uint32_t t = __builtin_amdgcn_readfirstlane(s_todo[kLongThreads - 1 - i]);
            const uint32_t start = ranges[2 * (int64_t)t], n = ranges[2 * (int64_t)t + 1] - start;
            const bool done =
                n <= 1u * kLongThreads   ? sort_run_parts<kLongThreads, 1>(s, sm.all.parts, in, t, start, (int)n, keys, vals)
                : n <= 2u * kLongThreads ? sort_run_parts<kLongThreads, 2>(s, sm.all.parts, in, t, start, (int)n, keys, vals)
                : n <= (uint32_t)kLargeCap
                    ? sort_run_parts<kLongThreads, 0>(s, sm.all.parts, in, t, start, (int)n, keys, vals)
                    : false;
            if (!done) {
                // the run's own slice of the key array is the radix passes' second
                // buffer; LDS holds their counters
                uint32_t* hist = reinterpret_cast<uint32_t*>(s);
                uint32_t* wcnt = hist + 256;
                uint32_t* flag = wcnt + (kLongThreads / 64) * 256;
                sort_run_global<kLongThreads>(in, reinterpret_cast<uint2*>(keys), t, start, n, keys, vals, hist, wcnt,
                                              flag);
            }
            __syncthreads();   // LDS is reused by the next run
        }
    }
}

}  // namespace

int64_t fs_sort_scan_parts(int64_t total_tiles) { return (total_tiles + kScanPart - 1) / kScanPart; }

hipError_t fs_launch_sort(uint64_t* keys, uint32_t* vals, int64_t capacity, const int64_t* num_pairs, int64_t hint,
                          int64_t total_tiles, uint32_t* ranges, const FsWorkspace& ws, hipStream_t s) {
    if (total_tiles >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    const int64_t pmax = hint >= 0 ? (hint < capacity ? hint : capacity) : capacity;
    const int64_t parts = fs_sort_scan_parts(total_tiles);
    {
        const int64_t work = total_tiles > parts ? total_tiles : parts;
        unsigned blocks = (unsigned)((work + 255) / 256);
        blocks = blocks < 1 ? 1 : (blocks > 2048 ? 2048 : blocks);
        hipLaunchKernelGGL(sort_clear_kernel, dim3(blocks), dim3(256), 0, s, ws.tile_cnt, ws.tile_fill, total_tiles,
                           ws.sort_status, parts, ws.sort_ticket);
    }
    const int64_t chunks = (pmax + kChunk - 1) / kChunk;
    if (chunks >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    const unsigned pblocks = (unsigned)(chunks < 1 ? 1 : chunks);
    hipLaunchKernelGGL(sort_count_kernel, dim3(pblocks), dim3(kChunkThreads), 0, s, keys, num_pairs, capacity,
                       total_tiles, ws.tile_cnt);
    hipLaunchKernelGGL(sort_scan_kernel, dim3((unsigned)parts), dim3(kThreads), 0, s, ws.tile_cnt, total_tiles, ranges,
                       ws.sort_status, ws.sort_ticket, parts, ws.long_list);
    hipLaunchKernelGGL(sort_scatter_kernel, dim3(pblocks), dim3(kChunkThreads), 0, s, keys, vals, num_pairs, capacity,
                       total_tiles, ranges, ws.tile_fill, ws.runs);
    const unsigned sblocks = (unsigned)((total_tiles + kThreads / 64 - 1) / (kThreads / 64));
    hipLaunchKernelGGL(sort_short_runs_kernel, dim3(sblocks), dim3(kThreads), 0, s, ws.runs, ranges, total_tiles, keys,
                       vals);
    hipLaunchKernelGGL(sort_long_runs_kernel, dim3(kLongGrid), dim3(kLongThreads), 0, s, ws.runs, ranges, ws.long_list,
                       ws.sort_ticket + 1, keys, vals);
    return hipGetLastError();
}
