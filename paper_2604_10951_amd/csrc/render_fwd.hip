// render_fwd.hip -- per-pixel front-to-back blending of C-channel features,
// full (Sec. 3.1 Eq. 2) or with Top-K hard selection (Sec. 3.4).
//
// Work decomposition.  A workgroup of four waves renders one 8x8 pixel block
// and one chunk of at most 128 channels, whatever the binning tile size; the
// block's depth-sorted entries are walked in batches of BG.  Tiles of 16x16 and
// 32x32 pixels hold 4 and 16 blocks, and a block meets only some of its tile's
// entries (about a third and a tenth on the clustered scenes), so for them the
// workgroup first tests the entries' pixel boxes, 256 at a time, and queues
// those that meet the block (FILTER).  The blocks of a tile repeat that test
// (12 B per entry), which costs far less than the walk it saves: one workgroup
// per 16x16 pixels, walking every entry of the tile, took 1.24 ms for the
// 300k-surfel, 640x480, C = 48 full-blend frame (16x16 tiles) against 0.27 ms
// with the queue alone and 0.17 ms with all that follows.  A block exits as soon
// as every pixel has stopped (T_stop, or K blended surfels), which is where Top-K
// saves work.  Feature images are written pixel-major (channels contiguous).
#include <type_traits>

#include "fs_internal.h"

namespace {

// One 16-byte vector of feature elements in LDS, widened to float32.
template <typename FT>
struct FeatVec;
template <>
struct FeatVec<float> {
    static constexpr int kElems = 4;
    FS_DEV static float at(const uint4& v, int i) {
        return __uint_as_float(i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w);
    }
};
template <>
struct FeatVec<uint16_t> {
    static constexpr int kElems = 8;
    FS_DEV static float at(const uint4& v, int i) {
        const uint32_t w = i < 2 ? v.x : i < 4 ? v.y : i < 6 ? v.z : v.w;
        return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
    }
};
typedef float f32x4 __attribute__((ext_vector_type(4)));

FS_DEV uint32_t wave_or(uint32_t x) { return __ockl_wfred_or_u32(x); }

// Per-entry data of the extended render (low-pass option, depth and normal
// outputs), staged once per batch by the entry's own thread.
FS_DEV void stage_ext(const FsRecord& r, const fs_camera& cam, const uint64_t* __restrict__ keys, uint32_t pos,
                      bool lowpass, bool geo, double2& mu, float4& g) {
    if (lowpass) {
        double mx, my;
        fs_record_centre(r, mx, my);
        mu = make_double2(mx, my);
    }
    if (geo) {
        const float3 nrm = fs_record_normal(r, cam);
        // the centre depth is needed (and keys given) only for the depth output
        g = make_float4(nrm.x, nrm.y, nrm.z, keys ? __uint_as_float((uint32_t)keys[pos]) : 0.f);
    }
}

// ---------------------------------------------------------------------------
// Render block: one 8x8 pixel block per workgroup of NW waves, so a long list
// is walked NW times faster than by one wave.  Per batch of BG entries:
//   a. alpha: NT / BG lanes per entry evaluate the pixels of its box inside the
//      block; each accepted pixel's alpha goes to LDS, with a bit per pixel and
//      entry (numbering the pairs over all threads by a scan and a bisection
//      balances them better, but its shuffles and per-pair record reads took
//      3,470 cycles a batch against 1,680 on the 1M-surfel 1280x720 frame);
//   b. walk (lanes = pixels): one wave runs the front-to-back transmittance
//      walk over the accepted entries in depth order (stop and Top-K tests,
//      FP64 T) and leaves the weights w = alpha T and the blended entries in
//      LDS, while the other waves accumulate the previous batch (d).  (The
//      kernel is half bound by vector issue, about 3,100 wave instructions a
//      batch with every wave repeating the walk to save the exchange);
//   c. rows: the feature rows of entries blended anywhere in the block go to
//      LDS by direct global -> LDS loads, issued after the walk and consumed
//      one batch later, so the load latency is hidden behind the next batch's
//      alpha pass;
//   d. accumulate: four lanes per pixel, each owning a quarter of the channels
//      as 16-byte vectors, so all pixels of a wave advance through their
//      entries together (pixel after pixel, all lanes on one pixel's channels:
//      the wave pays every pixel's LDS latency in turn, 0.346 ms for the
//      1M-surfel 1280x720 C = 128 full blend against 0.274).  The four pixels
//      of a 16-lane read phase take their vectors in rotated order, so that
//      their rows, which share banks, are read from different ones.
// Every pixel sees the same sequence of FP64 transmittance updates and FP32
// FMAs as in the split Top-K renderer, so the two give identical results.
constexpr int kQueue = 512;   // entries queued by the filter (a power of two)
template <int NVT, typename FT, int NW, int BG, bool EXT, bool FILTER>
struct WideShared {
    static constexpr int kChunk = 4 * NVT * FeatVec<FT>::kElems;   // channels of the workgroup
    FsRecord rec[BG];
    uint32_t recid[2][BG];        // per batch parity: record and surfel of the entries
    uint32_t sidx[2][BG];
    __align__(16) FT feat[BG][kChunk];   // the batch's feature rows, by entry; at the end the block's image
    float a[2][BG][64];           // per batch parity: alpha per accepted (entry, pixel), then the weight
    uint32_t amask[2][64];        // per pixel: the batch's accepted, then its blended entries
    uint32_t used;                // entries any pixel blends
    uint32_t active;              // some pixel still walks
    float z[EXT ? BG : 1][64];    // depth output: camera depth of the ray-plane point
    double2 mu[EXT ? BG : 1];
    float4 geo[EXT ? BG : 1];
    uint32_t qrid[FILTER ? kQueue : 1];   // tile-list entries whose boxes meet the block: record,
    uint32_t qpos[FILTER ? kQueue : 1];   // list position
    uint32_t qcount[NW];
    uint32_t item;
};

template <int NVT, typename FT, int NW, int BG, bool VEC, bool EXT, bool FILTER>
FS_DEV void render_block_wide(int64_t block, WideShared<NVT, FT, NW, BG, EXT, FILTER>& sm,
                              const FsRecord* __restrict__ records, const uint64_t* __restrict__ keys,
                              const uint32_t* __restrict__ vals, const uint32_t* __restrict__ ranges,
                              const FT* __restrict__ feats, int C, int64_t n, int64_t num_records,
                              const fs_camera* __restrict__ cams, int num_views, int S, const fs_opts& o,
                              float* __restrict__ out_feat, float* __restrict__ out_T, int32_t* __restrict__ out_n,
                              int32_t* __restrict__ out_last, int32_t* __restrict__ out_idx,
                              float* __restrict__ out_depth, float* __restrict__ out_normal,
                              uint64_t* __restrict__ counters) {
    static_assert(2 * BG + NW * 64 <= kQueue, "a refill fits the queue beside the batch in work and the next");
    static_assert(BG <= 32 && 64 % NW == 0, "batch masks are 32-bit; pixel groups split the 64 pixels evenly");
    constexpr int NT = NW * 64;
    constexpr int PPW = 64 / NW;                             // pixels accumulated per wave
    constexpr int kVE = FeatVec<FT>::kElems;                 // elements per 16-byte vector
    constexpr int kChunk = 4 * NVT * kVE;
    constexpr int kQ = FS_RECORD_BYTES / 16;
    constexpr int kRecSlots = (BG * kQ + NT - 1) / NT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const BlockPos bp = locate_block(block, S, 8, cams, num_views);
    if (!bp.valid) return;   // uniform across the workgroup
    const fs_camera& cam = cams[bp.view];
    const int chunk = blockIdx.y;
    const int c0 = chunk * kChunk;
    const int clen = C - c0 < kChunk ? C - c0 : kChunk;
    const int px = bp.x0 + (lane & 7), py = bp.y0 + (lane >> 3);
    const bool inside = px < cam.width && py < cam.height;
    const int64_t pix = cam.pixel_offset + (int64_t)py * cam.width + px;
    // the wave that walks: another one in each of the workgroups sharing a CU
    const int walker = (int)(blockIdx.x >> 8) & (NW - 1);
    const uint32_t start = ranges[2 * bp.tile], end = ranges[2 * bp.tile + 1];
    const int K = o.topk;
    const bool write_idx = out_idx != nullptr && chunk == 0 && K > 0;
    const bool lowpass = EXT && o.lowpass != 0;
    const bool geo = EXT && chunk == 0 && (out_depth != nullptr || out_normal != nullptr);
    float gD = 0.f, gN0 = 0.f, gN1 = 0.f, gN2 = 0.f;

    double T = 1.0;
    int cnt = 0;
    int last = -1;
    bool done = !inside;
    // accumulation: four lanes per pixel, each owning the vectors vec_of
    const int ap = wave * PPW + (lane >> 2);                 // pixel accumulated by this lane
    const int arot = (lane >> 2) & 3, avec = (lane & 3) + 4 * (arot % NVT);
    auto vec_of = [&](int v) {   // the lane's v-th vector
        return (NVT & (NVT - 1)) == 0 ? avec ^ (4 * v) : (lane & 3) + 4 * ((v + arot) % NVT);
    };
    float acc[NVT][kVE];
#pragma unroll
    for (int v = 0; v < NVT; ++v)
#pragma unroll
        for (int i = 0; i < kVE; ++i) acc[v][i] = 0.f;
    const double t_stop = o.t_stop;
    const float neg_half_log2e = -0.72134752044448170f;   // -log2(e) / 2
    uint32_t walked = 0, fetched = 0;   // 8x8 tiles (count_walk_kernel counts for larger ones)

    // records of batch i + 1 and list values of batch i + 2 are in flight
    // while batch i is processed
    float4 pre[kRecSlots];
    uint32_t pre_rid[kRecSlots];
    uint32_t nxt_rid[kRecSlots];
    auto fetch_vals = [&](uint32_t b0, uint32_t* rid) {
#pragma unroll
        for (int j = 0; j < kRecSlots; ++j) {
            const int e = (tid + j * NT) / kQ;
            rid[j] = (e < BG && b0 + (uint32_t)e < end) ? vals[b0 + e] : 0xffffffffu;
        }
    };
    auto fetch_records = [&](const uint32_t* rid) {
#pragma unroll
        for (int j = 0; j < kRecSlots; ++j) {
            const int q = (tid + j * NT) % kQ;
            pre_rid[j] = rid[j];
            pre[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if ((int64_t)rid[j] < num_records) pre[j] = reinterpret_cast<const float4*>(records + rid[j])[q];
        }
    };
    // FILTER: queue positions [qh, qt) hold the entries still to be walked;
    // thread t tests entry cp + t of the list, its value and box already in
    // c_rid and c_box (and the value after that in c_val)
    uint32_t qh = 0, qt = 0, cp = start;
    uint32_t c_rid = 0xffffffffu, c_val = 0xffffffffu;
    uint2 c_box = make_uint2(0u, 0u);
    auto load_box = [&]() {
        c_rid = c_val;
        if ((int64_t)c_rid < num_records)
            c_box = *reinterpret_cast<const uint2*>(&records[c_rid].x0);
        else
            c_rid = 0xffffffffu;
    };
    auto load_val = [&](uint32_t p) { c_val = p + (uint32_t)tid < end ? vals[p + tid] : 0xffffffffu; };
    // append the entries of the next NT list positions whose boxes meet the block
    auto refill = [&]() {
        const int x0 = (int16_t)(c_box.x & 0xffffu), x1 = (int16_t)(c_box.x >> 16);
        const int y0 = (int16_t)(c_box.y & 0xffffu), y1 = (int16_t)(c_box.y >> 16);
        const bool hit = c_rid != 0xffffffffu && x0 <= bp.x0 + 7 && x1 >= bp.x0 && y0 <= bp.y0 + 7 && y1 >= bp.y0 &&
                         x0 <= x1 && y0 <= y1;
        const uint64_t m = __ballot(hit);
        if (lane == 0) sm.qcount[wave] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t at = qt;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const uint32_t c = sm.qcount[w];
            at += w < wave ? c : 0u;
            qt += c;
        }
        if (hit) {
            const uint32_t i = (at + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))) & (kQueue - 1);
            sm.qrid[i] = c_rid;
            sm.qpos[i] = cp + (uint32_t)tid;
        }
        cp += NT;
        load_box();
        load_val(cp + NT);
        __syncthreads();
    };
    auto fetch_queued = [&](uint32_t h) {   // records of the batch at queue position h
#pragma unroll
        for (int j = 0; j < kRecSlots; ++j) {
            const int e = (tid + j * NT) / kQ;
            nxt_rid[j] = (e < BG && h + (uint32_t)e < qt) ? sm.qrid[(h + e) & (kQueue - 1)] : 0xffffffffu;
        }
        fetch_records(nxt_rid);
    };

    // accumulate the rows in sm.feat with the weights of parity par, each
    // pixel's entries in order; the next entry's weight is read ahead of the
    // current one's row
    auto accumulate = [&](int par) {
        uint32_t m = sm.amask[par][ap];
        int e = m ? __builtin_ctz(m) : 0;
        float w = sm.a[par][e][ap];
        while (m != 0u) {
            m &= m - 1u;
            const int en = m ? __builtin_ctz(m) : 0;
            const float wn = sm.a[par][en][ap];
            const uint4* __restrict__ row = reinterpret_cast<const uint4*>(&sm.feat[e][0]);
            constexpr int kHalf = NVT > 4 ? NVT / 2 : NVT;   // vectors in flight (registers)
#pragma unroll
            for (int h = 0; h < NVT; h += kHalf) {
                uint4 f[kHalf];
#pragma unroll
                for (int v = 0; v < kHalf; ++v) f[v] = row[vec_of(h + v)];
#pragma unroll
                for (int v = 0; v < kHalf; ++v)
#pragma unroll
                    for (int i = 0; i < kVE; ++i) acc[h + v][i] = fmaf(w, FeatVec<FT>::at(f[v], i), acc[h + v][i]);
            }
            e = en;
            w = wn;
        }
    };

    int pbuf = -1;                       // parity of the batch whose rows are in flight (-1: none)
    if constexpr (FILTER) {
        load_val(start);
        load_box();
        load_val(start + NT);
        while (qt < (uint32_t)BG && cp < end) refill();
        fetch_queued(0);
    } else if (start < end) {
        uint32_t r0[kRecSlots];
        fetch_vals(start, r0);
        fetch_records(r0);
        fetch_vals(start + BG, nxt_rid);
    }
    // stage the prefetched records of a batch of nbs entries (parity par)
    auto stage = [&](int par, int nbs) {
#pragma unroll
        for (int j = 0; j < kRecSlots; ++j) {
            const int t = tid + j * NT;
            const int e = t / kQ, q = t - e * kQ;
            if (e < nbs) {
                float4 v4 = pre[j];
                uint32_t rid = pre_rid[j];
                if ((int64_t)rid >= num_records) {   // never happens for a well-formed list
                    rid = 0u;
                    v4 = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (q == 4) v4.w = __int_as_float((int)0xbff00000);   // k2 = -1: never accepted
                    if (q == 5) v4.z = __int_as_float(1);                 // empty box
                }
                reinterpret_cast<float4*>(&sm.rec[e])[q] = v4;
                if (q == 0) {
                    sm.recid[par][e] = rid;
                    sm.sidx[par][e] = rid % (uint32_t)n;
                }
            }
        }
        if (tid < 64) sm.amask[par][tid] = 0u;
    };
    {
        const uint32_t left = FILTER ? qt - qh : end - start;
        stage(0, (int)(left < (uint32_t)BG ? left : (uint32_t)BG));
    }
    int it = 0;
    for (uint32_t b0 = start; FILTER ? qh != qt : b0 < end; b0 += BG, ++it) {
        const uint32_t left = FILTER ? qt - qh : end - b0;
        const int nb = (int)(left < (uint32_t)BG ? left : (uint32_t)BG);
        const int cur = it & 1;
        __syncthreads();   // A: records staged; every wave has finished the previous walk
        // list position of the batch's entry e
        auto pos_of = [&](int e) -> uint32_t { return FILTER ? sm.qpos[(qh + e) & (kQueue - 1)] : b0 + (uint32_t)e; };
        if constexpr (FILTER) {
            // the queue holds less than 2 BG entries before a refill adds at
            // most NT, so this batch's slots are not overwritten
            while (qt - qh - nb < (uint32_t)BG && cp < end) refill();
            fetch_queued(qh + nb);
        } else if (b0 + BG < end) {
            fetch_records(nxt_rid);
            fetch_vals(b0 + 2 * BG, nxt_rid);
        }
        if constexpr (EXT) {
            if ((lowpass || geo) && tid < nb)
                stage_ext(sm.rec[tid], cam, keys, pos_of(tid), lowpass, geo, sm.mu[tid], sm.geo[tid]);
            __syncthreads();
        }
        // a. alpha over the pixels of each entry's box inside the block: NT / BG
        //    lanes per entry, which read its record once, one lane per pixel
        //    of the box's longer side, stepping along the shorter one
        {
            constexpr int GL = NT / BG;
            static_assert(GL % 8 == 0, "a lane per pixel of a block's side");
            const int e = tid / GL, li = tid & 7, k0 = (tid % GL) >> 3;
            if (e < nb) {
                const FsRecord r = sm.rec[e];
                const int xa = r.x0 > bp.x0 ? r.x0 : bp.x0;
                const int ya = r.y0 > bp.y0 ? r.y0 : bp.y0;
                int xb = r.x1 < bp.x0 + 7 ? r.x1 : bp.x0 + 7;
                int yb = r.y1 < bp.y0 + 7 ? r.y1 : bp.y0 + 7;
                xb = xb < cam.width - 1 ? xb : cam.width - 1;
                yb = yb < cam.height - 1 ? yb : cam.height - 1;
                const int rw = xb - xa + 1, rh = yb - ya + 1;
                const bool along = rw >= rh;   // lanes along x
                const int steps = li < (along ? rw : rh) ? (along ? rh : rw) : 0;
                const int ix = along ? 0 : GL / 8, iy = along ? GL / 8 : 0;
                int ox = xa + (along ? li : k0) - r.ax, oy = ya + (along ? k0 : li) - r.ay;
                int p = (oy + r.ay - bp.y0) * 8 + (ox + r.ax - bp.x0);
                for (int k = k0; k < steps; k += GL / 8, ox += ix, oy += iy, p += ix + 8 * iy) {
                    FsResp rs = fs_response(r, (double)ox, (double)oy);
                    if constexpr (EXT)
                        if (lowpass) fs_lowpass_d2(rs, (double)ox, (double)oy, sm.mu[e].x, sm.mu[e].y);
                    if (rs.d2 <= r.k2) {
                        const float G = __builtin_amdgcn_exp2f(neg_half_log2e * (float)rs.d2);
                        sm.a[cur][e][p] = fminf(o.alpha_max, r.o * G);
                        atomicOr(&sm.amask[cur][p], 1u << e);
                        if constexpr (EXT)
                            if (geo) sm.z[e][p] = (float)((double)sm.geo[e].w * rs.rh);
                    }
                }
            }
        }
        // the previous batch's rows (issued before this batch's alpha pass)
        if (VEC) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();   // B: alpha of this batch and rows of the previous batch are in LDS
        // b. the transmittance walk of one wave: each lane visits its pixel's
        //    accepted entries, in depth order, with the next entry's alpha read
        //    ahead, and leaves its weights and its blended entries in place
        if (wave == walker) {
            uint32_t mask = 0u;
            uint32_t macc = done ? 0u : sm.amask[cur][lane];
            int e = macc ? __builtin_ctz(macc) : 0, laste = -1;
            float al = sm.a[cur][e][lane];
            while (macc != 0u && !done) {
                macc &= macc - 1u;
                const int en = macc ? __builtin_ctz(macc) : 0;
                const float aln = sm.a[cur][en][lane];
                const double Tn = T * (1.0 - (double)al);
                if (Tn < t_stop) {
                    done = true;
                } else {
                    const float w = (float)((double)al * T);
                    sm.a[cur][e][lane] = w;
                    if constexpr (EXT) {
                        if (geo) {
                            const float4 gg = sm.geo[e];
                            gD = fmaf(w, sm.z[e][lane], gD);
                            gN0 = fmaf(w, gg.x, gN0);
                            gN1 = fmaf(w, gg.y, gN1);
                            gN2 = fmaf(w, gg.z, gN2);
                        }
                    }
                    mask |= 1u << e;
                    T = Tn;
                    if (write_idx) out_idx[pix * K + cnt] = (int32_t)sm.recid[cur][e];
                    ++cnt;
                    laste = e;
                    if (K > 0 && cnt == K) done = true;
                }
                e = en;
                al = aln;
            }
            if (laste >= 0) last = (int)pos_of(laste);
            sm.amask[cur][lane] = mask;
            const uint32_t wused = wave_or(mask);
            const bool wactive = !__all(done);
            if (lane == 0) {
                sm.used = wused;
                sm.active = wactive ? 1u : 0u;
            }
            if constexpr (!FILTER) {
                walked += (uint32_t)nb;
                fetched += (uint32_t)__popc(wused);
            }
        }
        if (pbuf >= 0) accumulate(pbuf);
        __syncthreads();   // C: the walk is done, the previous batch's rows are no longer read
        const uint32_t used = sm.used;
        const bool wactive = sm.active != 0u;
        // the next batch's records, before the row loads: waiting for the former
        // would wait for the latter too (sm.rec's last reader, this batch's
        // alpha pass, ended before barrier B; the parity's masks, weights and ids
        // were last used before barrier C)
        if (wactive) {
            const uint32_t have = (FILTER ? qt - qh : left) - (uint32_t)nb;
            stage(cur ^ 1, (int)(have < (uint32_t)BG ? have : (uint32_t)BG));
        }
        // c. issue the rows of the blended entries
        if (VEC) {
            constexpr int kRowBytes = kChunk * (int)sizeof(FT);
            constexpr int kLanesPerRow = kRowBytes / 16;
            constexpr int kRowsPerInst = 64 / kLanesPerRow;
            const int lrow = lane / kLanesPerRow, lcol = lane - lrow * kLanesPerRow;
#pragma unroll
            for (int i0 = 0; i0 < BG; i0 += NW * kRowsPerInst) {
                const int r0 = i0 + wave * kRowsPerInst;
                const int e = r0 + lrow;
                // a row of 12 lanes (48 channels) leaves lanes over, and the last
                // instruction's rows may pass the batch
                if (lrow < kRowsPerInst && e < BG && ((used >> e) & 1u) && lcol * kVE < clen) {
                    const FT* src = feats + (int64_t)sm.sidx[cur][e] * C + c0 + lcol * kVE;
                    __builtin_amdgcn_global_load_lds((const void*)src,
                                                     (__attribute__((address_space(3))) void*)&sm.feat[r0][0], 16, 0,
                                                     0);
                }
            }
        } else {
            for (int t = tid; t < BG * kChunk; t += NT) {
                const int e = t / kChunk, c = t - e * kChunk;
                if (((used >> e) & 1u) && c < clen) sm.feat[e][c] = feats[(int64_t)sm.sidx[cur][e] * C + c0 + c];
            }
        }
        pbuf = cur;
        qh += (uint32_t)nb;
        if (!wactive) break;   // identical in every wave
    }
    if (pbuf >= 0) {
        if (VEC) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        accumulate(pbuf);
    }

    if (!FILTER && counters != nullptr && chunk == 0 && wave == walker) {
        int c = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) c += __shfl_xor(c, d, 64);
        if (lane == 0) {
            atomicAdd((unsigned long long*)&counters[2], (unsigned long long)c);
            atomicAdd((unsigned long long*)&counters[0], (unsigned long long)walked);
            atomicAdd((unsigned long long*)&counters[1], (unsigned long long)fetched);
            atomicAdd((unsigned long long*)&counters[3], 1ull);
        }
    }
    if (chunk == 0 && inside && wave == walker) {
        out_T[pix] = (float)T;
        out_n[pix] = cnt;
        if (out_last) out_last[pix] = last;
        if (write_idx)
            for (int j = cnt; j < K; ++j) out_idx[pix * K + j] = -1;
        if constexpr (EXT) {
            if (out_depth) out_depth[pix] = gD;
            if (out_normal) {
                out_normal[3 * pix] = gN0;
                out_normal[3 * pix + 1] = gN1;
                out_normal[3 * pix + 2] = gN2;
            }
        }
    }
    // the block's image goes out through LDS, as many pixels at a time as the
    // row buffers hold, so that every (non-temporal: it is not read back by
    // this kernel) store instruction fills whole lines
    constexpr int kImage = (int)sizeof(sm.feat) / (kChunk * 4);   // pixels per piece
    constexpr int kPiece = kImage < 64 ? kImage : 64;
    static_assert(kPiece % PPW == 0 || PPW % kPiece == 0, "pieces of whole waves or parts of one");
    float* __restrict__ image = reinterpret_cast<float*>(&sm.feat[0][0]);
    // rows of whole aligned float4 (c0 and clen are multiples of four when C is)
    const bool vec4 = (C & 3) == 0 && (reinterpret_cast<uintptr_t>(out_feat) & 15u) == 0u;
    if (pbuf < 0 && vec4 && clen == C) {
        // nothing blended: a pixel row's channels are contiguous
        const int w = cam.width - bp.x0 < 8 ? cam.width - bp.x0 : 8, h = cam.height - bp.y0 < 8 ? cam.height - bp.y0 : 8;
        for (int y = wave; y < h; y += NW) {
            float* __restrict__ row = out_feat + (cam.pixel_offset + (int64_t)(bp.y0 + y) * cam.width + bp.x0) * C;
            for (int t = lane; t < w * C >> 2; t += 64)
                __builtin_nontemporal_store(f32x4{0.f, 0.f, 0.f, 0.f}, reinterpret_cast<f32x4*>(row) + t);
        }
        return;
    }
    const int per = vec4 ? clen >> 2 : clen;
    const uint32_t inv = ((1u << 20) + (uint32_t)per - 1u) / (uint32_t)per;   // exact division of t < 64 * 128 by per
#pragma unroll 1
    for (int p0 = 0; p0 < 64; p0 += kPiece) {
        if (pbuf >= 0) {
            __syncthreads();   // rows, or the previous piece, no longer read
            if (ap >= p0 && ap < p0 + kPiece) {
#pragma unroll
                for (int v = 0; v < NVT; ++v)
#pragma unroll
                    for (int i = 0; i < kVE; i += 4)
                        *reinterpret_cast<f32x4*>(image + (ap - p0) * kChunk + vec_of(v) * kVE + i) =
                            f32x4{acc[v][i], acc[v][i + 1], acc[v][i + 2], acc[v][i + 3]};
            }
            __syncthreads();
        }
        for (int t = tid; t < kPiece * per; t += NT) {
            const int p = (int)(((uint64_t)t * inv) >> 20), c = t - p * per;
            const int qx = bp.x0 + ((p0 + p) & 7), qy = bp.y0 + ((p0 + p) >> 3);
            if (qx >= cam.width || qy >= cam.height) continue;
            float* dst = out_feat + (cam.pixel_offset + (int64_t)qy * cam.width + qx) * C + c0;
            if (vec4) {
                const f32x4 x = pbuf >= 0 ? *reinterpret_cast<const f32x4*>(image + p * kChunk + 4 * c)
                                          : f32x4{0.f, 0.f, 0.f, 0.f};
                __builtin_nontemporal_store(x, reinterpret_cast<f32x4*>(dst + 4 * c));
            } else {
                __builtin_nontemporal_store(pbuf >= 0 ? image[p * kChunk + c] : 0.f, dst + c);
            }
        }
    }
}

// Four waves per SIMD for up to four vectors per lane (64 channels, 128 bfloat16):
// a few registers over 128 let three (300k surfels, 1280x720, C = 64, tile 16: render
// 193 -> 163 us; with depth and normals, 200k, 640x480, C = 16: 88 -> 76).
template <int NVT, typename FT, int NW, int BG, bool VEC, bool EXT, bool FILTER>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(NVT <= 4 ? 4 : 1)))
render_wide_kernel(const FsRecord* __restrict__ records, const uint64_t* __restrict__ keys,
                   const uint32_t* __restrict__ vals, const uint32_t* __restrict__ ranges, const FT* __restrict__ feats,
                   int C, int64_t n, int64_t num_records, const fs_camera* __restrict__ cams, int num_views, int S,
                   fs_opts o, float* __restrict__ out_feat, float* __restrict__ out_T, int32_t* __restrict__ out_n,
                   int32_t* __restrict__ out_last, int32_t* __restrict__ out_idx, float* __restrict__ out_depth,
                   float* __restrict__ out_normal, uint64_t* __restrict__ counters,
                   const uint32_t* __restrict__ order, uint32_t* __restrict__ ticket, uint32_t nblocks) {
    __shared__ WideShared<NVT, FT, NW, BG, EXT, FILTER> sm;
    if (order == nullptr) {
        // the XCDs take one tile row of blocks each in turn: neighbouring
        // blocks share an L2 and dense regions are spread over all XCDs
        // (a launch row holds fewer than 2^32 threads; larger frames take several)
        const int64_t g = blockIdx.x + (int64_t)gridDim.x * blockIdx.z;
        if (g >= nblocks) return;
        const int64_t blk = xcd_remap_chunked(g, nblocks, block_row_chunk(cams, S));
        render_block_wide<NVT, FT, NW, BG, VEC, EXT, FILTER>(blk, sm, records, keys, vals, ranges, feats, C, n, num_records,
                                                     cams, num_views, S, o, out_feat, out_T, out_n, out_last,
                                                     out_idx, out_depth, out_normal, counters);
        return;
    }
    // nq queues: workgroup g takes items q, q + nq, q + 2 nq, .. (q = g mod
    // nq) from a ticket of its own, so the tickets (memory-side atomics,
    // each serialised per address) are shared by a grid's nq-th part only
    const uint32_t nq = gridDim.x < kRenderQueues ? gridDim.x : kRenderQueues;
    const uint32_t q = blockIdx.x % nq;
    // the first item is the workgroup's rank in its queue (taking the further
    // tickets one block ahead would hold back long blocks behind long ones:
    // 300k surfels, 640x480, C = 48: frame 0.214 -> 0.231 ms)
    const uint32_t ahead = (gridDim.x - q + nq - 1) / nq;   // workgroups of the queue
    uint32_t it = blockIdx.x;
    while (it < nblocks) {
        render_block_wide<NVT, FT, NW, BG, VEC, EXT, FILTER>(order[it], sm, records, keys, vals, ranges, feats, C, n,
                                                             num_records, cams, num_views, S, o, out_feat, out_T, out_n,
                                                             out_last, out_idx, out_depth, out_normal, counters);
        if (threadIdx.x == 0) sm.item = atomicAdd(ticket + q * kTicketStride, 1u);
        __syncthreads();   // every wave is done with the item; the next one is known
        it = (ahead + sm.item) * nq + q;
        __syncthreads();
    }
}

// The counters of a render with 16x16 or 32x32 tiles.  They are defined over
// 16x16 pixel blocks that walk their tile's whole list a batch of bg entries at a
// time until every pixel has stopped, and not over the blocks the render works
// in, so a pass of its own counts them, run only when they are asked for: one
// thread per pixel (a wave per 8x8 of them), with the render's response, stop and
// Top-K tests.
__global__ void __launch_bounds__(256)
count_walk_kernel(const FsRecord* __restrict__ records, const uint32_t* __restrict__ vals,
                  const uint32_t* __restrict__ ranges, int64_t num_records, const fs_camera* __restrict__ cams,
                  int num_views, int S, fs_opts o, int bg, int64_t nblocks, uint64_t* __restrict__ counters) {
    constexpr int kQ = FS_RECORD_BYTES / 16;
    __shared__ FsRecord s_rec[32];
    __shared__ double2 s_mu[32];
    __shared__ uint32_t s_used[4], s_active[4];
    __shared__ uint64_t s_pairs[4];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int K = o.topk;
    const double t_stop = o.t_stop;
    uint64_t walked = 0, rows = 0, blocks = 0, blended = 0;   // blended: this thread's pixels; the others uniform
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const BlockPos bp = locate_block(b, S, 16, cams, num_views);
        if (!bp.valid) continue;   // uniform across the workgroup, as every exit below
        const fs_camera& cam = cams[bp.view];
        const int x0 = bp.x0 + (wave & 1) * 8, y0 = bp.y0 + (wave >> 1) * 8;
        const int px = x0 + (lane & 7), py = y0 + (lane >> 3);
        const uint32_t start = ranges[2 * bp.tile], end = ranges[2 * bp.tile + 1];
        double T = 1.0;
        int cnt = 0;
        bool done = px >= cam.width || py >= cam.height;
        ++blocks;
        // record float4 pq of entry pe; the next batch's records and the list
        // values after those are in flight while a batch is walked
        const int pe = tid / kQ, pq = tid - pe * kQ;
        auto val_at = [&](uint32_t p) { return pe < bg && p + (uint32_t)pe < end ? vals[p + pe] : 0xffffffffu; };
        auto record_of = [&](uint32_t rid) {
            float4 v4 = make_float4(0.f, 0.f, 0.f, 0.f);
            if ((int64_t)rid < num_records)
                v4 = reinterpret_cast<const float4*>(records + rid)[pq];
            else if (pq == 5)   // past the list (never in a well-formed one)
                v4.z = __int_as_float(1);   // empty box
            return v4;
        };
        float4 pre = record_of(val_at(start));
        uint32_t nxt = val_at(start + (uint32_t)bg);
        for (uint32_t b0 = start; b0 < end; b0 += (uint32_t)bg) {
            const int nb = (int)(end - b0 < (uint32_t)bg ? end - b0 : (uint32_t)bg);
            __syncthreads();   // the previous batch is no longer read
            if (pe < nb) reinterpret_cast<float4*>(&s_rec[pe])[pq] = pre;
            pre = record_of(nxt);
            nxt = val_at(b0 + 2u * (uint32_t)bg);
            __syncthreads();
            if (o.lowpass != 0) {
                if (tid < nb) fs_record_centre(s_rec[tid], s_mu[tid].x, s_mu[tid].y);
                __syncthreads();
            }
            uint32_t mask = 0u;
            for (int e = 0; e < nb; ++e) {
                const FsRecord& r = s_rec[e];
                if (r.x1 < x0 || r.x0 > x0 + 7 || r.y1 < y0 || r.y0 > y0 + 7) continue;
                if (done || px < r.x0 || px > r.x1 || py < r.y0 || py > r.y1) continue;
                const double dx = (double)(px - r.ax), dy = (double)(py - r.ay);
                FsResp rs = fs_response(r, dx, dy);
                if (o.lowpass != 0) fs_lowpass_d2(rs, dx, dy, s_mu[e].x, s_mu[e].y);
                if (!(rs.d2 <= r.k2)) continue;
                const float G = __builtin_amdgcn_exp2f(-0.72134752044448170f * (float)rs.d2);
                const double Tn = T * (1.0 - (double)fminf(o.alpha_max, r.o * G));
                if (Tn < t_stop) {
                    done = true;
                } else {
                    T = Tn;
                    mask |= 1u << e;
                    ++cnt;
                    if (K > 0 && cnt == K) done = true;
                }
            }
            const uint32_t used = wave_or(mask);
            const bool active = !__all(done);
            if (lane == 0) {
                s_used[wave] = used;
                s_active[wave] = active ? 1u : 0u;
            }
            __syncthreads();
            walked += (uint64_t)nb;
            rows += (uint64_t)__popc(s_used[0] | s_used[1] | s_used[2] | s_used[3]);
            if ((s_active[0] | s_active[1] | s_active[2] | s_active[3]) == 0u) break;
        }
        blended += (uint64_t)cnt;
        __syncthreads();   // the last batch is no longer read
    }
    const uint64_t sum = __ockl_wfred_add_u64(blended);
    if (lane == 0) s_pairs[wave] = sum;
    __syncthreads();
    if (tid == 0) {
        const uint64_t pairs = s_pairs[0] + s_pairs[1] + s_pairs[2] + s_pairs[3];
        atomicAdd((unsigned long long*)&counters[0], (unsigned long long)walked);
        atomicAdd((unsigned long long*)&counters[1], (unsigned long long)rows);
        atomicAdd((unsigned long long*)&counters[2], (unsigned long long)pairs);
        atomicAdd((unsigned long long*)&counters[3], (unsigned long long)blocks);
    }
}

// Work order for the persistent launch: blocks bucketed by 4 log2(1 + list
// length) (64 buckets), longest bucket first.
FS_DEV int cost_bucket(uint32_t len) {
    const float b = 4.f * __log2f(1.f + (float)len);
    const int k = (int)b;
    return 63 - (k > 63 ? 63 : k);
}

// Pass 1: per group of 256 blocks, its blocks per cost bucket (no atomics
// outside LDS, nothing to clear beforehand); group 0 also zeroes the work
// queues' tickets.
__global__ void __launch_bounds__(256)
order_count_kernel(const uint32_t* __restrict__ ranges, int sb2, uint32_t nblocks, uint32_t* __restrict__ gcnt,
                   uint32_t* __restrict__ ticket) {
    __shared__ uint32_t h[64];
    const uint32_t tid = threadIdx.x;
    if (tid < 64) h[tid] = 0u;
    __syncthreads();
    const uint32_t b = blockIdx.x * 256u + tid;
    if (b < nblocks) {
        const uint32_t t = b / sb2;
        atomicAdd(&h[cost_bucket(ranges[2 * t + 1] - ranges[2 * t])], 1u);
    }
    __syncthreads();
    if (tid < 64) gcnt[blockIdx.x * 64u + tid] = h[tid];
    if (blockIdx.x == 0 && tid < kRenderQueues) ticket[tid * kTicketStride] = 0u;
}

// Pass 2: every group finds where its blocks of each bucket start -- the
// blocks of all groups in earlier buckets, then those of earlier groups in
// the same bucket -- and places them (ranks within the group by LDS
// cursors, so the order inside a bucket is not fixed).
__global__ void __launch_bounds__(256)
order_place_kernel(const uint32_t* __restrict__ ranges, int sb2, uint32_t nblocks, const uint32_t* __restrict__ gcnt,
                   uint32_t ngroups, uint32_t* __restrict__ order) {
    __shared__ uint32_t s_tot[4][64], s_bef[4][64], base[64];
    const uint32_t tid = threadIdx.x, k = tid & 63u, qtr = tid >> 6;
    uint32_t tot = 0u, bef = 0u;
    for (uint32_t w = qtr; w < ngroups; w += 4u) {
        const uint32_t c = gcnt[w * 64u + k];
        tot += c;
        bef += w < blockIdx.x ? c : 0u;
    }
    s_tot[qtr][k] = tot;
    s_bef[qtr][k] = bef;
    __syncthreads();
    if (tid < 64) {
        const uint32_t T = s_tot[0][k] + s_tot[1][k] + s_tot[2][k] + s_tot[3][k];
        const uint32_t B = s_bef[0][k] + s_bef[1][k] + s_bef[2][k] + s_bef[3][k];
        uint32_t incl = T;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, 64);
            if ((int)tid >= d) incl += y;
        }
        base[k] = incl - T + B;
    }
    __syncthreads();
    const uint32_t b = blockIdx.x * 256u + tid;
    if (b < nblocks) {
        const uint32_t t = b / sb2;
        const uint32_t pos = atomicAdd(&base[cost_bucket(ranges[2 * t + 1] - ranges[2 * t])], 1u);
        if (pos < nblocks) order[pos] = b;
    }
}

constexpr int64_t kMaxRow = int64_t(1) << 23;   // workgroups of 256 threads in one row of a launch

template <int NVT, typename FT, int NW, int BG, bool EXT, bool FILTER>
hipError_t launch_wide(const FsRecord* records, const uint64_t* keys, const uint32_t* vals, const uint32_t* ranges,
                       const void* feats, int C, int64_t n, const fs_camera* cams, int num_views, int64_t total_tiles,
                       const fs_opts& o, float* out_feat, float* out_T, int32_t* out_n, int32_t* out_last,
                       int32_t* out_idx, float* out_depth, float* out_normal, uint64_t* counters,
                       const FsWorkspace& ws, hipStream_t s) {
    const int sb = o.tile / 8;
    const int64_t blocks = total_tiles * sb * sb;   // 8x8 blocks
    if (blocks >= (int64_t(1) << 32)) return hipErrorInvalidValue;
    constexpr int kChunk = 4 * NVT * FeatVec<FT>::kElems;
    const int chunks = (C + kChunk - 1) / kChunk;
    const bool vec = (C % (16 / (int)sizeof(FT))) == 0;
    auto kern = vec ? render_wide_kernel<NVT, FT, NW, BG, true, EXT, FILTER>
                    : render_wide_kernel<NVT, FT, NW, BG, false, EXT, FILTER>;
    // workgroups the device holds at once: the work queue pays only beyond that
    // (with fewer blocks all of them start at once, in any order, and the two
    // ordering launches only cost: 19k surfels, 242x163, C = 76: frame 65.8 ->
    // 60.0 us)
    int64_t grid = 0;
    if (o.schedule == FS_SCHED_PERSISTENT && chunks == 1 && blocks <= ws.render_max_blocks) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), NW * 64, 0) !=
                hipSuccess || per_cu < 1)
            per_cu = 1;
        grid = (int64_t)fs_device_cus() * per_cu;
    }
    // and with enough lists to order: with fewer surfels than blocks most blocks
    // have none (2,000 surfels, 1280x720, C = 64, tile 16: render 61 us with the
    // queue, 49 without)
    if (grid > 0 && blocks > grid && n * num_views >= blocks) {
        const uint32_t nb = (uint32_t)blocks;
        const hipError_t e = fs_launch_block_order(ranges, sb * sb, nb, ws, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NW * 64), 0, s, records, keys, vals, ranges,
                           static_cast<const FT*>(feats), C, n, n * num_views, cams, num_views, o.tile, o, out_feat,
                           out_T, out_n, out_last, out_idx, out_depth, out_normal, counters, ws.render_order,
                           ws.render_ticket, nb);
        return hipGetLastError();
    }
    const int64_t row = blocks < kMaxRow ? blocks : kMaxRow;
    hipLaunchKernelGGL(kern, dim3((unsigned)row, (unsigned)chunks, (unsigned)((blocks + row - 1) / row)), dim3(NW * 64),
                       0, s, records, keys, vals,
                       ranges, static_cast<const FT*>(feats), C, n, n * num_views, cams, num_views, o.tile, o,
                       out_feat, out_T, out_n, out_last, out_idx, out_depth, out_normal, counters,
                       (const uint32_t*)nullptr, (uint32_t*)nullptr, (uint32_t)blocks);
    return hipGetLastError();
}

template <int NVT, typename FT>
hipError_t launch_waves(const FsRecord* records, const uint64_t* keys, const uint32_t* vals, const uint32_t* ranges,
                        const void* feats, int C, int64_t n, const fs_camera* cams, int num_views,
                        int64_t total_tiles, const fs_opts& o, float* out_feat, float* out_T, int32_t* out_n,
                        int32_t* out_last, int32_t* out_idx, float* out_depth, float* out_normal,
                        uint64_t* counters, const FsWorkspace& ws, hipStream_t s) {
    const bool bg16 = o.batch == 16;
    // the low-pass response and the depth / normal outputs run in their own
    // instantiations (32-entry batches), so the plain render carries none of
    // their registers
    const bool ext = o.lowpass != 0 || out_depth != nullptr || out_normal != nullptr;
#define FS_WIDE(B, X, F)                                                                                           \
    return launch_wide<NVT, FT, 4, B, X, F>(records, keys, vals, ranges, feats, C, n, cams, num_views, total_tiles, \
                                            o, out_feat, out_T, out_n, out_last, out_idx, out_depth, out_normal,    \
                                            counters, ws, s)
    if (o.tile > 8) {   // a block sees a part of its tile's list
        if (ext) FS_WIDE(32, true, true);
        if (bg16) FS_WIDE(16, false, true);
        FS_WIDE(32, false, true);
    }
    if (ext) FS_WIDE(32, true, false);
    if (bg16) FS_WIDE(16, false, false);
    FS_WIDE(32, false, false);
#undef FS_WIDE
}

}  // namespace

int fs_device_cus() {
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
        return n;
    }();
    return cus;
}

hipError_t fs_launch_block_order(const uint32_t* ranges, int sb2, uint32_t nblocks, const FsWorkspace& ws,
                                 hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    if ((int64_t)nblocks > ws.render_max_blocks || ws.render_order == nullptr) return hipErrorInvalidValue;
    const unsigned g = (nblocks + 255) / 256;
    if (ws.render_gcnt == nullptr || (int64_t)g * 64 > ws.render_gcnt_words) return hipErrorInvalidValue;
    hipLaunchKernelGGL(order_count_kernel, dim3(g), dim3(256), 0, s, ranges, sb2, nblocks, ws.render_gcnt,
                       ws.render_ticket);
    hipLaunchKernelGGL(order_place_kernel, dim3(g), dim3(256), 0, s, ranges, sb2, nblocks, ws.render_gcnt, g,
                       ws.render_order);
    return hipGetLastError();
}

hipError_t fs_launch_render_forward(const FsRecord* records, const uint64_t* keys, const uint32_t* vals,
                                    const uint32_t* ranges, const void* feats, int C, int64_t n,
                                    const fs_camera* cams, int num_views, int64_t total_tiles, const fs_opts& o,
                                    float* out_feat, float* out_T, int32_t* out_n, int32_t* out_last,
                                    int32_t* out_idx, float* out_depth, float* out_normal, uint64_t* counters,
                                    const FsWorkspace& ws, hipStream_t s) {
    if (total_tiles == 0) return hipSuccess;
    const bool bf16 = o.feat_dtype == FS_FEAT_BF16;
    if (counters != nullptr && o.tile > 8) {
        const bool ext = o.lowpass != 0 || out_depth != nullptr || out_normal != nullptr;
        const int64_t blocks = total_tiles * (o.tile / 16) * (o.tile / 16);
        // (the counters' atomics are serialised per address, about 50 ns each)
        const int64_t grid = blocks < 2048 ? blocks : 2048;
        hipLaunchKernelGGL(count_walk_kernel, dim3((unsigned)grid), dim3(256), 0, s, records, vals, ranges,
                           n * num_views, cams, num_views, o.tile, o, o.batch == 16 && !ext ? 16 : 32, blocks, counters);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        counters = nullptr;
    }
#define FS_WAVES(NVTv, FTv)                                                                                          \
    return launch_waves<NVTv, FTv>(records, keys, vals, ranges, feats, C, n, cams, num_views, total_tiles, o,      \
                                   out_feat, out_T, out_n, out_last, out_idx, out_depth, out_normal, counters, ws, s)
    // channels per workgroup: 16, 32, 48, 64 or 128 (more run in several, each
    // walking the lists again), so that narrow images take little LDS; 65 to 112
    // channels keep the LDS and accumulators of 128 (200k surfels, 640x480, tile 16:
    // render 71 us for 64, 87 for 76, 91 for 128)
    if (bf16) {
        if (C <= 32) FS_WAVES(1, uint16_t);
        if (C <= 64) FS_WAVES(2, uint16_t);
        FS_WAVES(4, uint16_t);
    }
    if (C <= 16) FS_WAVES(1, float);
    if (C <= 32) FS_WAVES(2, float);
    if (C <= 48) FS_WAVES(3, float);
    if (C <= 64) FS_WAVES(4, float);
    FS_WAVES(8, float);
#undef FS_WAVES
}
