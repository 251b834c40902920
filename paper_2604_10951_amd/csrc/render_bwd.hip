// render_bwd.hip -- gradients of L = sum_p g_p . F_p through the blend
// (Sec. 3.1 Eq. 2, Top-K of Sec. 3.4), the ray-splat intersection and the
// projection (Sec. 3.1 Eq. 1, Sec. 3.2 T) back to the surfel parameters.
//
// With contributors m of a pixel in depth order, w_m = alpha_m T_m:
//   dL/dc_m     = w_m g
//   dL/dalpha_m = T_m (g . c_m) - S_m / (1 - alpha_m),  S_m = sum_{l > m} w_l (g . c_l)
//   alpha = o exp(-d2 / 2) unless clamped at alpha_max (then no gradient)
//   d2 = u^2 + v^2, (u, v) = (h0 / h2, h1 / h2), h = L (1, dx, dy)
// where L is the anchored, normalised 3x3 coefficient matrix of the record.
// The blend's discrete choices are those of the forward pass: the same
// double-precision response decides acceptance, and entries after the
// pixel's last blended position are skipped.
//
// Kernel 1 (per 8x8 block, four waves): the block's entries are walked back to
// front in batches of 32.  All threads evaluate the (entry, pixel) pairs inside
// the entries' pixel boxes; lanes = pixels recover T by division from the
// forward's final transmittance and form the weights; groups of 16 threads own
// an entry each and form g . c_m and the sum of w g over its pixels from the
// block's upstream gradient, staged in LDS once; lanes = pixels run the suffix
// sums; the groups then run the scalar chain to dL/dL (9) and dL/do over
// their entries' accepted pixels.  Per-entry results go to global
// memory with atomics (float, so the sum order, hence the last bits, can vary).
// What bounds it is the serial chain of a long list's batches (five barriers
// each), not the arithmetic, so every phase spreads a batch's pairs over as
// many lanes as it can: one wave per block with a wave reduction per pair took
// 2.75 ms for the 200k-surfel, 640x480, C = 48 full blend (16x16 tiles), this
// form 0.28 ms.
// Kernel 2 (per surfel): dL/dL -> dL/dadj(T) -> dL/dT -> centre, scales,
// quaternion, summed over views, in double precision.
#include "fs_internal.h"

namespace {

constexpr int BG = 32;
constexpr int kGradFloats = FS_GRAD_RECORD_FLOATS;   // 9 (dL/dL) + 1 (dL/do) + 2 pad

FS_DEV float bf16_to_f32b(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
template <typename FT>
FS_DEV float to_f32(FT x);
template <>
FS_DEV float to_f32<float>(float x) { return x; }
template <>
FS_DEV float to_f32<uint16_t>(uint16_t x) { return bf16_to_f32b(x); }

// dL/dalpha of one (pixel, record) contribution -> dL/dL (9, rows of the
// record's coefficient matrix times (1, dx, dy)) and dL/do, through alpha = o
// exp(-d2 / 2) (no gradient when clamped at alpha_max), d2 = u^2 + v^2 and
// (u, v) = (h0, h1) / h2.
FS_DEV void blend_chain(const FsRecord& r, const FsResp& rs, double ddx, double ddy, float Gs, float dalpha,
                        float* g) {
    g[9] = Gs * dalpha;   // dL/do
    const float dG = r.o * dalpha;
    const float dd2 = -0.5f * Gs * dG;
    const float u = (float)rs.u, vv = (float)rs.v, rh = (float)rs.rh;
    const float du = 2.f * u * dd2, dv = 2.f * vv * dd2;
    const float dh0 = du * rh, dh1 = dv * rh, dh2 = -(u * du + vv * dv) * rh;
    const float fx = (float)ddx, fy = (float)ddy;
    g[0] = dh0;
    g[1] = dh0 * fx;
    g[2] = dh0 * fy;
    g[3] = dh1;
    g[4] = dh1 * fx;
    g[5] = dh1 * fy;
    g[6] = dh2;
    g[7] = dh2 * fx;
    g[8] = dh2 * fy;
}

__global__ void zero_f32_kernel(float* p, int64_t count) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = 0.f;
}

// Position of the m-th set bit of x (m < popcount).
FS_DEV int nth_bit(uint64_t x, int m) {
    int p = 0;
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) {
        const int c = __popcll(x & ((1ull << sh) - 1ull));
        if (m >= c) {
            m -= c;
            x >>= sh;
            p += sh;
        }
    }
    return p;
}

// Threads per entry and channels per thread of the feature phase: thread q of a
// group owns channels q, q + 16, ..., so that a group's atomics to a gradient
// row are contiguous.
constexpr int kBwdThreads = 256;
constexpr int kBwdGroup = 16;
constexpr int kBwdGroups = kBwdThreads / kBwdGroup;
constexpr int kBwdQueue = 512;   // entries queued by the filter (a power of two)
constexpr uint32_t kBwdLong = 64;   // blocks with longer lists are started first (200k surfels, 640x480, C = 48,
                                    // 8x8 tiles: 225 us, 245 from 16 and 248 from 256 entries, 260 without)

// FILTER (tiles larger than a block): only entries whose pixel boxes meet the
// block are walked, queued 256 list positions at a time.
template <int CPT, typename FT, bool FILTER>
struct BwdShared {
    static constexpr int kRow = kBwdGroup * CPT + (kBwdGroup * CPT % 64 == 0 ? 16 : 0);   // spread over the banks
    FsRecord rec[BG];
    uint32_t recid[BG];
    uint32_t sidx[BG];
    float g[64][kRow];             // upstream gradient of the block's pixels, zero past C and past the image
    float a[BG][64];               // alpha per accepted (entry, pixel)
    float w[BG][64];               // weight
    float d[BG][64];               // g . c, then dL/dalpha
    uint32_t amask[64];            // per pixel: accepted entries of the batch
    uint32_t emask[BG][2];         // per entry: accepted pixels
    int last[64];
    uint32_t qrid[FILTER ? kBwdQueue : 1];
    uint32_t qpos[FILTER ? kBwdQueue : 1];
    uint32_t qcount[kBwdThreads / 64];
};

template <int CPT, typename FT, bool FILTER>
__global__ void __launch_bounds__(kBwdThreads)
render_bwd_kernel(const FsRecord* __restrict__ records, const uint32_t* __restrict__ vals,
                  const uint32_t* __restrict__ ranges, const FT* __restrict__ feats, int C, int64_t n,
                  int64_t num_records, const fs_camera* __restrict__ cams, int num_views, int S, int64_t nblocks,
                  fs_opts o, const float* __restrict__ out_T, const int32_t* __restrict__ out_last,
                  const float* __restrict__ grad_feat, float* __restrict__ grad_records,
                  float* __restrict__ grad_feats) {
    constexpr int NT = kBwdThreads, NW = NT / 64;
    constexpr int kQ = FS_RECORD_BYTES / 16;
    constexpr int kRounds = BG / kBwdGroups;
    static_assert(BG * kQ <= NT, "one record float4 per thread");
    static_assert(2 * BG + NT <= kBwdQueue, "a refill fits the queue beside the batch in work and the next");
    __shared__ BwdShared<CPT, FT, FILTER> sm;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // grid row 0 (dispatched first) takes the blocks with long lists, row 1 the
    // others; the XCDs take one tile row of blocks each in turn
    const bool second = blockIdx.y != 0;
    // (a launch row holds fewer than 2^32 threads; larger frames take several)
    const int64_t g = blockIdx.x + (int64_t)gridDim.x * blockIdx.z;
    if (g >= nblocks) return;
    const int64_t block = xcd_remap_chunked(g, nblocks, block_row_chunk(cams, S));
    const BlockPos bp = locate_block(block, S, 8, cams, num_views);
    if (!bp.valid) return;
    const uint32_t start = ranges[2 * bp.tile], end = ranges[2 * bp.tile + 1];
    if ((end - start > kBwdLong) == second || start >= end) return;
    const fs_camera& cam = cams[bp.view];
    const int px = bp.x0 + (lane & 7), py = bp.y0 + (lane >> 3);
    const bool inside = px < cam.width && py < cam.height;
    const int64_t pix = cam.pixel_offset + (int64_t)py * cam.width + px;
    const int last = inside ? out_last[pix] : -1;
    // walk back from the block's last blended entry
    const int maxlast = __ockl_wfred_max_i32(last);
    if (maxlast < (int)start) return;   // nothing was blended in this block
    // a last position from another frame's lists must not walk past this
    // tile's run into the next tile's entries
    const uint32_t top = min((uint32_t)maxlast + 1u, end);
    const uint32_t len = top - start;   // entry i of the walk is list position top - 1 - i
    double T = inside ? (double)out_T[pix] : 1.0;   // wave 0's walk
    float suffix = 0.f;                             // S: sum over later contributors of w (g . c)
    if (tid < 64) sm.last[tid] = last;

    // records of the next batch are in flight while a batch is processed
    float4 pre = make_float4(0.f, 0.f, 0.f, 0.f);
    uint32_t pre_rid = 0xffffffffu;
    const int pe = tid / kQ, pq = tid - pe * kQ;    // record float4 of this thread: quarter pq of entry pe
    auto fetch_record = [&](uint32_t rid) {
        pre_rid = rid;
        pre = make_float4(0.f, 0.f, 0.f, 0.f);
        if ((int64_t)rid < num_records) pre = reinterpret_cast<const float4*>(records + rid)[pq];
    };
    auto val_at = [&](uint32_t i) { return i < len ? vals[top - 1u - i] : 0xffffffffu; };
    uint32_t nxt_rid = 0xffffffffu;
    uint32_t qh = 0, qt = 0, cp = 0;
    uint32_t c_rid = 0xffffffffu, c_val = 0xffffffffu;
    uint2 c_box = make_uint2(0u, 0u);
    auto load_box = [&]() {
        c_rid = c_val;
        if ((int64_t)c_rid < num_records)
            c_box = *reinterpret_cast<const uint2*>(&records[c_rid].x0);
        else
            c_rid = 0xffffffffu;
    };
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
            const uint32_t i = (at + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))) & (kBwdQueue - 1);
            sm.qrid[i] = c_rid;
            sm.qpos[i] = top - 1u - (cp + (uint32_t)tid);
        }
        cp += NT;
        load_box();
        c_val = val_at(cp + NT + (uint32_t)tid);
        __syncthreads();
    };
    auto fetch_queued = [&](uint32_t h) {
        fetch_record(pe < BG && h + (uint32_t)pe < qt ? sm.qrid[(h + pe) & (kBwdQueue - 1)] : 0xffffffffu);
    };

    if constexpr (FILTER) {
        c_val = val_at((uint32_t)tid);
        load_box();
        c_val = val_at((uint32_t)(NT + tid));
    } else {
        fetch_record(pe < BG ? val_at((uint32_t)pe) : 0xffffffffu);
        nxt_rid = pe < BG ? val_at((uint32_t)(BG + pe)) : 0xffffffffu;
    }
    for (int t = tid; t < 64 * BwdShared<CPT, FT, FILTER>::kRow; t += NT) {
        const int p = t / BwdShared<CPT, FT, FILTER>::kRow, c = t - p * BwdShared<CPT, FT, FILTER>::kRow;
        const int qx = bp.x0 + (p & 7), qy = bp.y0 + (p >> 3);
        const bool in = c < C && qx < cam.width && qy < cam.height;
        sm.g[p][c] = in ? grad_feat[(cam.pixel_offset + (int64_t)qy * cam.width + qx) * C + c] : 0.f;
    }
    if constexpr (FILTER) {
        while (qt < (uint32_t)BG && cp < len) refill();
        fetch_queued(0);
    }
    const int q = tid % kBwdGroup, grp = tid / kBwdGroup;

    for (uint32_t b0 = 0; FILTER ? qh != qt : b0 < len; b0 += BG) {
        const uint32_t left = FILTER ? qt - qh : len - b0;
        const int nb = (int)(left < (uint32_t)BG ? left : (uint32_t)BG);
        // 1. stage the records; clear the batch's masks (all of it was last read
        //    before the previous batch's final barrier)
        if (pe < nb) {
            uint32_t rid = pre_rid;
            if ((int64_t)rid >= num_records) {   // never happens for a well-formed list
                rid = 0u;
                if (pq == 4) pre.w = __int_as_float((int)0xbff00000);   // k2 = -1: never accepted
                if (pq == 5) pre.z = __int_as_float(1);                 // empty box
            }
            reinterpret_cast<float4*>(&sm.rec[pe])[pq] = pre;
            if (pq == 0) {
                sm.recid[pe] = rid;
                sm.sidx[pe] = rid % (uint32_t)n;
            }
        }
        if (tid < 64) sm.amask[tid] = 0u;
        if (tid < 2 * BG) (&sm.emask[0][0])[tid] = 0u;
        __syncthreads();
        // list position of the batch's entry e
        auto pos_of = [&](int e) -> int {
            return FILTER ? (int)sm.qpos[(qh + e) & (kBwdQueue - 1)] : (int)(top - 1u - (b0 + (uint32_t)e));
        };
        // the feature rows of the group's entries: in flight during the
        // response and weight phases
        float f[kRounds][CPT];
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int e = grp + r * kBwdGroups;
            const FT* __restrict__ row = feats + (int64_t)(e < nb ? sm.sidx[e] : 0u) * C;
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int c = q + i * kBwdGroup;
                f[r][i] = e < nb && c < C ? to_f32(row[c]) : 0.f;
            }
        }
        if constexpr (FILTER) {
            while (qt - qh - nb < (uint32_t)BG && cp < len) refill();
            fetch_queued(qh + nb);
        } else if (b0 + BG < len) {
            fetch_record(nxt_rid);
            nxt_rid = pe < BG ? val_at(b0 + 2u * BG + (uint32_t)pe) : 0xffffffffu;
        }
        // 2. responses of the pairs inside the entries' boxes (numbered by a
        //    prefix sum of the boxes' pixel counts, found by bisection)
        {
            int cnt_e = 0, packed = 0;
            if (lane < nb) {
                const FsRecord& r = sm.rec[lane];
                const int xa = r.x0 > bp.x0 ? r.x0 : bp.x0;
                const int ya = r.y0 > bp.y0 ? r.y0 : bp.y0;
                int xb = r.x1 < bp.x0 + 7 ? r.x1 : bp.x0 + 7;
                int yb = r.y1 < bp.y0 + 7 ? r.y1 : bp.y0 + 7;
                xb = xb < cam.width - 1 ? xb : cam.width - 1;
                yb = yb < cam.height - 1 ? yb : cam.height - 1;
                if (xb >= xa && yb >= ya) {
                    const int rw = xb - xa + 1, rh = yb - ya + 1;
                    cnt_e = rw * rh;
                    const int inv = (65536 + rw - 1) / rw;   // exact division of counts < 64 by rw <= 8
                    packed = (xa - bp.x0) | ((ya - bp.y0) << 3) | (rw << 6) | (inv << 10);
                }
            }
            const int Sc = __ockl_wfscan_add_i32(cnt_e, true);
            const int M = __builtin_amdgcn_readlane(Sc, 31);
            for (int base = wave * 64; base < M; base += NT) {   // uniform per wave: every lane shuffles
                const int m = base + lane;
                int e = 0;
#pragma unroll
                for (int step = BG / 2; step >= 1; step >>= 1)
                    if (__shfl(Sc, e + step - 1, 64) <= m) e += step;
                const int prev = __shfl(Sc, e > 0 ? e - 1 : 0, 64);
                const int pk = __shfl(packed, e, 64);
                if (m < M) {
                    const int local = m - (e > 0 ? prev : 0);
                    const int rw = (pk >> 6) & 15, inv = pk >> 10;
                    const int dy = (local * inv) >> 16, dx = local - dy * rw;
                    const int lx = (pk & 7) + dx, ly = ((pk >> 3) & 7) + dy, p = ly * 8 + lx;
                    const FsRecord& r = sm.rec[e];
                    const FsResp rs = fs_response(r, (double)(bp.x0 + lx - r.ax), (double)(bp.y0 + ly - r.ay));
                    if (rs.d2 <= r.k2 && pos_of(e) <= sm.last[p]) {
                        const float Gs = __builtin_amdgcn_exp2f(-0.72134752044448170f * (float)rs.d2);
                        sm.a[e][p] = fminf(o.alpha_max, r.o * Gs);
                        atomicOr(&sm.amask[p], 1u << e);
                        atomicOr(&sm.emask[e][p >> 5], 1u << (p & 31));
                    }
                }
            }
        }
        __syncthreads();
        // 3. weights, back to front (lanes = pixels)
        if (wave == 0) {
            uint32_t m = sm.amask[lane];
            while (m != 0u) {
                const int e = __builtin_ctz(m);
                m &= m - 1u;
                const double al = (double)sm.a[e][lane];
                T = T / (1.0 - al);
                sm.w[e][lane] = (float)(al * T);
            }
        }
        __syncthreads();
        // 4. D = g . c per contribution, dL/dc = sum of w g per entry: a group
        //    of 16 threads per entry, two of its pixels per step
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int e = grp + r * kBwdGroups;
            uint64_t m = (uint64_t)sm.emask[e][0] | (uint64_t)sm.emask[e][1] << 32;
            if (m == 0ull) continue;   // uniform inside the group
            float acc[CPT];
#pragma unroll
            for (int i = 0; i < CPT; ++i) acc[i] = 0.f;
            while (m != 0ull) {
                const int p0 = __builtin_ctzll(m);
                m &= m - 1ull;
                const bool two = m != 0ull;
                const int p1 = two ? __builtin_ctzll(m) : p0;
                if (two) m &= m - 1ull;
                const float w0 = sm.w[e][p0], w1 = two ? sm.w[e][p1] : 0.f;
                float d0 = 0.f, d1 = 0.f;
#pragma unroll
                for (int i = 0; i < CPT; ++i) {
                    const float g0 = sm.g[p0][q + i * kBwdGroup], g1 = sm.g[p1][q + i * kBwdGroup];
                    d0 = fmaf(g0, f[r][i], d0);
                    d1 = fmaf(g1, f[r][i], d1);
                    acc[i] = fmaf(w0, g0, acc[i]);
                    if (two) acc[i] = fmaf(w1, g1, acc[i]);
                }
#pragma unroll
                for (int s = 1; s < kBwdGroup; s <<= 1) {
                    d0 += __uint_as_float(lane_xor32(__float_as_uint(d0), s));
                    d1 += __uint_as_float(lane_xor32(__float_as_uint(d1), s));
                }
                if (q == 0) {
                    sm.d[e][p0] = d0;
                    if (two) sm.d[e][p1] = d1;
                }
            }
            float* __restrict__ dst = grad_feats + (int64_t)sm.sidx[e] * C;
#pragma unroll
            for (int i = 0; i < CPT; ++i)
                if (q + i * kBwdGroup < C) atomicAdd(dst + q + i * kBwdGroup, acc[i]);
        }
        __syncthreads();
        // 5. dL/dalpha, back to front (lanes = pixels)
        if (wave == 0) {
            uint32_t m = sm.amask[lane];
            while (m != 0u) {
                const int e = __builtin_ctz(m);
                m &= m - 1u;
                const float al = sm.a[e][lane], w = sm.w[e][lane], D = sm.d[e][lane];
                sm.d[e][lane] = w / al * D - suffix / (1.f - al);
                suffix = fmaf(w, D, suffix);
            }
        }
        __syncthreads();
        // 6. the chain to the record's coefficients: the entry's group takes its
        //    accepted pixels 16 at a time and sums over its lanes (a fixed order,
        //    so only the order of the blocks' atomics varies from run to run)
#pragma unroll 1
        for (int e = grp; e < BG; e += kBwdGroups) {
            const uint64_t m = (uint64_t)sm.emask[e][0] | (uint64_t)sm.emask[e][1] << 32;
            const int np = __popcll(m);
            if (np == 0) continue;   // uniform inside the group
            const FsRecord& r = sm.rec[e];
            float sum[10];
#pragma unroll
            for (int i = 0; i < 10; ++i) sum[i] = 0.f;
            for (int k = q; k < np; k += kBwdGroup) {
                const int p = nth_bit(m, k);
                const double ddx = (double)(bp.x0 + (p & 7) - r.ax), ddy = (double)(bp.y0 + (p >> 3) - r.ay);
                const FsResp rs = fs_response(r, ddx, ddy);
                const float Gs = __builtin_amdgcn_exp2f(-0.72134752044448170f * (float)rs.d2);
                if (r.o * Gs > o.alpha_max) continue;   // clamped: no gradient
                float gg[10];
                blend_chain(r, rs, ddx, ddy, Gs, sm.d[e][p], gg);
#pragma unroll
                for (int i = 0; i < 10; ++i) sum[i] += gg[i];
            }
#pragma unroll
            for (int s = 1; s < kBwdGroup; s <<= 1)
#pragma unroll
                for (int i = 0; i < 10; ++i) sum[i] += __uint_as_float(lane_xor32(__float_as_uint(sum[i]), s));
            float v = 0.f;   // component q of the sums
#pragma unroll
            for (int i = 0; i < 10; ++i) v = q == i ? sum[i] : v;
            if (v != 0.f) atomicAdd(&grad_records[(int64_t)sm.recid[e] * kGradFloats + q], v);
        }
        qh += (uint32_t)nb;
        __syncthreads();
    }
}

// dL/dL (anchored, normalised record coefficients; columns: constant, dx, dy)
// back to the surfel parameters.  L = adj(T) A / s with A mapping (1, dx, dy)
// to (x, y, 1) = (xa + dx, ya + dy, 1); since (u, v) does not change when L is
// scaled, the dependence of s on T contributes nothing and dL/dadj = dL/dL A^T / s.
__global__ void __launch_bounds__(256)
preprocess_bwd_kernel(const float* __restrict__ means, const float* __restrict__ scales,
                      const float* __restrict__ quats, const float* __restrict__ opacity, int64_t n,
                      const fs_camera* __restrict__ cams, int num_views, fs_opts o,
                      const float* __restrict__ grad_records, float* __restrict__ gm, float* __restrict__ gs,
                      float* __restrict__ gq, float* __restrict__ go) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double am[3] = {0, 0, 0}, as[2] = {0, 0}, aq[4] = {0, 0, 0, 0}, ao = 0.0;
    for (int v = 0; v < num_views; ++v) {
        const float* gr = grad_records + ((int64_t)v * n + i) * kGradFloats;
        double dl[9];
        bool any = false;
        for (int k = 0; k < 9; ++k) {
            dl[k] = gr[k];
            any = any || dl[k] != 0.0;
        }
        ao += gr[9];
        if (!any) continue;
        const fs_camera& cam = cams[v];
        FsGeo g;
        if (!fs_project(means + 3 * i, scales + 2 * i, quats + 4 * i, opacity[i], cam, (double)o.alpha_min, g))
            continue;
        FsFootprint fp;
        fs_footprint(g, cam.width, cam.height, fp);
        const double mx = g.T[2] / g.T[8], my = g.T[5] / g.T[8];
        const double s = (g.H[6] * mx + g.H[7] * my) + g.H[8];
        const double xa = fp.q.ax + 0.5, ya = fp.q.ay + 0.5;
        // dL/dH = dL/dL A^T / s ; A = [[xa,1,0],[ya,0,1],[1,0,0]]  (rows of H act on (x, y, 1))
        double dH[9];
        for (int r = 0; r < 3; ++r) {
            const double l0 = dl[3 * r], l1 = dl[3 * r + 1], l2 = dl[3 * r + 2];
            dH[3 * r + 0] = (l0 * xa + l1) / s;   // column x
            dH[3 * r + 1] = (l0 * ya + l2) / s;   // column y
            dH[3 * r + 2] = l0 / s;               // column 1
        }
        // H columns: T2 x Tw, Tw x T1, T1 x T2 ; for c = a x b: dL/da = b x g, dL/db = g x a
        const double* T1 = g.T;
        const double* T2 = g.T + 3;
        const double* Tw = g.T + 6;
        double gx[3], gy[3], g1[3];
        for (int r = 0; r < 3; ++r) {
            gx[r] = dH[3 * r];
            gy[r] = dH[3 * r + 1];
            g1[r] = dH[3 * r + 2];
        }
        double dT1[3], dT2[3], dTw[3], t0[3], t1[3];
        fs_cross(Tw, gx, t0);          // d(T2 x Tw)/dT2
        fs_cross(T1, g1, t1);          // d(T1 x T2)/dT2 = g1 x T1
        for (int k = 0; k < 3; ++k) dT2[k] = t0[k] - t1[k];
        fs_cross(gx, T2, t0);          // d(T2 x Tw)/dTw
        fs_cross(T1, gy, t1);          // d(Tw x T1)/dTw
        for (int k = 0; k < 3; ++k) dTw[k] = t0[k] + t1[k];
        fs_cross(gy, Tw, t0);          // d(Tw x T1)/dT1
        fs_cross(T2, g1, t1);          // d(T1 x T2)/dT1
        for (int k = 0; k < 3; ++k) dT1[k] = t0[k] + t1[k];
        // T = K [U | V | pc]: rows T1 = fx M0 + cx M2, T2 = fy M1 + cy M2, Tw = M2
        double dM0[3], dM1[3], dM2[3];
        for (int c = 0; c < 3; ++c) {
            dM0[c] = (double)cam.fx * dT1[c];
            dM1[c] = (double)cam.fy * dT2[c];
            dM2[c] = (double)cam.cx * dT1[c] + (double)cam.cy * dT2[c] + dTw[c];
        }
        const double dU[3] = {dM0[0], dM1[0], dM2[0]};
        const double dV[3] = {dM0[1], dM1[1], dM2[1]};
        const double dpc[3] = {dM0[2], dM1[2], dM2[2]};
        FsFrame fr;
        fs_frame(means + 3 * i, scales + 2 * i, quats + 4 * i, cam, fr);
        double Rtu[3], Rtv[3], dtu[3], dtv[3];
        for (int r = 0; r < 3; ++r) {
            const double R0 = cam.R[3 * r], R1 = cam.R[3 * r + 1], R2 = cam.R[3 * r + 2];
            Rtu[r] = (R0 * fr.tu[0] + R1 * fr.tu[1]) + R2 * fr.tu[2];
            Rtv[r] = (R0 * fr.tv[0] + R1 * fr.tv[1]) + R2 * fr.tv[2];
        }
        const double s0 = scales[2 * i], s1 = scales[2 * i + 1];
        for (int k = 0; k < 3; ++k) {
            const double Rk0 = cam.R[k], Rk1 = cam.R[3 + k], Rk2 = cam.R[6 + k];   // column k of R
            am[k] += (Rk0 * dpc[0] + Rk1 * dpc[1]) + Rk2 * dpc[2];
            dtu[k] = s0 * ((Rk0 * dU[0] + Rk1 * dU[1]) + Rk2 * dU[2]);
            dtv[k] = s1 * ((Rk0 * dV[0] + Rk1 * dV[1]) + Rk2 * dV[2]);
        }
        as[0] += fs_dot(Rtu, dU);
        as[1] += fs_dot(Rtv, dV);
        // quaternion: t_u = (1 - f a1, f a2, f a3), t_v = (f b1, 1 - f b2, f b3), f = 2 / |q|^2
        const double w = quats[4 * i], x = quats[4 * i + 1], y = quats[4 * i + 2], z = quats[4 * i + 3];
        const double f = fr.f;
        const double a1 = y * y + z * z, a2 = x * y + w * z, a3 = x * z - w * y;
        const double b1 = x * y - w * z, b2 = x * x + z * z, b3 = y * z + w * x;
        const double sf = -dtu[0] * a1 + dtu[1] * a2 + dtu[2] * a3 + dtv[0] * b1 - dtv[1] * b2 + dtv[2] * b3;
        const double q[4] = {w, x, y, z};
        const double da1[4] = {0, 0, 2 * y, 2 * z}, da2[4] = {z, y, x, w}, da3[4] = {-y, z, -w, x};
        const double db1[4] = {-z, y, x, -w}, db2[4] = {0, 2 * x, 0, 2 * z}, db3[4] = {x, w, z, y};
        for (int k = 0; k < 4; ++k) {
            const double inner = -dtu[0] * da1[k] + dtu[1] * da2[k] + dtu[2] * da3[k] + dtv[0] * db1[k] -
                                 dtv[1] * db2[k] + dtv[2] * db3[k];
            aq[k] += -f * f * q[k] * sf + f * inner;
        }
    }
    for (int k = 0; k < 3; ++k) gm[3 * i + k] += (float)am[k];
    gs[2 * i] += (float)as[0];
    gs[2 * i + 1] += (float)as[1];
    for (int k = 0; k < 4; ++k) gq[4 * i + k] += (float)aq[k];
    go[i] += (float)ao;
}

// ---------------------------------------------------------------------------
// Top-K backward.  The selection pass of the split forward recomputes every
// pixel's (row slot, weight) list and every block's row list; then one
// workgroup per 8x8 block:
//   1. D = g . c for every (pixel, contributor): feature rows are staged in
//      registers, TPP threads per row slot, over the slot's pixels; the same
//      pass sums w g, flushed once per (block, row) to dL/dc;
//   2. per pixel (LDS only) the forward's transmittance chain (double
//      precision, same order), the suffix sums S = sum_{l > m} w_l D_l and
//      dL/dalpha;
//   3. the chain to dL/dL and dL/do, a thread per pair of the slot, summed over
//      the slot's threads and flushed once per (block, slot).
// ---------------------------------------------------------------------------
constexpr int kGradThreads = 256;
constexpr int kGradMaxK = 16;
static_assert(kGradMaxK <= FS_TOPK_COMPACT_K, "the gradient pass reads compact lists");

template <typename FT, int TPP, int CPT>
__global__ void __launch_bounds__(kGradThreads)
topk_grad_kernel(const FsRecord* __restrict__ records, const uint2* __restrict__ pairs,
                 const int32_t* __restrict__ counts, const uint32_t* __restrict__ rows,
                 const uint32_t* __restrict__ nrows, const FT* __restrict__ feats, int C, int K, int64_t n,
                 const fs_camera* __restrict__ cams, int num_views, int S, int64_t nblocks, fs_opts o,
                 const float* __restrict__ grad_feat, float* __restrict__ grad_records,
                 float* __restrict__ grad_feats) {
    constexpr int kGroups = kGradThreads / TPP;   // row slots handled at once
    constexpr int kPairs = 64 * kGradMaxK;
    __shared__ uint2 s_pairs[kPairs];
    __shared__ float s_D[kPairs];    // g . c, then dL/dalpha
    __shared__ float s_al[kPairs];   // alpha
    __shared__ float s_T[kPairs];    // transmittance before the contribution
    __shared__ int s_soff[kPairs + 1];       // per row slot: first entry of its pair list
    __shared__ int s_sfill[kPairs];          // per row slot: pairs, then the fill cursor
    __shared__ uint16_t s_list[kPairs];      // pair indices p * K + j grouped by row slot
    __shared__ int s_cnt[64];
    __shared__ int s_off[64];                // first pair of each pixel's compact list
    __shared__ int s_wave[kGradThreads / 64];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t block = xcd_remap_chunked(blockIdx.x, nblocks, block_row_chunk(cams, S));
    const BlockPos bp = locate_block(block, S, 8, cams, num_views);
    if (!bp.valid) return;           // uniform
    const uint32_t R = nrows[block] & 0xffffu;   // rows (the high half counts the listed pairs)
    if (R == 0) return;              // no pixel of the block blended anything
    const fs_camera& cam = cams[bp.view];
    const int q = tid % TPP, grp = tid / TPP;
    const uint32_t* __restrict__ rowlist = rows + block * 64 * (int64_t)K;
    const int npairs = 64 * K;
    for (int t = tid; t < npairs; t += kGradThreads) s_sfill[t] = 0;
    if (tid < 64) {
        // counts, and the offsets of the pixels' lists in the block's compact
        // list area (the selection writes them back to back)
        const int px = bp.x0 + (tid & 7), py = bp.y0 + (tid >> 3);
        const int c = (px < cam.width && py < cam.height) ? counts[cam.pixel_offset + (int64_t)py * cam.width + px] : 0;
        const int incl = __ockl_wfscan_add_i32(c, true);
        s_cnt[tid] = c;
        s_off[tid] = incl - c;
    }
    __syncthreads();
    // pair j of pixel p at LDS p * K + j
    for (int t = tid; t < npairs; t += kGradThreads) {
        const int p = t / K, j = t - p * K;
        if (j < s_cnt[p]) s_pairs[t] = pairs[block * 64 * (int64_t)K + s_off[p] + j];
    }
    __syncthreads();
    // 1a. pairs grouped by row slot (counting sort in LDS)
    for (int t = tid; t < npairs; t += kGradThreads)
        if (t % K < s_cnt[t / K]) atomicAdd(&s_sfill[s_pairs[t].x], 1);
    __syncthreads();
    {
        constexpr int kPer = (kPairs + kGradThreads - 1) / kGradThreads;
        const int b0 = tid * kPer;
        int c[kPer];
        int sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            c[i] = b0 + i < (int)R ? s_sfill[b0 + i] : 0;
            sum += c[i];
        }
        const int incl = __ockl_wfscan_add_i32(sum, true);
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        int off = incl - sum;
        for (int w = 0; w < wave; ++w) off += s_wave[w];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (b0 + i < (int)R) {
                s_soff[b0 + i] = off;
                s_sfill[b0 + i] = 0;
            }
            off += c[i];
        }
        if (tid == kGradThreads - 1) s_soff[R] = off;
    }
    __syncthreads();
    for (int t = tid; t < npairs; t += kGradThreads)
        if (t % K < s_cnt[t / K]) {
            const uint32_t slot = s_pairs[t].x;
            s_list[s_soff[slot] + atomicAdd(&s_sfill[slot], 1)] = (uint16_t)t;
        }
    __syncthreads();
    // 1b. slot-major: a group of TPP threads owns a row slot, thread q the
    //     channels q, q + TPP, ...; it reads the feature row once and, over the
    //     slot's pixels, forms D = g . c (lane exchanges inside the group) and
    //     dL/dc = sum w g in registers, flushed once per (block, slot).  What
    //     bounds it is the latency of the upstream gradient's rows, so kAhead
    //     pixels' rows are in flight together, and the flush: the group's
    //     atomics to a row are contiguous (with four consecutive channels per
    //     thread each atomic instruction touched every line of the row, and one
    //     pixel's row was waited for at a time: 399 us for the 200k-surfel,
    //     640x480, C = 128 gradients against 235, and 166 with pass 3 below).
    constexpr int kAhead = 4;
    for (uint32_t s0 = 0; s0 < R; s0 += kGroups) {
        const uint32_t slot = s0 + (uint32_t)grp;
        if (slot >= R) break;   // uniform inside the group
        const uint32_t sidx = rowlist[slot];
        float f[CPT], acc[CPT];
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            acc[i] = 0.f;
            f[i] = q + i * TPP < C ? to_f32(feats[(int64_t)sidx * C + q + i * TPP]) : 0.f;
        }
        const int a = s_soff[slot], b = s_soff[slot + 1];
        // alpha of the slot's pairs (the forward's float value), one per thread
        {
            const FsRecord& r = records[(int64_t)bp.view * n + sidx];
            for (int i = a + q; i < b; i += TPP) {
                const int t = s_list[i], p = t / K;
                const FsResp rs = fs_response(r, (double)(bp.x0 + (p & 7) - r.ax), (double)(bp.y0 + (p >> 3) - r.ay));
                const float Gs = __builtin_amdgcn_exp2f(-0.72134752044448170f * (float)rs.d2);
                s_al[t] = fminf(o.alpha_max, r.o * Gs);
            }
        }
        for (int i0 = a; i0 < b; i0 += kAhead) {
            int tt[kAhead];
            float g[kAhead][CPT];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const bool on = i0 + u < b;
                tt[u] = s_list[on ? i0 + u : i0];
                const int p = tt[u] / K;
                const float* __restrict__ src =
                    grad_feat + (cam.pixel_offset + (int64_t)(bp.y0 + (p >> 3)) * cam.width + bp.x0 + (p & 7)) * C + q;
#pragma unroll
                for (int i = 0; i < CPT; ++i) g[u][i] = on && q + i * TPP < C ? src[i * TPP] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (i0 + u >= b) break;
                const float w = __uint_as_float(s_pairs[tt[u]].y);
                float part = 0.f;
#pragma unroll
                for (int i = 0; i < CPT; ++i) {
                    part = fmaf(g[u][i], f[i], part);
                    acc[i] = fmaf(w, g[u][i], acc[i]);
                }
#pragma unroll
                for (int d = 1; d < TPP; d <<= 1) part += __uint_as_float(lane_xor32(__float_as_uint(part), d));
                if (q == 0) s_D[tt[u]] = part;
            }
        }
        float* __restrict__ dst = grad_feats + (int64_t)sidx * C + q;
#pragma unroll
        for (int i = 0; i < CPT; ++i)
            if (q + i * TPP < C) atomicAdd(dst + i * TPP, acc[i]);
    }
    __syncthreads();
    // 2. per pixel, from LDS only: the transmittance before every contribution
    //    (the forward's double-precision product), then, back to front, the
    //    suffix sums and dL/dalpha, left in the place of D
    if (tid < 64) {
        const int c = s_cnt[tid], t0 = tid * K;
        double T = 1.0;
        for (int j = 0; j < c; ++j) {
            s_T[t0 + j] = (float)T;
            T = T * (1.0 - (double)s_al[t0 + j]);
        }
        float suffix = 0.f;
        for (int j = c - 1; j >= 0; --j) {
            const float D = s_D[t0 + j];
            s_D[t0 + j] = s_T[t0 + j] * D - suffix / (1.f - s_al[t0 + j]);
            suffix += __uint_as_float(s_pairs[t0 + j].y) * D;
        }
    }
    __syncthreads();
    // 3. the chain to dL/dL and dL/do, slot-major again: a thread per pair, sums
    //    over the group, one flush per (block, slot) (a thread per pair of the
    //    block with LDS float atomics per slot took 130 of the kernel's 235 us
    //    with the other passes in their present form)
    for (uint32_t s0 = 0; s0 < R; s0 += kGroups) {
        const uint32_t slot = s0 + (uint32_t)grp;
        if (slot >= R) break;   // uniform inside the group
        const int64_t rid = (int64_t)bp.view * n + rowlist[slot];
        const FsRecord& r = records[rid];
        float sum[10];
#pragma unroll
        for (int k = 0; k < 10; ++k) sum[k] = 0.f;
        const int b = s_soff[slot + 1];
        for (int i = s_soff[slot] + q; i < b; i += TPP) {
            const int t = s_list[i], p = t / K;
            const double ddx = (double)(bp.x0 + (p & 7) - r.ax), ddy = (double)(bp.y0 + (p >> 3) - r.ay);
            const FsResp rs = fs_response(r, ddx, ddy);
            const float Gs = __builtin_amdgcn_exp2f(-0.72134752044448170f * (float)rs.d2);
            if (r.o * Gs > o.alpha_max) continue;   // clamped: no gradient
            float gg[10];
            blend_chain(r, rs, ddx, ddy, Gs, s_D[t], gg);
#pragma unroll
            for (int k = 0; k < 10; ++k) sum[k] += gg[k];
        }
#pragma unroll
        for (int d = 1; d < TPP; d <<= 1)
#pragma unroll
            for (int k = 0; k < 10; ++k) sum[k] += __uint_as_float(lane_xor32(__float_as_uint(sum[k]), d));
        float v = 0.f;   // component q of the sums
#pragma unroll
        for (int k = 0; k < 10; ++k) v = q == k ? sum[k] : v;
        if (v != 0.f) atomicAdd(&grad_records[rid * kGradFloats + q], v);
    }
}

template <typename FT>
hipError_t launch_topk_grad(const FsRecord* records, const void* feats, int C, int64_t n, const fs_camera* cams,
                            int num_views, int64_t nblocks, const fs_opts& o, const float* grad_feat,
                            float* grad_records, float* grad_feats, const FsWorkspace& ws, hipStream_t s) {
    const FT* f = static_cast<const FT*>(feats);
#define FS_GRAD(TPP, CPT)                                                                                        \
    hipLaunchKernelGGL((topk_grad_kernel<FT, TPP, CPT>), dim3((unsigned)nblocks), dim3(kGradThreads), 0, s,        \
                       records, ws.topk_pairs, ws.topk_counts, ws.topk_rows, ws.topk_nrows, f, C, o.topk, n, cams,  \
                       num_views, o.tile, nblocks, o, grad_feat, grad_records, grad_feats)
    // 16 threads per row slot while a thread's channels stay few: the sums then
    // need no exchange beyond a 16-lane row
    if (C <= 16) FS_GRAD(16, 1);
    else if (C <= 32) FS_GRAD(16, 2);
    else if (C <= 48) FS_GRAD(16, 3);
    else if (C <= 64) FS_GRAD(16, 4);
    else if (C <= 128) FS_GRAD(16, 8);
    else if (C <= 256) FS_GRAD(32, 8);
    else FS_GRAD(64, 8);
#undef FS_GRAD
    return hipGetLastError();
}

template <int CPT, typename FT>
hipError_t launch_bwd(const FsRecord* records, const uint32_t* vals, const uint32_t* ranges, const void* feats,
                      int C, int64_t n, const fs_camera* cams, int num_views, int64_t total_tiles, const fs_opts& o,
                      const float* out_T, const int32_t* out_last, const float* grad_feat, float* grad_records,
                      float* grad_feats, hipStream_t s) {
    const int sb = o.tile / 8;
    const int64_t blocks = total_tiles * sb * sb;
    if (blocks >= (int64_t(1) << 32)) return hipErrorInvalidValue;
    const auto kern = sb > 1 ? render_bwd_kernel<CPT, FT, true> : render_bwd_kernel<CPT, FT, false>;
    const int64_t most = int64_t(1) << 23, row = blocks < most ? blocks : most;
    hipLaunchKernelGGL(kern, dim3((unsigned)row, 2, (unsigned)((blocks + row - 1) / row)), dim3(kBwdThreads), 0, s,
                       records, vals, ranges,
                       static_cast<const FT*>(feats), C, n, n * num_views, cams, num_views, o.tile, blocks, o, out_T,
                       out_last, grad_feat, grad_records, grad_feats);
    return hipGetLastError();
}

template <typename FT>
hipError_t launch_bwd_channels(const FsRecord* records, const uint32_t* vals, const uint32_t* ranges,
                               const void* feats, int C, int64_t n, const fs_camera* cams, int num_views,
                               int64_t total_tiles, const fs_opts& o, const float* out_T, const int32_t* out_last,
                               const float* grad_feat, float* grad_records, float* grad_feats, hipStream_t s) {
#define FS_BWD(CPT)                                                                                             \
    return launch_bwd<CPT, FT>(records, vals, ranges, feats, C, n, cams, num_views, total_tiles, o, out_T, out_last, \
                               grad_feat, grad_records, grad_feats, s)
    // channels per thread of a 16-thread group: the row is padded to 16 CPT
    if (C <= 16) FS_BWD(1);
    if (C <= 32) FS_BWD(2);
    if (C <= 48) FS_BWD(3);
    if (C <= 64) FS_BWD(4);
    if (C <= 128) FS_BWD(8);
#undef FS_BWD
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t fs_launch_render_backward(const float* means, const float* scales, const float* quats,
                                     const float* opacity, const FsRecord* records, const uint32_t* vals,
                                     const uint32_t* ranges, const void* feats, int C, int64_t n,
                                     const fs_camera* cams, int num_views, int64_t total_tiles, const fs_opts& o,
                                     const float* out_T, const int32_t* out_n, const int32_t* out_last,
                                     const float* grad_feat, float* grad_records, float* grad_means,
                                     float* grad_scales, float* grad_quats, float* grad_opacity, float* grad_feats,
                                     const FsWorkspace& ws, hipStream_t s) {
    (void)out_n;
    const int64_t nrec = n * num_views * kGradFloats;
    {
        unsigned blocks = (unsigned)((nrec + 255) / 256);
        blocks = blocks < 1 ? 1 : (blocks > 8192 ? 8192 : blocks);
        hipLaunchKernelGGL(zero_f32_kernel, dim3(blocks), dim3(256), 0, s, grad_records, nrec);
    }
    hipError_t e;
    const bool bf16 = o.feat_dtype == FS_FEAT_BF16;
    const int ve = bf16 ? 8 : 4;
    const int sb = o.tile / 8;
    const int64_t nblocks = total_tiles * sb * sb;
    if (o.topk > 0 && o.topk <= kGradMaxK && C % ve == 0 && C / ve <= 64 && ws.topk_pairs != nullptr &&
        ws.topk_counts != nullptr && nblocks < (int64_t(1) << 31)) {
        // recompute the selection, then the per-block gradient pass
        e = fs_launch_topk_select(records, nullptr, vals, ranges, n, cams, num_views, total_tiles, o, nullptr,
                                  ws.topk_counts, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, ws, s);
        if (e != hipSuccess) return e;
        e = bf16 ? launch_topk_grad<uint16_t>(records, feats, C, n, cams, num_views, nblocks, o, grad_feat,
                                              grad_records, grad_feats, ws, s)
                 : launch_topk_grad<float>(records, feats, C, n, cams, num_views, nblocks, o, grad_feat, grad_records,
                                           grad_feats, ws, s);
    } else {
        e = bf16 ? launch_bwd_channels<uint16_t>(records, vals, ranges, feats, C, n, cams, num_views, total_tiles, o,
                                                 out_T, out_last, grad_feat, grad_records, grad_feats, s)
                 : launch_bwd_channels<float>(records, vals, ranges, feats, C, n, cams, num_views, total_tiles, o, out_T,
                                              out_last, grad_feat, grad_records, grad_feats, s);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(preprocess_bwd_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, means, scales,
                       quats, opacity, n, cams, num_views, o, grad_records, grad_means, grad_scales, grad_quats,
                       grad_opacity);
    return hipGetLastError();
}
