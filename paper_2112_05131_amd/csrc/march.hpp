// march.hpp -- device helpers shared by the render kernels, and the
// sample-parallel march of rays in ray order.
#pragma once

#include <cmath>

#include "plx_internal.hpp"

namespace plx {

constexpr int kWave = 64;
constexpr float kSkipMargin = 0.05f;  // in steps

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Number of lanes below this one in the lane mask m.
__device__ __forceinline__ int lanes_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Orders this wave's LDS accesses before and after the call (the waves of a
// workgroup that use it share no LDS, so no barrier is needed).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The optional sparsity (Cauchy) and beta priors of Sec. 3.7, as the gradient
// kernels see them.
struct Priors {
    float lambda_s;    // Cauchy weight (0 = off)
    float lambda_b;    // beta weight (0 = off)
    float eps;         // beta epsilon
    double *loss;      // [2] (L_s, L_b) ADDED, or NULL
};

// Beta prior of one ray from its optical depth tau (FP64; 1 - T = -expm1(-tau)
// stays accurate for a nearly empty ray): returns dL_b/dsigma_k / delta_k =
// -T dL_b/dT, the factor of each of its samples' density gradient, and adds
// the ray's L_b to *loss.
__device__ inline float beta_factor(const Priors &p, double tau, double *loss) {
    const double T = exp(-tau), omT = -expm1(-tau), e = (double)p.eps;
    *loss += (double)p.lambda_b * (log(e + T) + log(e + omT));
    return (float)(-T * (double)p.lambda_b * (1.0 / (e + T) - 1.0 / (e + omT)));
}

// Cauchy prior at a sample with pre-activation density s > 0: the density
// gradient lambda_s 4 s / (1 + 2 s^2); log(1 + 2 s^2) goes to *ls.
__device__ __forceinline__ float cauchy_grad(const Priors &p, float s, float *ls) {
    if (p.lambda_s == 0.0f || !(s > 0.0f)) return 0.0f;
    *ls += log1pf(2.0f * s * s);
    return 4.0f * (p.lambda_s * s) / (1.0f + 2.0f * s * s);
}

// Adds a wave's prior losses to p.loss (one atomic per wave and term; the
// per-lane Cauchy sums are FP32, the wave sum FP64).
__device__ inline void add_prior_loss(const Priors &p, float ls_lane, double lb) {
    if (!p.loss) return;
    double ls = (double)ls_lane;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        ls += __shfl_xor(ls, m);
        lb += __shfl_xor(lb, m);
    }
    if ((threadIdx.x & 63) == 0) {
        if (ls != 0.0) unsafeAtomicAdd(p.loss, (double)p.lambda_s * ls);
        if (lb != 0.0) unsafeAtomicAdd(p.loss + 1, lb);
    }
}

// Background colour of a ray: its own when the call gives one per ray.
__device__ __forceinline__ void ray_background(const float *bg_rgb, const float bg[3], int64_t ray,
                                               float out[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) out[c] = bg_rgb ? bg_rgb[3 * ray + c] : bg[c];
}

__device__ __forceinline__ int64_t brick_id(const GridDev &g, const int b[3]) {
    return ((int64_t)b[0] * g.by + b[1]) * g.bz + b[2];
}

// Number of samples before sample k (at t = t_near + k*step), back along the
// ray, that certainly stay inside the box of bricks within R of brick b, where
// sample k lies: the box's entry parameter along the ray, less a margin of 5%
// of a step.
__device__ __forceinline__ int samples_behind(const GridDev &g, const RayGeom &r, int k, const int b[3], int R) {
#pragma clang fp contract(off)
    const int nb[3] = {g.bx, g.by, g.bz};
    const float t = r.t_near + (float)k * g.step;
    float t_edge = -__builtin_inff();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float dg = r.dg[a];
        if (dg == 0.0f) continue;
        // box faces on the grid boundary are never crossed by a sample
        const bool up = dg < 0.0f;
        const int bf = up ? b[a] + R : b[a] - R;
        if (up ? bf >= nb[a] - 1 : bf <= 0) continue;
        const float face = (float)((up ? bf + 1 : bf) * PLX_BRICK);
        t_edge = fmaxf(t_edge, (face - r.og[a]) / dg);
    }
    float q = (t - t_edge) / g.step - kSkipMargin;
    q = q < (float)kMaxSamples ? q : (float)kMaxSamples;
    return q > 0.0f ? (int)q : 0;
}

__device__ inline void sh_basis_all(const float d[3], float y[9]) {
#pragma unroll
    for (int l = 0; l < 9; ++l) y[l] = sh_basis_at(l, d[0], d[1], d[2]);
}

// ------------------------------------------------------------ sample-parallel march
//
// One wave marches R = 64 / P rays, P lanes each.  A round tests the next
// P*M samples of every ray against the cell bitmap (M consecutive ones per
// lane), packs the occupied ones of all the wave's rays into a list in LDS
// (position in the cell, cell), evaluates the list with lane groups, and
// composes: each lane its own samples, then a scan over the ray's lanes.
//
// A group of 8 lanes (FP32 records) or 4 lanes (16-bit records) takes one
// sample.  Lane j of the group reads the j-th 16 bytes of the record of each
// of the 8 corners, so a corner costs the vector cache one line instead of
// the 4 to 8 of a lane that reads whole records, interpolates its slots by
// the trilinear weights, multiplies them with its slots of the ray's SH basis
// and sums over the group.
//
// What bounds a lane-per-ray march is its serial chain (about 3 to 16 us a
// sample: index entries, then records, one sample after the other, a wave as
// long as the longest of its 64 rays); here the loads of up to 64 M samples
// are in flight together.

// Lanes that read one record.
template <int DT> struct Group {
    static constexpr int kLanes = DT == PLX_F32 ? 8 : 4;
    static constexpr int kSamples = kWave / kLanes;  // samples a wave evaluates at once
};

// A wave's part of LDS.
template <int P, int M> struct MarchLds {
    static constexpr int kRays = kWave / P;
    static constexpr int kEntries = kWave * M;
    float4 pos[kEntries];   // f0 f1 f2, ray slot; then the sample's density and projected colour
    int64_t cell[kEntries]; // storage id of the cell's lower corner
    float y[kRays][PLX_REC_SLOTS];  // SH basis of each ray at the record's slots (0 in unused ones)
};

// x + the value of the lane that DPP control CTRL names (all lanes active).
template <int CTRL> __device__ __forceinline__ float dpp_add(float x) {
    const int o = __builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, false);
    return x + __int_as_float(o);
}
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i of 8 <- lane 7 - i

// Fills a ray's basis row; called by the ray's P >= 4 lanes.
template <int P, int M>
__device__ __forceinline__ void march_basis(MarchLds<P, M> &sh, const float d[3]) {
    static_assert(P >= 4, "a lane per channel and one for the unused slots");
    const int part = lane_id() % P;
    float *row = sh.y[lane_id() / P];
    float y[9];
    sh_basis_all(d, y);
    if (part < 3) {
#pragma unroll
        for (int l = 0; l < 9; ++l) row[9 * part + l] = y[l];
    } else if (part == 3) {
#pragma unroll
        for (int s = PLX_NSH; s < PLX_REC_SLOTS; ++s) row[s] = 0.0f;
    }
}

// Buffer resource over n bytes at p: loads at a 32-bit offset, which return 0
// outside it.  A NULL id (-1) makes an offset in the last record below 4 GiB,
// past every table that the resource describes, so a NULL corner reads zeros
// without a test, and an address costs one instruction.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)n, 0x00020000);
}
__device__ __forceinline__ uint4 load_piece(__amdgpu_buffer_rsrc_t rsrc, uint32_t at) {
    const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 0, 0);
    return make_uint4(t[0], t[1], t[2], t[3]);
}
__device__ __forceinline__ void load_pair(__amdgpu_buffer_rsrc_t rsrc, uint32_t at, int uniform_offset,
                                          int out[2]) {
    const auto t = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)at, uniform_offset, 0);
    out[0] = (int)t[0];
    out[1] = (int)t[1];
}

// What a NULL corner reads in tables beyond 32-bit offsets.
static __device__ const uint4 zero_record[PLX_REC_SLOTS / 4] = {};

// A ray's reciprocal direction, for skipping.
struct RaySkip {
    float inv[3];
    float inv_step;
};

__device__ __forceinline__ RaySkip ray_skip(const GridDev &g, const RayGeom &r) {
    RaySkip s;
#pragma unroll
    for (int a = 0; a < 3; ++a) s.inv[a] = 1.0f / r.dg[a];
    s.inv_step = 1.0f / g.step;
    return s;
}

// Number of further samples after sample k, as samples_behind before it, with
// products by reciprocals for the quotients: the margin also covers the
// rounding of the exit parameter (a few ulps of t_edge, in steps).  The walks
// that count and emit a ray's segments must cut the same ones, so this runs
// without FMA contraction like the sample recipe: what the compiler would
// fuse may differ from kernel to kernel.
__device__ __forceinline__ int skip_box(const GridDev &g, const RayGeom &r, const RaySkip &q, int k,
                                        const int b[3], int R) {
#pragma clang fp contract(off)
    const int nb[3] = {g.bx, g.by, g.bz};
    const float t = r.t_near + (float)k * g.step;
    float t_edge = __builtin_inff();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool up = r.dg[a] > 0.0f;
        const int bf = up ? b[a] + R : b[a] - R;
        const float tf = ((float)((up ? bf + 1 : bf) * PLX_BRICK) - r.og[a]) * q.inv[a];
        // box faces on the grid boundary are never crossed by a sample
        const bool open = (up ? bf < nb[a] - 1 : bf > 0) && r.dg[a] != 0.0f;
        t_edge = fminf(t_edge, open ? tf : __builtin_inff());
    }
    float m = (t_edge - t) * q.inv_step - kSkipMargin - 6e-7f * (t_edge * q.inv_step);
    m = m < (float)kMaxSamples ? m : (float)kMaxSamples;  // also for an open box (inf - inf)
    return m > 0.0f ? (int)m : 0;
}

// Evaluates entries of the list in batches of Group::kSamples: pos becomes
// the sample's interpolated density and projected colour (x: density).  The
// ids of the next batch are loaded while a batch is summed, so that a batch
// waits for one load, not two that depend on each other.
template <int DT, int P, int M> struct Evaluator {
    static constexpr int G = Group<DT>::kLanes, NS = Group<DT>::kSamples;
    const GridDev &g;
    MarchLds<P, M> &sh;
    const int total;
    const int j = lane_id() % G, grp = lane_id() / G;
    const __amdgpu_buffer_rsrc_t index_rsrc = buffer_of(g.index, g.index_bytes);
    const __amdgpu_buffer_rsrc_t data_rsrc = buffer_of(g.data, g.data_bytes);

    // Positions and corner ids of the batch at b, two neighbours along z per
    // load; lanes past the end repeat the last entry.
    __device__ __forceinline__ void ids(float4 &ps, int id[8], int b) const {
        const int e = min(b + grp, total - 1);
        ps = sh.pos[e];
        const int64_t cell = sh.cell[e];
        const int64_t sy = g.nz, sx = (int64_t)g.ny * g.nz;
        if (g.data_bytes != 0u) {
            const uint32_t at = (uint32_t)cell * 4u;
#pragma unroll
            for (int c = 0; c < 8; c += 2)
                load_pair(index_rsrc, at, ((c & 4) ? (int)sx * 4 : 0) + ((c & 2) ? (int)sy * 4 : 0), id + c);
        } else {
            const int32_t *ip = g.index + cell;
#pragma unroll
            for (int c = 0; c < 8; c += 2)
                __builtin_memcpy(id + c, ip + ((c & 4) ? sx : 0) + ((c & 2) ? sy : 0), 8);
        }
    }

    // The lane's piece of the corners' records.
    __device__ __forceinline__ void records(uint4 v[8], const int id[8]) const {
        if (g.data_bytes != 0u) {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                v[c] = load_piece(data_rsrc, (uint32_t)id[c] * (uint32_t)Rec<DT>::bytes + 16u * j);
        } else {
            const char *const zeros = reinterpret_cast<const char *>(zero_record);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const char *p = static_cast<const char *>(g.data) + (int64_t)id[c] * Rec<DT>::bytes;
                v[c] = *reinterpret_cast<const uint4 *>((id[c] >= 0 ? p : zeros) + 16 * j);
            }
        }
    }

    // Interpolates the lane's slots, projects them on the ray's basis and
    // sums over the group; the lane that holds the density writes.
    __device__ __forceinline__ void sum(const uint4 v[8], const float4 &ps, int b) const {
        const float wx[2] = {1.0f - ps.x, ps.x}, wy[2] = {1.0f - ps.y, ps.y}, wz[2] = {1.0f - ps.z, ps.z};
        float w[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) w[c] = wx[(c >> 2) & 1] * wy[(c >> 1) & 1] * wz[c & 1];
        const float *y = sh.y[__float_as_int(ps.w)];
        float r, gr, bl, sig = 0.0f;
        if constexpr (DT == PLX_F32) {
            float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                a[0] += w[c] * __uint_as_float(v[c].x);
                a[1] += w[c] * __uint_as_float(v[c].y);
                a[2] += w[c] * __uint_as_float(v[c].z);
                a[3] += w[c] * __uint_as_float(v[c].w);
            }
            sig = a[0];  // lane 7: slot 28
            const float4 yv = *reinterpret_cast<const float4 *>(y + 4 * j);
            const float p0 = j < 7 ? a[0] * yv.x : 0.0f, p1 = j < 7 ? a[1] * yv.y : 0.0f;
            const float p2 = j < 7 ? a[2] * yv.z : 0.0f;
            const float p3 = j < 6 ? a[3] * yv.w : 0.0f;  // slot 27 and up are unused
            // red: slots 0..8 (lanes 0, 1 and lane 2's first), green 9..17
            // (the rest of lane 2, lane 3, two of lane 4), blue 18..26
            const float p01 = p0 + p1, p23 = p2 + p3, all = p01 + p23;
            r = j < 2 ? all : (j == 2 ? p0 : 0.0f);
            gr = j == 3 ? all : (j == 2 ? p1 + p23 : (j == 4 ? p01 : 0.0f));
            bl = j > 4 ? all : (j == 4 ? p23 : 0.0f);
            r = dpp_add<kDppHalfMirror>(dpp_add<kDppXor2>(dpp_add<kDppXor1>(r)));
            gr = dpp_add<kDppHalfMirror>(dpp_add<kDppXor2>(dpp_add<kDppXor1>(gr)));
            bl = dpp_add<kDppHalfMirror>(dpp_add<kDppXor2>(dpp_add<kDppXor1>(bl)));
        } else {
            float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const uint32_t h[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a[2 * i] += w[c] * Rec16<DT>::h2f(h[i] & 0xffffu);
                    a[2 * i + 1] += w[c] * Rec16<DT>::h2f(h[i] >> 16);
                }
                sig += w[c] * __uint_as_float(v[c].z);  // lane 3: byte 56
            }
            const float4 ya = *reinterpret_cast<const float4 *>(y + 8 * j);
            const float4 yb = *reinterpret_cast<const float4 *>(y + 8 * j + 4);
            const float p0 = a[0] * ya.x, p1 = a[1] * ya.y, p2 = a[2] * ya.z;
            // lane 0: red 0..7; lane 1: red 8, green 9..15; lane 2: green 16, 17,
            // blue 18..23; lane 3: blue 24..26 (its other slots are no colour)
            const float p01 = p0 + p1;
            const float rest = j < 3 ? a[3] * ya.w + a[4] * yb.x + a[5] * yb.y + a[6] * yb.z + a[7] * yb.w : 0.0f;
            const float all = p01 + p2 + rest;
            r = j == 0 ? all : (j == 1 ? p0 : 0.0f);
            gr = j == 1 ? p1 + p2 + rest : (j == 2 ? p01 : 0.0f);
            bl = j == 3 ? all : (j == 2 ? p2 + rest : 0.0f);
            r = dpp_add<kDppXor2>(dpp_add<kDppXor1>(r));
            gr = dpp_add<kDppXor2>(dpp_add<kDppXor1>(gr));
            bl = dpp_add<kDppXor2>(dpp_add<kDppXor1>(bl));
        }
        // every lane of the batch has read its entry before this write
        if (j == G - 1 && b + grp < total) sh.pos[b + grp] = make_float4(sig, r, gr, bl);
    }

    // Called by the whole wave; total > 0.
    __device__ __forceinline__ void run() const {
        float4 ps;
        int id[8];
        ids(ps, id, 0);
        for (int b = 0; b < total; b += NS) {
            uint4 v[8];
            records(v, id);
            const float4 pc = ps;
            if (b + NS < total) ids(ps, id, b + NS);
            sum(v, pc, b);
        }
    }
};

// Marches the wave's rays front to back (Eq. (1)); lane L works on ray slot
// L / P, whose geometry r and sample count n all its P lanes hold (n = 0: no
// ray).  march_basis must have filled the basis rows.  Returns, in every lane
// of a ray, the colour before the background is added and the optical depth.
// rec(i, k, v) gets the i-th occupied sample of a ray (sample index k, values
// v) in the lane that composes it, when REC::kOn; the ray's number of occupied
// samples goes to *count.  With REC::kOpaque a sample adds at most kOpaque to
// tau, and what it has beyond that goes to *over.  Called by the whole wave.
struct NoRecord {
    static constexpr bool kOn = false, kOpaque = false;
    __device__ __forceinline__ void operator()(int, int, const float4 &) const {}
};

// Optical depth beyond which FP32 has no transmittance left (expf(-104) is 0).
// Depths summed from samples cut here give the same transmittances, and can be
// taken off the sum again sample by sample, which a sum that an infinite (or
// huge) one has gone into cannot: the reverse walk of a ray needs that.
constexpr float kOpaque = 256.0f;

template <int DT, int P, int M, class REC>
__device__ __forceinline__ void march_rays(const GridDev &g, MarchLds<P, M> &sh, const RayGeom &r, int n,
                                           float C[3], double &tau, const REC &rec, int *count = nullptr,
                                           double *over = nullptr) {
    static_assert(P * M <= 64 && (P & (P - 1)) == 0, "window");
    int n_occ = 0;
    const int part = lane_id() % P, slot = lane_id() / P;
    C[0] = C[1] = C[2] = 0.0f;
    tau = 0.0;
    const RaySkip rs = ray_skip(g, r);
    int k = 0;         // first sample of the ray's next window
    bool skip = true;  // k may lie in an empty brick
    for (;;) {
        // the next window of each ray that holds an occupied sample: empty
        // boxes of bricks are skipped, then windows tested
        unsigned mask = 0u;
        bool open = k < n;
        // the lane's samples of the last window it tested: one is kept for
        // the list (5000 rays of 256^3, P = 64: 62 us, kept 52), several are
        // placed again, which costs less than their registers (65,536 rays of
        // 256^3, FP16, P = 16, M = 4: 174 us, kept 194)
        constexpr bool kKeep = M == 1;
        float f[kKeep ? M : 1][3];
        int64_t cell[kKeep ? M : 1];
        while (__ballot(open) != 0) {
            bool s = open && skip;
            while (__ballot(s) != 0) {
                if (s) {
                    const Sample sm = sample_at(g, r, k);
                    const int b[3] = {sm.cell[0] >> 3, sm.cell[1] >> 3, sm.cell[2] >> 3};
                    const int D = g.bdist[brick_id(g, b)];
                    s = D > 0;
                    if (s) {
                        k += skip_box(g, r, rs, k, b, D - 1) + 1;
                        s = open = k < n;
                    }
                }
            }
            if (open) {
                uint32_t word[M];
                int bit[M];
                const int kp = k + part * M;
#pragma unroll
                for (int i = 0; i < M; ++i) {
                    const Sample sm = sample_at(g, r, min(kp + i, n - 1));
                    if constexpr (kKeep) {
#pragma unroll
                        for (int a = 0; a < 3; ++a) f[i][a] = sm.f[a];
                        cell[i] = cell_id(g, sm.cell);
                    }
                    const int64_t b = ((int64_t)(sm.cell[0] >> 3) * g.by + (sm.cell[1] >> 3)) * g.bz + (sm.cell[2] >> 3);
                    const int bb = ((sm.cell[0] & 7) << 6) | ((sm.cell[1] & 7) << 3) | (sm.cell[2] & 7);
                    word[i] = g.occ[b * 16 + (bb >> 5)];
                    bit[i] = bb & 31;
                }
#pragma unroll
                for (int i = 0; i < M; ++i)
                    if (kp + i < n) mask |= ((word[i] >> bit[i]) & 1u) << i;
                const uint64_t some = __ballot(mask != 0u) >> (slot * P);
                const bool found = P == 64 ? some != 0 : (some & ((1ull << (P & 63)) - 1ull)) != 0;
                k += P * M;
                skip = !found;
                open = !found && k < n;
            }
        }
        // pack: a lane's entries follow those of the lanes below it
        const int cnt = __popc(mask);
        int before = 0, total = 0;
#pragma unroll
        for (int b = 0; (1 << b) <= M; ++b) {
            const uint64_t plane = __ballot((cnt >> b) & 1);
            before += lanes_below(plane) << b;
            total += __popcll(plane) << b;
        }
        if (total == 0) break;  // no ray found another occupied sample
        const int kp = k - P * M + part * M;  // the lane's first sample of the window
        {
            int e = before;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                if ((mask >> i) & 1u) {
                    if constexpr (kKeep) {
                        sh.pos[e] = make_float4(f[i][0], f[i][1], f[i][2], __int_as_float(slot));
                        sh.cell[e] = cell[i];
                    } else {
                        const Sample sm = sample_at(g, r, kp + i);
                        sh.pos[e] = make_float4(sm.f[0], sm.f[1], sm.f[2], __int_as_float(slot));
                        sh.cell[e] = cell_id(g, sm.cell);
                    }
                    ++e;
                }
            }
        }
        wave_lds_fence();
        Evaluator<DT, P, M>{g, sh, total}.run();
        wave_lds_fence();
        // compose the lane's samples, then the ray's lanes
        double tl = 0.0;
        float c[3] = {0.f, 0.f, 0.f};
        int at = 0;  // the ray's number of the entry at `before`
        if constexpr (REC::kOn) {
            const int first = P == 64 ? 0 : __shfl(before, 0, P);
            at = n_occ + before - first;
            n_occ += (P == 64 ? total : __shfl(before + cnt, P - 1, P)) - first;
        }
        {
            int e = before;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                if ((mask >> i) & 1u) {
                    const float4 v = sh.pos[e];
                    if constexpr (REC::kOn) rec(at + (e - before), kp + i, v);
                    ++e;
                    const float sd = fmaxf(v.x, 0.0f) * sample_delta(g, r.t_near, r.t_far, kp + i);
                    const float wk = expf(-(float)tl) * (-expm1f(-sd));
                    c[0] += wk * fmaxf(v.y, 0.0f);
                    c[1] += wk * fmaxf(v.z, 0.0f);
                    c[2] += wk * fmaxf(v.w, 0.0f);
                    if constexpr (REC::kOpaque) {
                        const float cut = fminf(sd, kOpaque);
                        if (over && sd > cut) *over += (double)sd - (double)cut;
                        tl += (double)cut;
                    } else {
                        tl += (double)sd;
                    }
                }
            }
        }
        double incl = tl;
#pragma unroll
        for (int o = 1; o < P; o <<= 1) {
            const double y = __shfl_up(incl, o, P);
            if (part >= o) incl += y;
        }
        // depth of the ray's lanes before this one, taken from the scan and not
        // as incl - tl: that is NaN where tl is infinite, and loses the lanes
        // before a depth beyond 2^53 of theirs
        double excl = __shfl_up(incl, 1, P);
        if (part == 0) excl = 0.0;
        const float T0 = expf(-(float)(tau + excl));
#pragma unroll
        for (int a = 0; a < 3; ++a) C[a] += T0 * c[a];
        tau += __shfl(incl, P - 1, P);
        wave_lds_fence();  // the list is rewritten by the next round
    }
#pragma unroll
    for (int o = 1; o < P; o <<= 1) {
#pragma unroll
        for (int a = 0; a < 3; ++a) C[a] += __shfl_xor(C[a], o, P);
    }
    if constexpr (REC::kOn) {
        *count = n_occ;
        if (over) {
#pragma unroll
            for (int o = 1; o < P; o <<= 1) *over += __shfl_xor(*over, o, P);
        }
    }
}

// ------------------------------------------------------------ host helpers

inline int validate_rays(const float *o, const float *d, int64_t n, const char *fn) {
    if (n < 0) return fail(PLX_EINVAL, "%s: n_rays < 0", fn);
    if (n > ((int64_t)1 << 34)) return fail(PLX_EINVAL, "%s: n_rays too large", fn);
    if (n > 0 && (!o || !d)) return fail(PLX_EINVAL, "%s: rays are NULL", fn);
    return PLX_OK;
}

// Priors of a gradient call from its options (validated).
inline int priors_from(const plx_render_opts *opts, Priors &p, const char *fn) {
    p.lambda_s = opts->lambda_sparsity;
    p.lambda_b = opts->lambda_beta;
    p.eps = opts->beta_eps;
    p.loss = opts->reg_loss_sum;
    if (!std::isfinite(p.lambda_s) || !std::isfinite(p.lambda_b))
        return fail(PLX_EINVAL, "%s: prior weights must be finite", fn);
    if (p.lambda_b != 0.0f && !(p.eps > 0.0f && std::isfinite(p.eps)))
        return fail(PLX_EINVAL, "%s: beta_eps must be > 0 when lambda_beta != 0", fn);
    return PLX_OK;
}

// Records the caller's timing event i (when given) on the stream.
inline int mark_event(void **events, int i, hipStream_t s, const char *fn) {
    if (!events || !events[i]) return PLX_OK;
    PLX_CHECK_HIP(hipEventRecord(static_cast<hipEvent_t>(events[i]), s), fn);
    return PLX_OK;
}
// Events first..last-1.
inline int mark_events(void **events, int first, int last, hipStream_t s, const char *fn) {
    for (int i = first; i < last; ++i)
        if (int rc = mark_event(events, i, s, fn)) return rc;
    return PLX_OK;
}

}  // namespace plx
