// ray_order.hip -- rendering and its backward pass in ray order, without
// segment lists (Sec. 3.1-3.3, Eq. (1); supplement B.1) for gfx950.
//
// The forward pass marches the rays (march.hpp: several lanes per ray) and can
// record the occupied samples (sample index, density and projected colour,
// 20 bytes).  The backward pass gives every ray a wave and every recorded
// sample a lane:
//  1. suffix scans over the wave give each sample the optical depth and the
//     radiance collected after it, hence its gradients with respect to its
//     density and projected colour (Eq. (1));
//  2. a voxel is a corner of consecutive samples of the ray, and the first of
//     them owns it: its lane sums the weighted gradients of the run;
//  3. the sums go through a queue in LDS to the gradient records, 32 lanes
//     per voxel, lane s sending slot s: its channel's sum times the ray's SH
//     basis, one 128-byte line of FP32 atomics per voxel and ray.
// The chain of a ray is then its windows of 64 samples, not its samples, and
// nothing is binned, counted or read back.  What bounds the backward pass is
// the rate of atomic requests (about three voxels per sample, two 64-byte
// requests each, at about 20G requests a second); with many rays the segment
// kernels (render.hip), which send one line per voxel and brick, send fewer.
#include <algorithm>

#include "march.hpp"

namespace plx {
namespace {

enum { MODE_FWD = 0, MODE_BWD = 1, MODE_TRAIN = 2 };
// What a forward keeps of its samples: nothing; the first ones of each ray;
// these, while it also returns depths (an instance of its own, as the sum of
// what kOpaque cuts off costs registers).
enum { REC_NONE = 0, REC_SAMPLES = 1, REC_DEPTHS = 2 };

// Per-ray values that a forward call hands to its backward.
struct RayVals {
    float4 g;      // dL/dC
    double tau;    // optical depth, of samples cut at kOpaque
    double loss;   // the ray's share of the loss
    double cauchy, beta;  // and of the priors' (backward; written where their losses are wanted)
};

struct RayArgs {
    const float *rays_o;
    const float *rays_d;
    const float *target;    // TRAIN
    const float *grad_rgb;  // BWD
    const float *tau_in;    // BWD
    float *rgb_out;         // FWD, TRAIN (optional)
    float *tau_out;         // FWD (optional)
    float *grad;            // BWD, TRAIN
    uint8_t *touched;       // BWD, TRAIN
    double *loss_sum;       // TRAIN
    RayVals *vals;          // TRAIN; FWD and BWD of the calls with a ray workspace
    int *st_count;          // recorded samples: occupied samples of each ray
    int *st_kidx;           // [n_rays][st_cap] their sample indices
    float4 *st_vals;        // [n_rays][st_cap] pre-activation density and projected colour
    int st_cap;
    int64_t n_rays;
    float bg[3];
    float loss_scale;
    const float *bg_rgb;    // optional per-ray background colours [n_rays][3]
    float *grad_bg;         // BWD, TRAIN, optional: T_final dL/dC per ray [n_rays][3]
    Priors pri;
};

__device__ __forceinline__ void load_ray(const RayArgs &a, int64_t ray, float o[3], float d[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        o[i] = a.rays_o[3 * ray + i];
        d[i] = a.rays_d[3 * ray + i];
    }
}

// Records the first st_cap occupied samples of a ray.
struct Record {
    static constexpr bool kOn = true, kOpaque = true;
    int *kidx;
    float4 *vals;
    int cap;
    __device__ __forceinline__ void operator()(int i, int k, const float4 &v) const {
        if (i < cap) {
            kidx[i] = k;
            vals[i] = v;
        }
    }
};

// Marches the wave's 64 / P rays; `ray` is the lane's.  TRAIN also forms the
// loss and dL/dC = 2 loss_scale (C - target).
template <int DT, int P, int M, int MODE, int REC>
__device__ __forceinline__ void forward_rays(const GridDev &g, const RayArgs &a, MarchLds<P, M> &sh, int64_t ray) {
    const bool in = ray < a.n_rays;
    float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f};
    if (in) load_ray(a, ray, o, d);
    RayGeom r;
    const int n = in ? ray_setup(g, o, d, r) : 0;
    march_basis(sh, d);
    float C[3];
    double tau;
    double over = 0.0;  // what tau lacks of the optical depth
    if constexpr (REC != REC_NONE) {
        int count = 0;
        const int64_t base = in ? ray * a.st_cap : 0;
        const Record rec{a.st_kidx + base, a.st_vals + base, a.st_cap};
        march_rays<DT>(g, sh, r, n, C, tau, rec, &count, REC == REC_DEPTHS ? &over : nullptr);
        if (in && lane_id() % P == 0) a.st_count[ray] = count;
    } else {
        march_rays<DT>(g, sh, r, n, C, tau, NoRecord{});
    }
    if (!in || lane_id() % P != 0) return;
    const float T = expf(-(float)tau);
    float bgc[3];
    ray_background(a.bg_rgb, a.bg, ray, bgc);
    float gr[3] = {0.f, 0.f, 0.f};
    double l2 = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float Cc = C[c] + T * bgc[c];
        if (MODE == MODE_FWD || a.rgb_out) a.rgb_out[3 * ray + c] = Cc;
        if (MODE == MODE_TRAIN) {
            const float diff = Cc - a.target[3 * ray + c];
            gr[c] = 2.0f * a.loss_scale * diff;
            l2 += (double)(diff * diff);
        }
    }
    if (MODE == MODE_FWD) {
        if (a.tau_out) a.tau_out[ray] = (float)(tau + over);
        if (REC != REC_NONE && a.vals) a.vals[ray].tau = tau;
    } else {
        RayVals v = {};
        v.g = make_float4(gr[0], gr[1], gr[2], 0.0f);
        v.tau = tau;
        v.loss = (double)a.loss_scale * l2;
        a.vals[ray] = v;
        if (a.grad_bg) {
#pragma unroll
            for (int c = 0; c < 3; ++c) a.grad_bg[3 * ray + c] = T * gr[c];
        }
    }
}

// Forward march of 64 / P rays per wave (one wave per workgroup).  At 128
// registers the 16-lane instances that record keep 1 to 14 in scratch, those
// with 64 lanes none.
template <int DT, int P, int M, int MODE, int REC>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4)))
void rays_fwd_kernel(GridDev g, RayArgs a) {
    __shared__ MarchLds<P, M> sh;
    constexpr int R = kWave / P;
    for (int64_t r0 = (int64_t)blockIdx.x * R; r0 < a.n_rays; r0 += (int64_t)gridDim.x * R)
        forward_rays<DT, P, M, MODE, REC>(g, a, sh, r0 + lane_id() / P);
}

constexpr int kQueue = 256;  // voxels queued per wave

struct BwdLds {
    MarchLds<64, 1> m;        // evaluation of samples that were not recorded; the basis row
    float4 geo[kWave];        // position in the cell of each sample of the window
    float4 grad[kWave];       // its gradients: density, projected colour
    int cell[3][kWave];       // its cell
    int q_id[kQueue];         // queued voxels and their sums
    float4 q_v[kQueue];
};

// Sends the queued voxels' gradients to their records: lanes 0..31 take one
// entry and lanes 32..63 the next, lane L & 31 = record slot (0..26 SH, 28
// density, 29 marks the voxel touched); y: the lane's slot of the ray's basis
// (1 for the density).  The LDS reads are unconditional (positions past the
// end are clamped and discarded), so a round's reads overlap.
__device__ __forceinline__ void drain(BwdLds &sh, int count, float y, float *grad, uint8_t *touched) {
    wave_lds_fence();
    const int L = lane_id(), s = L & 31, half = L >> 5;
    const int ch = s < PLX_NSH ? 1 + s / 9 : 0;
    const bool writes = s < PLX_NSH || s == PLX_SLOT_SIGMA;
    float *gs = grad + s;
    constexpr int U = 8;
    for (int b = 0; b < count; b += 2 * U) {
        int id[U];
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = min(b + 2 * u + half, kQueue - 1);
            id[u] = sh.q_id[e];
            v[u] = reinterpret_cast<const float *>(sh.q_v)[4 * e + ch];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = b + 2 * u + half < count;
            const float val = ok && writes ? y * v[u] : 0.0f;
            if (val != 0.0f) unsafeAtomicAdd(gs + (int64_t)id[u] * PLX_REC_SLOTS, val);
            if (ok && s == PLX_SLOT_SIGMA + 1) touched[id[u]] = 1;
        }
    }
    wave_lds_fence();
}

// State of a ray's reverse walk, the same in every lane.
struct Reverse {
    double tau;   // optical depth after the current window
    float gR;     // g . (radiance collected after it) less the beta factor
    float g[3];   // dL/dC
};

// One window of the reverse walk: lane e < total holds the e-th of `total`
// consecutive occupied samples (index k, values v).  Gradients of the
// samples, sums per voxel, queue.
template <bool PRI>
__device__ __forceinline__ void window_bwd(const GridDev &g, const RayArgs &a, BwdLds &sh, const RayGeom &r,
                                           Reverse &st, int total, int k, const float4 &v, float y, int &queued,
                                           float &ls) {
    const int e = lane_id();
    const bool on = e < total;
    const Sample sm = sample_at(g, r, on ? k : 0);
    const float sd = on ? fmaxf(v.x, 0.0f) * sm.delta : 0.0f;
    // optical depth after the sample (the samples above it in the window
    // taken off the end), and before it
    double dsum = (double)(a.vals ? fminf(sd, kOpaque) : sd);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const double t = __shfl_down(dsum, o);
        if (e + o < kWave) dsum += t;
    }
    const double tau_before = fmax(st.tau - dsum, 0.0);
    double above = __shfl_down(dsum, 1);
    if (e == kWave - 1) above = 0.0;
    const double tau_after = fmax(st.tau - above, 0.0);
    const float T_after = expf(-(float)tau_after), T_before = expf(-(float)tau_before);
    const float wk = T_before * (-expm1f(-sd));
    const float gc = st.g[0] * fmaxf(v.y, 0.0f) + st.g[1] * fmaxf(v.z, 0.0f) + st.g[2] * fmaxf(v.w, 0.0f);
    float rsum = on ? wk * gc : 0.0f;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const float t = __shfl_down(rsum, o);
        if (e + o < kWave) rsum += t;
    }
    float r_above = __shfl_down(rsum, 1);
    if (e == kWave - 1) r_above = 0.0f;
    if (on) {
        const float gR = st.gR + r_above;
        const float cs = PRI ? cauchy_grad(a.pri, v.x, &ls) : 0.0f;
        sh.geo[e] = make_float4(sm.f[0], sm.f[1], sm.f[2], 0.0f);
        sh.grad[e] = make_float4(v.x > 0.0f ? sm.delta * (T_after * gc - gR) + cs : 0.0f,
                                 v.y > 0.0f ? wk * st.g[0] : 0.0f, v.z > 0.0f ? wk * st.g[1] : 0.0f,
                                 v.w > 0.0f ? wk * st.g[2] : 0.0f);
#pragma unroll
        for (int c = 0; c < 3; ++c) sh.cell[c][e] = sm.cell[c];
    }
    st.tau = fmax(st.tau - __shfl(dsum, 0), 0.0);
    st.gR += __shfl(rsum, 0);
    wave_lds_fence();

    // the corners that the sample before does not have: this sample owns
    // them (cells are monotone along a ray, so a voxel's samples are
    // consecutive; a run that a window cuts is sent in two parts)
    unsigned own = 0u;
    int id[8];
    if (on) {
        int rel[3] = {2, 2, 2};
        if (e > 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) rel[c] = sm.cell[c] - sh.cell[c][e - 1];
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int x = ((c >> 2) & 1) + rel[0], yy = ((c >> 1) & 1) + rel[1], z = (c & 1) + rel[2];
            if ((unsigned)x > 1u || (unsigned)yy > 1u || (unsigned)z > 1u) own |= 1u << c;
        }
        const int32_t *ip = g.index + cell_id(g, sm.cell);
        const int64_t sy = g.nz, sx = (int64_t)g.ny * g.nz;
#pragma unroll
        for (int c = 0; c < 8; c += 2)
            __builtin_memcpy(id + c, ip + ((c & 4) ? sx : 0) + ((c & 2) ? sy : 0), 8);
    }
    float4 acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    unsigned alive = own;
    for (int i = e; alive != 0u && i < total; ++i) {
        const int rx = sh.cell[0][i] - sm.cell[0], ry = sh.cell[1][i] - sm.cell[1], rz = sh.cell[2][i] - sm.cell[2];
        const float4 f = sh.geo[i], gr = sh.grad[i];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            // corner c of the owner's cell is corner c - rel of sample i's
            const int x = ((c >> 2) & 1) - rx, yy = ((c >> 1) & 1) - ry, z = (c & 1) - rz;
            if ((unsigned)x > 1u || (unsigned)yy > 1u || (unsigned)z > 1u) alive &= ~(1u << c);
            if ((alive >> c) & 1u) {
                const float w = (x ? f.x : 1.0f - f.x) * (yy ? f.y : 1.0f - f.y) * (z ? f.z : 1.0f - f.z);
                acc[c].x += w * gr.x;
                acc[c].y += w * gr.y;
                acc[c].z += w * gr.z;
                acc[c].w += w * gr.w;
            }
        }
    }
    // queue them, one corner of all lanes at a time
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const bool has = on && ((own >> c) & 1u) && id[c] >= 0;
        const uint64_t m = __ballot(has);
        if (m == 0) continue;
        if (queued + kWave > kQueue) {
            drain(sh, queued, y, a.grad, a.touched);
            queued = 0;
        }
        if (has) {
            const int q = queued + lanes_below(m);
            sh.q_id[q] = id[c];
            sh.q_v[q] = acc[c];
        }
        queued += __popcll(m);
    }
    wave_lds_fence();  // geo, grad and cell are rewritten by the next window
}

// Backward pass of one ray per wave: the recorded samples from the last to the
// first, after those beyond the record's capacity, which are found and
// evaluated again.
template <int DT, int MODE, bool PRI>
__device__ __forceinline__ void backward_ray(const GridDev &g, const RayArgs &a, BwdLds &sh, int64_t ray,
                                             double prior_sum[2]) {
    const int L = lane_id();
    if (MODE == MODE_TRAIN && ray % kWave == 0) {
        // the losses of 64 rays with one atomic
        const int64_t i = ray + L;
        double l2 = i < a.n_rays ? a.vals[i].loss : 0.0;
#pragma unroll
        for (int m = kWave / 2; m >= 1; m >>= 1) l2 += __shfl_xor(l2, m);
        if (L == 0 && l2 != 0.0) unsafeAtomicAdd(a.loss_sum, l2);
    }
    Reverse st;
    float gw = 0.0f;
    double lb = 0.0;
    if (MODE == MODE_TRAIN) {
        const RayVals v = a.vals[ray];
        st.g[0] = v.g.x;
        st.g[1] = v.g.y;
        st.g[2] = v.g.z;
        st.tau = v.tau;
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) st.g[c] = a.grad_rgb[3 * ray + c];
        st.tau = a.vals ? a.vals[ray].tau : (double)a.tau_in[ray];
    }
    if (PRI && a.pri.lambda_b != 0.0f) gw = beta_factor(a.pri, st.tau, &lb);
    const float T = expf(-(float)st.tau);
    float bgc[3];
    ray_background(a.bg_rgb, a.bg, ray, bgc);
    if (MODE == MODE_BWD && a.grad_bg && L < 3) a.grad_bg[3 * ray + L] = T * st.g[L];
    // g . R_k less the beta factor: dC/dsigma_k's delta (T_{k+1} g.c_k - g.R_k)
    // and the beta term's delta gw share one running sum
    st.gR = T * (st.g[0] * bgc[0] + st.g[1] * bgc[1] + st.g[2] * bgc[2]) - gw;

    float ls = 0.0f;
    const int cnt = a.st_count[ray];
    if (cnt > 0) {
        float o[3], d[3];
        load_ray(a, ray, o, d);
        RayGeom r;
        const int n = ray_setup(g, o, d, r);
        march_basis(sh.m, d);
        wave_lds_fence();
        const int s = L & 31;
        const float y = s < PLX_NSH ? sh.m.y[0][s] : 1.0f;
        int queued = 0;
        const int stored = min(cnt, a.st_cap);
        const int64_t base = ray * a.st_cap;
        if (cnt > stored) {
            // windows of 64 samples from the ray's end down to the last
            // recorded one
            const int k_lo = stored > 0 ? a.st_kidx[base + stored - 1] + 1 : 0;
            int k_hi = n - 1;
            while (k_hi >= k_lo) {
                const int k = k_hi - (kWave - 1) + L;
                const bool in = k >= k_lo;
                const Sample sm = sample_at(g, r, in ? k : k_hi);
                const bool occ = in && cell_occupied(g, sm.cell);
                const uint64_t m = __ballot(occ);
                const int total = __popcll(m);
                int step = kWave;
                if (total > 0) {
                    const int e = lanes_below(m);
                    if (occ) {
                        sh.m.pos[e] = make_float4(sm.f[0], sm.f[1], sm.f[2], __int_as_float(0));
                        sh.m.cell[e] = cell_id(g, sm.cell);
                        sh.q_id[e] = k;  // the queue is empty between windows here
                    }
                    wave_lds_fence();
                    Evaluator<DT, 64, 1>{g, sh.m, total}.run();
                    wave_lds_fence();
                    const int ke = sh.q_id[min(L, total - 1)];
                    const float4 v = sh.m.pos[min(L, total - 1)];
                    wave_lds_fence();
                    window_bwd<PRI>(g, a, sh, r, st, total, ke, v, y, queued, ls);
                    drain(sh, queued, y, a.grad, a.touched);
                    queued = 0;
                } else {
                    const Sample s_hi = sample_at(g, r, k_hi);
                    const int b[3] = {s_hi.cell[0] >> 3, s_hi.cell[1] >> 3, s_hi.cell[2] >> 3};
                    const int D = g.bdist[brick_id(g, b)];
                    if (D > 0) step = max(step, samples_behind(g, r, k_hi, b, D - 1) + 1);
                }
                k_hi -= step;
            }
        }
        for (int i0 = (stored - 1) / kWave * kWave; stored > 0 && i0 >= 0; i0 -= kWave) {
            const int total = min(kWave, stored - i0);
            const int64_t i = base + i0 + min(L, total - 1);
            window_bwd<PRI>(g, a, sh, r, st, total, a.st_kidx[i], a.st_vals[i], y, queued, ls);
        }
        drain(sh, queued, y, a.grad, a.touched);
    }
    if (PRI && a.pri.loss) {
        double t = (double)ls;
#pragma unroll
        for (int m = kWave / 2; m >= 1; m >>= 1) t += __shfl_xor(t, m);
        if (a.vals) {
            if (L == 0) {
                a.vals[ray].cauchy = t;
                a.vals[ray].beta = lb;
            }
        } else {
            prior_sum[0] += t;
            prior_sum[1] += lb;
        }
    }
}

// 128 registers for four waves on a SIMD: the training pass fits, the backward
// alone keeps 2 in scratch, and the instances with priors, whose terms are
// FP64 over the scans, about 50 (168 and 208 bytes a lane).
template <int DT, int MODE, bool PRI>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4)))
void rays_bwd_kernel(GridDev g, RayArgs a) {
    __shared__ BwdLds sh;
    double prior_sum[2] = {0.0, 0.0};
    for (int64_t ray = blockIdx.x; ray < a.n_rays; ray += gridDim.x)
        backward_ray<DT, MODE, PRI>(g, a, sh, ray, prior_sum);
    if (PRI && a.pri.loss && !a.vals && lane_id() == 0) {
        if (prior_sum[0] != 0.0) unsafeAtomicAdd(a.pri.loss, (double)a.pri.lambda_s * prior_sum[0]);
        if (prior_sum[1] != 0.0) unsafeAtomicAdd(a.pri.loss + 1, prior_sum[1]);
    }
}

// Sums of the rays' prior losses: one atomic per workgroup and term (one per
// ray would queue up at one address).
__global__ __launch_bounds__(256) void rays_prior_kernel(const RayVals *vals, int64_t n, Priors pri) {
    __shared__ double part[2][4];
    double ls = 0.0, lb = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        ls += vals[i].cauchy;
        lb += vals[i].beta;
    }
#pragma unroll
    for (int m = kWave / 2; m >= 1; m >>= 1) {
        ls += __shfl_xor(ls, m);
        lb += __shfl_xor(lb, m);
    }
    if (lane_id() == 0) {
        part[0][threadIdx.x / kWave] = ls;
        part[1][threadIdx.x / kWave] = lb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        ls = part[0][0] + part[0][1] + part[0][2] + part[0][3];
        lb = part[1][0] + part[1][1] + part[1][2] + part[1][3];
        if (ls != 0.0) unsafeAtomicAdd(pri.loss, (double)pri.lambda_s * ls);
        if (lb != 0.0) unsafeAtomicAdd(pri.loss + 1, lb);
    }
}

// Rays from which 16 lanes per ray (4 rays per wave) are the better cut; below,
// each ray gets a wave.  Forward without record, 64 / 16 lanes (us), FP32:
// 5000 rays on 64^3 37 / 93, on 256^3 52 / 151; 65,536 rays on 128^3 143 / 152,
// on 256^3 176 / 231, on 512^3 233 / 366; 131,072 on 128^3 263 / 216, on 256^3
// 320 / 333, dense 64^3 432 / 407; 640,000 (an 800x800 image of 512^3)
// 1532 / 968.  16-bit records, which take half the lanes and loads: 32,768
// rays on 128^3 74 / 72, on 256^3 96 / 109, on 512^3 113 / 151; 65,536 on 128^3
// 128 / 101, on 256^3 158 / 143, on 512^3 192 / 195.  Fewer lanes only lose (8
// and 4 on that image: 1019 and 1308 FP32): the rays of a list do not form
// square tiles.
template <int DT> constexpr int64_t kWaveRays = DT == PLX_F32 ? 3 << 15 : 3 << 14;
// Workgroups of a launch; with more rays they stride (a grid holds fewer than
// 2^32 threads).
constexpr int64_t kMaxBlocks = 1 << 25;

template <int MODE, int REC>
int launch_fwd(const plx_grid *grid, const RayArgs &a, hipStream_t s, const char *fn) {
    const GridDev g = to_dev(grid);
    PLX_DISPATCH_DT(grid->sh_dtype, DT, {
        if (a.n_rays < kWaveRays<DT>) {
            const unsigned nb = (unsigned)a.n_rays;
            rays_fwd_kernel<DT, 64, 1, MODE, REC><<<nb, kWave, 0, s>>>(g, a);
        } else {
            const unsigned nb = (unsigned)std::min((a.n_rays + 3) / 4, kMaxBlocks);
            rays_fwd_kernel<DT, 16, 4, MODE, REC><<<nb, kWave, 0, s>>>(g, a);
        }
    });
    return check_launch(fn);
}

// The forward that records.
int launch_record(const plx_grid *grid, const RayArgs &a, hipStream_t s, const char *fn) {
    return a.tau_out ? launch_fwd<MODE_FWD, REC_DEPTHS>(grid, a, s, fn) : launch_fwd<MODE_FWD, REC_SAMPLES>(grid, a, s, fn);
}

// Workgroups of a backward whose prior losses no per-ray values hold: as many
// as the chip runs at once, each adding its own.  An atomic per ray, one after
// the other at one address, took most of the time: 300,000 rays on 256^3 4.94 ms,
// now 1.87, without the priors 1.64.  With values, where a pass over them
// sums the losses, a workgroup per ray evens out rays of different length:
// 20,000 rays on 512^3 0.50 ms a step, on 4096 workgroups 0.60.
constexpr int64_t kPriorBlocks = 1 << 12;

template <int MODE>
int launch_bwd(const plx_grid *grid, const RayArgs &a, hipStream_t s, const char *fn) {
    const GridDev g = to_dev(grid);
    const bool loss = a.pri.loss != nullptr;
    // the priors' terms only in an instance of their own
    if (a.pri.lambda_s != 0.0f || a.pri.lambda_b != 0.0f) {
        const unsigned nb = (unsigned)std::min(a.n_rays, loss && !a.vals ? kPriorBlocks : kMaxBlocks);
        PLX_DISPATCH_DT(grid->sh_dtype, DT, rays_bwd_kernel<DT, MODE, true><<<nb, kWave, 0, s>>>(g, a));
        int rc = check_launch(fn);
        if (rc || !loss || !a.vals) return rc;
        rays_prior_kernel<<<(unsigned)std::min<int64_t>((a.n_rays + 255) / 256, 64), 256, 0, s>>>(a.vals, a.n_rays, a.pri);
    } else {
        const unsigned nb = (unsigned)std::min(a.n_rays, kMaxBlocks);
        PLX_DISPATCH_DT(grid->sh_dtype, DT, rays_bwd_kernel<DT, MODE, false><<<nb, kWave, 0, s>>>(g, a));
    }
    return check_launch(fn);
}

RayArgs base_args(const plx_render_opts *opts, const float *o, const float *d, int64_t n) {
    RayArgs a = {};
    a.rays_o = o;
    a.rays_d = d;
    a.n_rays = n;
    for (int i = 0; i < 3; ++i) a.bg[i] = opts->background[i];
    a.bg_rgb = opts->background_rgb;
    a.grad_bg = opts->grad_background;
    return a;
}

// Layout of the per-sample state buffer: per-ray counts, then sample indices,
// then float4 values, each part 256-byte aligned.
struct StateLayout {
    int64_t kidx, vals, bytes;
};

StateLayout state_layout(int64_t n_rays, int32_t cap) {
    auto up = [](int64_t x) { return (x + 255) / 256 * 256; };
    StateLayout l;
    l.kidx = up(n_rays * 4);
    l.vals = l.kidx + up(n_rays * (int64_t)cap * 4);
    l.bytes = l.vals + n_rays * (int64_t)cap * 16;
    return l;
}

int attach_state(RayArgs &a, void *state, int64_t state_bytes, int32_t cap, const char *fn) {
    if (!state) return fail(PLX_EINVAL, "%s: state is NULL", fn);
    if (cap < 0 || cap > (1 << 20)) return fail(PLX_EINVAL, "%s: cap %d out of range", fn, (int)cap);
    if (reinterpret_cast<uintptr_t>(state) % 256)
        return fail(PLX_EINVAL, "%s: state must be 256-byte aligned", fn);
    const StateLayout l = state_layout(a.n_rays, cap);
    if (state_bytes < l.bytes)
        return fail(PLX_EINVAL, "%s: state of %lld bytes, need %lld", fn, (long long)state_bytes,
                    (long long)l.bytes);
    char *base = static_cast<char *>(state);
    a.st_count = reinterpret_cast<int *>(base);
    a.st_kidx = reinterpret_cast<int *>(base + l.kidx);
    a.st_vals = reinterpret_cast<float4 *>(base + l.vals);
    a.st_cap = cap;
    return PLX_OK;
}

// Workspaces of the fused call: the rays' values and counts, and the records.
struct WorkLayout {
    int64_t count, ray_bytes;
    int64_t vals, samp_bytes;
};

WorkLayout work_layout(int64_t n_rays, int32_t cap) {
    auto up = [](int64_t x) { return (x + 255) / 256 * 256; };
    WorkLayout l;
    l.count = up(n_rays * (int64_t)sizeof(RayVals));
    l.ray_bytes = l.count + up(n_rays * 4);
    l.vals = up(n_rays * (int64_t)cap * 4);
    l.samp_bytes = l.vals + up(n_rays * (int64_t)cap * 16);
    return l;
}

int check_work(const void *p, int64_t have, int64_t need, const char *what, const char *fn) {
    if (!p) return fail(PLX_EINVAL, "%s: %s is NULL", fn, what);
    if (reinterpret_cast<uintptr_t>(p) % 256) return fail(PLX_EINVAL, "%s: %s must be 256-byte aligned", fn, what);
    if (have < need)
        return fail(PLX_EINVAL, "%s: %s of %lld bytes, need %lld", fn, what, (long long)have, (long long)need);
    return PLX_OK;
}

int attach_work(RayArgs &a, void *ray_ws, int64_t ray_ws_bytes, void *samp_ws, int64_t samp_ws_bytes, int32_t cap,
                const char *fn) {
    if (cap < 1 || cap > (1 << 20)) return fail(PLX_EINVAL, "%s: cap %d out of range", fn, (int)cap);
    const WorkLayout l = work_layout(a.n_rays, cap);
    int rc = check_work(ray_ws, ray_ws_bytes, l.ray_bytes, "ray workspace", fn);
    if (rc || (rc = check_work(samp_ws, samp_ws_bytes, l.samp_bytes, "sample workspace", fn))) return rc;
    a.vals = static_cast<RayVals *>(ray_ws);
    a.st_count = reinterpret_cast<int *>(static_cast<char *>(ray_ws) + l.count);
    a.st_kidx = static_cast<int *>(samp_ws);
    a.st_vals = reinterpret_cast<float4 *>(static_cast<char *>(samp_ws) + l.vals);
    a.st_cap = cap;
    return PLX_OK;
}

}  // namespace

int render_fwd_rays(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o, const float *rays_d,
                    int64_t n_rays, float *rgb_out, float *tau_out, hipStream_t s, const char *fn) {
    RayArgs a = base_args(opts, rays_o, rays_d, n_rays);
    a.rgb_out = rgb_out;
    a.tau_out = tau_out;
    int rc = mark_event(opts->kernel_events, 0, s, fn);
    if (rc || (rc = launch_fwd<MODE_FWD, REC_NONE>(grid, a, s, fn))) return rc;
    return mark_events(opts->kernel_events, 1, 4, s, fn);
}

}  // namespace plx

using namespace plx;

extern "C" {

int64_t plx_render_state_bytes(int64_t n_rays, int32_t cap) {
    if (n_rays < 0 || cap < 0 || cap > (1 << 20)) return 0;
    return state_layout(n_rays, cap).bytes;
}

int plx_render_fwd_state(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                         const float *rays_d, int64_t n_rays, float *rgb_out, float *tau_out,
                         void *state, int64_t state_bytes, int32_t cap, plx_stream stream) {
    const char *fn = "plx_render_fwd_state";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!rgb_out) return fail(PLX_EINVAL, "%s: rgb_out is NULL", fn);
    RayArgs a = base_args(opts, rays_o, rays_d, n_rays);
    if ((rc = attach_state(a, state, state_bytes, cap, fn))) return rc;
    a.rgb_out = rgb_out;
    a.tau_out = tau_out;
    return launch_record(grid, a, as_stream(stream), fn);
}

int plx_render_bwd_state(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                         const float *rays_d, int64_t n_rays, const float *grad_rgb,
                         const float *tau_fwd, const void *state, int64_t state_bytes, int32_t cap,
                         float *grad, uint8_t *touched, plx_stream stream) {
    const char *fn = "plx_render_bwd_state";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!grad_rgb || !tau_fwd || (grid->n_vox > 0 && (!grad || !touched)))
        return fail(PLX_EINVAL, "%s: NULL grad_rgb/tau_fwd/grad/touched", fn);
    RayArgs a = base_args(opts, rays_o, rays_d, n_rays);
    if ((rc = priors_from(opts, a.pri, fn))) return rc;
    if ((rc = attach_state(a, const_cast<void *>(state), state_bytes, cap, fn))) return rc;
    a.grad_rgb = grad_rgb;
    a.tau_in = tau_fwd;
    a.grad = grad;
    a.touched = touched;
    return launch_bwd<MODE_BWD>(grid, a, as_stream(stream), fn);
}

int64_t plx_rays_ray_bytes(int64_t n_rays) {
    if (n_rays < 0 || n_rays > ((int64_t)1 << 34)) return 0;
    return work_layout(n_rays, 0).ray_bytes;
}

int64_t plx_rays_samp_bytes(int64_t n_rays, int32_t cap) {
    if (n_rays < 0 || n_rays > ((int64_t)1 << 34) || cap < 1 || cap > (1 << 20)) return 0;
    return work_layout(n_rays, cap).samp_bytes;
}

int plx_render_fwd_rays(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                        const float *rays_d, int64_t n_rays, float *rgb_out, float *tau_out, void *ray_ws,
                        int64_t ray_ws_bytes, void *samp_ws, int64_t samp_ws_bytes, int32_t cap,
                        plx_stream stream) {
    const char *fn = "plx_render_fwd_rays";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!rgb_out) return fail(PLX_EINVAL, "%s: rgb_out is NULL", fn);
    hipStream_t s = as_stream(stream);
    if (!ray_ws && !samp_ws) return render_fwd_rays(grid, opts, rays_o, rays_d, n_rays, rgb_out, tau_out, s, fn);
    RayArgs a = base_args(opts, rays_o, rays_d, n_rays);
    if ((rc = attach_work(a, ray_ws, ray_ws_bytes, samp_ws, samp_ws_bytes, cap, fn))) return rc;
    a.rgb_out = rgb_out;
    a.tau_out = tau_out;
    if ((rc = mark_event(opts->kernel_events, 0, s, fn))) return rc;
    if ((rc = launch_record(grid, a, s, fn))) return rc;
    return mark_events(opts->kernel_events, 1, 4, s, fn);
}

int plx_render_bwd_rays(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                        const float *rays_d, int64_t n_rays, const float *grad_rgb, void *ray_ws,
                        int64_t ray_ws_bytes, void *samp_ws, int64_t samp_ws_bytes, int32_t cap, float *grad,
                        uint8_t *touched, plx_stream stream) {
    const char *fn = "plx_render_bwd_rays";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!grad_rgb || (grid->n_vox > 0 && (!grad || !touched)))
        return fail(PLX_EINVAL, "%s: NULL grad_rgb/grad/touched", fn);
    RayArgs a = base_args(opts, rays_o, rays_d, n_rays);
    if ((rc = priors_from(opts, a.pri, fn))) return rc;
    if ((rc = attach_work(a, ray_ws, ray_ws_bytes, samp_ws, samp_ws_bytes, cap, fn))) return rc;
    a.grad_rgb = grad_rgb;
    a.grad = grad;
    a.touched = touched;
    hipStream_t s = as_stream(stream);
    if ((rc = mark_events(opts->kernel_events, 0, 3, s, fn))) return rc;
    if ((rc = launch_bwd<MODE_BWD>(grid, a, s, fn))) return rc;
    return mark_event(opts->kernel_events, 3, s, fn);
}

int plx_render_train_rays(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                          const float *rays_d, const float *target, int64_t n_rays, void *ray_ws,
                          int64_t ray_ws_bytes, void *samp_ws, int64_t samp_ws_bytes, int32_t cap,
                          float loss_scale, float *rgb_out, float *grad, uint8_t *touched, double *loss_sum,
                          plx_stream stream) {
    const char *fn = "plx_render_train_rays";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!target || !loss_sum || (grid->n_vox > 0 && (!grad || !touched)))
        return fail(PLX_EINVAL, "%s: NULL target/grad/touched/loss_sum", fn);
    RayArgs a = base_args(opts, rays_o, rays_d, n_rays);
    if ((rc = priors_from(opts, a.pri, fn))) return rc;
    if ((rc = attach_work(a, ray_ws, ray_ws_bytes, samp_ws, samp_ws_bytes, cap, fn))) return rc;
    a.target = target;
    a.loss_scale = loss_scale;
    a.rgb_out = rgb_out;
    a.grad = grad;
    a.touched = touched;
    a.loss_sum = loss_sum;
    hipStream_t s = as_stream(stream);
    void **ev = opts->kernel_events;
    if ((rc = mark_event(ev, 0, s, fn))) return rc;
    if ((rc = launch_fwd<MODE_TRAIN, REC_SAMPLES>(grid, a, s, fn))) return rc;
    if ((rc = mark_events(ev, 1, 3, s, fn))) return rc;
    if ((rc = launch_bwd<MODE_TRAIN>(grid, a, s, fn))) return rc;
    return mark_event(ev, 3, s, fn);
}

}  // extern "C"
