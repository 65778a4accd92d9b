// optim.hip -- RMSProp with sparse (active-voxel) updates (Sec. 3.5 and
// Sec. 3.8: the gradient is very sparse, so only voxels that received a
// gradient term are updated) for gfx950.
//
// A workgroup takes kVox voxels, lists those whose touched byte is set in LDS
// and then updates them, 32 at a time: 8 lanes per voxel, 4 FP32 slots per
// lane (16-byte accesses, one 128-byte line per voxel and array).  An inactive
// voxel costs one byte read of the touched map, so the cost of a step follows
// the active set, not the grid.
//
// Memory bounds it: three lines read and three written per active voxel, at
// 5.5-6 TB/s.  Lanes of untouched voxels that idle beside a touched one (no
// list) took 340 us for 1.67M touched of 8.39M background voxels, with the
// list 236.  64 voxels a list keep a fully touched grid's accesses as
// dense as without it: 963 us for 6.71M voxels, 975 with 128, 985 with 256.
#include "plx_internal.hpp"

namespace plx {
namespace {

constexpr int kVox = 64;
// Grids from this size on do not keep the optimiser's state in the 256 MB of
// last-level cache from step to step (3 lines a voxel), so where most voxels
// are touched the second moments and gradients, which nothing reads again
// before they are evicted, are streamed past the caches: 804 us against 868 for
// 6.27M touched of 8.39M voxels, 910 against 963 for 6.71M of 6.71M.  Small
// active sets stay in the cache and are slower without it: 235k touched of
// 1.68M voxels 40 us against 32, 241k of 262k voxels 32 against 30.
constexpr int64_t kStreamVox = (256ll << 20) / (3 * PLX_REC_SLOTS * 4);

typedef float float_x4 __attribute__((ext_vector_type(4)));

template <bool STREAM>
__device__ __forceinline__ float4 load_state(const float4 *p) {
    if (!STREAM) return *p;
    const float_x4 x = __builtin_nontemporal_load(reinterpret_cast<const float_x4 *>(p));
    return make_float4(x[0], x[1], x[2], x[3]);
}

template <bool STREAM>
__device__ __forceinline__ void store_state(float4 *p, float x, float y, float z, float w) {
    if (STREAM) __builtin_nontemporal_store(float_x4{x, y, z, w}, reinterpret_cast<float_x4 *>(p));
    else *p = make_float4(x, y, z, w);
}

// One voxel's four slots of lane L (0-7).  zero_keeps: the learning rates and
// eps are such that a gradient of +0 leaves a parameter as it is.
template <int DT, bool STREAM>
__device__ __forceinline__ void update(int64_t m, int L, void *data, float *master, float *vstate,
                                       float *grad, float lr_sigma, float lr_sh, float beta,
                                       float eps, bool zero_keeps) {
    float *P = DT == PLX_F32 ? static_cast<float *>(data) : master;
    float4 *pp = reinterpret_cast<float4 *>(P + m * PLX_REC_SLOTS) + L;
    float4 *gp = reinterpret_cast<float4 *>(grad + m * PLX_REC_SLOTS) + L;
    float4 *vp = reinterpret_cast<float4 *>(vstate + m * PLX_REC_SLOTS) + L;
    const float4 g4 = load_state<STREAM>(gp), v4 = load_state<STREAM>(vp);
    const float g[4] = {g4.x, g4.y, g4.z, g4.w};
    float v[4] = {v4.x, v4.y, v4.z, v4.w};
    bool on = true, decay = true;
    if (DT == PLX_F32 && zero_keeps) {
        // A 64-byte half of a record whose gradients are all +0 and whose
        // second moments are all >= 0 (not NaN): p - lr * 0 / (sqrt(v') + eps)
        // is p, so only v decays, where there is any.  The colour-only records
        // of a background have one such half: 1.67M of them 340 us to 310
        // without lists.  Whole halves, as partly written ones cost more.
        bool zero = true, pos = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            zero = zero && __float_as_uint(g[e]) == 0u && v[e] >= 0.0f;
            pos = pos || v[e] > 0.0f;
        }
        const int half = threadIdx.x & 60;
        on = (__ballot(zero) >> half & 15) != 15;
        decay = (__ballot(pos) >> half & 15) != 0;
    }
    if (!on && !decay) return;
    float p[4] = {};
    if (on) {
        const float4 p4 = *pp;
        p[0] = p4.x, p[1] = p4.y, p[2] = p4.z, p[3] = p4.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int s = 4 * L + e;
        if (s < PLX_NSH || s == PLX_SLOT_SIGMA) {
            const float lr = s == PLX_SLOT_SIGMA ? lr_sigma : lr_sh;
            v[e] = fmaf(beta, v[e], (1.0f - beta) * g[e] * g[e]);
            p[e] = p[e] - lr * g[e] / (sqrtf(v[e]) + eps);
        }
    }
    store_state<STREAM>(vp, v[0], v[1], v[2], v[3]);
    if (!on) return;
    *pp = make_float4(p[0], p[1], p[2], p[3]);
    store_state<STREAM>(gp, 0.0f, 0.0f, 0.0f, 0.0f);
    if (DT != PLX_F32) {
        uint2 w;
        if (L == 7) {
            w.x = __float_as_uint(p[0]);
            w.y = 0u;
        } else {
            w.x = to16<DT>(p[0]) | (to16<DT>(p[1]) << 16);
            w.y = to16<DT>(p[2]) | (to16<DT>(p[3]) << 16);
            if (L == 6) w.y &= 0xffffu;
        }
        reinterpret_cast<uint2 *>(static_cast<char *>(data) + m * kRec16Bytes)[L] = w;
    }
}

template <int DT>
__global__ __launch_bounds__(256) void rmsprop_kernel(void *data, float *master, float *vstate,
                                                      float *grad, uint8_t *touched,
                                                      int64_t n_vox, float lr_sigma, float lr_sh,
                                                      float beta, float eps, bool zero_keeps) {
    __shared__ uint8_t list[kVox];  // the workgroup's touched voxels, in order
    __shared__ int count;
    const int64_t base = (int64_t)blockIdx.x * kVox;
    if (threadIdx.x < kVox) {
        const int64_t m = base + threadIdx.x;
        const bool on = m < n_vox && touched[m];
        if (on) touched[m] = 0;
        const uint64_t mask = __ballot(on);
        if (on) list[__popcll(mask & ((1ull << threadIdx.x) - 1))] = (uint8_t)threadIdx.x;
        if (threadIdx.x == 0) count = __popcll(mask);
    }
    __syncthreads();
    const int n = count, L = threadIdx.x & 7;
    if (n_vox >= kStreamVox && n > kVox / 2) {
        for (int e = threadIdx.x >> 3; e < n; e += 32)
            update<DT, true>(base + list[e], L, data, master, vstate, grad, lr_sigma, lr_sh, beta, eps, zero_keeps);
    } else {
        for (int e = threadIdx.x >> 3; e < n; e += 32)
            update<DT, false>(base + list[e], L, data, master, vstate, grad, lr_sigma, lr_sh, beta, eps, zero_keeps);
    }
}

}  // namespace
}  // namespace plx

using namespace plx;

extern "C" int plx_rmsprop_step(const plx_grid *grid, float *master, float *vstate, float *grad,
                                uint8_t *touched, float lr_sigma, float lr_sh, float beta,
                                float eps, plx_stream stream) {
    const char *fn = "plx_rmsprop_step";
    int rc = validate_grid(grid, false, fn);
    if (rc) return rc;
    if (grid->n_vox == 0) return PLX_OK;
    if (!vstate || !grad || !touched) return fail(PLX_EINVAL, "%s: NULL vstate/grad/touched", fn);
    if (grid->sh_dtype == PLX_F32 && master)
        return fail(PLX_EINVAL, "%s: master must be NULL for FP32 grids", fn);
    if (grid->sh_dtype != PLX_F32 && !master)
        return fail(PLX_EINVAL, "%s: 16-bit grids need the FP32 master records", fn);
    if (!(beta >= 0.0f && beta < 1.0f)) return fail(PLX_EINVAL, "%s: beta must be in [0, 1)", fn);
    const int64_t nw = (grid->n_vox + kVox - 1) / kVox;
    if (nw > 0x7fffffff) return fail(PLX_EINVAL, "%s: grid too large", fn);
    hipStream_t s = as_stream(stream);
    // the difference quotient of a +0 gradient is +0
    const bool zero_keeps = lr_sigma >= 0.0f && lr_sh >= 0.0f && std::isfinite(lr_sigma) &&
                            std::isfinite(lr_sh) && eps > 0.0f;
    PLX_DISPATCH_DT(grid->sh_dtype, DT,
                    rmsprop_kernel<DT><<<(unsigned)nw, 256, 0, s>>>(grid->data, master, vstate, grad,
                                                                    touched, grid->n_vox, lr_sigma,
                                                                    lr_sh, beta, eps, zero_keeps));
    return check_launch(fn);
}
