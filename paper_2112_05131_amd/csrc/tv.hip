// tv.hip -- total-variation regulariser over a contiguous segment of cells
// (Sec. 3.5, the loss below Eq. (2); supplement B.1: stochastic TV on
// random contiguous segments of the pointer grid, differences normalised by
// D/256, and the SH rule that empty cells and edges count as equal to the
// current cell) for gfx950.
//
// Density term: one thread per cell of the segment, reading the cell and
// its three forward neighbours (NULL or out of range = 0).  SH terms exist
// only for a non-NULL cell (a NULL or out-of-range neighbour gives a zero
// difference): the block collects its non-NULL cells in LDS and then handles
// each with 32 lanes, lane q = coefficient q, so the four records are read and
// the four gradient records updated with one line-wide access each.
// The MSI background's instance uses its three colour coefficients as the
// colour terms and wraps its last (azimuth) axis.
// Gradients go to the cell and its neighbours with float atomics
// (neighbouring cells share voxels); the loss is reduced per workgroup and
// added once in FP64.
#include <algorithm>

#include "plx_internal.hpp"

namespace plx {
namespace {

// BG: the MSI background grid's TV, whose colour terms are its three colour
// coefficients (record slots 24-26) and whose last (azimuth) axis wraps.
constexpr int kBgSlot = 24;

// CELLS: cells a workgroup takes at a time, with its first CELLS threads for
// the density terms and then all 32 groups of 32 lanes for the SH terms.  The
// SH terms are a serial chain per group (record reads, then atomics), so the
// number of groups against the number of cells bounds a small segment; the
// loss bounds a large one, whose atomics all meet at one address (about 12 ns
// each, one after the other).  Hence wide workgroups, no more of them than
// the chip holds at once, each walking its share of the segment: with 256
// threads and a workgroup (an atomic) for every 256 cells 34 us for the 2,622
// cells of 64^3's segment, 39 for 20,972 of a unit-cube foreground, 60 for
// its background's 83,887 and 100 for 512^3's 1,342,178; so 14, 18, 43 and 61.
constexpr int kThreads = 1024;
constexpr int64_t kMaxGroups = 512;  // two workgroups on each of 256 CUs
constexpr int64_t kMaxBlocks = 1 << 21;  // a grid holds fewer than 2^32 threads; beyond, they stride
template <int DT, bool BG, int CELLS>
__global__ __launch_bounds__(kThreads) void tv_kernel(GridDev g, int64_t start, int64_t count,
                                                      int64_t ncell, float lam_sig_v, float lam_sh_v,
                                                      float eps, float s0, float s1, float s2,
                                                      float *grad, uint8_t *touched, double *loss_sum) {
    __shared__ int4 cells[CELLS];  // non-NULL cells of the block: id and forward neighbours
    __shared__ int n_cells_sh;
    __shared__ double part[kThreads / 64];
    const float sa[3] = {s0, s1, s2};
    double local = 0.0;
    for (int64_t base = (int64_t)blockIdx.x * CELLS; base < count;
         base += (int64_t)gridDim.x * CELLS) {
        __syncthreads();  // the previous cells are done
        if (threadIdx.x == 0) n_cells_sh = 0;
        __syncthreads();
        const int64_t c = base + threadIdx.x;
        if (threadIdx.x < CELLS && c < count) {
            int64_t v = start + c;
            v = v < ncell ? v : v % ncell;
            const int k = (int)(v % g.nz);
            const int64_t r = v / g.nz;
            const int j = (int)(r % g.ny);
            const int i = (int)(r / g.ny);
            const int64_t sy = g.nz, sx = (int64_t)g.ny * g.nz;
            const int id = g.index[v];
            const int nid[3] = {i + 1 < g.nx ? g.index[v + sx] : -1, j + 1 < g.ny ? g.index[v + sy] : -1,
                                k + 1 < g.nz ? g.index[v + 1] : (BG ? g.index[v - k] : -1)};

            // density channel: NULL or out-of-range reads 0
            {
                const float x0 = id >= 0 ? rec_sigma<DT>(g.data, id) : 0.0f;
                float dl[3], ss = 0.0f;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float xa = nid[a] >= 0 ? rec_sigma<DT>(g.data, nid[a]) : 0.0f;
                    dl[a] = sa[a] * (xa - x0);
                    ss += dl[a] * dl[a];
                }
                const float term = sqrtf(ss + eps);
                local += (double)lam_sig_v * (double)term;
                const float coef = lam_sig_v / term;
                if (id >= 0) {
                    const float gsum = sa[0] * dl[0] + sa[1] * dl[1] + sa[2] * dl[2];
                    const float gv = -coef * gsum;
                    if (gv != 0.0f) unsafeAtomicAdd(grad + (int64_t)id * PLX_REC_SLOTS + PLX_SLOT_SIGMA, gv);
                    touched[id] = 1;
                }
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    if (nid[a] < 0) continue;
                    const float gv = coef * sa[a] * dl[a];
                    if (gv != 0.0f)
                        unsafeAtomicAdd(grad + (int64_t)nid[a] * PLX_REC_SLOTS + PLX_SLOT_SIGMA, gv);
                    touched[nid[a]] = 1;
                }
            }
            if (id >= 0) cells[atomicAdd(&n_cells_sh, 1)] = make_int4(id, nid[0], nid[1], nid[2]);
        }
        __syncthreads();

        // SH channels of the non-NULL cells: groups of 32 lanes, lane q = slot q
        const int q = threadIdx.x & 31, grp = threadIdx.x >> 5;
        const int nc = n_cells_sh;
        for (int e = grp; e < nc; e += kThreads / 32) {
            const int4 cl = cells[e];
            const int nb[3] = {cl.y, cl.z, cl.w};
            float term = 0.0f;
            if (BG ? (q >= kBgSlot && q < kBgSlot + 3) : q < PLX_NSH) {
                const float x0 = rec_slot<DT>(g.data, cl.x, q);
                float dl[3], ss = 0.0f;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    dl[a] = nb[a] >= 0 ? sa[a] * (rec_slot<DT>(g.data, nb[a], q) - x0) : 0.0f;
                    ss += dl[a] * dl[a];
                }
                term = sqrtf(ss + eps);
                const float coef = lam_sh_v / term;
                float gsum = 0.0f;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    if (nb[a] < 0) continue;
                    const float gv = coef * sa[a] * dl[a];
                    gsum += sa[a] * dl[a];
                    if (gv != 0.0f) unsafeAtomicAdd(grad + (int64_t)nb[a] * PLX_REC_SLOTS + q, gv);
                }
                const float gv = -coef * gsum;
                if (gv != 0.0f) unsafeAtomicAdd(grad + (int64_t)cl.x * PLX_REC_SLOTS + q, gv);
            }
            local += (double)lam_sh_v * (double)term;
        }
    }

    // block reduction of the loss, one FP64 atomic per block
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) local += __shfl_xor(local, m);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = local;
    __syncthreads();
    if (threadIdx.x == 0 && loss_sum) {
        double t = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) t += part[w];
        if (t != 0.0) unsafeAtomicAdd(loss_sum, t);
    }
}

}  // namespace
}  // namespace plx

using namespace plx;

namespace plx {
namespace {

int tv_launch(const plx_grid *grid, int64_t cell_start, int64_t cell_count, float lambda_sigma,
              float lambda_sh, float eps, float *grad, uint8_t *touched, double *loss_sum,
              plx_stream stream, bool bg, const char *fn) {
    int rc = validate_grid(grid, false, fn);
    if (rc) return rc;
    if (bg && grid->sh_dtype != PLX_F32) return fail(PLX_EINVAL, "%s: background records must be FP32", fn);
    if (cell_count < 0) return fail(PLX_EINVAL, "%s: cell_count < 0", fn);
    if (cell_count == 0) return PLX_OK;
    if (!grad || !touched) return fail(PLX_EINVAL, "%s: grad/touched is NULL", fn);
    // eps > 0 keeps the square root and its derivative finite where all three
    // differences vanish (constant regions, the uniform initial grid)
    if (!(eps > 0.0f) || !std::isfinite(eps)) return fail(PLX_EINVAL, "%s: eps must be positive and finite", fn);
    const int64_t ncell = n_cells(grid->reso);
    const int64_t start = ((cell_start % ncell) + ncell) % ncell;
    const float inv = (float)(1.0 / (double)cell_count);
    hipStream_t s = as_stream(stream);
    GridDev g = to_dev(grid);
    const float sc[3] = {grid->reso[0] / 256.0f, grid->reso[1] / 256.0f, grid->reso[2] / 256.0f};
    auto launch = [&](auto kernel, int cells, int64_t most = kMaxGroups) {
        const int64_t nb = std::min((cell_count + cells - 1) / cells, most);
        kernel<<<(unsigned)nb, kThreads, 0, s>>>(g, start, cell_count, ncell, lambda_sigma * inv,
                                                 lambda_sh * inv, eps, sc[0], sc[1], sc[2], grad,
                                                 touched, loss_sum);
    };
    // 128 cells at a time spread a segment over twice the workgroups of 256:
    // 14 us against 18 for 2,622 cells, 43 against 46 for 83,887, the same 23
    // for 167,773; above, where every workgroup has several shares either way,
    // 256 halve the barriers: 61 against 74 for 1,342,178
    const bool wide = cell_count > 2 * 128 * kMaxGroups;
    // without a loss nothing queues up: a workgroup for every 1024 cells takes
    // 1.00 ms against 1.19 for the 16M cells of a 256^3 grid at 10%, 20 us
    // against 28 for 3M empty ones
    const bool huge = !loss_sum && cell_count > 1024 * kMaxGroups;
    if (bg) {
        if (huge) launch(tv_kernel<PLX_F32, true, 1024>, 1024, kMaxBlocks);
        else if (wide) launch(tv_kernel<PLX_F32, true, 256>, 256);
        else launch(tv_kernel<PLX_F32, true, 128>, 128);
    } else {
        PLX_DISPATCH_DT(grid->sh_dtype, DT, {
            if (huge) launch(tv_kernel<DT, false, 1024>, 1024, kMaxBlocks);
            else if (wide) launch(tv_kernel<DT, false, 256>, 256);
            else launch(tv_kernel<DT, false, 128>, 128);
        });
    }
    return check_launch(fn);
}

}  // namespace
}  // namespace plx

extern "C" int plx_tv_grad(const plx_grid *grid, int64_t cell_start, int64_t cell_count,
                           float lambda_sigma, float lambda_sh, float eps, float *grad,
                           uint8_t *touched, double *loss_sum, plx_stream stream) {
    return tv_launch(grid, cell_start, cell_count, lambda_sigma, lambda_sh, eps, grad, touched, loss_sum,
                     stream, false, "plx_tv_grad");
}

extern "C" int plx_bg_tv_grad(const plx_grid *bg_grid, int64_t cell_start, int64_t cell_count,
                              float lambda_sigma, float lambda_color, float eps, float *grad,
                              uint8_t *touched, double *loss_sum, plx_stream stream) {
    return tv_launch(bg_grid, cell_start, cell_count, lambda_sigma, lambda_color, eps, grad, touched,
                     loss_sum, stream, true, "plx_bg_tv_grad");
}
