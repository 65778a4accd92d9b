// render.hip -- differentiable volume rendering over the sparse voxel grid
// (Sec. 3.1-3.3, Eq. (1); supplement B.1) for gfx950.
//
// Work mapping: two orders of the same work.  In ray order several lanes march
// a ray (march.hpp): the views here, and the batches of ray_order.hip.  In
// brick order, for large batches, a ray is cut into segments, one per occupied
// brick of 8^3 cells, and the segments are sorted by brick: a lane, or a
// workgroup per brick, takes them, so that rays crossing the same voxels share
// their records and send their gradients as one.
//
// SH factorisation.  The SH basis depends only on the ray direction, so the
// pre-activation colour of a sample is sum_c w_c (sum_l y_l k_{c,l}): when a
// corner voxel is loaded its coefficients are projected on the ray's basis
// once, and each sample interpolates four numbers per corner (density and
// the three projected channels).  In the backward pass the gradient of a
// coefficient is y_l times the gradient of its channel's projected value,
// so a lane accumulates four numbers per corner.
//
// Exact empty-space skipping, two levels.  A sample whose lower-corner cell
// has no non-NULL corner reads only zeros: it changes neither colour nor
// transmittance and has no gradient.
//  - Brick level: every 8^3-cell brick stores its Chebyshev distance D (in
//    bricks) to the nearest brick with an occupied cell.  From a sample in a
//    brick with D > 0, every cell of the box of bricks within D-1 of it is
//    empty, so the ray jumps to the box's exit point along its own direction
//    (less a margin of 5% of a step, far above FP32 rounding of t and g).
//  - Cell level: near occupied bricks a lane tests 16 candidate samples at a
//    time against the cell bitmap (16 independent loads) and processes only
//    the occupied ones.
// The corner ids and projected values of the current cell stay in registers
// while consecutive samples stay in one cell; a move to a face-adjacent cell
// keeps the 4 shared corners and loads only the other 4.
//
// Transmittance is exp(-tau) of the FP64 optical depth in both passes.
//
// Backward.  The ray is replayed from its last sample to its first.  With
// tau_after the optical depth after sample k (starting from the forward
// total), T_{k+1} = exp(-tau_after), T_k = exp(-(tau_after - sigma delta))
// and the rest of the ray R_k = sum_{j>k} w_j c_j + T_n bg is a running sum;
// dC/dsigma_k = delta (T_{k+1} c_k - R_k), dC/dc_k = w_k.  Corner gradients
// are accumulated in registers for as long as a voxel stays a corner of the
// current cell.  When it stops being one, the lane appends (voxel, four
// accumulated values, lane) to a queue in LDS; after every step of the
// replay the wave drains the queue two voxels at a time, 32 lanes per voxel,
// so that each voxel's 28 gradient values go out as one float atomic
// instruction covering its 128-byte gradient record (the access pattern for
// which the L2 float atomics are fastest).
//
// Priors (Sec. 3.7).  The Cauchy sparsity prior adds
// lambda_s 4 sigma / (1 + 2 sigma^2) to each sample's density gradient; the
// beta prior on T = T_final adds delta_k times one factor per ray,
// -T dL_b/dT, computed once from the ray's optical depth.  Both ride on the
// density slot of the same corner accumulators.
#include <string.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "march.hpp"

namespace plx {
namespace {

constexpr int kThreads = 256;          // rays per block
constexpr int kWavesPerBlock = kThreads / kWave;
constexpr int kChunk = 16;             // candidate samples tested per round
constexpr int kQCap = 8 * kWave;       // queue entries per wave (8 corners per lane per step)

enum { MODE_FWD = 0, MODE_BWD = 1, MODE_TRAIN = 2, MODE_MAXW = 3 };

// Wave-uniform copies (readfirstlane) of values the compiler cannot prove
// uniform, so that they live in scalar registers.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uni(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ int64_t uni64(int64_t v) {
    const uint64_t u = (uint64_t)v;
    const uint32_t lo = (uint32_t)uni((int)(uint32_t)u), hi = (uint32_t)uni((int)(uint32_t)(u >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <class T> __device__ __forceinline__ T *uni_ptr(T *p) {
    return reinterpret_cast<T *>(uni64((int64_t)reinterpret_cast<uintptr_t>(p)));
}

__device__ inline GridDev uniform_grid(const GridDev &s) {
    GridDev g;
    g.nx = uni(s.nx);
    g.ny = uni(s.ny);
    g.nz = uni(s.nz);
    g.bx = uni(s.bx);
    g.by = uni(s.by);
    g.bz = uni(s.bz);
    for (int a = 0; a < 3; ++a) {
        g.scale[a] = uni(s.scale[a]);
        g.offset[a] = uni(s.offset[a]);
    }
    g.step = uni(s.step);
    g.index = uni_ptr(s.index);
    g.data = uni_ptr(s.data);
    g.occ = uni_ptr(s.occ);
    g.bdist = uni_ptr(s.bdist);
    g.n_vox = uni64(s.n_vox);
    g.index_bytes = (uint32_t)uni((int)s.index_bytes);
    g.data_bytes = (uint32_t)uni((int)s.data_bytes);
    return g;
}

// ------------------------------------------------------------ voxel records

// Density and the three colour channels projected on the ray's SH basis y.
struct Q4 {
    float s, r, g, b;
};

__device__ __forceinline__ Q4 q4_zero() { return Q4{0.0f, 0.0f, 0.0f, 0.0f}; }

template <int DT> struct Project;
template <> struct Project<PLX_F32> {
    // slots 0..27 as seven 16-byte loads, sigma (slot 28) as one 4-byte load
    __device__ static inline Q4 run(const void *data, int id, const float y[9]) {
        const float *rec = static_cast<const float *>(data) + (int64_t)id * PLX_REC_SLOTS;
        const float4 *p = reinterpret_cast<const float4 *>(rec);
        float v[28];
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const float4 t = p[i];
            v[4 * i] = t.x;
            v[4 * i + 1] = t.y;
            v[4 * i + 2] = t.z;
            v[4 * i + 3] = t.w;
        }
        Q4 q;
        q.s = rec[PLX_SLOT_SIGMA];
        q.r = 0.0f;
        q.g = 0.0f;
        q.b = 0.0f;
#pragma unroll
        for (int l = 0; l < 9; ++l) {
            q.r += y[l] * v[l];
            q.g += y[l] * v[9 + l];
            q.b += y[l] * v[18 + l];
        }
        return q;
    }
};
template <int DT> struct Project16 {
    // the 64-byte record as four 16-byte loads: 16-bit slot s in word s/2,
    // the FP32 density in word 14
    __device__ static inline float h2f(uint32_t h) {
        return DT == PLX_BF16 ? bf16_to_f32(h) : f16_to_f32(h);
    }
    __device__ static inline float slot(const uint32_t w[16], int s) {
        return h2f((s & 1) ? (w[s >> 1] >> 16) : (w[s >> 1] & 0xffffu));
    }
    __device__ static inline Q4 run(const void *data, int id, const float y[9]) {
        const uint4 *p = reinterpret_cast<const uint4 *>(static_cast<const char *>(data) +
                                                         (int64_t)id * kRec16Bytes);
        uint32_t w[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 t = p[i];
            w[4 * i] = t.x;
            w[4 * i + 1] = t.y;
            w[4 * i + 2] = t.z;
            w[4 * i + 3] = t.w;
        }
        Q4 q;
        q.s = __uint_as_float(w[14]);
        q.r = 0.0f;
        q.g = 0.0f;
        q.b = 0.0f;
#pragma unroll
        for (int l = 0; l < 9; ++l) {
            q.r += y[l] * slot(w, l);
            q.g += y[l] * slot(w, 9 + l);
            q.b += y[l] * slot(w, 18 + l);
        }
        return q;
    }
};
template <> struct Project<PLX_BF16> : Project16<PLX_BF16> {};
template <> struct Project<PLX_F16> : Project16<PLX_F16> {};

// ------------------------------------------------------------ flush queue

// The lane's current cell: corner ids and projected values.
struct CornerCache {
    int cell[3];  // lower corner; cell[0] < 0 = empty cache
    int ids[8];
    Q4 q[8];
};


// Per-wave queue of flushed corners in LDS (structure of arrays).
struct Queue {
    int *count;     // entries in use
    int *id;        // [kQCap] voxel id
    uint8_t *src;   // [kQCap] lane that flushed it (selects the SH basis)
    float4 *v;      // [kQCap] accumulated density, R, G, B gradients
    float *y;       // [64][9] SH basis of each lane's ray
};

// Appends, for every active lane, its corners in `mask` (bit c = corner c)
// that are not NULL, with their accumulators.  One offset reservation per
// call: a lane's entries start at the sum of the counts of the active lanes
// below it (from the bit planes of the counts); only this wave uses the
// queue, and its LDS accesses are ordered.
__device__ __forceinline__ void push_corners(const Queue &qu, const CornerCache &cc,
                                             const Q4 acc[8], unsigned mask) {
    unsigned m = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c)
        if (((mask >> c) & 1u) && cc.ids[c] >= 0) m |= 1u << c;
    const int cnt = __popc(m);
    int before = 0, total = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const uint64_t plane = __ballot((cnt >> b) & 1);
        before += lanes_below(plane) << b;
        total += __popcll(plane) << b;
    }
    if (total == 0) return;
    const uint64_t act = __ballot(1);
    const int leader = __builtin_ctzll(act);
    int base = 0;
    if (lane_id() == leader) {
        base = *qu.count;
        *qu.count = base + total;
    }
    base = __builtin_amdgcn_readlane(base, leader);
    int e = base + before;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if ((m >> c) & 1u) {
            qu.id[e] = cc.ids[c];
            qu.src[e] = (uint8_t)lane_id();
            qu.v[e] = make_float4(acc[c].s, acc[c].r, acc[c].g, acc[c].b);
            ++e;
        }
    }
}

// Sends every queued voxel's gradient to its FP32 record: lanes 0..31 take
// one entry and lanes 32..63 the next, lane L & 31 = record slot (0..26 SH,
// 28 density, 29 marks the voxel touched).  Called by the whole wave.  The
// LDS reads are unconditional (positions past the count are clamped into the
// queue and their values discarded), so the reads of a round overlap and
// the only branches are the ones around the stores.
__device__ __forceinline__ void drain(const Queue &qu, float *grad, uint8_t *touched) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int E = __builtin_amdgcn_readfirstlane(*qu.count);
    if (E == 0) return;
    const int L = lane_id();
    const int s = L & 31;
    const bool sh = s < PLX_NSH;
    const int ch = sh ? 1 + s / 9 : 0;  // v component: 0 density, 1..3 colour
    const int l = sh ? s % 9 : 0;
    const bool writes = sh || s == PLX_SLOT_SIGMA;
    const bool marks = s == PLX_SLOT_SIGMA + 1;
    float *gs = grad + s;
    const int half = L >> 5;
    // eight pairs of entries per round
    constexpr int U = 8;
    for (int b0 = 0; b0 < E; b0 += 2 * U) {
        const int e0 = b0 + half;
        int id[U], src[U];
        float a[U], yv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = min(e0 + 2 * u, kQCap - 1);
            id[u] = qu.id[e];
            src[u] = (int)qu.src[e] & (kWave - 1);
            a[u] = reinterpret_cast<const float *>(qu.v)[4 * e + ch];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) yv[u] = qu.y[src[u] * 9 + l];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = e0 + 2 * u < E;
            const float val = (ok && writes) ? (sh ? yv[u] : 1.0f) * a[u] : 0.0f;
            if (val != 0.0f) unsafeAtomicAdd(gs + (int64_t)id[u] * PLX_REC_SLOTS, val);
            if (ok && marks) touched[id[u]] = 1;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (L == 0) *qu.count = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------ corner cache


__device__ inline int64_t corner_offset(const GridDev &g, int c) {
    return ((c >> 2) & 1) * ((int64_t)g.ny * g.nz) + ((c >> 1) & 1) * (int64_t)g.nz + (c & 1);
}

template <class T> __device__ __forceinline__ void swap2(T &a, T &b) {
    const T t = a;
    a = b;
    b = t;
}

// Exchanges the corners at positions c and c ^ BIT (the two faces of the cell
// across axis BIT).  After a move by +-1 along that axis, the shared corners
// then sit at their new positions; the other four positions are reloaded.
template <int BIT, bool BWD>
__device__ __forceinline__ void swap_faces(CornerCache &cc, Q4 acc[8]) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (c & BIT) continue;
        swap2(cc.ids[c], cc.ids[c | BIT]);
        swap2(cc.q[c], cc.q[c | BIT]);
        if (BWD) swap2(acc[c], acc[c | BIT]);
    }
}

// Makes `cell` the lane's cached cell.  On a move to a face-adjacent cell the
// four shared corners change position (positions `keep` receive the corner
// at position ^ bit) and only the other four are loaded; on any other move
// all eight are.  Corners that stop being corners are flushed first
// (backward).  Without `project` only the corner ids are loaded (the replay
// of stored samples needs them for the scatter, not the values).
template <int DT, bool BWD>
__device__ __forceinline__ void move_to(const GridDev &g, CornerCache &cc, const int cell[3],
                                        Q4 acc[8], const Queue &qu, const float y[9],
                                        bool project = true) {
    const int dx = cell[0] - cc.cell[0], dy = cell[1] - cc.cell[1], dz = cell[2] - cc.cell[2];
    if (dx == 0 && dy == 0 && dz == 0) return;
    const bool had = cc.cell[0] >= 0;
    const bool adj = had && abs(dx) + abs(dy) + abs(dz) == 1;
    const int bit = dx != 0 ? 4 : (dy != 0 ? 2 : 1);
    const bool plus = dx + dy + dz > 0;
    unsigned keep = 0;
    if (adj) {
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (((c & bit) != 0) != plus) keep |= 1u << c;
    }
    if (BWD && had) {
        // corners leaving: those at `keep` positions (shift) or all (jump)
        push_corners(qu, cc, acc, adj ? keep : 0xffu);
    }
    if (adj) {
        if (bit == 4) swap_faces<4, BWD>(cc, acc);
        else if (bit == 2) swap_faces<2, BWD>(cc, acc);
        else swap_faces<1, BWD>(cc, acc);
    }
    cc.cell[0] = cell[0];
    cc.cell[1] = cell[1];
    cc.cell[2] = cell[2];
    const int64_t lin = cell_id(g, cc.cell);
    int nid[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) nid[c] = ((keep >> c) & 1u) ? cc.ids[c] : g.index[lin + corner_offset(g, c)];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (!((keep >> c) & 1u)) {
            cc.ids[c] = nid[c];
            cc.q[c] = (project && nid[c] >= 0) ? Project<DT>::run(g.data, nid[c], y) : q4_zero();
            if (BWD) acc[c] = q4_zero();
        }
    }
}

__device__ inline void corner_weights(const float f[3], float w[8]) {
    const float ax[2] = {1.0f - f[0], f[0]};
    const float ay[2] = {1.0f - f[1], f[1]};
    const float az[2] = {1.0f - f[2], f[2]};
#pragma unroll
    for (int c = 0; c < 8; ++c) w[c] = ax[(c >> 2) & 1] * ay[(c >> 1) & 1] * az[c & 1];
}

// Interpolated (pre-activation) density and projected colour at weights w.
__device__ __forceinline__ Q4 interpolate(const CornerCache &cc, const float w[8]) {
    Q4 v = q4_zero();
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        v.s += w[c] * cc.q[c].s;
        v.r += w[c] * cc.q[c].r;
        v.g += w[c] * cc.q[c].g;
        v.b += w[c] * cc.q[c].b;
    }
    return v;
}

// ------------------------------------------------------------ sample cursor

// Occupancy of samples k0 .. k0+M-1 (bit i: sample k0+i exists and its cell
// is occupied); the M bitmap loads are independent.
// The loads are unconditional (indices outside [0, n) are clamped and their
// bits masked off afterwards): a load under a per-sample branch would be
// waited for inside that branch, serialising the 16 round trips.
template <int M = kChunk>
__device__ __forceinline__ uint32_t chunk_bits(const GridDev &g, const RayGeom &r, int n, int k0) {
    static_assert(M >= 1 && M < 32, "chunk size");
    constexpr uint32_t kFull = (1u << M) - 1u;
    const int k_max = n > 0 ? n - 1 : 0;
    uint32_t word[M];
    int bit[M];
#pragma unroll
    for (int i = 0; i < M; ++i) {
        int k = k0 + i;
        k = k < 0 ? 0 : (k > k_max ? k_max : k);
        const Sample s = sample_at(g, r, k);
        const int64_t b = ((int64_t)(s.cell[0] >> 3) * g.by + (s.cell[1] >> 3)) * g.bz + (s.cell[2] >> 3);
        const int bb = ((s.cell[0] & 7) << 6) | ((s.cell[1] & 7) << 3) | (s.cell[2] & 7);
        word[i] = g.occ[b * 16 + (bb >> 5)];
        bit[i] = bb & 31;
    }
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < M; ++i) m |= ((word[i] >> bit[i]) & 1u) << i;
    // samples k0 + i inside [0, n)
    const int lo = k0 < 0 ? -k0 : 0;
    const int hi = n - k0;  // first i past the end
    uint32_t valid = hi <= 0 ? 0u : (hi >= M ? kFull : ((1u << hi) - 1u));
    valid &= lo >= M ? 0u : ((kFull << lo) & kFull);
    return m & valid;
}

// ------------------------------------------------------------ brick-binned training
//
// plx_render_fwd, plx_render_bwd and plx_render_train run the batch in brick
// order.  Rays sampled from many
// cameras share few voxels with their neighbours in the batch, so a ray-order
// pass fetches every voxel record (and read-modify-writes every gradient
// line) about as often as rays cross it.  Here each ray is cut into segments,
// one per 8^3-cell brick with occupied cells that its samples pass through
// (a ray crosses a brick at most once: cell indices are monotone along it);
// the segments are sorted by brick, and the forward and backward passes run
// one lane per segment in that order, so the lanes of a wave read and update
// the same few hundred voxels.  Per ray, the segment results compose exactly
// as the samples do: the colour is sum_s T_in(s) C_s + T_n bg with
// T_in(s) = exp(-sum_{s'<s} tau_s'), and the backward replay of a segment
// starts from the optical depth after it and the radiance the ray collects
// after it (g . R), so every sample sees the same T_k, w_k and R_k.
//
// The lanes of a wave march in step, so a wave takes as many trips as its
// longest segment.  Inside a brick the segments are therefore ordered by
// length class (the segment's number of samples in steps of kLenStep): the
// bins are keyed by (brick, class).  A wave's segments then have closer
// lengths while the order stays by brick (ordering by class first, across
// bricks, evens the lengths out further but loses more to the scattered
// record reads than it gains).

//
// The bricks themselves are ordered by tiles of kTile^3 bricks (tiles in
// storage order, bricks inside a tile in storage order), so that the
// segments of consecutive waves stay within a compact block of the grid
// rather than a row of bricks along z.

constexpr int kLenClasses = 8;
constexpr int kLenStep = 4;
constexpr int kTile = 4;
constexpr int kBrickCells = PLX_BRICK * PLX_BRICK * PLX_BRICK;           // 512
constexpr int kBrickVox = (PLX_BRICK + 1) * (PLX_BRICK + 1) * (PLX_BRICK + 1);  // 729 corner voxels

inline int tiles_along(int bricks) { return (bricks + kTile - 1) / kTile; }
// Number of (brick, class) bins: brick order positions times classes.
inline int64_t n_bins(const GridDev &g) {
    return (int64_t)tiles_along(g.bx) * tiles_along(g.by) * tiles_along(g.bz) * (kTile * kTile * kTile) *
           kLenClasses;
}

// Position of brick b in the binning order.
__device__ __forceinline__ int64_t brick_order(const GridDev &g, const int b[3]) {
    const int nty = (g.by + kTile - 1) / kTile, ntz = (g.bz + kTile - 1) / kTile;
    const int64_t tile = ((int64_t)(b[0] / kTile) * nty + b[1] / kTile) * ntz + b[2] / kTile;
    return tile * (kTile * kTile * kTile) + ((b[0] % kTile) * kTile + b[1] % kTile) * kTile + b[2] % kTile;
}

// Brick at position jo of the binning order.
__device__ __forceinline__ void brick_at(const GridDev &g, int64_t jo, int b[3]) {
    const int nty = (g.by + kTile - 1) / kTile, ntz = (g.bz + kTile - 1) / kTile;
    const int64_t tile = jo / (kTile * kTile * kTile);
    const int in = (int)(jo % (kTile * kTile * kTile));
    b[0] = (int)(tile / ((int64_t)nty * ntz)) * kTile + in / (kTile * kTile);
    b[1] = (int)((tile / ntz) % nty) * kTile + (in / kTile) % kTile;
    b[2] = (int)(tile % ntz) * kTile + in % kTile;
}

__device__ __forceinline__ int64_t seg_bin(int64_t order, int k0, int k1) {
    const int c = min((k1 - k0) / kLenStep, kLenClasses - 1);
    return order * kLenClasses + c;
}

constexpr int kScanT = 256, kScanI = 16, kScanTile = kScanT * kScanI;

// Exclusive block-wide scan of one int64 per thread; *total gets the sum.
template <int NT = kScanT>
__device__ int64_t block_scan_excl(int64_t v, int64_t *total) {
    __shared__ int64_t wsum[NT / kWave];
    const int L = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int64_t x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t y = __shfl_up(x, o);
        if (L >= o) x += y;
    }
    if (L == kWave - 1) wsum[w] = x;
    __syncthreads();
    int64_t before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i) {
        if (i < w) before += wsum[i];
        tot += wsum[i];
    }
    __syncthreads();
    *total = tot;
    return before + x - v;
}

// Up to three arrays of counts scanned by the same three launches (one array
// each took nine, about 5 us apiece whatever the batch).  The counts of an
// array are c[0], c[stride], c[2*stride], ... (stride 2 reads one half of an
// array of 64-bit counter pairs).
struct ScanOf {
    const unsigned *c;
    int64_t n, nb;       // counts, and blocks of them
    int stride;
    int64_t *bsum, *boff;  // [nb], [nb + 1]
    int64_t *out;        // [n + 1]: out[i] = sum of c[0..i)
    int64_t *total;      // optional second copy of out[n]
};
struct ScanArgs {
    ScanOf of[3];
    int n_of;
};

// The array of a block (nb[0] blocks of the first, then those of the second
// ...); *blk gets its number there.
__device__ __forceinline__ const ScanOf &scan_of(const ScanArgs &a, int64_t *blk) {
    int64_t b = blockIdx.x;
    int k = 0;
    while (k + 1 < a.n_of && b >= a.of[k].nb) b -= a.of[k++].nb;
    *blk = b;
    return a.of[k];
}

__global__ __launch_bounds__(kScanT) void count_sum_kernel(ScanArgs a) {
    int64_t blk;
    const ScanOf &q = scan_of(a, &blk);
    const int64_t base = blk * kScanTile + (int64_t)threadIdx.x * kScanI;
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanI; ++i)
        if (base + i < q.n) s += q.c[(base + i) * q.stride];
    int64_t tot;
    block_scan_excl(s, &tot);
    if (threadIdx.x == 0) q.bsum[blk] = tot;
}

// One block per array.
__global__ __launch_bounds__(kScanT) void block_offsets_kernel(ScanArgs a) {
    const ScanOf &q = a.of[blockIdx.x];
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < q.nb; b0 += kScanT) {
        const int64_t b = b0 + threadIdx.x;
        int64_t tot;
        const int64_t ex = block_scan_excl(b < q.nb ? q.bsum[b] : 0, &tot);
        if (b < q.nb) q.boff[b] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) {
        q.out[q.n] = carry;
        if (q.total) *q.total = carry;
    }
}

__global__ __launch_bounds__(kScanT) void count_scan_kernel(ScanArgs a) {
    int64_t blk;
    const ScanOf &q = scan_of(a, &blk);
    const int64_t base = blk * kScanTile + (int64_t)threadIdx.x * kScanI;
    unsigned v[kScanI];
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanI; ++i) {
        v[i] = base + i < q.n ? q.c[(base + i) * q.stride] : 0u;
        s += v[i];
    }
    int64_t tot;
    int64_t r = q.boff[blk] + block_scan_excl(s, &tot);
#pragma unroll
    for (int i = 0; i < kScanI; ++i) {
        if (base + i < q.n) q.out[base + i] = r;
        r += v[i];
    }
}

__global__ void zero_u32_kernel(unsigned *p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// One occupied sample of the sample buffer, as the forward pass leaves it:
// its position in its cell, its sample index and cell, and the interpolated
// (pre-activation) density and projected colour.
struct SampleRec {
    float4 pos;   // f[0], f[1], f[2], (k << 9 | cell x*64 + y*8 + z) as integer bits
    float4 val;   // sigma, r, g, b
};

struct BinArgs {
    const float *rays_o;
    const float *rays_d;
    const float *target;    // TRAIN
    const float *grad_rgb;  // BWD
    float *tau_out;         // FWD (optional)
    float *rgb_out;
    double *loss_sum;
    float *grad;
    uint8_t *touched;
    int64_t n_rays;
    int64_t n_seg;
    float bg[3];
    const float *bg_rgb;    // optional per-ray background colours [n_rays][3]
    float *grad_bg;         // TRAIN/BWD, optional: T_final dL/dC per ray [n_rays][3]
    float loss_scale;
    int n_blocks;  // blocks of the launch at hand (rays or segments)
    int nb8;
    unsigned *nseg;      // [n_rays] segments of each ray
    int64_t *seg_off;    // [n_rays + 1] first ray-major slot of each ray
    unsigned *bcount;    // [n_bins] segments in each (length class, brick) bin
    unsigned *bcursor;   // [n_bins] placement cursors
    int64_t *boff;       // [n_bins + 1] first bin-major position of each bin
    int4 *bseg;          // [n_seg] bin-major: ray, first sample, last sample, ray-major slot
    double *tau_seg;     // [n_seg] ray-major: optical depth of the segment
    float4 *c_seg;       // [n_seg] ray-major: colour the segment adds (before T_in)
    double *tau_in;      // [n_seg] ray-major: optical depth before the segment
    float *gr_after;     // [n_seg] ray-major: g . (radiance collected after the segment)
    float4 *g_ray;       // [n_rays] dL/dC of each ray; w: beta factor of its samples
    unsigned *status;    // set to 1 when the emitting walk disagrees with the counting walk
    const int64_t *n_seg_dev;  // when set, the segment count is read here instead of n_seg
    void **events;       // optional hipEvent_t[4] recorded between the render kernels
    int64_t seg_cap;     // segment records the segment buffer holds
    // per-bin sample counts and the recorded backward (NULL when the bins
    // carry no sample buffer)
    unsigned long long *bcnt64;  // [n_bins] segments (low half) and sample slots (high half) per bin
    unsigned long long *bcur64;  // [n_bins] segment and sample placement cursors, packed the same way
    int64_t *bsoff;      // [n_bins + 1] first sample slot of each bin
    unsigned *blist;     // [n_brick] binning-order positions of the bricks with segments
    unsigned *nbrick;    // device count of blist entries
    int64_t *totals;     // [2] segments and sample slots (after nbrick)
    int64_t n_brick;
    int64_t *soff;       // [n_seg] bin-major: first sample slot of each segment
    int *nocc;           // [n_seg] bin-major: occupied samples the replay recorded
    SampleRec *srec;     // [samp_cap] sample records
    int64_t samp_cap;
    Priors pri;
    float *wmax;         // MAXW: [M] per-voxel maximum sample weight
};

// Number of segments of the call: the host's count, or the device copy when
// the launch was sized by a bound instead.
__device__ __forceinline__ int64_t seg_count_of(const BinArgs &a) {
    return a.n_seg_dev ? min(*a.n_seg_dev, a.n_seg) : a.n_seg;
}

// A segment record with its ray and slot inside the call's arrays.  The emit
// walk repeats the count walk exactly, so every position holds a valid
// record; the check keeps a record that is not (a disagreement, which the
// emit kernel reports in the status word) from indexing outside the arrays.
__device__ __forceinline__ bool seg_valid(const BinArgs &a, const int4 &sg, int64_t n_seg) {
    return (uint64_t)(int64_t)sg.x < (uint64_t)a.n_rays && (uint64_t)(int64_t)sg.w < (uint64_t)n_seg;
}

__device__ __forceinline__ void load_ray_lane(const BinArgs &a, int64_t ray, float o[3], float d[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        o[i] = a.rays_o[3 * ray + i];
        d[i] = a.rays_d[3 * ray + i];
    }
}

// Calls f(brick order position, first sample, last sample) for every brick
// with an occupied cell that the ray's samples enter with a first sample in
// [ks, ke), in ray order; boxes of empty bricks are skipped with the distance
// field, and inside a brick only the samples near its exit face are placed.
// A segment is a maximal run of the ray's samples in one occupied brick, so
// the parts of a ray, walked apart, give the segments of the whole.
template <class F>
__device__ __forceinline__ void walk_bricks(const GridDev &g, const RayGeom &r, int n, int ks, int ke, F &&f) {
    const RaySkip rs = ray_skip(g, r);
    int k = ks;
    // a brick that the part begins in the middle of belongs to the part before
    bool inside = false;
    if (k > 0 && k < ke) {
        const Sample s0 = sample_at(g, r, k - 1), s1 = sample_at(g, r, k);
        inside = s0.cell[0] / PLX_BRICK == s1.cell[0] / PLX_BRICK && s0.cell[1] / PLX_BRICK == s1.cell[1] / PLX_BRICK &&
                 s0.cell[2] / PLX_BRICK == s1.cell[2] / PLX_BRICK;
    }
    while (k < ke) {
        const Sample s = sample_at(g, r, k);
        const int b[3] = {s.cell[0] / PLX_BRICK, s.cell[1] / PLX_BRICK, s.cell[2] / PLX_BRICK};
        const int64_t bid = brick_id(g, b);
        const int D = g.bdist[bid];
        const int m = skip_box(g, r, rs, k, b, D > 0 ? D - 1 : 0);
        if (D > 0) {
            k += m + 1;
            inside = false;
            continue;
        }
        int kl = m < n - 1 - k ? k + m : n - 1;
        while (kl + 1 < n) {
            const Sample s2 = sample_at(g, r, kl + 1);
            if (s2.cell[0] / PLX_BRICK != b[0] || s2.cell[1] / PLX_BRICK != b[1] ||
                s2.cell[2] / PLX_BRICK != b[2])
                break;
            ++kl;
        }
        if (!inside) f(brick_order(g, b), k, kl);
        inside = false;
        k = kl + 1;
    }
}

// Lanes that walk a ray, each an eighth of its samples: a walk is a chain of
// distance reads, which a lane per ray leaves bare with few rays.  Count and
// emit in us: 5,000 rays inside 128^3 58 + 81, now 16 + 19; 20,011 through
// 256x256x128 42 + 57, now 25 + 30.  1M rays on 256^3 would still gain (180 +
// 191 with a lane per ray, 160 + 179 with eight), but a batch that large is
// binned beside the step before it, whose kernels the eightfold threads slow
// (two steps of 1M rays on 512^3 10.28 ms, with eight lanes 10.44).
// The lanes' segment counts, 16 bits each, wait for the emit walk in the ray's
// dL/dC, which the render calls write later; a part has no more segments than
// a line crosses bricks.
constexpr int kWalkParts = 8;
constexpr int64_t kWalkPartRays = 1 << 17;
inline int walk_parts(const GridDev &g, int64_t n_rays) {
    return n_rays <= kWalkPartRays && (int64_t)g.bx + g.by + g.bz < (1 << 16) ? kWalkParts : 1;
}

template <int PARTS>
__global__ __launch_bounds__(kThreads) void seg_count_kernel(GridDev g, BinArgs a) {
    const int blk = xcd_logical_block(blockIdx.x, a.nb8);
    if (blk >= a.n_blocks) return;
    const int64_t t = (int64_t)blk * kThreads + threadIdx.x, ray = t / PARTS;
    if (ray >= a.n_rays) return;
    const int part = (int)(t % PARTS);
    float o[3], d[3];
    load_ray_lane(a, ray, o, d);
    RayGeom r;
    const int n = ray_setup(g, o, d, r);
    unsigned cnt = 0;
    walk_bricks(g, r, n, (int)((int64_t)n * part / PARTS), (int)((int64_t)n * (part + 1) / PARTS),
                [&](int64_t bid, int k0, int k1) {
                    ++cnt;
                    const int64_t bin = seg_bin(bid, k0, k1);
                    if (a.bcnt64) atomicAdd(a.bcnt64 + bin, 1ull | ((unsigned long long)(k1 - k0 + 1) << 32));
                    else atomicAdd(a.bcount + bin, 1u);
                });
    if (PARTS > 1) {
        reinterpret_cast<uint16_t *>(a.g_ray + ray)[part] = (uint16_t)cnt;
#pragma unroll
        for (int m = 1; m < PARTS; m <<= 1) cnt += __shfl_xor(cnt, m, PARTS);
    }
    if (part == 0) a.nseg[ray] = cnt;
}

template <int PARTS>
__global__ __launch_bounds__(kThreads) void seg_emit_kernel(GridDev g, BinArgs a) {
    const int blk = xcd_logical_block(blockIdx.x, a.nb8);
    if (blk >= a.n_blocks) return;
    const int64_t t = (int64_t)blk * kThreads + threadIdx.x, ray = t / PARTS;
    if (ray >= a.n_rays) return;
    const int part = (int)(t % PARTS);
    float o[3], d[3];
    load_ray_lane(a, ray, o, d);
    RayGeom r;
    const int n = ray_setup(g, o, d, r);
    int64_t slot = a.seg_off[ray];
    int64_t slot_end = a.seg_off[ray + 1];
    bool bad = false;
    if (PARTS > 1) {
        const int own = reinterpret_cast<const uint16_t *>(a.g_ray + ray)[part];
        int incl = own;
#pragma unroll
        for (int m = 1; m < PARTS; m <<= 1) {
            const int y = __shfl_up(incl, m, PARTS);
            if (part >= m) incl += y;
        }
        bad = slot + __shfl(incl, PARTS - 1, PARTS) != slot_end;
        slot += incl - own;
        slot_end = min(slot_end, slot + own);
    }
    walk_bricks(g, r, n, (int)((int64_t)n * part / PARTS), (int)((int64_t)n * (part + 1) / PARTS),
                [&](int64_t bid, int k0, int k1) {
        const int64_t bin = seg_bin(bid, k0, k1);
        const unsigned len = (unsigned)(k1 - k0 + 1);
        // one cursor update gives the segment's position and (with a sample
        // buffer) its first sample slot
        unsigned long long cur = 0;
        if (a.bcur64) cur = atomicAdd(a.bcur64 + bin, 1ull | ((unsigned long long)len << 32));
        const int64_t pos = a.boff[bin] + (a.bcur64 ? (int64_t)(unsigned)cur : (int64_t)atomicAdd(a.bcursor + bin, 1u));
        // positions and slots stay inside the ranges the count reserved
        // and inside the segment buffer
        if (pos < a.boff[bin + 1] && slot < slot_end && pos < a.seg_cap && slot < a.seg_cap) {
            a.bseg[pos] = make_int4((int)ray, k0, k1, (int)slot);
            if (a.soff) {
                // the segment's sample slots, inside its bin's and the buffer's
                const int64_t sp = a.bsoff[bin] + (int64_t)(cur >> 32);
                const bool fits = sp + len <= a.bsoff[bin + 1] && sp + len <= a.samp_cap;
                a.soff[pos] = fits ? sp : -1;
                bad |= !fits;
            }
        } else {
            bad = true;
        }
        ++slot;
    });
    if (bad || slot != slot_end) *a.status = 1u;
}

// Appends the binning-order position of every brick with segments to
// a.blist (one counter update per wave; the order across waves is free).
__global__ __launch_bounds__(kThreads) void brick_list_kernel(BinArgs a, int64_t n_bricks) {
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool has = j < n_bricks && a.boff[(j + 1) * kLenClasses] > a.boff[j * kLenClasses];
    const uint64_t m = __ballot(has);
    if (m == 0) return;
    unsigned base = 0;
    if (lane_id() == 0) base = atomicAdd(a.nbrick, (unsigned)__popcll(m));
    base = __shfl(base, 0);
    if (has) a.blist[base + lanes_below(m)] = (unsigned)j;
}

// Occupied samples of [k_lo, k_hi] in increasing / decreasing order.
struct SpanCursor {
    int k;          // next sample to examine
    int k0;         // first sample of the current chunk
    uint32_t mask;  // occupied samples of the chunk not yet returned
};

__device__ __forceinline__ int span_next_up(const GridDev &g, const RayGeom &r, int n, int k_hi,
                                            SpanCursor &c) {
    while (c.mask == 0u) {
        if (c.k > k_hi) return -1;
        c.k0 = c.k;
        c.mask = chunk_bits(g, r, n, c.k);
        if (k_hi - c.k < kChunk - 1) c.mask &= (2u << (k_hi - c.k)) - 1u;
        c.k += kChunk;
    }
    const int b = __builtin_ctz(c.mask);
    c.mask &= c.mask - 1u;
    return c.k0 + b;
}

__device__ __forceinline__ int span_next_down(const GridDev &g, const RayGeom &r, int n, int k_lo,
                                              SpanCursor &c) {
    while (c.mask == 0u) {
        if (c.k < k_lo) return -1;
        c.k0 = c.k - (kChunk - 1);
        c.mask = chunk_bits(g, r, n, c.k0);
        if (c.k0 < k_lo) c.mask &= ~0u << (k_lo - c.k0);
        c.k -= kChunk;
    }
    const int b = 31 - __builtin_clz(c.mask);
    c.mask &= ~(1u << b);
    return c.k0 + b;
}

// Forward over one segment (transmittance relative to its start).  REC
// (the training and backward calls with a sample buffer) also stores every
// occupied sample's position in its cell, cell, sample index and
// interpolated values, in the segment's slots of the sample buffer.
template <int DT, bool REC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
void seg_fwd_kernel(GridDev g, BinArgs a) {
    const int blk = xcd_logical_block(blockIdx.x, a.nb8);
    if (blk >= a.n_blocks) return;
    const int64_t i = (int64_t)blk * kThreads + threadIdx.x;
    const int64_t n_seg = seg_count_of(a);
    if (i >= n_seg) return;
    const int4 sg = a.bseg[i];
    if (!seg_valid(a, sg, n_seg)) return;
    float o[3], d[3];
    load_ray_lane(a, sg.x, o, d);
    RayGeom r;
    const int n = ray_setup(g, o, d, r);
    float y[9];
    sh_basis_all(d, y);
    CornerCache cc;
    cc.cell[0] = cc.cell[1] = cc.cell[2] = -1;
    Q4 none[8];
    Queue noq{};
    SpanCursor cur{sg.y, 0, 0u};
    double tau = 0.0;
    float C[3] = {0.0f, 0.0f, 0.0f};
    int64_t base = 0, room = 0;
    if (REC) {
        base = a.soff[i];
        room = (int64_t)sg.z - sg.y + 1;  // the slots the count reserved
        if (base < 0 || base + room > a.samp_cap) room = 0;
    }
    int j = 0;
    while (true) {
        const int k = span_next_up(g, r, n, sg.z, cur);
        if (k < 0) break;
        const Sample s = sample_at(g, r, k);
        move_to<DT, false>(g, cc, s.cell, none, noq, y);
        float w[8];
        corner_weights(s.f, w);
        const Q4 v = interpolate(cc, w);
        if (REC && j < room) {
            const int code = (k << 9) | ((s.cell[0] & (PLX_BRICK - 1)) << 6) |
                             ((s.cell[1] & (PLX_BRICK - 1)) << 3) | (s.cell[2] & (PLX_BRICK - 1));
            SampleRec *rec = a.srec + base + j;
            rec->pos = make_float4(s.f[0], s.f[1], s.f[2], __int_as_float(code));
            rec->val = make_float4(v.s, v.r, v.g, v.b);
        }
        ++j;
        const float sd = fmaxf(v.s, 0.0f) * s.delta;
        const float wk = expf(-(float)tau) * (-expm1f(-sd));
        C[0] += wk * fmaxf(v.r, 0.0f);
        C[1] += wk * fmaxf(v.g, 0.0f);
        C[2] += wk * fmaxf(v.b, 0.0f);
        tau += (double)sd;
    }
    a.tau_seg[sg.w] = tau;
    a.c_seg[sg.w] = make_float4(C[0], C[1], C[2], 0.0f);
    if (REC) a.nocc[i] = (int)min((int64_t)j, room);
}

// ------------------------------------------------------------ brick-staged forward
//
// The segments of one brick read the same (at most 9^3) corner records, and
// at the training workload about 240 bricks are in flight per XCD at once,
// several times what its 4 MB L2 holds, so the lane-per-segment forward
// fetches each record from HBM several times.  The staged forward gives each
// brick with segments one workgroup: the brick's corner records are loaded
// once, coalesced, into LDS, and the workgroup's lanes march the brick's
// segments (one lane each) with the corner fetches served from LDS.  The
// arithmetic is that of seg_fwd.  It serves the forward renders of the
// 16-bit storage types, and their recording forward where bricks hold few
// segments (with many, the sample-parallel one below); FP32 records need
// 82 KB of LDS per brick, which leaves one workgroup (about two busy waves)
// per CU, and there the lane-per-segment kernel wins.

// 16-byte words of a staged record: FP32 slots 0..26 and the density in
// word 6's last float (28 floats); the 64-byte 16-bit record as stored.
template <int DT> struct StagedRec {
    static constexpr int kWords = DT == PLX_F32 ? 7 : 4;
};

template <int DT>
__device__ __forceinline__ Q4 project_staged(const uint4 *w4, const float y[9]) {
    if constexpr (DT == PLX_F32) {
        float v[28];
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const uint4 t = w4[i];
            v[4 * i] = __uint_as_float(t.x);
            v[4 * i + 1] = __uint_as_float(t.y);
            v[4 * i + 2] = __uint_as_float(t.z);
            v[4 * i + 3] = __uint_as_float(t.w);
        }
        Q4 q;
        q.s = v[27];
        q.r = 0.0f;
        q.g = 0.0f;
        q.b = 0.0f;
#pragma unroll
        for (int l = 0; l < 9; ++l) {
            q.r += y[l] * v[l];
            q.g += y[l] * v[9 + l];
            q.b += y[l] * v[18 + l];
        }
        return q;
    } else {
        uint32_t w[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 t = w4[i];
            w[4 * i] = t.x;
            w[4 * i + 1] = t.y;
            w[4 * i + 2] = t.z;
            w[4 * i + 3] = t.w;
        }
        Q4 q;
        q.s = __uint_as_float(w[14]);
        q.r = 0.0f;
        q.g = 0.0f;
        q.b = 0.0f;
#pragma unroll
        for (int l = 0; l < 9; ++l) {
            q.r += y[l] * Project16<DT>::slot(w, l);
            q.g += y[l] * Project16<DT>::slot(w, 9 + l);
            q.b += y[l] * Project16<DT>::slot(w, 18 + l);
        }
        return q;
    }
}

// move_to of the staged forward: cc.ids hold brick-local lattice positions
// (x*81 + y*9 + z) of non-NULL corners, -1 for NULL ones.
template <int DT>
__device__ __forceinline__ void move_staged(CornerCache &cc, const int cell[3], const int b0[3],
                                            const uint4 *s_rec, const int *s_id, const float y[9]) {
    const int dx = cell[0] - cc.cell[0], dy = cell[1] - cc.cell[1], dz = cell[2] - cc.cell[2];
    if (dx == 0 && dy == 0 && dz == 0) return;
    const bool had = cc.cell[0] >= 0;
    const bool adj = had && abs(dx) + abs(dy) + abs(dz) == 1;
    const int bit = dx != 0 ? 4 : (dy != 0 ? 2 : 1);
    const bool plus = dx + dy + dz > 0;
    unsigned keep = 0;
    if (adj) {
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (((c & bit) != 0) != plus) keep |= 1u << c;
        Q4 unused[8];
        if (bit == 4) swap_faces<4, false>(cc, unused);
        else if (bit == 2) swap_faces<2, false>(cc, unused);
        else swap_faces<1, false>(cc, unused);
    }
    cc.cell[0] = cell[0];
    cc.cell[1] = cell[1];
    cc.cell[2] = cell[2];
    const int lx = cell[0] - b0[0], ly = cell[1] - b0[1], lz = cell[2] - b0[2];
    const bool inside = (unsigned)lx < PLX_BRICK && (unsigned)ly < PLX_BRICK && (unsigned)lz < PLX_BRICK;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (!((keep >> c) & 1u)) {
            const int p = (lx + ((c >> 2) & 1)) * 81 + (ly + ((c >> 1) & 1)) * 9 + (lz + (c & 1));
            const bool has = inside && s_id[p] >= 0;
            cc.ids[c] = has ? p : -1;
            cc.q[c] = has ? project_staged<DT>(s_rec + p * StagedRec<DT>::kWords, y) : q4_zero();
        }
    }
}

template <int DT, bool REC>
__global__ __launch_bounds__(kThreads) void seg_fwd_brick_kernel(GridDev g, BinArgs a) {
    constexpr int W = StagedRec<DT>::kWords;
    __shared__ uint4 s_rec[kBrickVox * W];
    __shared__ int s_id[kBrickVox];
    if (blockIdx.x >= (unsigned)a.n_brick) return;
    const int t = threadIdx.x;
    const int64_t jo = a.blist[blockIdx.x];
    int b[3];
    brick_at(g, jo, b);
    const int b0[3] = {b[0] * PLX_BRICK, b[1] * PLX_BRICK, b[2] * PLX_BRICK};
    const int64_t seg0 = a.boff[jo * kLenClasses], seg1 = a.boff[(jo + 1) * kLenClasses];

    // stage the brick's corner records
    for (int p = t; p < kBrickVox; p += kThreads) {
        const int X = b0[0] + p / 81, Y = b0[1] + (p / 9) % 9, Z = b0[2] + p % 9;
        s_id[p] = (X < g.nx && Y < g.ny && Z < g.nz) ? g.index[((int64_t)X * g.ny + Y) * g.nz + Z] : -1;
    }
    __syncthreads();
    for (int k = t; k < kBrickVox * W; k += kThreads) {
        const int p = k / W, w = k - p * W;
        const int id = s_id[p];
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (id >= 0) {
            if constexpr (DT == PLX_F32) {
                const float *rec = static_cast<const float *>(g.data) + (int64_t)id * PLX_REC_SLOTS;
                v = reinterpret_cast<const uint4 *>(rec)[w];
                if (w == 6) v.w = __float_as_uint(rec[PLX_SLOT_SIGMA]);  // slot 27 is padding
            } else {
                v = reinterpret_cast<const uint4 *>(static_cast<const char *>(g.data) +
                                                    (int64_t)id * kRec16Bytes)[w];
            }
        }
        s_rec[k] = v;
    }
    __syncthreads();

    // march the brick's segments, one lane each
    for (int64_t i = seg0 + t; i < seg1; i += kThreads) {
        const int4 sg = a.bseg[i];
        if (!seg_valid(a, sg, a.n_seg)) continue;
        float o[3], d[3];
        load_ray_lane(a, sg.x, o, d);
        RayGeom r;
        const int n = ray_setup(g, o, d, r);
        float y[9];
        sh_basis_all(d, y);
        CornerCache cc;
        cc.cell[0] = cc.cell[1] = cc.cell[2] = -1;
        SpanCursor cur{sg.y, 0, 0u};
        double tau = 0.0;
        float C[3] = {0.0f, 0.0f, 0.0f};
        int64_t base = 0, room = 0;
        if (REC) {
            base = a.soff[i];
            room = (int64_t)sg.z - sg.y + 1;
            if (base < 0 || base + room > a.samp_cap) room = 0;
        }
        int j = 0;
        while (true) {
            const int k = span_next_up(g, r, n, sg.z, cur);
            if (k < 0) break;
            const Sample s = sample_at(g, r, k);
            move_staged<DT>(cc, s.cell, b0, s_rec, s_id, y);
            float w[8];
            corner_weights(s.f, w);
            const Q4 v = interpolate(cc, w);
            if (REC && j < room) {
                const int code = (k << 9) | ((s.cell[0] & (PLX_BRICK - 1)) << 6) |
                                 ((s.cell[1] & (PLX_BRICK - 1)) << 3) | (s.cell[2] & (PLX_BRICK - 1));
                SampleRec *rec = a.srec + base + j;
                rec->pos = make_float4(s.f[0], s.f[1], s.f[2], __int_as_float(code));
                rec->val = make_float4(v.s, v.r, v.g, v.b);
            }
            ++j;
            const float sd = fmaxf(v.s, 0.0f) * s.delta;
            const float wk = expf(-(float)tau) * (-expm1f(-sd));
            C[0] += wk * fmaxf(v.r, 0.0f);
            C[1] += wk * fmaxf(v.g, 0.0f);
            C[2] += wk * fmaxf(v.b, 0.0f);
            tau += (double)sd;
        }
        a.tau_seg[sg.w] = tau;
        a.c_seg[sg.w] = make_float4(C[0], C[1], C[2], 0.0f);
        if (REC) a.nocc[i] = (int)min((int64_t)j, room);
    }
}

// ------------------------------------------------------------ sample-parallel forward
//
// The recording forward of the training call, one workgroup per brick with
// segments, in three phases per group of up to kFwdSegs of its segments:
//  1. two or four lanes per segment (one for a large group) walk its
//     samples in runs of kWalkRun and store each occupied one's position
//     record (position in its cell, sample index, cell) in the segment's
//     slots of the sample buffer, in sample order; the waves with no
//     segment meanwhile load the brick's corner ids and first staging;
//  2. every lane takes samples of the group (all lanes busy, whatever the
//     segments' lengths) and interpolates them from the brick's corner
//     records, staged in LDS (FP32 in two halves along x of 5 x 9 x 9
//     corners, 45 KB, so that two workgroups fit on a CU, with the samples
//     listed by half first, as lanes that pass over the other half's samples
//     idle: 1.84 -> 1.76 ms for 1M rays through 512^3; 16-bit records whole),
//     storing the values in the sample's record (0.66 ms of that time is the
//     interpolation: 56 16-byte LDS reads per sample);
//  3. the lanes of a segment compose runs of its records, each with the
//     transmittance from the run's start, and chain the runs (a run's colour
//     times the transmittance of the runs before it).
// The values and the composition are those of seg_fwd (project each corner
// on the ray's SH basis, trilinear weights, Eq. (1) with the FP64 optical
// depth); the assignment of work to lanes and the grouping of the
// composition's products differ.

constexpr int kFwdThreads = 512;  // threads of a forward workgroup
constexpr int kFwdSegs = 384;     // segments per group
constexpr int kFwdList = 2048;    // samples listed by half at a time (FP32)
constexpr int kWalkRun = 8;       // consecutive samples a walking lane tests at once
// Segments per brick (on average over the call) from which the training call
// takes this forward: with fewer, most of a 512-thread workgroup idles in the
// walk and the composition, and the lane-per-segment forward is faster (on
// the 512^3 / 5% grid: 0.35 against 0.72 ms at 65,536 rays, about 9
// segments per brick; even at 262,144 rays, about 36; 2.66 against 1.81 ms
// at 1M rays, 138)
constexpr int64_t kFwdParMinSegs = 40;

template <int DT> struct FwdStage {
    static constexpr int kHalves = DT == PLX_F32 ? 2 : 1;
    static constexpr int kPlanes = PLX_BRICK / kHalves + 1;  // corner planes along x per half
    static constexpr int kWords = StagedRec<DT>::kWords;
    static constexpr int kVox = kPlanes * 81;
    static constexpr int kPer = 4;  // samples a thread finds at a time
    static constexpr int kChunk = kPer * kFwdThreads;
    static_assert(kHalves == 1 || kChunk <= kFwdList, "a chunk's samples fit the list");
};

// Stages the corner records of planes x = x0 .. x0 + kPlanes - 1 of the
// brick's 9^3 lattice (NULL corners as zeros).
template <int DT>
__device__ __forceinline__ void stage_planes(const GridDev &g, uint4 *s_rec, const int *s_id, int x0) {
    constexpr int W = FwdStage<DT>::kWords;
    for (int k = threadIdx.x; k < FwdStage<DT>::kVox * W; k += kFwdThreads) {
        const int p = k / W, w = k - p * W;
        const int id = s_id[x0 * 81 + p];
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (id >= 0) {
            if constexpr (DT == PLX_F32) {
                const float *rec = static_cast<const float *>(g.data) + (int64_t)id * PLX_REC_SLOTS;
                v = reinterpret_cast<const uint4 *>(rec)[w];
                if (w == 6) v.w = __float_as_uint(rec[PLX_SLOT_SIGMA]);  // slot 27 is padding
            } else {
                v = reinterpret_cast<const uint4 *>(static_cast<const char *>(g.data) +
                                                    (int64_t)id * kRec16Bytes)[w];
            }
        }
        s_rec[k] = v;
    }
}

// The staged words of the corner record with id `id` (NULL: zeros).
template <int DT>
__device__ __forceinline__ void load_corner_words(const GridDev &g, int id, uint4 wv[]) {
    constexpr int W = StagedRec<DT>::kWords;
#pragma unroll
    for (int w = 0; w < W; ++w) wv[w] = make_uint4(0u, 0u, 0u, 0u);
    if (id < 0) return;
    if constexpr (DT == PLX_F32) {
        const float *rec = static_cast<const float *>(g.data) + (int64_t)id * PLX_REC_SLOTS;
#pragma unroll
        for (int w = 0; w < W; ++w) wv[w] = reinterpret_cast<const uint4 *>(rec)[w];
        wv[W - 1].w = __float_as_uint(rec[PLX_SLOT_SIGMA]);  // slot 27 is padding
    } else {
        const uint4 *rec = reinterpret_cast<const uint4 *>(static_cast<const char *>(g.data) +
                                                           (int64_t)id * kRec16Bytes);
#pragma unroll
        for (int w = 0; w < W; ++w) wv[w] = rec[w];
    }
}

// Loads the ids of the brick's 9^3 corners into s_id and the records of the
// first staging (planes 0 .. kPlanes-1) into s_rec; thread `start` of
// `stride` threads takes corners start, start + stride, ...
template <int DT>
__device__ __forceinline__ void stage_ids_first(const GridDev &g, const int b0[3], int *s_id, uint4 *s_rec,
                                                int start, int stride) {
    constexpr int W = StagedRec<DT>::kWords;
    for (int p = start; p < kBrickVox; p += stride) {
        const int X = b0[0] + p / 81, Y = b0[1] + (p / 9) % 9, Z = b0[2] + p % 9;
        const int id = (X < g.nx && Y < g.ny && Z < g.nz) ? g.index[((int64_t)X * g.ny + Y) * g.nz + Z] : -1;
        s_id[p] = id;
        if (p < FwdStage<DT>::kVox) {
            uint4 wv[W];
            load_corner_words<DT>(g, id, wv);
#pragma unroll
            for (int w = 0; w < W; ++w) s_rec[p * W + w] = wv[w];
        }
    }
}

template <int DT>
__global__ __launch_bounds__(kFwdThreads) __attribute__((amdgpu_waves_per_eu(4)))
void seg_fwd_samples_kernel(GridDev g, BinArgs a) {
    using FS = FwdStage<DT>;
    constexpr int W = FS::kWords;
    __shared__ uint4 s_rec[FS::kVox * W];
    __shared__ int s_id[kBrickVox];
    __shared__ float4 s_y4[kFwdSegs * 3];      // SH basis of each segment's ray (9 of 12 floats)
    __shared__ int s_pre[kFwdSegs + 1];        // first sample of each segment in the group's numbering
    __shared__ int64_t s_soff[kFwdSegs];       // its first sample slot
    // a chunk's samples (segment << 11 | number in the chunk): those of the
    // lower half from the front, those of the upper from the back
    __shared__ uint32_t s_list[FS::kHalves == 2 ? kFwdList : 1];
    __shared__ int s_nlist[2];
    if (blockIdx.x >= (unsigned)a.n_brick) return;
    const int t = threadIdx.x;
    float *s_y = reinterpret_cast<float *>(s_y4);
    const int64_t jo = a.blist[blockIdx.x];
    int b[3];
    brick_at(g, jo, b);
    const int b0[3] = {b[0] * PLX_BRICK, b[1] * PLX_BRICK, b[2] * PLX_BRICK};
    const int64_t seg0 = a.boff[jo * kLenClasses], seg1 = a.boff[(jo + 1) * kLenClasses];
    int cur_half = -1;  // half whose corners are in LDS

    for (int64_t c0 = seg0; c0 < seg1; c0 += kFwdSegs) {
        const int ns = (int)min((int64_t)kFwdSegs, seg1 - c0);
        // 1. walk: kL lanes per segment (lane t: segment t / kL, part t % kL),
        // each taking runs of kWalkRun consecutive samples, store the
        // segment's occupied sample positions in order
        const int kL = ns * 4 <= kFwdThreads - 2 * kWave ? 4 : (ns * 2 <= kFwdThreads - 2 * kWave ? 2 : 1);
        const int sx = t / kL, part = t % kL;
        const bool mine = sx < ns;
        const int64_t i = c0 + sx;
        int4 sg = make_int4(0, 0, -1, 0);
        bool live = false;
        RayGeom r = {};
        int occ = 0;
        int64_t base = 0;
        // the waves with no segment of the first group load the corner ids
        // and the first staging meanwhile
        const int st0 = (ns * kL + kWave - 1) / kWave * kWave;
        const bool pre_stage = cur_half < 0 && st0 < kFwdThreads;
        if (pre_stage && t >= st0) stage_ids_first<DT>(g, b0, s_id, s_rec, t - st0, kFwdThreads - st0);
        if (mine) {
            sg = a.bseg[i];
            base = a.soff[i];
            float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f};
            live = seg_valid(a, sg, a.n_seg);
            if (live) {
                load_ray_lane(a, sg.x, o, d);
                const int n = ray_setup(g, o, d, r);
                const int64_t room = (int64_t)sg.z - sg.y + 1;  // the slots the count reserved
                if (base >= 0 && base + room <= a.samp_cap) {
                    // the kL lanes of a segment are adjacent and loop together
                    for (int kr = sg.y; kr <= sg.z; kr += kL * kWalkRun) {
                        const int ks = kr + part * kWalkRun;
                        uint32_t bits = 0u;
                        if (ks <= sg.z) {
                            bits = chunk_bits<kWalkRun>(g, r, n, ks);
                            if (sg.z - ks < kWalkRun - 1) bits &= (2u << (sg.z - ks)) - 1u;
                        }
                        const int c = __popc(bits);
                        int incl = c;  // inclusive prefix over the segment's parts
                        for (int dd = 1; dd < kL; dd <<= 1) {
                            const int y = __shfl_up(incl, dd, kL);
                            if (part >= dd) incl += y;
                        }
                        const int all = __shfl(incl, kL - 1, kL);
                        int at = occ + incl - c;
                        while (bits != 0u) {
                            const int k = ks + __builtin_ctz(bits);
                            bits &= bits - 1u;
                            const Sample sm = sample_at(g, r, k);
                            const int code = (k << 9) | ((sm.cell[0] & (PLX_BRICK - 1)) << 6) |
                                             ((sm.cell[1] & (PLX_BRICK - 1)) << 3) | (sm.cell[2] & (PLX_BRICK - 1));
                            a.srec[base + at].pos = make_float4(sm.f[0], sm.f[1], sm.f[2], __int_as_float(code));
                            ++at;
                        }
                        occ += all;
                    }
                }
            }
            if (part == 0) {
                sh_basis_all(d, s_y + sx * 12);
                s_soff[sx] = base;
            }
        }
        if (cur_half < 0) {
            if (!pre_stage) {
                // no wave was free during the walk: all threads stage
                stage_ids_first<DT>(g, b0, s_id, s_rec, t, kFwdThreads);
            }
            cur_half = 0;
        }
        int64_t tot64;
        const int pre = (int)block_scan_excl<kFwdThreads>(mine && part == 0 ? occ : 0, &tot64);
        const int tot = (int)tot64;
        if (mine && part == 0) s_pre[sx] = pre;
        if (t == 0) s_pre[kFwdSegs] = tot;
        __syncthreads();  // positions stored, s_pre / s_soff / s_y / the staging written

        // 2. values.  The segment of sample q of the group:
        auto seg_of = [&](int q) {
            int lo = 0, hi = ns - 1;  // last segment whose first sample is <= q
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_pre[mid] <= q) lo = mid;
                else hi = mid - 1;
            }
            return lo;
        };
        // interpolates a sample whose corners are staged from plane x0 on
        auto evaluate = [&](int seg, const float4 &pos, int x0, SampleRec *rec) {
            const int code = __float_as_int(pos.w);
            const int lx = ((code >> 6) & (PLX_BRICK - 1)) - x0, cy = (code >> 3) & (PLX_BRICK - 1),
                      cz = code & (PLX_BRICK - 1);
            float y[9];
#pragma unroll
            for (int l = 0; l < 9; ++l) y[l] = s_y[seg * 12 + l];
            const float f[3] = {pos.x, pos.y, pos.z};
            float w[8];
            corner_weights(f, w);
            Q4 v = q4_zero();
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int p = (lx + ((c >> 2) & 1)) * 81 + (cy + ((c >> 1) & 1)) * 9 + (cz + (c & 1));
                const Q4 qc = project_staged<DT>(s_rec + p * W, y);
                v.s += w[c] * qc.s;
                v.r += w[c] * qc.r;
                v.g += w[c] * qc.g;
                v.b += w[c] * qc.b;
            }
            rec->val = make_float4(v.s, v.r, v.g, v.b);
        };
        for (int q0 = 0; q0 < tot; q0 += FS::kChunk) {
            int seg_u[FS::kPer];
            SampleRec *rec_u[FS::kPer];
#pragma unroll
            for (int u = 0; u < FS::kPer; ++u) {
                const int q = q0 + u * kFwdThreads + t;
                seg_u[u] = -1;
                rec_u[u] = a.srec;
                if (q < tot) {
                    seg_u[u] = seg_of(q);
                    rec_u[u] = a.srec + s_soff[seg_u[u]] + (q - s_pre[seg_u[u]]);
                }
            }
            if constexpr (FS::kHalves == 1) {
                float4 pos_u[FS::kPer];
#pragma unroll
                for (int u = 0; u < FS::kPer; ++u)
                    if (seg_u[u] >= 0) pos_u[u] = rec_u[u]->pos;
#pragma unroll
                for (int u = 0; u < FS::kPer; ++u)
                    if (seg_u[u] >= 0) evaluate(seg_u[u], pos_u[u], 0, rec_u[u]);
            } else {
                // list the chunk's samples by half, so that the lanes that
                // take a half's are all busy
                int code_u[FS::kPer];
#pragma unroll
                for (int u = 0; u < FS::kPer; ++u)
                    if (seg_u[u] >= 0) code_u[u] = __float_as_int(rec_u[u]->pos.w);
                if (q0 > 0) __syncthreads();  // the previous chunk's list and counts read
                if (t < 2) s_nlist[t] = 0;
                __syncthreads();
#pragma unroll
                for (int u = 0; u < FS::kPer; ++u) {
                    const int q = u * kFwdThreads + t;
                    const bool upper = seg_u[u] >= 0 && ((code_u[u] >> 6) & (PLX_BRICK - 1)) >= FS::kPlanes - 1;
                    const uint64_t m1 = __ballot(upper), m0 = __ballot(seg_u[u] >= 0 && !upper);
                    int at0 = 0, at1 = 0;
                    if (lane_id() == 0) {
                        if (m0) at0 = atomicAdd(&s_nlist[0], __popcll(m0));
                        if (m1) at1 = atomicAdd(&s_nlist[1], __popcll(m1));
                    }
                    at0 = __shfl(at0, 0) + lanes_below(m0);
                    at1 = kFwdList - 1 - __shfl(at1, 0) - lanes_below(m1);
                    if (seg_u[u] >= 0) s_list[upper ? at1 : at0] = (uint32_t)seg_u[u] << 11 | (uint32_t)q;
                }
                __syncthreads();
                for (int hh = 0; hh < FS::kHalves; ++hh) {
                    const int h = hh == 0 ? cur_half : 1 - cur_half;
                    const int n_h = s_nlist[h];
                    if (hh == 1) {
                        if (n_h == 0) break;  // the same in every thread
                        __syncthreads();      // the other half's reads are done
                        stage_planes<DT>(g, s_rec, s_id, h * (FS::kPlanes - 1));
                        __syncthreads();
                        cur_half = h;
                    }
                    for (int e = t; e < n_h; e += kFwdThreads) {
                        const uint32_t ent = s_list[h ? kFwdList - 1 - e : e];
                        const int seg = (int)(ent >> 11);
                        SampleRec *rec = a.srec + s_soff[seg] + (q0 + (int)(ent & 2047u) - s_pre[seg]);
                        evaluate(seg, rec->pos, h * (FS::kPlanes - 1), rec);
                    }
                    if (hh == 1) break;
                }
            }
        }
        __syncthreads();  // every value stored before the segments compose

        // 3. composition: the kL lanes of a segment each compose a run of its
        // samples (transmittance from the run's start, record loads kCompU at
        // a time), then the runs are chained: run q's colour is scaled by the
        // transmittance of the runs before it (a segment without slots, which
        // the emit walk reports in the status word, contributes nothing)
        if (mine && live) {
            constexpr int kCompU = 4;
            const int per = (occ + kL - 1) / kL;
            const int j_lo = min(occ, part * per), j_hi = min(occ, j_lo + per);
            double tau = 0.0;
            float C[3] = {0.0f, 0.0f, 0.0f};
            for (int j0 = j_lo; j0 < j_hi; j0 += kCompU) {
                SampleRec rb[kCompU];
#pragma unroll
                for (int u = 0; u < kCompU; ++u)
                    if (j0 + u < j_hi) rb[u] = a.srec[base + j0 + u];
#pragma unroll
                for (int u = 0; u < kCompU; ++u) {
                    if (j0 + u >= j_hi) break;
                    const int k = (int)((unsigned)__float_as_int(rb[u].pos.w) >> 9);
                    const float delta = sample_at(g, r, k).delta;
                    const float sd = fmaxf(rb[u].val.x, 0.0f) * delta;
                    const float wk = expf(-(float)tau) * (-expm1f(-sd));
                    C[0] += wk * fmaxf(rb[u].val.y, 0.0f);
                    C[1] += wk * fmaxf(rb[u].val.z, 0.0f);
                    C[2] += wk * fmaxf(rb[u].val.w, 0.0f);
                    tau += (double)sd;
                }
            }
            if (kL > 1) {
                double incl = tau;  // optical depth up to the end of this run
                for (int dd = 1; dd < kL; dd <<= 1) {
                    const double y = __shfl_up(incl, dd, kL);
                    if (part >= dd) incl += y;
                }
                // the depth before the run from the scan, not as incl - tau,
                // which is NaN after an infinite density
                double excl = __shfl_up(incl, 1, kL);
                if (part == 0) excl = 0.0;
                const float T0 = expf(-(float)excl);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    C[c] *= T0;
                    for (int dd = 1; dd < kL; dd <<= 1) C[c] += __shfl_xor(C[c], dd, kL);
                }
                tau = __shfl(incl, kL - 1, kL);
            }
            if (part == 0) {
                a.tau_seg[sg.w] = tau;
                a.c_seg[sg.w] = make_float4(C[0], C[1], C[2], 0.0f);
                a.nocc[i] = occ;
            }
        }
        __syncthreads();  // s_y / s_pre / s_soff are rewritten by the next group
    }
}

// Segments of a ray are walked kSegU at a time: the loads of a group are
// issued together (positions past the last segment are clamped to it and
// their values unused), then the group is composed in order.
constexpr int kSegU = 4;

// Per ray: composes its segments into the colour (and optical depth).  FWD
// writes them out; TRAIN also forms the loss and dL/dC = 2 loss_scale (C -
// target), BWD takes dL/dC as given; both then record, for every segment,
// the optical depth before it and g . R after it.
template <int MODE>
__global__ __launch_bounds__(kThreads) void seg_combine_kernel(BinArgs a) {
    __shared__ double blk_loss[kWavesPerBlock];
    const int64_t ray = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double l2 = 0.0, lb = 0.0;
    if constexpr (MODE == MODE_MAXW) {
        if (ray < a.n_rays) {
            const int64_t s0 = a.seg_off[ray], s1 = min(a.seg_off[ray + 1], a.seg_cap);
            double tau = 0.0;
            for (int64_t s = s0; s < s1; s += kSegU) {
                double ts[kSegU];
#pragma unroll
                for (int u = 0; u < kSegU; ++u) ts[u] = a.tau_seg[min(s + u, s1 - 1)];
#pragma unroll
                for (int u = 0; u < kSegU; ++u) {
                    if (s + u < s1) {
                        a.tau_in[s + u] = tau;
                        tau += ts[u];
                    }
                }
            }
        }
        return;
    }
    if (ray < a.n_rays) {
        const int64_t s0 = a.seg_off[ray], s1 = min(a.seg_off[ray + 1], a.seg_cap);
        double tau = 0.0;
        float C[3] = {0.0f, 0.0f, 0.0f};
        for (int64_t s = s0; s < s1; s += kSegU) {
            double ts[kSegU];
            float4 cs[kSegU];
#pragma unroll
            for (int u = 0; u < kSegU; ++u) {
                const int64_t sc = min(s + u, s1 - 1);
                ts[u] = a.tau_seg[sc];
                cs[u] = a.c_seg[sc];
            }
#pragma unroll
            for (int u = 0; u < kSegU; ++u) {
                if (s + u < s1) {
                    if (MODE != MODE_FWD) a.tau_in[s + u] = tau;
                    const float T = expf(-(float)tau);
                    C[0] += T * cs[u].x;
                    C[1] += T * cs[u].y;
                    C[2] += T * cs[u].z;
                    tau += ts[u];
                }
            }
        }
        const float T_final = expf(-(float)tau);
        float gr[3], R[3], bgc[3];
        ray_background(a.bg_rgb, a.bg, ray, bgc);
#pragma unroll
        for (int c3 = 0; c3 < 3; ++c3) {
            const float Cc = C[c3] + T_final * bgc[c3];
            if (MODE != MODE_BWD && a.rgb_out) a.rgb_out[3 * ray + c3] = Cc;
            if (MODE == MODE_TRAIN) {
                const float diff = Cc - a.target[3 * ray + c3];
                gr[c3] = 2.0f * a.loss_scale * diff;
                l2 += (double)(diff * diff);
            } else if (MODE == MODE_BWD) {
                gr[c3] = a.grad_rgb[3 * ray + c3];
            }
            R[c3] = T_final * bgc[c3];
        }
        if (MODE == MODE_FWD) {
            if (a.tau_out) a.tau_out[ray] = (float)tau;
        } else {
            const float gw = a.pri.lambda_b != 0.0f ? beta_factor(a.pri, tau, &lb) : 0.0f;
            a.g_ray[ray] = make_float4(gr[0], gr[1], gr[2], gw);
            if (a.grad_bg) {
#pragma unroll
                for (int c3 = 0; c3 < 3; ++c3) a.grad_bg[3 * ray + c3] = T_final * gr[c3];
            }
            for (int64_t s = s1 - 1; s >= s0; s -= kSegU) {
                double ti[kSegU];
                float4 cs[kSegU];
#pragma unroll
                for (int u = 0; u < kSegU; ++u) {
                    const int64_t sc = max(s - u, s0);
                    ti[u] = a.tau_in[sc];
                    cs[u] = a.c_seg[sc];
                }
#pragma unroll
                for (int u = 0; u < kSegU; ++u) {
                    if (s - u >= s0) {
                        a.gr_after[s - u] = gr[0] * R[0] + gr[1] * R[1] + gr[2] * R[2];
                        const float T = expf(-(float)ti[u]);
                        R[0] += T * cs[u].x;
                        R[1] += T * cs[u].y;
                        R[2] += T * cs[u].z;
                    }
                }
            }
        }
    }
    if (MODE != MODE_FWD) add_prior_loss(a.pri, 0.0f, lb);
    if (MODE == MODE_TRAIN) {
        double wl = (double)a.loss_scale * l2;
#pragma unroll
        for (int m = kWave / 2; m >= 1; m >>= 1) wl += __shfl_xor(wl, m);
        if ((threadIdx.x & (kWave - 1)) == 0) blk_loss[threadIdx.x / kWave] = wl;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w = 0; w < kWavesPerBlock; ++w) t += blk_loss[w];
            if (t != 0.0) unsafeAtomicAdd(a.loss_sum, t);
        }
    }
}

// Backward replay of one segment, from its last occupied sample to its first.
template <int DT, bool CAUCHY>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3)))
void seg_bwd_kernel(GridDev g, BinArgs a) {
    __shared__ int q_count[kWavesPerBlock];
    __shared__ int q_id[kWavesPerBlock * kQCap];
    __shared__ uint8_t q_src[kWavesPerBlock * kQCap];
    __shared__ float4 q_v[kWavesPerBlock * kQCap];
    __shared__ float q_y[kWavesPerBlock * kWave * 9];

    const int blk = xcd_logical_block(blockIdx.x, a.nb8);
    if (blk >= a.n_blocks) return;
    const int wid = threadIdx.x / kWave;
    const int L = lane_id();
    if (L == 0) q_count[wid] = 0;
    __syncthreads();
    Queue qu;
    qu.count = q_count + wid;
    qu.id = q_id + wid * kQCap;
    qu.src = q_src + wid * kQCap;
    qu.v = q_v + wid * kQCap;
    qu.y = q_y + wid * kWave * 9;

    const int64_t i = (int64_t)blk * kThreads + threadIdx.x;
    const int64_t n_seg = seg_count_of(a);
    int4 sg = make_int4(0, 0, -1, 0);
    if (i < n_seg) sg = a.bseg[i];
    const bool live = i < n_seg && seg_valid(a, sg, n_seg);
    float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f};
    if (live) load_ray_lane(a, sg.x, o, d);
    RayGeom r;
    const int n = live ? ray_setup(g, o, d, r) : 0;
    float *y = qu.y + L * 9;
    sh_basis_all(d, y);

    CornerCache cc;
    cc.cell[0] = cc.cell[1] = cc.cell[2] = -1;
    Q4 acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = q4_zero();

    float gr[3] = {0.f, 0.f, 0.f};
    double tau_after = 0.0;
    float gR = 0.0f, ls = 0.0f;
    if (live) {
        const float4 gg = a.g_ray[sg.x];
        gr[0] = gg.x;
        gr[1] = gg.y;
        gr[2] = gg.z;
        tau_after = a.tau_in[sg.w] + a.tau_seg[sg.w];
        gR = a.gr_after[sg.w] - gg.w;  // the beta factor joins the running sum
    }
    float T_after = expf(-(float)tau_after);
    SpanCursor cur{sg.z, 0, 0u};
    bool active = live && n > 0;
    while (__any(active)) {
        if (active) {
            const int k = span_next_down(g, r, n, sg.y, cur);
            if (k < 0) {
                if (cc.cell[0] >= 0) push_corners(qu, cc, acc, 0xffu);
                active = false;
            } else {
                const Sample s = sample_at(g, r, k);
                move_to<DT, true>(g, cc, s.cell, acc, qu, y);
                float w[8];
                corner_weights(s.f, w);
                const Q4 v = interpolate(cc, w);
                const float sd = fmaxf(v.s, 0.0f) * s.delta;
                const double tau_before = fmax(tau_after - (double)sd, 0.0);
                const float T_before = expf(-(float)tau_before);
                const float wk = T_before * (-expm1f(-sd));
                const float gc = gr[0] * fmaxf(v.r, 0.0f) + gr[1] * fmaxf(v.g, 0.0f) +
                                 gr[2] * fmaxf(v.b, 0.0f);
                const float cs = CAUCHY ? cauchy_grad(a.pri, v.s, &ls) : 0.0f;
                const float dsig = v.s > 0.0f ? s.delta * (T_after * gc - gR) + cs : 0.0f;
                const float g_r = v.r > 0.0f ? wk * gr[0] : 0.0f;
                const float g_g = v.g > 0.0f ? wk * gr[1] : 0.0f;
                const float g_b = v.b > 0.0f ? wk * gr[2] : 0.0f;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    acc[c].s += w[c] * dsig;
                    acc[c].r += w[c] * g_r;
                    acc[c].g += w[c] * g_g;
                    acc[c].b += w[c] * g_b;
                }
                gR += wk * gc;
                tau_after = tau_before;
                T_after = T_before;
            }
        }
        drain(qu, a.grad, a.touched);
    }
    if (CAUCHY) add_prior_loss(a.pri, ls, 0.0);
}

// ------------------------------------------------------------ recorded backward
//
// The scatter of seg_bwd sends about nine partial gradients to every voxel a
// batch reaches (one per segment that has it as a corner), each a 128-B line
// of FP32 atomics, and global atomics are the slowest path on the chip (about
// 20G 64-byte requests per second, whatever the lanes' pattern); its replay
// also repeats the forward's corner gathers.  The recorded backward instead:
//  1. seg_fwd (REC) stores, per occupied sample, its position in the cell,
//     sample index, cell and interpolated values (32 B) in the segment's
//     slots of the sample buffer;
//  2. seg_combine forms the per-ray and per-segment quantities as before;
//  3. seg_scatter (one workgroup per brick with segments) loads the brick's
//     samples, forms their gradients with respect to density and projected
//     colour (the lane that has a sample finds its weight and gradients; one
//     lane per segment runs the reverse recurrence's two chains, the FP64
//     optical depth before each sample and the radiance after it), sorts
//     them in LDS by cell, and then each lane owns one of the brick's stored
//     corner voxels and sums the contributions of the samples of the (up to) 8 cells around
//     it, so every voxel gets one 128-B line of atomics per brick instead of
//     one per segment, and no corner record is read a second time.
// The terms are those of seg_bwd (Sec. 3.3, Eq. (1) and the chain rule
// through the trilinear weights and the SH basis); only the order of the
// additions differs.

// Its phases are short and latency shows between them (two workgroups a CU,
// 1,100 samples each on 1M rays through 512^3): so no long chain runs on the
// few lanes that own a segment -- exponentials, weights and gradients are
// found by the lane that has the sample, and a segment's lane only subtracts
// depths and sums g . R -- and only the brick's stored voxels are given
// lanes, in one round where a brick of mostly empty corners took two.
// 2.24 -> 2.07 ms; its 21M 64-byte atomic requests, which overlap the rest, would
// take 1.07 alone (20 G/s).

constexpr int kScatterThreads = 512;       // threads of a scatter workgroup
constexpr int kScatterSegs = 256;          // segments per pass
constexpr int kVoxRounds = (kBrickVox + kScatterThreads - 1) / kScatterThreads;
constexpr int kScatterCap = 1536;          // samples in LDS per pass
constexpr int kScatterPer = kScatterCap / kScatterThreads;
constexpr int kChainU = 4;                 // chain steps whose LDS reads are issued together
constexpr int kStageRows = 8;              // rows a wave stages per flush round
constexpr int kStageStride = 29;           // 28 values and the voxel id per staged row

// A sample in the scatter's LDS, sorted by cell: its position in the cell, the
// gradients of its values and the pass-local number of its segment.
struct LdsSample {
    float f[3];
    float v[4];
    int seg;
};
static_assert(sizeof(LdsSample) == 32, "two 16-byte words per sample");

// Sends the 28 gradient values of every lane's voxel (id < 0: none) to the
// FP32 records, kStageRows rows at a time through the wave's staging rows:
// lanes 0..31 then take one row and lanes 32..63 the next, lane s of a half
// the record slot s (0..26 SH, 28 density, 29 the touched byte), so every
// instruction covers two 128-B gradient lines.  Called by the whole wave.
__device__ __forceinline__ void flush_voxel_rows(float *stage, const float acc[28], int id, float *grad,
                                                 uint8_t *touched) {
    const int L = lane_id();
    const int s = L & 31;
    const int half = L >> 5;
    const int col = s < PLX_NSH ? s : PLX_NSH;  // staged column of the lane's slot
#pragma unroll
    for (int h = 0; h < kWave / kStageRows; ++h) {
        const bool mine = L / kStageRows == h;
        if (__ballot(id >= 0 && mine) == 0) continue;
        if (mine) {
            float *row = stage + (L % kStageRows) * kStageStride;
#pragma unroll
            for (int v = 0; v < 28; ++v) row[v] = acc[v];
            row[28] = __int_as_float(id);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < kStageRows / 2; ++u) {
            const float *row = stage + (2 * u + half) * kStageStride;
            const int rid = __float_as_int(row[28]);
            const float val = row[col];
            if (rid >= 0) {
                if ((s < PLX_NSH || s == PLX_SLOT_SIGMA) && val != 0.0f)
                    unsafeAtomicAdd(grad + (int64_t)rid * PLX_REC_SLOTS + s, val);
                if (s == PLX_SLOT_SIGMA + 1) touched[rid] = 1;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Reverse recurrence of one segment (the state a lane carries along it).
struct SegState {
    double tau_after;  // optical depth after the current sample
    float gR;          // g . (radiance collected after the current sample)
};

// What the samples of a segment read while the pass's gradients are formed;
// the flush stages its rows in the same LDS afterwards.
struct SegParts {
    float4 g[kScatterSegs];     // dL/dC of the ray; w: t_near
    float t_far[kScatterSegs];
    float tau[kScatterSegs];    // optical depth after the segment's last sample of the pass
};
constexpr int kStageFloats = kScatterThreads / kWave * kStageRows * kStageStride;
static_assert(sizeof(SegParts) <= kStageFloats * sizeof(float), "the parts fit the staging rows");

// 128 registers, for two workgroups on a CU, with 23 more in scratch (80 bytes a
// lane; 27 and 96 with the Cauchy term).
template <bool CAUCHY>
__global__ __launch_bounds__(kScatterThreads) __attribute__((amdgpu_waves_per_eu(4)))
void seg_scatter_kernel(GridDev g, BinArgs a) {
    __shared__ int64_t s_soff[kScatterSegs];   // sample slot of each segment of the group
    __shared__ int s_pre[kScatterSegs + 1];    // its first sample in the group's numbering
    __shared__ float4 s_y4[kScatterSegs * 3];  // SH basis of its ray (9 of 12 floats)
    __shared__ int s_cnt[kBrickCells];         // samples per cell
    __shared__ int s_coff[kBrickCells + 1];    // first sorted position of each cell
    __shared__ __align__(16) LdsSample s_rec[kScatterCap];   // the pass's samples
    __shared__ __align__(16) float s_stage[kStageFloats];
    __shared__ int s_vid[kBrickVox];           // the brick's stored corner voxels: id
    __shared__ uint16_t s_vpos[kBrickVox];     // and position x*81 + y*9 + z in the 9^3 lattice

    if (blockIdx.x >= (unsigned)a.n_brick) return;
    const int t = threadIdx.x;
    float *s_y = reinterpret_cast<float *>(s_y4);
    float *stage = s_stage + (t / kWave) * kStageRows * kStageStride;
    SegParts &parts = *reinterpret_cast<SegParts *>(s_stage);
    // per sample of the pass, before the sort: optical thickness, then the
    // depth before the sample; its weight, then g . R after it; its g . colour
    float *s_tau = reinterpret_cast<float *>(s_rec), *s_w = s_tau + kScatterCap, *s_gc = s_w + kScatterCap;
    const int64_t jo = a.blist[blockIdx.x];
    int bxyz[3];
    brick_at(g, jo, bxyz);
    const int64_t seg0 = a.boff[jo * kLenClasses], seg1 = a.boff[(jo + 1) * kLenClasses];

    // list the stored corner voxels, in lattice order
    int n_vox = 0;
#pragma unroll
    for (int rr = 0; rr < kVoxRounds; ++rr) {
        const int p = t + rr * kScatterThreads;
        int id = -1;
        if (p < kBrickVox) {
            const int X = bxyz[0] * PLX_BRICK + p / 81, Y = bxyz[1] * PLX_BRICK + (p / 9) % 9,
                      Z = bxyz[2] * PLX_BRICK + p % 9;
            if (X < g.nx && Y < g.ny && Z < g.nz) id = g.index[((int64_t)X * g.ny + Y) * g.nz + Z];
        }
        int64_t on;
        const int at = n_vox + (int)block_scan_excl<kScatterThreads>(id >= 0 ? 1 : 0, &on);
        if (id >= 0) {
            s_vid[at] = id;
            s_vpos[at] = (uint16_t)p;
        }
        n_vox += (int)on;
    }
    float ls = 0.0f;

    for (int64_t c0 = seg0; c0 < seg1; c0 += kScatterSegs) {
        // a group of up to kScatterSegs segments; lane t < ns walks segment t
        const int ns = (int)min((int64_t)kScatterSegs, seg1 - c0);
        int occ = 0;
        SegState st = {};
        // the lane's segment: SH basis and parts to LDS (the flush of a pass
        // overwrites the parts)
        auto load_parts = [&](bool first) {
            if (t >= ns) return;
            const int64_t i = c0 + t;
            const int4 sg = a.bseg[i];
            float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 1.f};
            float4 gg = make_float4(0.f, 0.f, 0.f, 0.f);
            RayGeom r = {};
            if (seg_valid(a, sg, a.n_seg)) {
                load_ray_lane(a, sg.x, o, d);
                gg = a.g_ray[sg.x];
                (void)ray_setup(g, o, d, r);
                if (first) {
                    occ = a.nocc[i];
                    st.tau_after = a.tau_in[sg.w] + a.tau_seg[sg.w];
                    st.gR = a.gr_after[sg.w] - gg.w;  // the beta factor joins the running sum
                }
            }
            parts.g[t] = make_float4(gg.x, gg.y, gg.z, r.t_near);
            parts.t_far[t] = r.t_far;
            if (first) {
                s_soff[t] = a.soff[i];
                sh_basis_all(d, s_y + t * 12);
            }
        };
        load_parts(true);
        int64_t tot64;
        const int pre = (int)block_scan_excl<kScatterThreads>(occ, &tot64);
        const int tot = (int)tot64;
        if (t < kScatterSegs) s_pre[t] = pre;  // segments past ns hold the total
        if (t == 0) s_pre[kScatterSegs] = tot;
        __syncthreads();

        // passes over the group's samples from the last one back, so that a
        // segment longer than a pass meets its samples in reverse order
        for (int q0 = ((tot - 1) / kScatterCap) * kScatterCap; tot > 0 && q0 >= 0; q0 -= kScatterCap) {
            const int nq = min(kScatterCap, tot - q0);
            for (int c = t; c < kBrickCells; c += kScatterThreads) s_cnt[c] = 0;
            const int e_lo = max(pre, q0) - q0, e_hi = min(pre + occ, q0 + nq) - q0;  // the lane's segment
            if (q0 + nq < tot) load_parts(false);
            if (t < ns) parts.tau[t] = (float)st.tau_after;
            // load the pass's samples (slots first, then all loads)
            int seg_u[kScatterPer];
            float4 val_u[kScatterPer];
            int code_u[kScatterPer];
            auto slot_of = [&](int u) {
                return s_soff[seg_u[u]] + (q0 + u * kScatterThreads + t - s_pre[seg_u[u]]);
            };
#pragma unroll
            for (int u = 0; u < kScatterPer; ++u) {
                const int q = u * kScatterThreads + t;
                seg_u[u] = -1;
                if (q < nq) {
                    const int qq = q0 + q;
                    int lo = 0, hi = ns - 1;  // last segment whose first sample is <= qq
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (s_pre[mid] <= qq) lo = mid;
                        else hi = mid - 1;
                    }
                    seg_u[u] = lo;
                }
            }
#pragma unroll
            for (int u = 0; u < kScatterPer; ++u) {
                if (seg_u[u] < 0) continue;
                const SampleRec *rec = a.srec + slot_of(u);
                val_u[u] = rec->val;
                code_u[u] = __float_as_int(rec->pos.w);
            }
            __syncthreads();  // s_cnt cleared, the parts written; the previous pass's LDS reads done
            // count the samples per cell; the thread that has a sample finds
            // its optical thickness
            int rank_u[kScatterPer];
            float delta_u[kScatterPer];
#pragma unroll
            for (int u = 0; u < kScatterPer; ++u) {
                if (seg_u[u] < 0) continue;
                rank_u[u] = atomicAdd(&s_cnt[code_u[u] & (kBrickCells - 1)], 1);
                delta_u[u] = sample_delta(g, parts.g[seg_u[u]].w, parts.t_far[seg_u[u]], (unsigned)code_u[u] >> 9);
                s_tau[u * kScatterThreads + t] = fmaxf(val_u[u].x, 0.0f) * delta_u[u];
            }
            __syncthreads();
            {
                static_assert(kScatterThreads == kBrickCells, "one cell per thread");
                int64_t all;
                s_coff[t] = (int)block_scan_excl<kScatterThreads>(s_cnt[t], &all);
                if (t == 0) s_coff[kBrickCells] = (int)all;
            }
            // the depth before each sample, back along each segment
            for (int e = e_hi - 1; e >= e_lo; e -= kChainU) {
                float x[kChainU];
#pragma unroll
                for (int u = 0; u < kChainU; ++u) x[u] = s_tau[max(e - u, e_lo)];
#pragma unroll
                for (int u = 0; u < kChainU; ++u) {
                    if (e - u < e_lo) break;
                    st.tau_after = fmax(st.tau_after - (double)x[u], 0.0);
                    s_tau[e - u] = (float)st.tau_after;
                }
            }
            __syncthreads();
            // each sample's weight and g . colour
            float em_u[kScatterPer];
#pragma unroll
            for (int u = 0; u < kScatterPer; ++u) {
                if (seg_u[u] < 0) continue;
                const int q = u * kScatterThreads + t;
                const float4 gr = parts.g[seg_u[u]], v = val_u[u];
                em_u[u] = -expm1f(-(fmaxf(v.x, 0.0f) * delta_u[u]));
                s_w[q] = expf(-s_tau[q]) * em_u[u];
                s_gc[q] = gr.x * fmaxf(v.y, 0.0f) + gr.y * fmaxf(v.z, 0.0f) + gr.z * fmaxf(v.w, 0.0f);
            }
            __syncthreads();
            // g . R after each sample, back along each segment
            for (int e = e_hi - 1; e >= e_lo; e -= kChainU) {
                float x[kChainU], y[kChainU];
#pragma unroll
                for (int u = 0; u < kChainU; ++u) {
                    x[u] = s_w[max(e - u, e_lo)];
                    y[u] = s_gc[max(e - u, e_lo)];
                }
#pragma unroll
                for (int u = 0; u < kChainU; ++u) {
                    if (e - u < e_lo) break;
                    s_w[e - u] = st.gR;
                    st.gR += x[u] * y[u];
                }
            }
            __syncthreads();
            LdsSample mine[kScatterPer];
#pragma unroll
            for (int u = 0; u < kScatterPer; ++u) {
                if (seg_u[u] < 0) continue;
                const int q = u * kScatterThreads + t;
                const float4 gr = parts.g[seg_u[u]], v = val_u[u], pos = a.srec[slot_of(u)].pos;
                // the segment's next sample, or the end of its part of the pass
                const bool last = q + 1 >= nq || q0 + q + 1 >= s_pre[seg_u[u] + 1];
                const float T_after = expf(-(last ? parts.tau[seg_u[u]] : s_tau[q + 1]));
                const float wk = expf(-s_tau[q]) * em_u[u];
                const float cs = CAUCHY ? cauchy_grad(a.pri, v.x, &ls) : 0.0f;
                mine[u].f[0] = pos.x;
                mine[u].f[1] = pos.y;
                mine[u].f[2] = pos.z;
                mine[u].v[0] = v.x > 0.0f ? delta_u[u] * (T_after * s_gc[q] - s_w[q]) + cs : 0.0f;
                mine[u].v[1] = v.y > 0.0f ? wk * gr.x : 0.0f;
                mine[u].v[2] = v.z > 0.0f ? wk * gr.y : 0.0f;
                mine[u].v[3] = v.w > 0.0f ? wk * gr.z : 0.0f;
                mine[u].seg = seg_u[u];
            }
            __syncthreads();  // the chains' values read
            // sort by cell: every sample into its cell's range
#pragma unroll
            for (int u = 0; u < kScatterPer; ++u)
                if (seg_u[u] >= 0) s_rec[s_coff[code_u[u] & (kBrickCells - 1)] + rank_u[u]] = mine[u];
            __syncthreads();

            // each lane sums its voxels' contributions and flushes them
#pragma unroll 1
            for (int v0 = 0; v0 < n_vox; v0 += kScatterThreads) {
                const int vi = v0 + t;
                const int id = vi < n_vox ? s_vid[vi] : -1, p = vi < n_vox ? s_vpos[vi] : 0;
                float acc[28];
#pragma unroll
                for (int v = 0; v < 28; ++v) acc[v] = 0.0f;
                // the sample ranges of the voxel's (up to) 8 cells, the
                // non-empty ones first in corner order (start | count << 11 |
                // corner << 22), walked as one list: a wave then runs as long
                // as its busiest lane's total, not the sum over the corners of
                // each corner's busiest lane
                unsigned qr[8];
                int nne = 0;
                {
                    const int px = p / 81, py = (p / 9) % 9, pz = p % 9;
#pragma unroll
                    for (int j = 0; j < 8; ++j) qr[j] = 0u;
#pragma unroll
                    for (int o = 0; o < 8; ++o) {
                        // the voxel is corner o (x: bit 2) of the cell p - o
                        const int cx = px - ((o >> 2) & 1), cy = py - ((o >> 1) & 1), cz = pz - (o & 1);
                        unsigned ent = 0u;
                        if (id >= 0 && cx >= 0 && cy >= 0 && cz >= 0 && cx < PLX_BRICK && cy < PLX_BRICK &&
                            cz < PLX_BRICK) {
                            const int cell = (cx << 6) | (cy << 3) | cz;
                            const int r0 = s_coff[cell], n = s_coff[cell + 1] - r0;
                            if (n > 0) ent = (unsigned)r0 | ((unsigned)n << 11) | ((unsigned)o << 22);
                        }
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if (ent != 0u && j == nne) qr[j] = ent;
                        nne += ent != 0u ? 1 : 0;
                    }
                }
                const bool any = nne > 0;
                int e = (int)(qr[0] & 0x7ffu), cnt = (int)((qr[0] >> 11) & 0x7ffu), oc = (int)(qr[0] >> 22);
#pragma unroll
                for (int j = 0; j < 7; ++j) qr[j] = qr[j + 1];
                qr[7] = 0u;
#pragma unroll 1
                for (;;) {
                    // the wave leaves together; a lane that is done adds nothing
                    const bool live = cnt > 0;
                    if (__ballot(live) == 0) break;
                    // the whole sample in two 16-byte reads, f0 f1 f2 v0 | v1 v2 v3 seg
                    // (a done lane reads sorted sample 0, a valid one)
                    const float4 *sp = reinterpret_cast<const float4 *>(s_rec + (live ? e : 0));
                    const float4 sa = sp[0], sb = sp[1];
                    const float wx = (oc & 4) ? sa.x : 1.0f - sa.x;
                    const float wy = (oc & 2) ? sa.y : 1.0f - sa.y;
                    const float wz = (oc & 1) ? sa.z : 1.0f - sa.z;
                    const float w = wx * wy * wz;
                    const int sy = __float_as_int(sb.w) * 3;
                    const float4 y0 = s_y4[sy], y1 = s_y4[sy + 1], y2 = s_y4[sy + 2];
                    const float yy[9] = {y0.x, y0.y, y0.z, y0.w, y1.x, y1.y, y1.z, y1.w, y2.x};
                    const float a_r = live ? w * sb.x : 0.0f, a_g = live ? w * sb.y : 0.0f,
                                a_b = live ? w * sb.z : 0.0f;
#pragma unroll
                    for (int l = 0; l < 9; ++l) {
                        acc[l] += a_r * yy[l];
                        acc[9 + l] += a_g * yy[l];
                        acc[18 + l] += a_b * yy[l];
                    }
                    const float s27 = acc[27] + w * sa.w;
                    acc[27] = live ? s27 : acc[27];
                    ++e;
                    cnt -= live ? 1 : 0;
                    if (live && cnt == 0) {
                        // next range (an empty entry leaves the lane done)
                        e = (int)(qr[0] & 0x7ffu);
                        cnt = (int)((qr[0] >> 11) & 0x7ffu);
                        oc = (int)(qr[0] >> 22);
#pragma unroll
                        for (int j = 0; j < 7; ++j) qr[j] = qr[j + 1];
                        qr[7] = 0u;
                    }
                }
                flush_voxel_rows(stage, acc, any ? id : -1, a.grad, a.touched);
            }
            __syncthreads();
        }
    }
    if (CAUCHY && a.pri.loss) {
        // the lanes that have samples, not those that own segments, hold the
        // loss: one atomic per workgroup, as one of every wave queued up at
        // the address (65,536 rays through a dense 200^3 grid 3.13 ms a call,
        // now 2.39, without the priors 2.33)
        double *part = reinterpret_cast<double *>(s_stage);  // the last flush is done
        double sum = (double)ls;
#pragma unroll
        for (int m = kWave / 2; m >= 1; m >>= 1) sum += __shfl_xor(sum, m);
        if (lane_id() == 0) part[t / kWave] = sum;
        __syncthreads();
        if (t == 0) {
            for (int w = 1; w < kScatterThreads / kWave; ++w) sum += part[w];
            if (sum != 0.0) unsafeAtomicAdd(a.pri.loss, (double)a.pri.lambda_s * sum);
        }
    }
}

// ------------------------------------------------------------ maximum sample weight

// Position, in a brick's 9^3 corner lattice, of corner c relative to corner 0
// of its cell.
__device__ __forceinline__ constexpr int corner_position(int c) {
    return ((c >> 2) & 1) * 81 + ((c >> 1) & 1) * 9 + (c & 1);
}

// Raises the maxima of the corners of the cell at position p.
__device__ __forceinline__ void raise_corners(unsigned *s_max, int p, float w) {
    const unsigned cand = __float_as_uint(w);
#pragma unroll
    for (int c = 0; c < 8; ++c)
        if (s_max[p + corner_position(c)] < cand) atomicMax(&s_max[p + corner_position(c)], cand);
}

// The weight pass runs in brick order in two phases over the same segments.
// Phase 0 gives each segment's optical depth (density only; no colour is
// needed), the combine step turns those into the depth before each segment,
// and phase 1 replays the segment from there: sample k's weight is
// T_k (1 - exp(-sigma_k delta_k)) with T_k from the ray's running optical
// depth, exactly as the forward pass composites, and every non-NULL corner of
// the sample's cell is raised to the largest weight it sees.
//
// One workgroup per brick: the cell bits, the densities of the 9^3 corners
// and their maxima sit in LDS (6 KB), a lane walks a segment (segments of one
// length class side by side), and a voxel gets one atomic maximum per brick.
// With one lane per segment on global memory the chains of index entries,
// densities (one 4-byte read of a 128-byte record each) and the maxima
// bounded both phases: 1M rays on 256^3 0.81 + 2.73 ms, now 0.14 + 0.19.
//
// SPARSE, for bricks with few segments: a wave per brick, which first marks
// the corners that its samples read and loads only these.  Loading them all
// costs a brick 729 lines of 128 bytes however few rays cross it (5,000 rays
// through a dense 256x256x128 grid, 6 segments a brick, 0.59 ms; so 0.24, and
// 0.32 with a lane per segment).  In us, all / SPARSE, by segments a brick:
// 16,000 bricks 5 499 / 228, 18 535 / 389, 24 653 / 447, 55 568 / 591, 71 677 /
// 671, 184 675 / 890; 4,096 bricks 11 172 / 117, 29 180 / 167, 45 178 / 190.
// Too few waves are left with fewer bricks: 1,733 92 / 67, 794 66 / 62, 832 with
// 4 segments 63 / 68, 300 40 / 60.
constexpr int64_t kSparseSegs = 32, kSparseBricks = 1024;
template <int DT, int PHASE, bool SPARSE>
__global__ __launch_bounds__(SPARSE ? kWave : kThreads) void seg_weight_kernel(GridDev g, BinArgs a) {
    constexpr int T = SPARSE ? kWave : kThreads;
    constexpr int kRounds = (kBrickVox + T - 1) / T;
    __shared__ float s_sigma[kBrickVox];
    __shared__ unsigned s_max[kBrickVox];
    __shared__ uint32_t s_occ[kBrickCells / 32];
    __shared__ uint32_t s_need[SPARSE ? (kBrickVox + 31) / 32 : 1];
    if (blockIdx.x >= (unsigned)a.n_brick) return;
    const int t = threadIdx.x;
    const int64_t jo = a.blist[blockIdx.x];
    int b[3];
    brick_at(g, jo, b);
    const int b0[3] = {b[0] * PLX_BRICK, b[1] * PLX_BRICK, b[2] * PLX_BRICK};
    const int64_t seg0 = a.boff[jo * kLenClasses], seg1 = a.boff[(jo + 1) * kLenClasses];
    // calls f(corner position of the cell, sample) for the occupied samples of a segment
    auto walk = [&](const int4 &sg, auto &&f) {
        float o[3], d[3];
        load_ray_lane(a, sg.x, o, d);
        RayGeom r;
        ray_setup(g, o, d, r);
        for (int k = sg.y; k <= sg.z; ++k) {
            const Sample smp = sample_at(g, r, k);
            const int lx = smp.cell[0] - b0[0], ly = smp.cell[1] - b0[1], lz = smp.cell[2] - b0[2];
            if ((unsigned)lx >= PLX_BRICK || (unsigned)ly >= PLX_BRICK || (unsigned)lz >= PLX_BRICK) continue;
            const int cell = (lx << 6) | (ly << 3) | lz;
            if ((s_occ[cell >> 5] >> (cell & 31)) & 1u) f(lx * 81 + ly * 9 + lz, smp);
        }
    };
    if (t < kBrickCells / 32) s_occ[t] = g.occ[brick_id(g, b) * (kBrickCells / 32) + t];
    if constexpr (SPARSE) {
        if (t < (kBrickVox + 31) / 32) s_need[t] = 0u;
        __syncthreads();
        for (int64_t i = seg0 + t; i < seg1; i += T) {
            const int4 sg = a.bseg[i];
            if (!seg_valid(a, sg, a.n_seg)) continue;
            int cur = -1;
            walk(sg, [&](int p, const Sample &) {
                if (p == cur) return;
                cur = p;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const int q = p + corner_position(c);
                    atomicOr(&s_need[q >> 5], 1u << (q & 31));
                }
            });
        }
        __syncthreads();
    }
    int vid[kRounds];
#pragma unroll
    for (int rr = 0; rr < kRounds; ++rr) {
        const int p = t + rr * T;
        vid[rr] = -1;
        if (p < kBrickVox && (!SPARSE || ((s_need[p >> 5] >> (p & 31)) & 1u))) {
            const int X = b0[0] + p / 81, Y = b0[1] + (p / 9) % 9, Z = b0[2] + p % 9;
            if (X < g.nx && Y < g.ny && Z < g.nz) vid[rr] = g.index[((int64_t)X * g.ny + Y) * g.nz + Z];
        }
    }
#pragma unroll
    for (int rr = 0; rr < kRounds; ++rr) {
        const int p = t + rr * T;
        if (p < kBrickVox) {
            s_sigma[p] = vid[rr] >= 0 ? rec_sigma<DT>(g.data, vid[rr]) : 0.0f;
            s_max[p] = 0u;
        }
    }
    __syncthreads();

    for (int64_t i = seg0 + t; i < seg1; i += T) {
        const int4 sg = a.bseg[i];
        if (!seg_valid(a, sg, a.n_seg)) continue;
        double tau = PHASE == 0 ? 0.0 : a.tau_in[sg.w];
        int cur = -1;      // corner position of the current cell's lower corner
        float wmax = 0.0f; // largest weight of the run of samples in it
        walk(sg, [&](int p, const Sample &smp) {
            const float wx[2] = {1.0f - smp.f[0], smp.f[0]}, wy[2] = {1.0f - smp.f[1], smp.f[1]},
                        wz[2] = {1.0f - smp.f[2], smp.f[2]};
            float sp = 0.0f;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                sp += wx[(c >> 2) & 1] * wy[(c >> 1) & 1] * wz[c & 1] * s_sigma[p + corner_position(c)];
            const float sd = fmaxf(sp, 0.0f) * smp.delta;
            if (PHASE == 1) {
                const float wk = expf(-(float)tau) * (-expm1f(-sd));
                if (p != cur) {
                    if (cur >= 0) raise_corners(s_max, cur, wmax);
                    cur = p;
                    wmax = 0.0f;
                }
                wmax = fmaxf(wmax, wk);
            }
            tau += (double)sd;
        });
        if (PHASE == 0) a.tau_seg[sg.w] = tau;
        else if (cur >= 0) raise_corners(s_max, cur, wmax);
    }
    if (PHASE == 0) return;
    __syncthreads();
    // non-negative floats order as their bit patterns; wmax only grows, so a
    // value already at least the candidate makes the atomic unnecessary
#pragma unroll
    for (int rr = 0; rr < kRounds; ++rr) {
        const int p = t + rr * T;
        if (p >= kBrickVox || vid[rr] < 0) continue;
        const unsigned cand = s_max[p];
        unsigned *q = reinterpret_cast<unsigned *>(a.wmax) + vid[rr];
        if (cand > 0u && __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < cand) atomicMax(q, cand);
    }
}

// ------------------------------------------------------------------ novel views

// Pixel-centred pinhole ray of pixel (px, py) of a view, in FP64 with a fixed
// operation order (no contraction), rounded to FP32 once.
__device__ inline void camera_ray(const plx_view &v, int px, int py, float o[3], float d[3]) {
#pragma clang fp contract(off)
    const double x = ((double)px + 0.5 - 0.5 * (double)v.width) / v.focal;
    const double yv = -(((double)py + 0.5 - 0.5 * (double)v.height) / v.focal);
    const double z = -1.0;
    double dv[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) dv[a] = v.c2w[4 * a + 0] * x + v.c2w[4 * a + 1] * yv + v.c2w[4 * a + 2] * z;
    const double nrm = sqrt(dv[0] * dv[0] + dv[1] * dv[1] + dv[2] * dv[2]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        d[a] = (float)(dv[a] / nrm);
        o[a] = (float)v.c2w[4 * a + 3];
    }
}

// How a view is cut: a workgroup is one wave and marches kW x kH pixels, P
// lanes each.  One wave per workgroup and one workgroup per tile let the
// dispatcher even out tiles of very different cost (with four waves and 256
// pixels per workgroup and a queue of tiles, an 800x800 view of a 512^3 scene
// had 18% of its wave slots filled on average).  Many lanes a ray shorten the
// chain of rounds of a view that does not fill the chip, few lanes share a
// wave's set-up among more rays.  Measured with 16 / 8 / 4 lanes (ms, FP16
// records): 200x200 on 512^3 0.15 / 0.25 / 0.56, 400x400 on 512^3 0.24 / 0.32 /
// 0.65, 800x800 on 512^3 0.70 / 0.66 / 0.72, 1280x720 on 256^3 0.90 / 0.76 /
// 0.70, 1920x1080 on 256^3 1.81 / 1.50 / 1.26.  From 256x256 pixels on 16
// lanes fill the chip alone, and 8 leave room for another stream's launch
// (two 288x288 views on two streams: 0.49 ms together, 0.67 one after the
// other).  The choice follows the view, not its launch: the order of a ray's
// additions depends on the cut, and a view has the same bits whatever it is
// batched with.
template <int P_> struct ViewsCut {
    static constexpr int P = P_, M = 4;
    static constexpr int kW = P == 16 ? 2 : 4, kH = kWave / P / kW;
};
inline int view_lanes(const plx_view &v) {
    const int64_t n = (int64_t)v.width * v.height;
    return n < (1 << 16) ? 16 : (n < (3 << 18) ? 8 : 4);
}

constexpr int kLaneTile = 8;  // pixels of a PLX_VIEW_LANE view's tiles along x and y

// Tiles of a view (host), by its lanes per ray.
template <class CUT> inline int64_t tiles_of(const plx_view &v) {
    return (int64_t)((v.width + CUT::kW - 1) / CUT::kW) * ((v.height + CUT::kH - 1) / CUT::kH);
}
// Workgroups of a launch; beyond it (16.7M pixels) they stride over the tiles
// (a grid holds fewer than 2^32 threads, a view may have 2^32 pixels).
constexpr int64_t kViewsMaxBlocks = 1 << 20;

// Scene table (device, written by plx_scene_table_set): a 256-byte header,
// then one GridDev per scene.
constexpr unsigned kSceneMagic = 0x504c5853u;
struct SceneTableHeader {
    unsigned magic;
    int n_scenes;
    int sh_dtype;
};
constexpr int64_t kSceneTableHead = 256;

// Views reach the device as kernel arguments (no copy engine, no setup
// launch, no host buffer that must outlive the call): one launch renders up
// to kViewsPerLaunch views, and a longer list is split into several.
constexpr int kViewsPerLaunch = 24;

// The caller's queue buffer (PLX_VIEWS_QUEUE_BYTES, zero before first use)
// holds a sticky status word; the dispatcher hands out the tiles.
struct ViewsQueue {
    unsigned reserved[3];
    unsigned status;
};

struct ViewsArgs {
    const SceneTableHeader *table;
    const GridDev *scenes;
    plx_view v[kViewsPerLaunch];
    int64_t tile_start[kViewsPerLaunch + 1];
    int lanes[kViewsPerLaunch];  // per ray (view_lanes)
    int n_views;
    unsigned *status;
    float bg[3];
    float *rgb_out;
};

// Descriptors of the scene table reach the device the same way.
constexpr int kSetupItems = 24;

struct SceneSetupArgs {
    GridDev g[kSetupItems];
    int first, count, n_scenes, sh_dtype;
    SceneTableHeader *table;
    GridDev *scenes;
};

__global__ void scene_setup_kernel(SceneSetupArgs a) {
    const int i = threadIdx.x;
    if (i < a.count) a.scenes[a.first + i] = a.g[i];
    if (a.first == 0 && i == 0) {
        a.table->magic = kSceneMagic;
        a.table->n_scenes = a.n_scenes;
        a.table->sh_dtype = a.sh_dtype;
    }
}

// One tile of a view: the wave generates the rays of its pixels and marches
// them.
template <int DT, class CUT>
__device__ __forceinline__ void render_tile(const GridDev &g, const plx_view &v, int64_t tile, const float bg[3],
                                            float *rgb_out, void *lds) {
    constexpr int P = CUT::P, M = CUT::M;
    MarchLds<P, M> &sh = *static_cast<MarchLds<P, M> *>(lds);
    const int tpr = (v.width + CUT::kW - 1) / CUT::kW;
    const int slot = lane_id() / P;
    const int px = (int)(tile % tpr) * CUT::kW + slot % CUT::kW;
    const int py = (int)(tile / tpr) * CUT::kH + slot / CUT::kW;
    const bool in = px < v.width && py < v.height;
    float o[3], d[3];
    camera_ray(v, min(px, v.width - 1), min(py, v.height - 1), o, d);
    RayGeom r;
    const int n = in ? ray_setup(g, o, d, r) : 0;
    march_basis(sh, d);
    float C[3];
    double tau;
    march_rays<DT>(g, sh, r, n, C, tau, NoRecord{});
    if (in && lane_id() % P == 0) {
        const float T_final = expf(-(float)tau);
        float *out = rgb_out + 3 * (v.out_offset + (int64_t)py * v.width + px);
#pragma unroll
        for (int c3 = 0; c3 < 3; ++c3) out[c3] = C[c3] + T_final * bg[c3];
    }
}

// Front-to-back march of one ray by one lane (Eq. (1)): the colour before the
// background is added and the optical depth.
template <int DT>
__device__ __forceinline__ void march_lane(const GridDev &g, const RayGeom &r, int n, const float y[9], float C[3],
                                           double &tau) {
    C[0] = C[1] = C[2] = 0.0f;
    tau = 0.0;
    CornerCache cc;
    cc.cell[0] = cc.cell[1] = cc.cell[2] = -1;
    Q4 none[8];
    Queue noq{};
    const RaySkip rs = ray_skip(g, r);
    for (int k = 0; k < n;) {
        {
            const Sample s = sample_at(g, r, k);
            const int b[3] = {s.cell[0] / PLX_BRICK, s.cell[1] / PLX_BRICK, s.cell[2] / PLX_BRICK};
            const int D = g.bdist[brick_id(g, b)];
            if (D > 0) {
                k += skip_box(g, r, rs, k, b, D - 1) + 1;
                continue;
            }
        }
        for (uint32_t mask = chunk_bits(g, r, n, k); mask != 0u; mask &= mask - 1u) {
            const Sample s = sample_at(g, r, k + __builtin_ctz(mask));
            move_to<DT, false>(g, cc, s.cell, none, noq, y);
            float w[8];
            corner_weights(s.f, w);
            const Q4 v = interpolate(cc, w);
            const float sd = fmaxf(v.s, 0.0f) * s.delta;
            const float wk = expf(-(float)tau) * (-expm1f(-sd));
            C[0] += wk * fmaxf(v.r, 0.0f);
            C[1] += wk * fmaxf(v.g, 0.0f);
            C[2] += wk * fmaxf(v.b, 0.0f);
            tau += (double)sd;
        }
        k += kChunk;
    }
}

// Novel views, a tile per workgroup (one wave).  128 registers for four waves
// on a SIMD, with 3 (FP32) to 7 (16-bit) in scratch.
template <int DT>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(4)))
void views_kernel(ViewsArgs a) {
    constexpr size_t kLds = sizeof(MarchLds<4, ViewsCut<4>::M>);  // the largest of the cuts
    __shared__ __align__(16) unsigned char lds[kLds];
    // a table of other scenes' storage type (or not a scene table): nothing
    // is rendered and the status word says so
    const bool ok = a.table->magic == kSceneMagic && a.table->sh_dtype == DT;
    for (int64_t tile = blockIdx.x; tile < a.tile_start[a.n_views]; tile += gridDim.x) {
        int lo = 0;  // the view of the tile
        for (int i = 1; i < a.n_views; ++i)
            if (a.tile_start[i] <= tile) lo = i;
        const plx_view &v = a.v[lo];
        if (!ok || v.scene >= a.table->n_scenes) {
            if (threadIdx.x == 0) atomicOr(a.status, 1u);
            continue;
        }
        const GridDev g = uniform_grid(a.scenes[v.scene]);
        const int64_t tl = tile - a.tile_start[lo];
        if (a.lanes[lo] == 16)
            render_tile<DT, ViewsCut<16>>(g, v, tl, a.bg, a.rgb_out, lds);
        else if (a.lanes[lo] == 8)
            render_tile<DT, ViewsCut<8>>(g, v, tl, a.bg, a.rgb_out, lds);
        else
            render_tile<DT, ViewsCut<4>>(g, v, tl, a.bg, a.rgb_out, lds);
    }
}

// Views with PLX_VIEW_LANE: a lane per ray, a tile of kLaneTile^2 pixels per
// workgroup (one wave).  A kernel of its own, as the march's 128 registers do
// not hold both (4 to 5 times slower, spilled), and launched only for such
// views: waves that find nothing to do still wait for their place behind other
// streams' launches (p50 of a half-loaded server 1.46 -> 2.11 ms).
template <int DT>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(3)))
void views_lane_kernel(ViewsArgs a) {
    const bool ok = a.table->magic == kSceneMagic && a.table->sh_dtype == DT;
    for (int64_t tile = blockIdx.x; tile < a.tile_start[a.n_views]; tile += gridDim.x) {
        int lo = 0;  // the view of the tile
        for (int i = 1; i < a.n_views; ++i)
            if (a.tile_start[i] <= tile) lo = i;
        const plx_view &v = a.v[lo];
        if (!ok || v.scene >= a.table->n_scenes) {
            if (threadIdx.x == 0) atomicOr(a.status, 1u);
            continue;
        }
        const GridDev g = uniform_grid(a.scenes[v.scene]);
        const int64_t tl = tile - a.tile_start[lo];
        const int tpr = (v.width + kLaneTile - 1) / kLaneTile;
        const int px = (int)(tl % tpr) * kLaneTile + lane_id() % kLaneTile;
        const int py = (int)(tl / tpr) * kLaneTile + lane_id() / kLaneTile;
        if (px >= v.width || py >= v.height) continue;
        float o[3], d[3];
        camera_ray(v, px, py, o, d);
        RayGeom r;
        const int n = ray_setup(g, o, d, r);
        float y[9];
        sh_basis_all(d, y);
        float C[3];
        double tau;
        march_lane<DT>(g, r, n, y, C, tau);
        const float T_final = expf(-(float)tau);
        float *out = a.rgb_out + 3 * (v.out_offset + (int64_t)py * v.width + px);
#pragma unroll
        for (int c3 = 0; c3 < 3; ++c3) out[c3] = C[c3] + T_final * a.bg[c3];
    }
}


// Work counters (one thread per ray; diagnostic, not a hot path).
__global__ void stats_kernel(GridDev g, const float *rays_o, const float *rays_d, int64_t n_rays,
                             uint32_t *cell_mark, uint32_t *vox_mark, unsigned long long *cnt) {
    const int64_t ray = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long n_all = 0, n_occ = 0;
    if (ray < n_rays) {
        float o[3], d[3];
        for (int i = 0; i < 3; ++i) {
            o[i] = rays_o[3 * ray + i];
            d[i] = rays_d[3 * ray + i];
        }
        RayGeom r;
        const int n = ray_setup(g, o, d, r);
        n_all = n;
        int64_t last = -1;
        for (int k = 0; k < n; ++k) {
            const Sample s = sample_at(g, r, k);
            const int64_t lin = cell_id(g, s.cell);
            if (!cell_occupied(g, s.cell)) continue;
            ++n_occ;
            if (lin == last) continue;
            last = lin;
            for (int c = 0; c < 8; ++c) {
                const int64_t v = lin + corner_offset(g, c);
                atomicOr(cell_mark + (v >> 5), 1u << (v & 31));
                const int id = g.index[v];
                if (id >= 0) atomicOr(vox_mark + (id >> 5), 1u << (id & 31));
            }
        }
    }
    for (int m = 32; m >= 1; m >>= 1) {
        n_all += __shfl_xor(n_all, m);
        n_occ += __shfl_xor(n_occ, m);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&cnt[0], n_all);
        atomicAdd(&cnt[1], n_occ);
    }
}

// Adds the exclusive scan of n counts into out[0..n] (out[n] = total) to a.
// tmp: 2*nb+1 int64 where nb = ceil(n / kScanTile).
int add_scan(ScanArgs &a, const unsigned *c, int64_t n, int stride, int64_t *out, int64_t *tmp, int64_t *total,
             const char *fn) {
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb < 1 || nb > 0x1fffffff) return fail(PLX_EINVAL, "%s: bad scan size", fn);
    a.of[a.n_of++] = {c, n, nb, stride, tmp, tmp + nb, out, total};
    return PLX_OK;
}

int run_scans(const ScanArgs &a, hipStream_t s, const char *fn) {
    int64_t nb = 0;
    for (int k = 0; k < a.n_of; ++k) nb += a.of[k].nb;
    count_sum_kernel<<<(unsigned)nb, kScanT, 0, s>>>(a);
    int rc = check_launch(fn);
    if (rc) return rc;
    block_offsets_kernel<<<(unsigned)a.n_of, kScanT, 0, s>>>(a);
    if ((rc = check_launch(fn))) return rc;
    count_scan_kernel<<<(unsigned)nb, kScanT, 0, s>>>(a);
    return check_launch(fn);
}

inline int64_t scan_tmp_words(int64_t n) { return 2 * ((n + kScanTile - 1) / kScanTile) + 1; }
inline int64_t align256(int64_t x) { return (x + 255) / 256 * 256; }

// ------------------------------------------------------------ caller-owned bins
//
// The work lists of a batch live in two caller-owned buffers (plx_bins):
// the ray buffer holds the per-ray segment counts and offsets, the per-bin
// counts, cursors and offsets, the scan temporaries and a status word; the
// segment buffer holds the bin-major segment records and the per-segment
// values the render passes hand from one kernel to the next.

struct RayBufLayout {
    int64_t nseg, segoff, gray, bcount, bcursor, status, boff, scan;
    // per-bin sample counts (samples == true only)
    int64_t nbrick, bsoff, blist;
    int64_t bytes;
    bool samples;
};

// samples: with the per-bin sample counts and the brick list that the
// recorded backward needs (every caller-owned ray buffer has them; the
// fixed scratch of plx_render_train_static does not).
RayBufLayout ray_buf_layout(int64_t n_rays, int64_t nbk, bool samples = true) {
    RayBufLayout l = {};
    l.samples = samples;
    int64_t off = 0;
    l.nseg = off; off += align256(n_rays * 4);
    l.segoff = off; off += align256((n_rays + 1) * 8);
    l.gray = off; off += align256(n_rays * 16);
    // bin counts, cursors and the status word are cleared by one launch
    if (samples) {
        // 64-bit (segments, sample slots) counters and cursors, the status
        // word and the brick counter, cleared by one launch
        l.bcount = off; off += nbk * 8;
        l.bcursor = off; off += nbk * 8;
        l.status = off; off += 4;
        l.nbrick = off; off = align256(off + 4);
    } else {
        l.bcount = off; off += nbk * 4;
        l.bcursor = off; off += nbk * 4;
        l.status = off; off += align256(2 * nbk * 4 + 4) - 2 * nbk * 4;
    }
    l.boff = off; off += align256((nbk + 1) * 8);
    if (samples) {
        l.bsoff = off; off += align256((nbk + 1) * 8);
        l.blist = off; off += align256(nbk / kLenClasses * 4);
    }
    // (the segment and the sample offsets of the bins are scanned together;
    // the second has its temporaries in the list of bricks, made afterwards)
    l.scan = off; off += align256((scan_tmp_words(n_rays) + scan_tmp_words(nbk)) * 8);
    l.bytes = off;
    return l;
}

struct SampBufLayout {
    int64_t soff, nocc, srec, bytes;
};

SampBufLayout samp_buf_layout(int64_t n_seg, int64_t n_samp) {
    SampBufLayout l;
    int64_t off = 0;
    l.soff = off; off += align256(n_seg * 8);
    l.nocc = off; off += align256(n_seg * 4);
    l.srec = off; off += align256(n_samp * (int64_t)sizeof(SampleRec));
    l.bytes = off;
    return l;
}

// Sample slots one call handles (the scatter numbers a pass's samples with
// 32-bit integers; the records are addressed with 64-bit offsets).
constexpr int64_t kMaxSampBinned = (int64_t)1 << 40;

struct SegBufLayout {
    int64_t bseg, tseg, cseg, tin, gra, bytes;
};

SegBufLayout seg_buf_layout(int64_t n_seg) {
    SegBufLayout l;
    int64_t off = 0;
    l.bseg = off; off += align256(n_seg * 16);
    l.tseg = off; off += align256(n_seg * 8);
    l.cseg = off; off += align256(n_seg * 16);
    l.tin = off; off += align256(n_seg * 8);
    l.gra = off; off += align256(n_seg * 4);
    l.bytes = off;
    return l;
}

constexpr int64_t kMaxRaysBinned = 0x7fffffffLL - kThreads;

// Points a's per-ray and per-bin arrays into a ray buffer.
void attach_ray_buf(BinArgs &a, void *ray_buf, const RayBufLayout &l) {
    char *base = static_cast<char *>(ray_buf);
    a.nseg = reinterpret_cast<unsigned *>(base + l.nseg);
    a.seg_off = reinterpret_cast<int64_t *>(base + l.segoff);
    a.g_ray = reinterpret_cast<float4 *>(base + l.gray);
    a.status = reinterpret_cast<unsigned *>(base + l.status);
    a.boff = reinterpret_cast<int64_t *>(base + l.boff);
    if (l.samples) {
        a.bcnt64 = reinterpret_cast<unsigned long long *>(base + l.bcount);
        a.bcur64 = reinterpret_cast<unsigned long long *>(base + l.bcursor);
        a.bcount = reinterpret_cast<unsigned *>(base + l.bcount);  // the low halves, read at stride 2
        a.nbrick = reinterpret_cast<unsigned *>(base + l.nbrick);
        a.totals = reinterpret_cast<int64_t *>(base + l.nbrick + 4);
        a.bsoff = reinterpret_cast<int64_t *>(base + l.bsoff);
        a.blist = reinterpret_cast<unsigned *>(base + l.blist);
    } else {
        a.bcount = reinterpret_cast<unsigned *>(base + l.bcount);
        a.bcursor = reinterpret_cast<unsigned *>(base + l.bcursor);
    }
}

// Points a's recorded-backward arrays into a sample buffer.
void attach_samp_buf(BinArgs &a, void *samp_buf, const SampBufLayout &l) {
    char *b = static_cast<char *>(samp_buf);
    a.soff = reinterpret_cast<int64_t *>(b + l.soff);
    a.nocc = reinterpret_cast<int *>(b + l.nocc);
    a.srec = reinterpret_cast<SampleRec *>(b + l.srec);
}

// Points a's per-segment arrays into a segment buffer.
void attach_seg_buf(BinArgs &a, void *seg_buf, const SegBufLayout &l) {
    char *b2 = static_cast<char *>(seg_buf);
    a.bseg = reinterpret_cast<int4 *>(b2 + l.bseg);
    a.tau_seg = reinterpret_cast<double *>(b2 + l.tseg);
    a.c_seg = reinterpret_cast<float4 *>(b2 + l.cseg);
    a.tau_in = reinterpret_cast<double *>(b2 + l.tin);
    a.gr_after = reinterpret_cast<float *>(b2 + l.gra);
}

int check_buf(const void *p, int64_t have, int64_t need, const char *what, const char *fn) {
    if (!p) return fail(PLX_EINVAL, "%s: %s is NULL", fn, what);
    if (reinterpret_cast<uintptr_t>(p) % 256) return fail(PLX_EINVAL, "%s: %s must be 256-byte aligned", fn, what);
    if (have < need)
        return fail(PLX_EINVAL, "%s: %s of %lld bytes, need %lld", fn, what, (long long)have, (long long)need);
    return PLX_OK;
}

// Validates bins against the grid and batch of a render call and points a's
// arrays into them.
int attach_bins(const plx_grid *grid, const plx_bins *bins, int64_t n_rays, BinArgs &a, const char *fn) {
    if (!bins) return fail(PLX_EINVAL, "%s: bins is NULL", fn);
    if (bins->n_rays != n_rays)
        return fail(PLX_EINVAL, "%s: bins were made for %lld rays, the call has %lld", fn,
                    (long long)bins->n_rays, (long long)n_rays);
    if (bins->n_seg < 0 || bins->n_seg > kMaxRaysBinned)
        return fail(PLX_EINVAL, "%s: bins->n_seg = %lld out of range", fn, (long long)bins->n_seg);
    const RayBufLayout rl = ray_buf_layout(n_rays, n_bins(to_dev(grid)));
    int rc = check_buf(bins->ray_buf, bins->ray_buf_bytes, rl.bytes, "bins->ray_buf", fn);
    if (rc) return rc;
    attach_ray_buf(a, bins->ray_buf, rl);
    a.n_seg = bins->n_seg;
    a.seg_cap = bins->n_seg;
    if (bins->n_seg > 0) {
        const SegBufLayout sl = seg_buf_layout(bins->n_seg);
        if ((rc = check_buf(bins->seg_buf, bins->seg_buf_bytes, sl.bytes, "bins->seg_buf", fn))) return rc;
        attach_seg_buf(a, bins->seg_buf, sl);
    }
    const int64_t n_bricks = n_bins(to_dev(grid)) / kLenClasses;
    if (bins->n_brick < 0 || bins->n_brick > n_bricks || (bins->n_seg > 0) != (bins->n_brick > 0))
        return fail(PLX_EINVAL, "%s: bins->n_brick = %lld out of range", fn, (long long)bins->n_brick);
    if (bins->n_samp < 0 || bins->n_samp > kMaxSampBinned || (bins->n_seg > 0 && bins->n_samp < bins->n_seg))
        return fail(PLX_EINVAL, "%s: bins->n_samp = %lld out of range", fn, (long long)bins->n_samp);
    a.n_brick = bins->n_brick;
    if (bins->samp_buf && bins->n_seg > 0) {
        const SampBufLayout pl = samp_buf_layout(bins->n_seg, bins->n_samp);
        if ((rc = check_buf(bins->samp_buf, bins->samp_buf_bytes, pl.bytes, "bins->samp_buf", fn))) return rc;
        attach_samp_buf(a, bins->samp_buf, pl);
        a.samp_cap = bins->n_samp;
    }
    return PLX_OK;
}

// Blocks of the count and emit walks of a's rays; returns the lanes per ray.
int walk_blocks(const GridDev &g, BinArgs &a) {
    const int parts = walk_parts(g, a.n_rays);
    const int64_t nbr = (a.n_rays * parts + kThreads - 1) / kThreads;
    a.n_blocks = (int)nbr;
    a.nb8 = round_up8(nbr);
    return parts;
}

int emit_launch(const GridDev &g, BinArgs &a, hipStream_t s, const char *fn) {
    if (walk_blocks(g, a) == 1) seg_emit_kernel<1><<<a.nb8, kThreads, 0, s>>>(g, a);
    else seg_emit_kernel<kWalkParts><<<a.nb8, kThreads, 0, s>>>(g, a);
    return check_launch(fn);
}

// Counting phase: per-ray and per-bin segment counts and their scans.
// Leaves the total at seg_off[n_rays] on the device.
int bin_count_launch(const GridDev &g, BinArgs &a, int64_t nbk, int64_t *scan_tmp, hipStream_t s,
                     const char *fn) {
    const int64_t n_rays = a.n_rays;
    // counters, cursors, the status word (and the brick counter)
    const int64_t nz = a.bcnt64 ? 4 * nbk + 2 : 2 * nbk + 1;
    zero_u32_kernel<<<(unsigned)((nz + 255) / 256), 256, 0, s>>>(
        a.bcnt64 ? reinterpret_cast<unsigned *>(a.bcnt64) : a.bcount, nz);
    int rc = check_launch(fn);
    if (rc) return rc;
    const int parts = walk_blocks(g, a);
    if (parts == 1) seg_count_kernel<1><<<a.nb8, kThreads, 0, s>>>(g, a);
    else seg_count_kernel<kWalkParts><<<a.nb8, kThreads, 0, s>>>(g, a);
    if ((rc = check_launch(fn))) return rc;
    ScanArgs q = {};
    int64_t *bin_tmp = scan_tmp + scan_tmp_words(n_rays);
    if ((rc = add_scan(q, a.nseg, n_rays, 1, a.seg_off, scan_tmp, a.bcnt64 ? a.totals : nullptr, fn))) return rc;
    if (!a.bcnt64) {
        if ((rc = add_scan(q, a.bcount, nbk, 1, a.boff, bin_tmp, nullptr, fn))) return rc;
        return run_scans(q, s, fn);
    }
    const unsigned *halves = reinterpret_cast<const unsigned *>(a.bcnt64);
    if ((rc = add_scan(q, halves, nbk, 2, a.boff, bin_tmp, nullptr, fn))) return rc;
    if ((rc = add_scan(q, halves + 1, nbk, 2, a.bsoff, reinterpret_cast<int64_t *>(a.blist), a.totals + 1, fn))) return rc;
    if ((rc = run_scans(q, s, fn))) return rc;
    const int64_t n_bricks = nbk / kLenClasses;
    brick_list_kernel<<<(unsigned)((n_bricks + kThreads - 1) / kThreads), kThreads, 0, s>>>(a, n_bricks);
    return check_launch(fn);
}

// Render passes over binned segments: MODE_FWD renders, MODE_BWD and
// MODE_TRAIN also run the backward replay, MODE_MAXW the weight passes.
// Launch sizes come from a.n_seg, an upper bound when a.n_seg_dev is set.
template <int MODE>
int render_binned(const plx_grid *grid, BinArgs a, hipStream_t s, const char *fn) {
    GridDev g = to_dev(grid);
    const int64_t nbr = (a.n_rays + kThreads - 1) / kThreads;
    const int64_t nbs = (a.n_seg + kThreads - 1) / kThreads;
    BinArgs as = a;
    as.n_blocks = (int)nbs;
    as.nb8 = round_up8(nbs);
    int rc;
    if ((rc = mark_event(a.events, 0, s, fn))) return rc;
    if constexpr (MODE == MODE_MAXW) {
        if (a.n_seg == 0) return PLX_OK;
        const bool sparse = a.n_brick >= kSparseBricks && a.n_seg < kSparseSegs * a.n_brick;
        PLX_DISPATCH_DT(grid->sh_dtype, DT, {
            if (sparse) seg_weight_kernel<DT, 0, true><<<(unsigned)a.n_brick, kWave, 0, s>>>(g, as);
            else seg_weight_kernel<DT, 0, false><<<(unsigned)a.n_brick, kThreads, 0, s>>>(g, as);
        });
        if ((rc = check_launch(fn))) return rc;
        seg_combine_kernel<MODE><<<(unsigned)nbr, kThreads, 0, s>>>(a);
        if ((rc = check_launch(fn))) return rc;
        PLX_DISPATCH_DT(grid->sh_dtype, DT, {
            if (sparse) seg_weight_kernel<DT, 1, true><<<(unsigned)a.n_brick, kWave, 0, s>>>(g, as);
            else seg_weight_kernel<DT, 1, false><<<(unsigned)a.n_brick, kThreads, 0, s>>>(g, as);
        });
        return check_launch(fn);
    }
    if (a.n_seg > 0) {
        const bool rec = MODE != MODE_FWD && a.srec;
        const bool lists = a.blist && a.n_brick > 0;
        if (rec && lists && a.n_seg >= kFwdParMinSegs * a.n_brick) {
            // recording forward: sample-parallel, one workgroup per brick
            PLX_DISPATCH_DT(grid->sh_dtype, DT,
                            seg_fwd_samples_kernel<DT><<<(unsigned)a.n_brick, kFwdThreads, 0, s>>>(g, as));
        } else if (lists && grid->sh_dtype != PLX_F32) {
            // brick-staged (16-bit records: 47 KB of LDS per brick, three
            // workgroups per CU; FP32's 82 KB leave one, and the lane-per-
            // segment kernel with its L2 traffic is then twice as fast)
            const unsigned nb = (unsigned)a.n_brick;
            if (rec) {
                PLX_DISPATCH_DT(grid->sh_dtype, DT, seg_fwd_brick_kernel<DT, true><<<nb, kThreads, 0, s>>>(g, as));
            } else {
                PLX_DISPATCH_DT(grid->sh_dtype, DT, seg_fwd_brick_kernel<DT, false><<<nb, kThreads, 0, s>>>(g, as));
            }
        } else if (rec) {
            PLX_DISPATCH_DT(grid->sh_dtype, DT, seg_fwd_kernel<DT, true><<<as.nb8, kThreads, 0, s>>>(g, as));
        } else {
            PLX_DISPATCH_DT(grid->sh_dtype, DT, seg_fwd_kernel<DT, false><<<as.nb8, kThreads, 0, s>>>(g, as));
        }
        if ((rc = check_launch(fn))) return rc;
    }
    if ((rc = mark_event(a.events, 1, s, fn))) return rc;
    seg_combine_kernel<MODE><<<(unsigned)nbr, kThreads, 0, s>>>(a);
    if ((rc = check_launch(fn))) return rc;
    if ((rc = mark_event(a.events, 2, s, fn))) return rc;
    if (MODE != MODE_FWD && a.n_seg > 0 && a.srec) {
        // recorded backward: one scatter workgroup per brick (the Cauchy
        // prior's per-sample terms only in an instance of their own)
        if (a.n_brick > 0) {
            if (as.pri.lambda_s != 0.0f)
                seg_scatter_kernel<true><<<(unsigned)a.n_brick, kScatterThreads, 0, s>>>(g, as);
            else
                seg_scatter_kernel<false><<<(unsigned)a.n_brick, kScatterThreads, 0, s>>>(g, as);
            if ((rc = check_launch(fn))) return rc;
        }
    } else if (MODE != MODE_FWD && a.n_seg > 0) {
        // the Cauchy prior's per-sample terms only in an instance of their own
        if (as.pri.lambda_s != 0.0f) {
            PLX_DISPATCH_DT(grid->sh_dtype, DT, seg_bwd_kernel<DT, true><<<as.nb8, kThreads, 0, s>>>(g, as));
        } else {
            PLX_DISPATCH_DT(grid->sh_dtype, DT, seg_bwd_kernel<DT, false><<<as.nb8, kThreads, 0, s>>>(g, as));
        }
        if ((rc = check_launch(fn))) return rc;
    }
    return mark_event(a.events, 3, s, fn);
}

// ------------------------------------------------------------ fixed scratch
//
// plx_render_train_static serves callers that cannot allocate (code under
// graph capture, serving loops): its segment lists live in a fixed device
// array instead of caller buffers, sized for the worst case of the batch
// (every ray crossing the most bricks a line can cross), and the segment
// kernels read the true segment count on the device, so the call neither
// allocates nor synchronises.  The array is per device and kept until the
// process ends; calls that overlap on one device share it and race.
constexpr int64_t kStaticScratchBytes = (int64_t)64 << 20;
constexpr int kMaxDevices = 64;

std::mutex g_static_mu;
void *g_static_ptr[kMaxDevices] = {};

}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

// Device address of this device's fixed scratch, looked up once per device
// (the array's name is a host-side stand-in, never passed to a kernel).
int static_scratch(void **out, const char *fn) {
    int dev = 0;
    PLX_CHECK_HIP(hipGetDevice(&dev), fn);
    if (dev < 0 || dev >= kMaxDevices) return fail(PLX_EDEVICE, "%s: device %d out of range", fn, dev);
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
        void *p = nullptr;
        PLX_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), fn);
        if (!p) return fail(PLX_EDEVICE, "%s: no address for the fixed scratch", fn);
        g_static_ptr[dev] = p;
    }
    *out = g_static_ptr[dev];
    return PLX_OK;
}

// Whether a batch whose lists exist is rendered over them (the march in ray
// order needs none).  Ray order / lists in us:
// - 16-bit records: a workgroup stages its brick's records once, which pays
//   when many samples share them and there are bricks enough to fill the chip.
//   Samples per brick 1,150 (512^3 at 5%) 1044 / 1517, 1,580 (dense 128^3) 358 / 386,
//   1,860 (256x256x128) 1151 / 1210; 2,000 (200^3) 1669 / 1430, 2,840 (256x256x128)
//   1730 / 1542, 4,150 (128^3 from inside) 812 / 668, 19,100 (128^3) 3548 / 2010; but
//   with 1,728 bricks 697 / 725 at 10,500, 1,000 bricks 1023 / 1275 at 39,300.
// - FP32: the bricks in order share what the caches hold, which counts when
//   the grid's records do not fit (8,192 bricks with stored corners are some
//   512 MB): 98,304 rays on 512^3 417 / 325, 400,000 984 / 911, 786,000 on dense 200^3
//   8961 / 7722; 65,536 226 / 235; with 4,096 bricks 4939 / 4743 at 786,000 rays of
//   dense 128^3, 3194 / 3190 at 200,000 from inside, 5,000 bricks 1195 / 1330.
// - from 786,432 rays on the lists, whose order does not depend on the rays'
//   (512^3, 1M rays: 2.12 / 1.92 ms, shuffled 2.46 / 1.92).
bool forward_over_lists(int32_t sh_dtype, int64_t n_rays, const plx_bins *bins) {
    if (n_rays >= 3 << 18) return true;
    if (sh_dtype == PLX_F32) return n_rays >= 3 << 15 && bins->n_brick >= 1 << 13;
    return bins->n_brick >= 1 << 11 && bins->n_samp >= 2000 * bins->n_brick;
}

}  // namespace
}  // namespace plx

using namespace plx;

extern "C" {

int64_t plx_bins_ray_bytes(const int32_t reso[3], int64_t n_rays) {
    if (!reso || reso[0] < 2 || reso[1] < 2 || reso[2] < 2 || n_rays < 0 || n_rays > kMaxRaysBinned)
        return 0;
    plx_grid tmp = {};
    for (int a = 0; a < 3; ++a) tmp.reso[a] = reso[a];
    return ray_buf_layout(n_rays, n_bins(to_dev(&tmp))).bytes;
}

int64_t plx_bins_seg_bytes(int64_t n_seg) {
    if (n_seg < 0 || n_seg > kMaxRaysBinned) return 0;
    return seg_buf_layout(n_seg).bytes;
}

int64_t plx_bins_samp_bytes(int64_t n_seg, int64_t n_samp) {
    if (n_seg < 0 || n_seg > kMaxRaysBinned || n_samp < 0 || n_samp > kMaxSampBinned) return 0;
    return samp_buf_layout(n_seg, n_samp).bytes;
}

int plx_bins_count(const plx_grid *grid, const float *rays_o, const float *rays_d, int64_t n_rays,
                   void *ray_buf, int64_t ray_buf_bytes, plx_bins *bins, plx_stream stream) {
    const char *fn = "plx_bins_count";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!bins) return fail(PLX_EINVAL, "%s: bins is NULL", fn);
    if (n_rays > kMaxRaysBinned) return fail(PLX_EINVAL, "%s: too many rays", fn);
    const GridDev g = to_dev(grid);
    const int64_t nbk = n_bins(g);
    const RayBufLayout l = ray_buf_layout(n_rays, nbk);
    if ((rc = check_buf(ray_buf, ray_buf_bytes, l.bytes, "ray_buf", fn))) return rc;
    *bins = plx_bins{};
    bins->n_rays = n_rays;
    bins->ray_buf = ray_buf;
    bins->ray_buf_bytes = ray_buf_bytes;
    if (n_rays == 0) return PLX_OK;
    hipStream_t s = as_stream(stream);
    BinArgs a = {};
    a.rays_o = rays_o;
    a.rays_d = rays_d;
    a.n_rays = n_rays;
    attach_ray_buf(a, ray_buf, l);
    int64_t *scan_tmp = reinterpret_cast<int64_t *>(static_cast<char *>(ray_buf) + l.scan);
    if ((rc = bin_count_launch(g, a, nbk, scan_tmp, s, fn))) return rc;
    // the status word, the brick count and the two totals lie side by side
    struct {
        unsigned status, bricks;
        int64_t total, samples;
    } h = {};
    static_assert(sizeof(h) == 24, "as in the ray buffer");
    PLX_CHECK_HIP(hipMemcpyAsync(&h, a.status, sizeof(h), hipMemcpyDeviceToHost, s), fn);
    PLX_CHECK_HIP(hipStreamSynchronize(s), fn);
    const int64_t total = h.total, samples = h.samples;
    const unsigned bricks = h.bricks;
    if (total < 0 || total > kMaxRaysBinned)
        return fail(PLX_EINVAL, "%s: %lld ray segments, more than one call handles", fn, (long long)total);
    if (samples < 0 || samples > kMaxSampBinned)
        return fail(PLX_EINVAL, "%s: %lld sample slots, more than one call handles", fn, (long long)samples);
    bins->n_seg = total;
    bins->n_samp = samples;
    bins->n_brick = bricks;
    return PLX_OK;
}

int plx_bins_apply(const plx_grid *grid, const float *rays_o, const float *rays_d,
                   const plx_bins *bins, plx_stream stream) {
    const char *fn = "plx_bins_apply";
    int rc = validate_grid(grid, true, fn);
    if (rc) return rc;
    if (!bins) return fail(PLX_EINVAL, "%s: bins is NULL", fn);
    if ((rc = validate_rays(rays_o, rays_d, bins->n_rays, fn))) return rc;
    BinArgs a = {};
    if ((rc = attach_bins(grid, bins, bins->n_rays, a, fn))) return rc;
    if (bins->n_seg == 0) return PLX_OK;
    a.rays_o = rays_o;
    a.rays_d = rays_d;
    a.n_rays = bins->n_rays;
    return emit_launch(to_dev(grid), a, as_stream(stream), fn);
}

int plx_bins_verify(const plx_grid *grid, const plx_bins *bins, plx_stream stream) {
    const char *fn = "plx_bins_verify";
    int rc = validate_grid(grid, true, fn);
    if (rc) return rc;
    BinArgs a = {};
    if (!bins) return fail(PLX_EINVAL, "%s: bins is NULL", fn);
    if ((rc = attach_bins(grid, bins, bins->n_rays, a, fn))) return rc;
    if (bins->n_rays == 0) return PLX_OK;
    hipStream_t s = as_stream(stream);
    unsigned st = 0;
    PLX_CHECK_HIP(hipMemcpyAsync(&st, a.status, sizeof(st), hipMemcpyDeviceToHost, s), fn);
    PLX_CHECK_HIP(hipStreamSynchronize(s), fn);
    if (st != 0) return fail(PLX_EDEVICE, "%s: the segment walk of plx_bins_apply disagreed with plx_bins_count", fn);
    return PLX_OK;
}

int plx_render_fwd(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                   const float *rays_d, int64_t n_rays, const plx_bins *bins, float *rgb_out,
                   float *tau_out, plx_stream stream) {
    const char *fn = "plx_render_fwd";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!rgb_out) return fail(PLX_EINVAL, "%s: rgb_out is NULL", fn);
    BinArgs a = {};
    if ((rc = attach_bins(grid, bins, n_rays, a, fn))) return rc;
    a.events = opts->kernel_events;
    a.rays_o = rays_o;
    a.rays_d = rays_d;
    a.rgb_out = rgb_out;
    a.tau_out = tau_out;
    a.n_rays = n_rays;
    for (int i = 0; i < 3; ++i) a.bg[i] = opts->background[i];
    a.bg_rgb = opts->background_rgb;
    a.grad_bg = opts->grad_background;
    if (!forward_over_lists(grid->sh_dtype, n_rays, bins))
        return render_fwd_rays(grid, opts, rays_o, rays_d, n_rays, rgb_out, tau_out, as_stream(stream), fn);
    return render_binned<MODE_FWD>(grid, a, as_stream(stream), fn);
}

int plx_render_bwd(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                   const float *rays_d, int64_t n_rays, const plx_bins *bins, const float *grad_rgb,
                   const float *tau_fwd, float *grad, uint8_t *touched, plx_stream stream) {
    const char *fn = "plx_render_bwd";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!grad_rgb || !tau_fwd || (grid->n_vox > 0 && (!grad || !touched)))
        return fail(PLX_EINVAL, "%s: NULL grad_rgb/tau_fwd/grad/touched", fn);
    BinArgs a = {};
    if ((rc = priors_from(opts, a.pri, fn))) return rc;
    if ((rc = attach_bins(grid, bins, n_rays, a, fn))) return rc;
    a.events = opts->kernel_events;
    a.rays_o = rays_o;
    a.rays_d = rays_d;
    a.grad_rgb = grad_rgb;
    a.grad = grad;
    a.touched = touched;
    a.n_rays = n_rays;
    for (int i = 0; i < 3; ++i) a.bg[i] = opts->background[i];
    a.bg_rgb = opts->background_rgb;
    a.grad_bg = opts->grad_background;
    return render_binned<MODE_BWD>(grid, a, as_stream(stream), fn);
}

int plx_render_max_weight(const plx_grid *grid, const float *rays_o, const float *rays_d,
                          int64_t n_rays, const plx_bins *bins, float *wmax, plx_stream stream) {
    const char *fn = "plx_render_max_weight";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (n_rays == 0) return PLX_OK;
    if (!wmax) return fail(PLX_EINVAL, "%s: wmax is NULL", fn);
    BinArgs a = {};
    if ((rc = attach_bins(grid, bins, n_rays, a, fn))) return rc;
    a.rays_o = rays_o;
    a.rays_d = rays_d;
    a.wmax = wmax;
    a.n_rays = n_rays;
    return render_binned<MODE_MAXW>(grid, a, as_stream(stream), fn);
}

int plx_render_train(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                     const float *rays_d, const float *target, int64_t n_rays, const plx_bins *bins,
                     float loss_scale, float *rgb_out, float *grad, uint8_t *touched,
                     double *loss_sum, plx_stream stream) {
    const char *fn = "plx_render_train";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!target || !loss_sum || (grid->n_vox > 0 && (!grad || !touched)))
        return fail(PLX_EINVAL, "%s: NULL target/grad/touched/loss_sum", fn);
    BinArgs a = {};
    if ((rc = priors_from(opts, a.pri, fn))) return rc;
    if ((rc = attach_bins(grid, bins, n_rays, a, fn))) return rc;
    a.events = opts->kernel_events;
    a.rays_o = rays_o;
    a.rays_d = rays_d;
    a.target = target;
    a.rgb_out = rgb_out;
    a.loss_sum = loss_sum;
    a.grad = grad;
    a.touched = touched;
    a.n_rays = n_rays;
    for (int i = 0; i < 3; ++i) a.bg[i] = opts->background[i];
    a.bg_rgb = opts->background_rgb;
    a.grad_bg = opts->grad_background;
    a.loss_scale = loss_scale;
    return render_binned<MODE_TRAIN>(grid, a, as_stream(stream), fn);
}

int plx_render_train_static(const plx_grid *grid, const plx_render_opts *opts, const float *rays_o,
                            const float *rays_d, const float *target, int64_t n_rays,
                            float loss_scale, float *rgb_out, float *grad, uint8_t *touched,
                            double *loss_sum, plx_stream stream) {
    const char *fn = "plx_render_train_static";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_rays == 0) return PLX_OK;
    if (!target || !loss_sum || (grid->n_vox > 0 && (!grad || !touched)))
        return fail(PLX_EINVAL, "%s: NULL target/grad/touched/loss_sum", fn);
    const GridDev g = to_dev(grid);
    const int64_t nbk = n_bins(g);
    // a ray enters each brick at most once and a line crosses at most
    // bx + by + bz - 2 bricks of the lattice
    const int64_t per_ray = (int64_t)g.bx + g.by + g.bz;
    const int64_t cap = n_rays * per_ray;
    const RayBufLayout rl = ray_buf_layout(n_rays, nbk, false);
    const SegBufLayout sl = seg_buf_layout(cap);
    if (n_rays > kMaxRaysBinned || cap > kMaxRaysBinned || rl.bytes + sl.bytes > kStaticScratchBytes)
        return fail(PLX_ENOMEM,
                    "%s: %lld rays on a %dx%dx%d grid need %lld bytes of scratch, more than the fixed %lld "
                    "(the bound is ray buffer + %lld segments per ray)",
                    fn, (long long)n_rays, grid->reso[0], grid->reso[1], grid->reso[2],
                    (long long)(rl.bytes + sl.bytes), (long long)kStaticScratchBytes, (long long)per_ray);
    BinArgs a = {};
    if ((rc = priors_from(opts, a.pri, fn))) return rc;
    void *base = nullptr;
    if ((rc = static_scratch(&base, fn))) return rc;
    hipStream_t s = as_stream(stream);
    a.rays_o = rays_o;
    a.rays_d = rays_d;
    a.n_rays = n_rays;
    attach_ray_buf(a, base, rl);
    attach_seg_buf(a, static_cast<char *>(base) + rl.bytes, sl);
    int64_t *scan_tmp = reinterpret_cast<int64_t *>(static_cast<char *>(base) + rl.scan);
    // counts, scans and records: the previous call's contents are cleared
    // by the counting phase (bin counters, cursors, status)
    if ((rc = bin_count_launch(g, a, nbk, scan_tmp, s, fn))) return rc;
    a.n_seg = cap;  // launch bound; the kernels read the count itself
    a.seg_cap = cap;
    a.n_seg_dev = a.seg_off + n_rays;
    if ((rc = emit_launch(g, a, s, fn))) return rc;
    a.events = opts->kernel_events;
    a.target = target;
    a.rgb_out = rgb_out;
    a.loss_sum = loss_sum;
    a.grad = grad;
    a.touched = touched;
    for (int i = 0; i < 3; ++i) a.bg[i] = opts->background[i];
    a.bg_rgb = opts->background_rgb;
    a.grad_bg = opts->grad_background;
    a.loss_scale = loss_scale;
    return render_binned<MODE_TRAIN>(grid, a, s, fn);
}

int64_t plx_scene_table_bytes(int32_t n_scenes) {
    if (n_scenes < 1) return 0;
    return kSceneTableHead + (int64_t)n_scenes * (int64_t)sizeof(GridDev);
}

int plx_scene_table_set(const plx_grid *scenes, int32_t n_scenes, void *table, int64_t table_bytes,
                        plx_stream stream) {
    const char *fn = "plx_scene_table_set";
    if (!scenes || n_scenes < 1) return fail(PLX_EINVAL, "%s: need at least one scene", fn);
    if (!table || reinterpret_cast<uintptr_t>(table) % 256)
        return fail(PLX_EINVAL, "%s: table must be a 256-byte aligned device pointer", fn);
    if (table_bytes < plx_scene_table_bytes(n_scenes))
        return fail(PLX_EINVAL, "%s: table of %lld bytes, need %lld", fn, (long long)table_bytes,
                    (long long)plx_scene_table_bytes(n_scenes));
    const int32_t dt = scenes[0].sh_dtype;
    for (int32_t i = 0; i < n_scenes; ++i) {
        int rc = validate_grid(&scenes[i], true, fn);
        if (rc) return rc;
        if (scenes[i].sh_dtype != dt) return fail(PLX_EINVAL, "%s: scenes must share one sh_dtype", fn);
    }
    hipStream_t s = as_stream(stream);
    SceneSetupArgs a = {};
    a.n_scenes = n_scenes;
    a.sh_dtype = dt;
    a.table = static_cast<SceneTableHeader *>(table);
    a.scenes = reinterpret_cast<GridDev *>(static_cast<char *>(table) + kSceneTableHead);
    for (int32_t first = 0; first < n_scenes; first += kSetupItems) {
        a.first = first;
        a.count = std::min(kSetupItems, n_scenes - first);
        for (int i = 0; i < a.count; ++i) a.g[i] = to_dev(&scenes[first + i]);
        scene_setup_kernel<<<1, 32, 0, s>>>(a);
        int rc = check_launch(fn);
        if (rc) return rc;
    }
    return PLX_OK;
}

int plx_render_views(const void *scene_table, int32_t n_scenes, int32_t sh_dtype, const plx_view *views,
                     int32_t n_views, const plx_render_opts *opts, float *rgb_out, void *queue,
                     plx_stream stream) {
    const char *fn = "plx_render_views";
    if (!scene_table || n_scenes < 1) return fail(PLX_EINVAL, "%s: need a scene table of at least one scene", fn);
    if (sh_dtype != PLX_F32 && sh_dtype != PLX_BF16 && sh_dtype != PLX_F16)
        return fail(PLX_EINVAL, "%s: bad sh_dtype %d", fn, sh_dtype);
    if (n_views < 0) return fail(PLX_EINVAL, "%s: n_views < 0", fn);
    if (!opts) return fail(PLX_EINVAL, "%s: opts is NULL", fn);
    if (n_views == 0) return PLX_OK;
    if (!views || !rgb_out || !queue) return fail(PLX_EINVAL, "%s: NULL views/rgb_out/queue", fn);
    if (reinterpret_cast<uintptr_t>(queue) % 256)
        return fail(PLX_EINVAL, "%s: queue must be 256-byte aligned", fn);
    for (int32_t i = 0; i < n_views; ++i) {
        const plx_view &v = views[i];
        if (v.scene < 0 || v.scene >= n_scenes) return fail(PLX_EINVAL, "%s: view %d: bad scene", fn, i);
        if (v.width < 1 || v.height < 1 || v.width > 65536 || v.height > 65536)
            return fail(PLX_EINVAL, "%s: view %d: bad size %dx%d", fn, i, v.width, v.height);
        if (!(v.focal > 0.0) || !std::isfinite(v.focal) || v.out_offset < 0)
            return fail(PLX_EINVAL, "%s: view %d: bad focal or out_offset", fn, i);
    }
    hipStream_t s = as_stream(stream);
    ViewsArgs va;
    va.table = static_cast<const SceneTableHeader *>(scene_table);
    va.scenes = reinterpret_cast<const GridDev *>(static_cast<const char *>(scene_table) + kSceneTableHead);
    va.status = &static_cast<ViewsQueue *>(queue)->status;
    va.rgb_out = rgb_out;
    for (int i = 0; i < 3; ++i) va.bg[i] = opts->background[i];
    for (int32_t first = 0; first < n_views; first += kViewsPerLaunch) {
        va.n_views = std::min(kViewsPerLaunch, n_views - first);
        // the tiles of the views that take `lane` (or not), none for the others
        auto tiles_for = [&](bool lane) {
            int64_t tiles = 0;
            for (int i = 0; i < va.n_views; ++i) {
                const plx_view &v = views[first + i];
                va.v[i] = v;
                va.lanes[i] = view_lanes(v);
                va.tile_start[i] = tiles;
                if (((v.reserved & PLX_VIEW_LANE) != 0) != lane) continue;
                if (lane) tiles += (int64_t)((v.width + kLaneTile - 1) / kLaneTile) * ((v.height + kLaneTile - 1) / kLaneTile);
                else tiles += va.lanes[i] == 16 ? tiles_of<ViewsCut<16>>(v)
                                                : (va.lanes[i] == 8 ? tiles_of<ViewsCut<8>>(v) : tiles_of<ViewsCut<4>>(v));
            }
            va.tile_start[va.n_views] = tiles;
            return (unsigned)std::min(tiles, kViewsMaxBlocks);
        };
        int rc;
        if (const unsigned nb = tiles_for(false)) {
            PLX_DISPATCH_DT(sh_dtype, DT, views_kernel<DT><<<nb, kWave, 0, s>>>(va));
            if ((rc = check_launch(fn))) return rc;
        }
        if (const unsigned nb = tiles_for(true)) {
            PLX_DISPATCH_DT(sh_dtype, DT, views_lane_kernel<DT><<<nb, kWave, 0, s>>>(va));
            if ((rc = check_launch(fn))) return rc;
        }
    }
    return PLX_OK;
}

int plx_render_views_status(const void *queue, plx_stream stream) {
    const char *fn = "plx_render_views_status";
    if (!queue) return fail(PLX_EINVAL, "%s: queue is NULL", fn);
    hipStream_t s = as_stream(stream);
    unsigned st = 0;
    PLX_CHECK_HIP(hipMemcpyAsync(&st, &static_cast<const ViewsQueue *>(queue)->status, sizeof(st),
                                 hipMemcpyDeviceToHost, s), fn);
    PLX_CHECK_HIP(hipStreamSynchronize(s), fn);
    if (st != 0)
        return fail(PLX_EINVAL, "%s: a launch on this queue met a scene table of another storage type, or "
                                "a view naming a scene beyond it; those views were not rendered", fn);
    return PLX_OK;
}

int plx_render_stats(const plx_grid *grid, const float *rays_o, const float *rays_d,
                     int64_t n_rays, uint32_t *cell_mark, uint32_t *vox_mark, void *ws,
                     int64_t ws_bytes, int64_t counts[4], plx_stream stream) {
    const char *fn = "plx_render_stats";
    int rc = validate_grid(grid, true, fn);
    if (rc || (rc = validate_rays(rays_o, rays_d, n_rays, fn))) return rc;
    if (!cell_mark || !vox_mark || !counts) return fail(PLX_EINVAL, "%s: NULL argument", fn);
    if ((rc = check_buf(ws, ws_bytes, PLX_COUNT_WORKSPACE_BYTES, "workspace", fn))) return rc;
    hipStream_t s = as_stream(stream);
    const int64_t cw = (n_cells(grid->reso) + 31) / 32, vw = (grid->n_vox + 31) / 32;
    zero_u32_kernel<<<(unsigned)((cw + 255) / 256), 256, 0, s>>>(cell_mark, cw);
    if ((rc = check_launch(fn))) return rc;
    if (vw) {
        zero_u32_kernel<<<(unsigned)((vw + 255) / 256), 256, 0, s>>>(vox_mark, vw);
        if ((rc = check_launch(fn))) return rc;
    }
    // two sample counters at the start of the workspace (the bit counts
    // below reuse its first word after these are read back)
    auto *cnt = static_cast<unsigned long long *>(ws);
    zero_u32_kernel<<<1, 256, 0, s>>>(static_cast<unsigned *>(ws), 4);
    if ((rc = check_launch(fn))) return rc;
    if (n_rays > 0) {
        stats_kernel<<<(unsigned)((n_rays + 255) / 256), 256, 0, s>>>(to_dev(grid), rays_o, rays_d,
                                                                      n_rays, cell_mark, vox_mark, cnt);
        if ((rc = check_launch(fn))) return rc;
    }
    unsigned long long h[2];
    PLX_CHECK_HIP(hipMemcpyAsync(h, cnt, sizeof(h), hipMemcpyDeviceToHost, s), fn);
    PLX_CHECK_HIP(hipStreamSynchronize(s), fn);
    counts[0] = (int64_t)h[0];
    counts[1] = (int64_t)h[1];
    int64_t cells = 0, vox = 0;
    if ((rc = count_set_bits(cell_mark, n_cells(grid->reso), ws, &cells, s, fn))) return rc;
    if ((rc = count_set_bits(vox_mark, grid->n_vox, ws, &vox, s, fn))) return rc;
    counts[2] = cells;
    counts[3] = vox;
    return PLX_OK;
}

}  // extern "C"
