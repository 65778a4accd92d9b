// grid.hip -- grid create / pack / occupancy / prune / upsample (Sec. 3.2,
// Sec. 3.4, supplement B.1) for gfx950.
//
// Size-changing operations are stream compactions over the cells in storage
// order: a three-phase scan (per-block flag counts, one-block scan of the
// counts, per-block local scan and write).  Table ids therefore follow
// increasing storage id, as the index-grid definition requires.  A block
// of the last phase also makes the records of its occupied cells, 8 lanes (16
// bytes each) per record: its table ids are consecutive, so the stores are
// too.  Memory bounds these passes; a thread per cell that copied or
// interpolated a whole record by itself took 545 us (copy) and 1413 us (index
// and trilinear values) for 256x256x128 cells refined to 512x512x128, now
// 146 and 473.
#include "plx_internal.hpp"

namespace plx {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;  // cells per thread
constexpr int kScanTile = kScanThreads * kScanItems;

// Exclusive scan of one int per thread over a block of THREADS.
template <int THREADS = kScanThreads>
__device__ inline int block_exclusive_scan(int x, int *total) {
    __shared__ int wsum[THREADS / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < THREADS / 64; ++i) {
        off += (i < w) ? wsum[i] : 0;
        tot += wsum[i];
    }
    __syncthreads();
    *total = tot;
    return off + inc - x;
}

// ---- predicates over cells: flags<ITEMS>(v, n), the flags of the ITEMS cells
// from v on (bit i: cell v + i; cells from n on are 0)
struct MaskPred {
    const uint8_t *mask;
    bool aligned;  // mask is 16-byte aligned
    template <int ITEMS>
    __device__ uint32_t flags(int64_t v, int64_t n) const {
        uint32_t f = 0;
        if (ITEMS == 16 && aligned && v + ITEMS <= n) {
            const uint4 q = *reinterpret_cast<const uint4 *>(mask + v);
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int i = 0; i < 16; ++i) f |= ((w[i >> 2] >> (8 * (i & 3)) & 0xffu) != 0u ? 1u : 0u) << i;
        } else {
            for (int i = 0; i < ITEMS; ++i)
                if (v + i < n && mask[v + i] != 0) f |= 1u << i;
        }
        return f;
    }
};

// New cell occupied iff its parent cell is occupied: along each axis the
// parent of cell k of nn is floor((2k + 1) on / (2 nn)).  Along the last axis
// quotient and remainder go from cell to cell by additions; a division per
// cell and axis took 115 us per pass over 33.6M cells, so 38 to 54.
struct ParentPred {
    const int32_t *old_index;
    int on[3], nn[3];
    bool narrow;  // every product, and every cell, fits 32 bits
    __device__ uint32_t quotient(uint64_t a, uint64_t b) const {
        return narrow ? (uint32_t)a / (uint32_t)b : (uint32_t)(a / b);
    }
    __device__ void decode(int64_t v, int &i, int &j, int &k) const {
        if (narrow) {
            const uint32_t r = (uint32_t)v / (uint32_t)nn[2];
            k = (int)((uint32_t)v - r * nn[2]);
            i = (int)(r / (uint32_t)nn[1]);
            j = (int)(r - (uint32_t)i * nn[1]);
        } else {
            const int64_t r = v / nn[2];
            k = (int)(v - r * nn[2]);
            i = (int)(r / nn[1]);
            j = (int)(r - (int64_t)i * nn[1]);
        }
    }
    __device__ const int32_t *row(int i, int j) const {
        const int pi = (int)quotient((uint64_t)(2 * (int64_t)i + 1) * on[0], 2 * (uint64_t)nn[0]);
        const int pj = (int)quotient((uint64_t)(2 * (int64_t)j + 1) * on[1], 2 * (uint64_t)nn[1]);
        return old_index + ((int64_t)pi * on[1] + pj) * on[2];
    }
    template <int ITEMS>
    __device__ uint32_t flags(int64_t v, int64_t n) const {
        if (v >= n) return 0u;
        int i, j, k;
        decode(v, i, j, k);
        const int32_t *p = row(i, j);
        const uint64_t den = 2 * (uint64_t)nn[2], num = (uint64_t)(2 * (int64_t)k + 1) * on[2];
        const uint32_t q0 = quotient((uint64_t)on[2], den), dq = quotient(2 * (uint64_t)on[2], den);
        const uint64_t r0 = on[2] - q0 * den, dr = 2 * (uint64_t)on[2] - dq * den;
        uint32_t q = quotient(num, den);
        uint64_t rem = num - q * den;
        int32_t id[ITEMS];
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) {
            id[e] = v + e < n ? p[q] : -1;
            q += dq;
            rem += dr;
            if (rem >= den) {
                rem -= den;
                ++q;
            }
            if (++k == nn[2]) {
                k = 0;
                q = q0;
                rem = r0;
                if (++j == nn[1]) {
                    j = 0;
                    ++i;
                }
                if (v + e + 1 < n) p = row(i, j);
            }
        }
        uint32_t f = 0;
#pragma unroll
        for (int e = 0; e < ITEMS; ++e) f |= (id[e] >= 0 ? 1u : 0u) << e;
        return f;
    }
};

// Flag counts of the tiles of kScanThreads * ITEMS cells, 16 cells a thread
// whatever ITEMS is (ITEMS <= 4: several tiles a workgroup).
template <int ITEMS, class Pred>
__global__ __launch_bounds__(kScanThreads) void scan_count_kernel(Pred pred, int64_t n, int64_t nb,
                                                                  int *counts) {
    constexpr int kWidth = kScanThreads * ITEMS / kScanItems;  // threads of a tile
    static_assert(kWidth <= 64 || kWidth == kScanThreads, "a tile is a wave's lanes or a workgroup");
    const int64_t t = (int64_t)blockIdx.x * kScanThreads + threadIdx.x;
    int c = __popc(pred.template flags<kScanItems>(t * kScanItems, n));
    if (kWidth == kScanThreads) {
        int tot;
        block_exclusive_scan(c, &tot);
        c = tot;
    } else {
#pragma unroll
        for (int m = kWidth / 2; m >= 1; m >>= 1) c += __shfl_xor(c, m);
    }
    if (threadIdx.x % kWidth == 0 && t / kWidth < nb) counts[t / kWidth] = c;
}

// One block: exclusive scan of nb block counts into offsets[0..nb], offsets[nb]
// = total.  8 counts a thread, moved in and out through LDS so that the
// accesses are whole lines (one compute unit does them all: 62 us for 65,536
// counts with 16 consecutive ones read by each thread, now 36).
constexpr int kOffsetThreads = 1024, kOffsetItems = 8, kOffsetTile = kOffsetThreads * kOffsetItems;

__global__ __launch_bounds__(kOffsetThreads) void scan_offsets_kernel(const int *counts, int64_t nb,
                                                                      int64_t *offsets) {
    __shared__ int sh[kOffsetTile + kOffsetThreads];  // count i at i + i / kOffsetItems
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kOffsetTile) {
#pragma unroll
        for (int u = 0; u < kOffsetItems; ++u) {
            const int i = u * kOffsetThreads + threadIdx.x;
            sh[i + i / kOffsetItems] = b0 + i < nb ? counts[b0 + i] : 0;
        }
        __syncthreads();
        int *mine = sh + threadIdx.x * (kOffsetItems + 1);
        int sum = 0, tot;
#pragma unroll
        for (int u = 0; u < kOffsetItems; ++u) {
            const int c = mine[u];
            mine[u] = sum;
            sum += c;
        }
        const int before = block_exclusive_scan<kOffsetThreads>(sum, &tot);
#pragma unroll
        for (int u = 0; u < kOffsetItems; ++u) mine[u] += before;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kOffsetItems; ++u) {
            const int i = u * kOffsetThreads + threadIdx.x;
            if (b0 + i < nb) offsets[b0 + i] = carry + sh[i + i / kOffsetItems];
        }
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) offsets[nb] = carry;
}

// Index entries of the tile's cells, and its records through wr: wr.item(v, e)
// (what the list keeps of occupied cell v, the e-th of the tile) and
// wr.records(list, n, first): the n records with ids from `first` on.
template <int ITEMS, class Pred, class Writer>
__global__ __launch_bounds__(kScanThreads) void scan_write_kernel(Pred pred, Writer wr, int64_t n,
                                                                  int32_t *index_out,
                                                                  const int64_t *offsets) {
    constexpr int kTile = kScanThreads * ITEMS;
    __shared__ uint32_t flags_sh[kScanThreads];
    __shared__ int rank_sh[kScanThreads];
    __shared__ typename Writer::Item list[kTile];
    const int64_t base = (int64_t)blockIdx.x * kTile;
    const uint32_t flags = pred.template flags<ITEMS>(base + threadIdx.x * ITEMS, n);
    int tot;
    rank_sh[threadIdx.x] = block_exclusive_scan(__popc(flags), &tot);
    flags_sh[threadIdx.x] = flags;
    __syncthreads();
    const int64_t first = offsets[blockIdx.x];
#pragma unroll 4
    for (int e = threadIdx.x; e < kTile; e += kScanThreads) {
        if (base + e >= n) break;
        const uint32_t f = flags_sh[e / ITEMS];
        const int i = e % ITEMS;
        const int local = rank_sh[e / ITEMS] + __popc(f & ((1u << i) - 1u));
        const bool on = f >> i & 1u;
        index_out[base + e] = on ? (int32_t)(first + local) : -1;
        if (Writer::kRecords && on) list[local] = wr.item(base + e, e);
    }
    if (!Writer::kRecords) return;
    __syncthreads();
    wr.records(list, tot, first);
}

// Workspace of the grid calls (caller-owned, plx_grid_workspace_bytes): a
// 256-byte block of counters, then a byte per cell, where the prune keeps two
// bits a cell (occupied, stored) and a compaction, which needs none of these,
// its offsets and counts per block; the size also has the room that the
// counts and offsets had behind the bytes.
struct WsLayout {
    int64_t counters, bytes8, scan, bytes;
};
inline int64_t up256(int64_t x) { return (x + 255) / 256 * 256; }
inline int64_t scan_blocks(int64_t n) { return (n + kScanTile - 1) / kScanTile; }
WsLayout ws_layout(int64_t ncell) {
    WsLayout l;
    l.counters = 0;
    l.bytes8 = 256;
    l.scan = l.bytes8 + up256(ncell);
    const int64_t nb = scan_blocks(ncell);
    l.bytes = l.scan + up256((nb + 1) * 8) + up256(nb * 4);
    return l;
}

int check_ws(const void *ws, int64_t ws_bytes, int64_t need, const char *fn) {
    if (!ws) return fail(PLX_EINVAL, "%s: workspace is NULL", fn);
    if (reinterpret_cast<uintptr_t>(ws) % 256) return fail(PLX_EINVAL, "%s: workspace must be 256-byte aligned", fn);
    if (ws_bytes < need)
        return fail(PLX_EINVAL, "%s: workspace of %lld bytes, need %lld", fn, (long long)ws_bytes, (long long)need);
    return PLX_OK;
}

__global__ void zero_u64_kernel(unsigned long long *p, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) p[i] = 0ull;
}

// Clears the workspace's counters (a kernel rather than a memset node, so
// that a captured graph replays it like any other launch).
int zero_counters(void *ws, hipStream_t s, const char *fn) {
    zero_u64_kernel<<<1, 32, 0, s>>>(static_cast<unsigned long long *>(ws), 32);
    return check_launch(fn);
}

// The counts and offsets lie where the prune keeps its bits: a compaction
// needs one or the other.
template <int ITEMS = kScanItems, class Pred, class Writer>
int run_scan(Pred pred, Writer wr, int64_t n, int32_t *index_out, void *ws, hipStream_t s, const char *what) {
    if (n <= 0) return PLX_OK;
    constexpr int64_t tile = kScanThreads * ITEMS;
    const int64_t nb = (n + tile - 1) / tile;
    if (scan_blocks(n) > 0x7fffffff / (kScanItems / ITEMS)) return fail(PLX_EINVAL, "%s: too many cells", what);
    char *scan = static_cast<char *>(ws) + ws_layout(n).bytes8;
    int64_t *offsets = reinterpret_cast<int64_t *>(scan);
    int *counts = reinterpret_cast<int *>(scan + up256((nb + 1) * 8));
    int rc;
    scan_count_kernel<ITEMS><<<(unsigned)scan_blocks(n), kScanThreads, 0, s>>>(pred, n, nb, counts);
    if ((rc = check_launch(what))) return rc;
    scan_offsets_kernel<<<1, kOffsetThreads, 0, s>>>(counts, nb, offsets);
    if ((rc = check_launch(what))) return rc;
    scan_write_kernel<ITEMS><<<(unsigned)nb, kScanThreads, 0, s>>>(pred, wr, n, index_out, offsets);
    return check_launch(what);
}

// ---- writers
struct IndexWriter {
    static constexpr bool kRecords = false;
    using Item = uint8_t;
    __device__ uint8_t item(int64_t, int) const { return 0; }
    __device__ void records(const uint8_t *, int, int64_t) const {}
};

// CHUNKS: 16-byte chunks per record, one lane each.
template <int CHUNKS>
struct PruneWriter {
    static constexpr bool kRecords = true;
    using Item = int32_t;
    const int32_t *old_index;
    const uint4 *old_data;
    uint4 *new_data;
    __device__ int32_t item(int64_t v, int) const { return old_index[v]; }
    __device__ void records(const int32_t *list, int n, int64_t first) const {
        const int L = threadIdx.x % CHUNKS;
        constexpr int step = kScanThreads / CHUNKS;
        int e = threadIdx.x / CHUNKS;
        // four records in flight per lane
        for (; e + 3 * step < n; e += 4 * step) {
            uint4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = old_data[(int64_t)list[e + u * step] * CHUNKS + L];
#pragma unroll
            for (int u = 0; u < 4; ++u) new_data[(first + e + u * step) * CHUNKS + L] = x[u];
        }
        for (; e < n; e += step) new_data[(first + e) * CHUNKS + L] = old_data[(int64_t)list[e] * CHUNKS + L];
    }
};

// Old-grid coordinate of new voxel j (FP64, same operation order as the
// definition): ((j + 0.5) N_old / N_new) - 0.5, clamped to [0, N_old - 1].
__device__ inline void upsample_coord(int j, int n_old, int n_new, int &i0, double &f) {
    double g = ((double)j + 0.5) * (double)n_old / (double)n_new - 0.5;
    if (g < 0.0) g = 0.0;
    if (g > (double)(n_old - 1)) g = (double)(n_old - 1);
    int c = (int)floor(g);
    if (c > n_old - 2) c = n_old - 2;
    if (c < 0) c = 0;
    i0 = c;
    f = g - (double)c;
}

// Trilinear values in FP64.  The thread that writes a cell's index entry finds
// its lower corner and fractions, once for the record's 8 lanes; these hold
// slots 4L..4L+3 each and the id of one corner for all of them.
template <int DT>
struct UpsampleWriter {
    static constexpr bool kRecords = true;
    // A tile's records are made in turn, 32 at a time, so small tiles: 16, 4 and
    // 2 cells a thread took 830, 562 and 469 us for the 6.1M records of
    // 512x512x128 cells, 18% of them occupied in clusters.
    static constexpr int kItems = 2;
    struct Item {
        int64_t corner;  // the lower corner's place in the old index
        double f[3];
    };
    GridDev go;
    ParentPred pred;
    void *new_data;
    __device__ Item item(int64_t v, int) const {
        int x[3], c[3];
        Item it;
        pred.decode(v, x[0], x[1], x[2]);
        upsample_coord(x[0], go.nx, pred.nn[0], c[0], it.f[0]);
        upsample_coord(x[1], go.ny, pred.nn[1], c[1], it.f[1]);
        upsample_coord(x[2], go.nz, pred.nn[2], c[2], it.f[2]);
        it.corner = ((int64_t)c[0] * go.ny + c[1]) * go.nz + c[2];
        return it;
    }
    __device__ void records(const Item *list, int n, int64_t first) const {
        const int L = threadIdx.x & 7;
        const int64_t my_corner = ((int64_t)(L >> 2) * go.ny + (L >> 1 & 1)) * go.nz + (L & 1);
        for (int e = threadIdx.x >> 3; e < n; e += kScanThreads / 8) {
            const Item it = list[e];
            const double fx = it.f[0], fy = it.f[1], fz = it.f[2];
            const int my = go.index[it.corner + my_corner];
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            int id[8];
            typename Rec<DT>::Raw raw[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                id[q] = __shfl(my, q, 8);
                raw[q] = Rec<DT>::raw(go.data, id[q] < 0 ? 0 : id[q], L);  // the parent's record exists
            }
            auto add = [&](int q) {
                const double w = (q & 4 ? fx : 1.0 - fx) * (q & 2 ? fy : 1.0 - fy) * (q & 1 ? fz : 1.0 - fz);
                const float4 v = Rec<DT>::cvt(raw[q], L);
                acc[0] += w * (double)v.x;
                acc[1] += w * (double)v.y;
                acc[2] += w * (double)v.z;
                acc[3] += w * (double)v.w;
            };
            if (__all(my >= 0)) {  // no NULL corner in the wave's records
#pragma unroll
                for (int q = 0; q < 8; ++q) add(q);
            } else {
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (id[q] >= 0) add(q);
            }
            float o[4] = {(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
            if (L == 6) o[3] = 0.0f;                  // slot 27 is unused,
            if (L == 7) o[1] = o[2] = o[3] = 0.0f;    // as are those after the density
            const int64_t m = first + e;
            if (DT == PLX_F32) {
                reinterpret_cast<float4 *>(static_cast<char *>(new_data) + m * kRecF32Bytes)[L] =
                    make_float4(o[0], o[1], o[2], o[3]);
            } else {
                uint2 w;
                if (L == 7) {
                    w.x = __float_as_uint(o[0]);
                    w.y = 0u;
                } else {
                    w.x = to16<DT>(o[0]) | (to16<DT>(o[1]) << 16);
                    w.y = to16<DT>(o[2]) | (to16<DT>(o[3]) << 16);
                    if (L == 6) w.y &= 0xffffu;
                }
                reinterpret_cast<uint2 *>(static_cast<char *>(new_data) + m * kRec16Bytes)[L] = w;
            }
        }
    }
};

// ---- small kernels

// Counting kernels run a fixed grid of kCountBlocks x kCountThreads threads
// that stride over the input; each block adds its total to the counter with
// one atomic (one atomic per wave on a single address serialises: 2M of them
// for a 512^3 mask).
constexpr int kCountThreads = 256;
constexpr int64_t kCountBlocks = 2048;

inline unsigned count_blocks(int64_t n) {
    const int64_t b = (n + kCountThreads - 1) / kCountThreads;
    return (unsigned)(b < 1 ? 1 : (b > kCountBlocks ? kCountBlocks : b));
}

__device__ void block_add(unsigned long long v, unsigned long long *out) {
    __shared__ unsigned long long part[kCountThreads / 64];
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < kCountThreads / 64; ++w) t += part[w];
        if (t) atomicAdd(out, t);
    }
}

// Adds the block's totals of v0 and v1 to out[0] and out[1].
__device__ void block_add2(unsigned long long v0, unsigned long long v1, unsigned long long *out) {
    __shared__ unsigned long long part[2][kCountThreads / 64];
    for (int o = 32; o >= 1; o >>= 1) {
        v0 += __shfl_xor(v0, o);
        v1 += __shfl_xor(v1, o);
    }
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = v0;
        part[1][threadIdx.x >> 6] = v1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t0 = 0, t1 = 0;
        for (int w = 0; w < kCountThreads / 64; ++w) {
            t0 += part[0][w];
            t1 += part[1][w];
        }
        if (t0) atomicAdd(out, t0);
        if (t1) atomicAdd(out + 1, t1);
    }
}

// Number of non-zero bytes of m[0..n).
__global__ __launch_bounds__(kCountThreads) void count_nonzero_kernel(const uint8_t *m, int64_t n,
                                                                      unsigned long long *out) {
    const int64_t stride = (int64_t)gridDim.x * kCountThreads;
    unsigned long long c = 0;
    for (int64_t i = (int64_t)blockIdx.x * kCountThreads + threadIdx.x; i < n; i += stride)
        c += m[i] != 0;
    block_add(c, out);
}

// Number of set bits among the first nbits bits of w[0..nw).
__global__ __launch_bounds__(kCountThreads) void popcount_kernel(const uint32_t *w, int64_t nw,
                                                                 int64_t nbits,
                                                                 unsigned long long *out) {
    const int64_t stride = (int64_t)gridDim.x * kCountThreads;
    unsigned long long c = 0;
    for (int64_t i = (int64_t)blockIdx.x * kCountThreads + threadIdx.x; i < nw; i += stride) {
        uint32_t x = w[i];
        const int64_t first = i * 32;
        if (first + 32 > nbits) {
            const int keep = (int)(nbits - first);
            x &= keep >= 32 ? 0xffffffffu : ((1u << keep) - 1u);
        }
        c += __popc(x);
    }
    block_add(c, out);
}

template <int DT>
__global__ void pack_kernel(int64_t n, const float *density, const float *sh, float sigma0,
                            float dc, void *out) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * 8) return;
    int64_t m = t >> 3;
    int L = (int)(t & 7);
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        int s = 4 * L + e;
        float x = 0.0f;
        if (s < PLX_NSH)
            x = sh ? sh[m * PLX_NSH + s] : ((s % 9) == 0 ? dc : 0.0f);
        else if (s == PLX_SLOT_SIGMA)
            x = density ? density[m] : sigma0;
        v[e] = x;
    }
    if (DT == PLX_F32) {
        reinterpret_cast<float4 *>(static_cast<char *>(out) + m * kRecF32Bytes)[L] =
            make_float4(v[0], v[1], v[2], v[3]);
    } else {
        uint2 w;
        if (L == 7) {
            w.x = __float_as_uint(v[0]);
            w.y = 0u;
        } else {
            w.x = to16<DT>(v[0]) | (to16<DT>(v[1]) << 16);
            w.y = to16<DT>(v[2]) | (to16<DT>(v[3]) << 16);
            if (L == 6) w.y &= 0xffffu;  // slot 27 unused
        }
        reinterpret_cast<uint2 *>(static_cast<char *>(out) + m * kRec16Bytes)[L] = w;
    }
}

template <int DT>
__global__ void unpack_kernel(int64_t n, const void *rec, float *density, float *sh) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * 32) return;
    int64_t m = t >> 5;
    int s = (int)(t & 31);
    if (s < PLX_NSH) {
        if (sh) sh[m * PLX_NSH + s] = rec_slot<DT>(rec, m, s);
    } else if (s == PLX_SLOT_SIGMA) {
        if (density) density[m] = rec_sigma<DT>(rec, m);
    }
}

// Cell occupancy bits in brick-major order (bit t of brick b is its cell t/64,
// (t/8)%8, t%8; cells outside the lattice, of partial bricks, get 0) and the
// seed of the brick's distance, 0 when any of its bits is set, else far.  One
// wave per brick: the 9x9 rows of 9 index entries that its cells' corners
// share become one bit each (16 lanes a row, four rows at a time), and lane (i, j) combines four
// rows into a byte.  A thread per cell, which read all eight corners and
// divided by the extents, took 150 us for 512x512x128 and 256x256x128 cells
// together; so 93.
__global__ __launch_bounds__(256) void occupancy_kernel(GridDev g, int64_t n_brick, uint8_t *occ,
                                                        uint8_t *bd) {
    __shared__ uint16_t rows_sh[4][9 * 12];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t b = (int64_t)blockIdx.x * 4 + w;
    if (b >= n_brick) return;
    uint16_t *rows = rows_sh[w];
    // (as many bricks as 32 bits count would have 2^41 cells)
    const uint32_t br = (uint32_t)b / (uint32_t)g.bz;
    const int bk = (int)((uint32_t)b - br * g.bz), bi = (int)(br / (uint32_t)g.by), bj = (int)(br - (uint32_t)bi * g.by);
    const int kk = lane & 15, jj = lane >> 4, left_i = g.nx - bi * PLX_BRICK;
    const int left_j = (kk < 9 && bk * PLX_BRICK + kk < g.nz) ? min(9, g.ny - bj * PLX_BRICK) : 0;
    const int64_t sy = g.nz, sx = sy * g.ny;
    const int32_t *p = g.index + ((int64_t)bi * sx + bj * sy + bk) * PLX_BRICK;
    const int64_t off = jj * sy + kk;
    int32_t id[27];
#pragma unroll
    for (int it = 0; it < 27; ++it) {  // entries off the lattice: the brick's first one instead
        const int i = it / 3, j0 = it % 3 * 4;
        id[it] = p[i < left_i && j0 + jj < left_j ? i * sx + j0 * sy + off : 0];
    }
#pragma unroll
    for (int it = 0; it < 27; ++it) {
        const uint64_t m = __ballot(it / 3 < left_i && it % 3 * 4 + jj < left_j && id[it] >= 0);
        if (kk == 0) rows[it * 4 + jj] = (uint16_t)(m >> (lane & 48));
    }
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
    const int i = lane >> 3, j = lane & 7;
    const uint32_t m = rows[i * 12 + j] | rows[i * 12 + j + 1] | rows[i * 12 + j + 12] | rows[i * 12 + j + 13];
    uint32_t bits = (m | m >> 1) & 0xffu;
    const int nk = g.nz - 1 - bk * PLX_BRICK;  // cells of the lattice along k
    if (nk < PLX_BRICK) bits &= (1u << nk) - 1u;
    if (bi * PLX_BRICK + i >= g.nx - 1 || bj * PLX_BRICK + j >= g.ny - 1) bits = 0u;
    occ[b * 64 + lane] = (uint8_t)bits;
    const uint64_t any = __ballot(bits != 0u);
    if (lane == 0) bd[b] = any ? 0 : 255;
}

// Chebyshev distance over bricks, one axis: d(p) <- min over q of max(|p - q|,
// d(q)) along every line of that axis, capped; z, y and x in turn give the
// distance in the three-dimensional maximum norm (three launches instead of
// one relaxation pass per unit of the cap: 174 us to 28 for the bricks
// of 512x512x128 and 256x256x128 cells).  In place: a workgroup owns 8 lines and
// walks them 64 bricks at a time, keeping the old values behind it in LDS.
constexpr int kDistLines = 8, kDistRun = 64, kDistWin = kDistRun + 2 * PLX_BRICK_DIST_CAP;

__global__ __launch_bounds__(256) void brick_dist_kernel(uint8_t *bd, int64_t n_line, int len,
                                                         int64_t stride) {
    __shared__ uint8_t win[kDistWin][kDistLines];
    constexpr int cap = PLX_BRICK_DIST_CAP;
    const int ln = threadIdx.x % kDistLines, t = threadIdx.x / kDistLines;
    constexpr int nt = 256 / kDistLines;
    const int64_t l = (int64_t)blockIdx.x * kDistLines + ln;
    uint8_t *line = bd + (l / stride) * (stride * len) + l % stride;
    const bool live = l < n_line;
    for (int p0 = 0; p0 < len; p0 += kDistRun) {
        // window rows 0..2cap-1 are rows kDistRun.. of the window before
        // (rows of the run behind, then the first `cap` of this one)
        uint8_t keep[2 * cap / nt];
#pragma unroll
        for (int u = 0; u < 2 * cap / nt; ++u) {
            const int r = t + u * nt, p = p0 - cap + r;
            if (p0 > 0) keep[u] = win[kDistRun + r][ln];
            else keep[u] = live && p >= 0 && p < len ? line[p * stride] : 255;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2 * cap / nt; ++u) win[t + u * nt][ln] = keep[u];
        for (int r = 2 * cap + t; r < kDistWin; r += nt) {
            const int p = p0 - cap + r;
            win[r][ln] = live && p < len ? line[p * stride] : 255;
        }
        __syncthreads();
        for (int r = cap + t; r < cap + kDistRun; r += nt) {
            int d = win[r][ln] < cap ? win[r][ln] : cap;
            for (int o = 1; o < d; ++o) {
                const int a = win[r - o][ln], c = win[r + o][ln];
                const int m = a < c ? a : c, x = m > o ? m : o;
                d = x < d ? x : d;
            }
            if (live && p0 + r - cap < len) line[(p0 + r - cap) * stride] = (uint8_t)d;
        }
        __syncthreads();
    }
}

// Occupied and stored cells as one bit each, 32 cells a word: bits[0 ..
// 2 nw64) and the same number of words after them (nw64 = 64-cell words).
// Occupied: a voxel with density (value == NULL) or value[id] >= thresh.
template <int DT>
__global__ __launch_bounds__(256) void prune_bits_kernel(GridDev g, int64_t ncell, const float *value,
                                                         float thresh, unsigned long long *bits) {
    constexpr int kCells = 4;  // per thread, their reads in flight together
    const int lane = threadIdx.x & 63;
    const int64_t nw = (ncell + 63) / 64, w0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kCells;
    int32_t id[kCells];
    float x[kCells];
#pragma unroll
    for (int u = 0; u < kCells; ++u) {
        const int64_t v = (w0 + u) * 64 + lane;
        id[u] = v < ncell ? g.index[v] : -1;
    }
#pragma unroll
    for (int u = 0; u < kCells; ++u)
        x[u] = id[u] < 0 ? 0.0f : value ? value[id[u]] : rec_sigma<DT>(g.data, id[u]);
#pragma unroll
    for (int u = 0; u < kCells; ++u) {
        const uint64_t stored = __ballot(id[u] >= 0), occ = __ballot(id[u] >= 0 && x[u] >= thresh);
        if (lane == 0 && w0 + u < nw) {
            bits[w0 + u] = occ;
            bits[nw + w0 + u] = stored;
        }
    }
}

// 34 bits of a bit string of n words from bit b on (b >= -1; bits before and
// after the string are 0).
__device__ inline uint64_t bits34(const uint32_t *w, int64_t n, int64_t b) {
    const int64_t i = b >> 5;  // floor
    const int s = (int)(b & 31);
    const uint64_t a = i >= 0 && i < n ? w[i] : 0u, c = i + 1 < n ? w[i + 1] : 0u, d = i + 2 < n ? w[i + 2] : 0u;
    uint64_t x = (a | c << 32) >> s;
    if (s > 30) x |= d << (64 - s);
    return x & 0x3ffffffffull;
}

// keep = stored with an occupied voxel in the 3x3x3 neighbourhood, for 32
// cells of a row at a time: the nine rows' bits, unaligned, ORed and spread by
// one cell.  Reading 27 bytes for every cell took 207 us for 256x256x128
// cells; so 31.
__global__ __launch_bounds__(kCountThreads) void prune_keep_kernel(GridDev g, int64_t ncell,
                                                                   const uint32_t *bits, uint8_t *keep,
                                                                   unsigned long long *counts) {
    __shared__ uint32_t word_sh[kCountThreads];
    __shared__ int64_t cell_sh[kCountThreads];
    __shared__ uint8_t cells_sh[kCountThreads];
    const int64_t nw = 2 * ((ncell + 63) / 64);
    const int per_row = (g.nz + 31) / 32;
    const int64_t n_grp = (int64_t)g.nx * g.ny * per_row;
    unsigned long long n_kept = 0, n_stored = 0;
    for (int64_t g0 = (int64_t)blockIdx.x * kCountThreads; g0 < n_grp; g0 += (int64_t)gridDim.x * kCountThreads) {
        const int64_t grp = g0 + threadIdx.x;
        uint32_t kept = 0u;
        int64_t cell = 0;
        int cells = 0;
        if (grp < n_grp) {
            const int k0 = (int)(grp % per_row) * 32;
            const int64_t r = grp / per_row;
            const int j = (int)(r % g.ny), i = (int)(r / g.ny);
            uint64_t near = 0;
            for (int a = -1; a <= 1; ++a)
                for (int c = -1; c <= 1; ++c)
                    if (i + a >= 0 && i + a < g.nx && j + c >= 0 && j + c < g.ny)
                        near |= bits34(bits, nw, (r + (int64_t)a * g.ny + c) * g.nz + k0 - 1);
            if (k0 == 0) near &= ~1ull;  // the row's own cells only
            const int left = g.nz - k0;
            if (left < 33) near &= (1ull << (left + 1)) - 1;
            uint32_t stored = (uint32_t)(bits34(bits + nw, nw, r * g.nz + k0 - 1) >> 1);
            if (left < 32) stored &= (1u << left) - 1u;
            kept = (uint32_t)(near | near >> 1 | near >> 2) & stored;
            n_kept += __popc(kept);
            n_stored += __popc(stored);
            cell = r * g.nz + k0;
            cells = left < 32 ? left : 32;
        }
        __syncthreads();  // the words before are written
        word_sh[threadIdx.x] = kept;
        cell_sh[threadIdx.x] = cell;
        cells_sh[threadIdx.x] = (uint8_t)cells;
        __syncthreads();
#pragma unroll 4
        for (int c = threadIdx.x; c < kCountThreads * 32; c += kCountThreads)
            if (c % 32 < cells_sh[c / 32]) keep[cell_sh[c / 32] + c % 32] = word_sh[c / 32] >> (c % 32) & 1u;
    }
    block_add2(n_kept, n_stored, counts);
}

__global__ __launch_bounds__(kCountThreads) void upsample_count_kernel(ParentPred pred, int64_t n,
                                                                       unsigned long long *out) {
    unsigned long long c = 0;
    for (int64_t v = ((int64_t)blockIdx.x * kCountThreads + threadIdx.x) * kScanItems; v < n;
         v += (int64_t)gridDim.x * kCountThreads * kScanItems)
        c += __popc(pred.flags<kScanItems>(v, n));
    block_add(c, out);
}

template <int DS, int DD>
__global__ void convert_kernel(int64_t n, const void *src, void *dst) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * 8) return;
    int64_t m = t >> 3;
    int L = (int)(t & 7);
    float4 x = Rec<DS>::load4(src, m, L);
    float v[4] = {x.x, x.y, x.z, x.w};
    if (DD == PLX_F32) {
        reinterpret_cast<float4 *>(static_cast<char *>(dst) + m * kRecF32Bytes)[L] =
            make_float4(v[0], v[1], v[2], v[3]);
    } else {
        uint2 w;
        if (L == 7) {
            w.x = __float_as_uint(v[0]);
            w.y = 0u;
        } else {
            w.x = to16<DD>(v[0]) | (to16<DD>(v[1]) << 16);
            w.y = to16<DD>(v[2]) | (to16<DD>(v[3]) << 16);
            if (L == 6) w.y &= 0xffffu;
        }
        reinterpret_cast<uint2 *>(static_cast<char *>(dst) + m * kRec16Bytes)[L] = w;
    }
}

int sync_read_u64(const unsigned long long *dev, int n, int64_t *host, hipStream_t s,
                  const char *what) {
    unsigned long long tmp[4] = {0, 0, 0, 0};
    PLX_CHECK_HIP(hipMemcpyAsync(tmp, dev, n * sizeof(unsigned long long), hipMemcpyDeviceToHost, s),
                  what);
    PLX_CHECK_HIP(hipStreamSynchronize(s), what);
    for (int i = 0; i < n; ++i) host[i] = (int64_t)tmp[i];
    return PLX_OK;
}

inline unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

MaskPred mask_pred(const uint8_t *mask) {
    return {mask, reinterpret_cast<uintptr_t>(mask) % 16 == 0};
}

ParentPred parent_pred(const plx_grid *grid, const int32_t new_reso[3]) {
    ParentPred p{grid->index, {}, {}, n_cells(new_reso) < (1ll << 32)};
    for (int a = 0; a < 3; ++a) {
        p.on[a] = grid->reso[a];
        p.nn[a] = new_reso[a];
        p.narrow = p.narrow && 2 * (uint64_t)new_reso[a] * (uint64_t)grid->reso[a] < (1ull << 32);
    }
    return p;
}

// Shared by both prune counts: occupied = non-NULL with density (value ==
// NULL) or value[id] at least thresh; kept = non-NULL with an occupied voxel
// in its 3x3x3 neighbourhood.
int prune_count(const plx_grid *grid, const float *value, float thresh, uint8_t *keep_out, void *ws,
                int64_t ws_bytes, int64_t *n_kept, int64_t *n_pruned, plx_stream stream,
                const char *fn) {
    int rc = validate_grid(grid, false, fn);
    if (rc) return rc;
    if (!keep_out || !n_kept || !n_pruned) return fail(PLX_EINVAL, "%s: NULL argument", fn);
    hipStream_t s = as_stream(stream);
    int64_t ncell = n_cells(grid->reso);
    const WsLayout l = ws_layout(ncell);
    if ((rc = check_ws(ws, ws_bytes, l.bytes, fn))) return rc;
    auto *counts = static_cast<unsigned long long *>(ws);
    auto *bits = reinterpret_cast<unsigned long long *>(static_cast<char *>(ws) + l.bytes8);
    if ((rc = zero_counters(ws, s, fn))) return rc;
    GridDev g = to_dev(grid);
    PLX_DISPATCH_DT(grid->sh_dtype, DT,
                    prune_bits_kernel<DT><<<blocks_for(ncell, 1024), 256, 0, s>>>(g, ncell, value, thresh, bits));
    if ((rc = check_launch(fn))) return rc;
    prune_keep_kernel<<<count_blocks(ncell), kCountThreads, 0, s>>>(g, ncell, reinterpret_cast<const uint32_t *>(bits),
                                                                         keep_out, counts);
    if ((rc = check_launch(fn))) return rc;
    int64_t h[2];
    if ((rc = sync_read_u64(counts, 2, h, s, fn))) return rc;
    *n_kept = h[0];
    *n_pruned = h[1] - h[0];
    return PLX_OK;
}

}  // namespace
}  // namespace plx

using namespace plx;

extern "C" {

int64_t plx_grid_workspace_bytes(const int32_t reso[3]) {
    if (!reso || reso[0] < 2 || reso[1] < 2 || reso[2] < 2) return 0;
    return ws_layout(n_cells(reso)).bytes;
}

int plx_mask_count(const uint8_t *mask, int64_t n, void *ws, int64_t ws_bytes, int64_t *count_out,
                   plx_stream stream) {
    if (!count_out) return fail(PLX_EINVAL, "plx_mask_count: count_out is NULL");
    if (n < 0) return fail(PLX_EINVAL, "plx_mask_count: n < 0");
    int rc = check_ws(ws, ws_bytes, PLX_COUNT_WORKSPACE_BYTES, "plx_mask_count");
    if (rc) return rc;
    if (n == 0) {
        *count_out = 0;
        return PLX_OK;
    }
    if (!mask) return fail(PLX_EINVAL, "plx_mask_count: mask is NULL");
    hipStream_t s = as_stream(stream);
    auto *cnt = static_cast<unsigned long long *>(ws);
    if ((rc = zero_counters(ws, s, "plx_mask_count"))) return rc;
    count_nonzero_kernel<<<count_blocks(n), kCountThreads, 0, s>>>(mask, n, cnt);
    if ((rc = check_launch("plx_mask_count"))) return rc;
    return sync_read_u64(cnt, 1, count_out, s, "plx_mask_count");
}

int plx_grid_create(const uint8_t *mask, const int32_t reso[3], int32_t *index_out, void *ws,
                    int64_t ws_bytes, plx_stream stream) {
    if (!mask || !reso || !index_out) return fail(PLX_EINVAL, "plx_grid_create: NULL argument");
    for (int a = 0; a < 3; ++a)
        if (reso[a] < 2) return fail(PLX_EINVAL, "plx_grid_create: reso[%d] < 2", a);
    int64_t n = n_cells(reso);
    int rc = check_ws(ws, ws_bytes, ws_layout(n).bytes, "plx_grid_create");
    if (rc) return rc;
    return run_scan(mask_pred(mask), IndexWriter{}, n, index_out, ws, as_stream(stream), "plx_grid_create");
}

int plx_records_pack(int32_t sh_dtype, int64_t n, const float *density, const float *sh,
                     float sigma0, float dc, void *out, plx_stream stream) {
    if (n < 0) return fail(PLX_EINVAL, "plx_records_pack: n < 0");
    if (n == 0) return PLX_OK;
    if (!out) return fail(PLX_EINVAL, "plx_records_pack: out is NULL");
    hipStream_t s = as_stream(stream);
    PLX_DISPATCH_DT(sh_dtype, DT,
                    pack_kernel<DT><<<blocks_for(n * 8, 256), 256, 0, s>>>(n, density, sh, sigma0,
                                                                           dc, out));
    return check_launch("plx_records_pack");
}

int plx_records_unpack(int32_t sh_dtype, int64_t n, const void *records, float *density,
                       float *sh, plx_stream stream) {
    if (n < 0) return fail(PLX_EINVAL, "plx_records_unpack: n < 0");
    if (n == 0) return PLX_OK;
    if (!records) return fail(PLX_EINVAL, "plx_records_unpack: records is NULL");
    hipStream_t s = as_stream(stream);
    PLX_DISPATCH_DT(sh_dtype, DT,
                    unpack_kernel<DT><<<blocks_for(n * 32, 256), 256, 0, s>>>(n, records, density, sh));
    return check_launch("plx_records_unpack");
}

int plx_records_convert(int32_t src_dtype, const void *src, int32_t dst_dtype, void *dst,
                        int64_t n, plx_stream stream) {
    if (n < 0) return fail(PLX_EINVAL, "plx_records_convert: n < 0");
    if (n == 0) return PLX_OK;
    if (!src || !dst) return fail(PLX_EINVAL, "plx_records_convert: NULL argument");
    hipStream_t s = as_stream(stream);
    unsigned nb = blocks_for(n * 8, 256);
    PLX_DISPATCH_DT(src_dtype, DS,
                    PLX_DISPATCH_DT(dst_dtype, DD,
                                    convert_kernel<DS, DD><<<nb, 256, 0, s>>>(n, src, dst)));
    return check_launch("plx_records_convert");
}

int plx_grid_build_occupancy(const plx_grid *grid, uint32_t *occ_out, plx_stream stream) {
    int rc = validate_grid(grid, false, "plx_grid_build_occupancy");
    if (rc) return rc;
    if (!occ_out) return fail(PLX_EINVAL, "plx_grid_build_occupancy: occ_out is NULL");
    hipStream_t s = as_stream(stream);
    plx_grid gd = *grid;
    gd.occ = occ_out;
    GridDev g = to_dev(&gd);
    uint8_t *bd = reinterpret_cast<uint8_t *>(occ_out) + occ_brick_offset(grid->reso);
    const int64_t nb = n_bricks(grid->reso);
    occupancy_kernel<<<blocks_for(nb, 4), 256, 0, s>>>(g, nb, reinterpret_cast<uint8_t *>(occ_out), bd);
    if ((rc = check_launch("plx_grid_build_occupancy"))) return rc;
    const int len[3] = {g.bz, g.by, g.bx};
    int64_t stride = 1;
    for (int a = 0; a < 3; ++a) {
        const int64_t lines = nb / len[a];
        brick_dist_kernel<<<blocks_for(lines, kDistLines), 256, 0, s>>>(bd, lines, len[a], stride);
        if ((rc = check_launch("plx_grid_build_occupancy"))) return rc;
        stride *= len[a];
    }
    return PLX_OK;
}

int plx_grid_prune_count(const plx_grid *grid, float sigma_thresh, uint8_t *keep_out, void *ws,
                         int64_t ws_bytes, int64_t *n_kept, int64_t *n_pruned, plx_stream stream) {
    return plx::prune_count(grid, nullptr, sigma_thresh, keep_out, ws, ws_bytes, n_kept, n_pruned,
                            stream, "plx_grid_prune_count");
}

int plx_grid_prune_weight_count(const plx_grid *grid, const float *wmax, float w_thresh,
                                uint8_t *keep_out, void *ws, int64_t ws_bytes, int64_t *n_kept,
                                int64_t *n_pruned, plx_stream stream) {
    if (!wmax) return plx::fail(PLX_EINVAL, "plx_grid_prune_weight_count: wmax is NULL");
    return plx::prune_count(grid, wmax, w_thresh, keep_out, ws, ws_bytes, n_kept, n_pruned, stream,
                            "plx_grid_prune_weight_count");
}

int plx_grid_prune_apply(const plx_grid *grid, const uint8_t *keep, plx_grid *out, void *ws,
                         int64_t ws_bytes, plx_stream stream) {
    int rc = validate_grid(grid, false, "plx_grid_prune_apply");
    if (rc) return rc;
    if (!keep || !out || !out->index) return fail(PLX_EINVAL, "plx_grid_prune_apply: NULL argument");
    for (int a = 0; a < 3; ++a)
        if (out->reso[a] != grid->reso[a])
            return fail(PLX_EINVAL, "plx_grid_prune_apply: out->reso differs from grid->reso");
    if (out->sh_dtype != grid->sh_dtype)
        return fail(PLX_EINVAL, "plx_grid_prune_apply: out->sh_dtype differs");
    if (out->n_vox > 0 && !out->data) return fail(PLX_EINVAL, "plx_grid_prune_apply: out->data is NULL");
    if ((rc = check_ws(ws, ws_bytes, ws_layout(n_cells(grid->reso)).bytes, "plx_grid_prune_apply"))) return rc;
    auto run = [&](auto writer) {
        return run_scan(mask_pred(keep), writer, n_cells(grid->reso), const_cast<int32_t *>(out->index), ws,
                        as_stream(stream), "plx_grid_prune_apply");
    };
    const auto *src = static_cast<const uint4 *>(grid->data);
    auto *dst = static_cast<uint4 *>(const_cast<void *>(static_cast<const void *>(out->data)));
    if (grid->sh_dtype == PLX_F32) return run(PruneWriter<kRecF32Bytes / 16>{grid->index, src, dst});
    return run(PruneWriter<kRec16Bytes / 16>{grid->index, src, dst});
}

int plx_grid_upsample_count(const plx_grid *grid, const int32_t new_reso[3], void *ws,
                            int64_t ws_bytes, int64_t *n_out, plx_stream stream) {
    int rc = validate_grid(grid, false, "plx_grid_upsample_count");
    if (rc) return rc;
    if (!new_reso || !n_out) return fail(PLX_EINVAL, "plx_grid_upsample_count: NULL argument");
    for (int a = 0; a < 3; ++a)
        if (new_reso[a] < 2) return fail(PLX_EINVAL, "plx_grid_upsample_count: new_reso[%d] < 2", a);
    hipStream_t s = as_stream(stream);
    const ParentPred pred = parent_pred(grid, new_reso);
    int64_t n = n_cells(new_reso);
    if ((rc = check_ws(ws, ws_bytes, PLX_COUNT_WORKSPACE_BYTES, "plx_grid_upsample_count"))) return rc;
    auto *cnt = static_cast<unsigned long long *>(ws);
    if ((rc = zero_counters(ws, s, "plx_grid_upsample_count"))) return rc;
    upsample_count_kernel<<<count_blocks((n + kScanItems - 1) / kScanItems), kCountThreads, 0, s>>>(pred, n, cnt);
    if ((rc = check_launch("plx_grid_upsample_count"))) return rc;
    return sync_read_u64(cnt, 1, n_out, s, "plx_grid_upsample_count");
}

int plx_grid_upsample_apply(const plx_grid *grid, plx_grid *out, void *ws, int64_t ws_bytes,
                            plx_stream stream) {
    int rc = validate_grid(grid, false, "plx_grid_upsample_apply");
    if (rc) return rc;
    if (!out || !out->index) return fail(PLX_EINVAL, "plx_grid_upsample_apply: NULL argument");
    for (int a = 0; a < 3; ++a)
        if (out->reso[a] < 2) return fail(PLX_EINVAL, "plx_grid_upsample_apply: out->reso[%d] < 2", a);
    if (out->sh_dtype != grid->sh_dtype)
        return fail(PLX_EINVAL, "plx_grid_upsample_apply: out->sh_dtype differs from grid->sh_dtype");
    if (out->n_vox > 0 && !out->data) return fail(PLX_EINVAL, "plx_grid_upsample_apply: out->data is NULL");
    hipStream_t s = as_stream(stream);
    const ParentPred pred = parent_pred(grid, out->reso);
    int64_t n = n_cells(out->reso);
    if ((rc = check_ws(ws, ws_bytes, ws_layout(n).bytes, "plx_grid_upsample_apply"))) return rc;
    GridDev g = to_dev(grid);
    PLX_DISPATCH_DT(grid->sh_dtype, DT,
                    return run_scan<UpsampleWriter<DT>::kItems>(pred, UpsampleWriter<DT>{g, pred, const_cast<void *>(out->data)},
                                    n, const_cast<int32_t *>(out->index), ws, s, "plx_grid_upsample_apply"));
    return PLX_OK;
}

int plx_touched_count(const uint8_t *touched, int64_t n_vox, void *ws, int64_t ws_bytes,
                      int64_t *count_out, plx_stream stream) {
    if (!count_out) return fail(PLX_EINVAL, "plx_touched_count: count_out is NULL");
    if (n_vox < 0) return fail(PLX_EINVAL, "plx_touched_count: n_vox < 0");
    int rc = check_ws(ws, ws_bytes, PLX_COUNT_WORKSPACE_BYTES, "plx_touched_count");
    if (rc) return rc;
    if (n_vox == 0) {
        *count_out = 0;
        return PLX_OK;
    }
    if (!touched) return fail(PLX_EINVAL, "plx_touched_count: touched is NULL");
    hipStream_t s = as_stream(stream);
    auto *cnt = static_cast<unsigned long long *>(ws);
    if ((rc = zero_counters(ws, s, "plx_touched_count"))) return rc;
    count_nonzero_kernel<<<count_blocks(n_vox), kCountThreads, 0, s>>>(touched, n_vox, cnt);
    if ((rc = check_launch("plx_touched_count"))) return rc;
    return sync_read_u64(cnt, 1, count_out, s, "plx_touched_count");
}

}  // extern "C"

namespace plx {

int count_set_bits(const uint32_t *words, int64_t n_bits, void *ws, int64_t *count_out,
                   hipStream_t s, const char *fn) {
    if (n_bits <= 0) {
        *count_out = 0;
        return PLX_OK;
    }
    const int64_t nw = (n_bits + 31) / 32;
    auto *cnt = static_cast<unsigned long long *>(ws);
    int rc = zero_counters(ws, s, fn);
    if (rc) return rc;
    popcount_kernel<<<count_blocks(nw), kCountThreads, 0, s>>>(words, nw, n_bits, cnt);
    if ((rc = check_launch(fn))) return rc;
    return sync_read_u64(cnt, 1, count_out, s, fn);
}

}  // namespace plx
