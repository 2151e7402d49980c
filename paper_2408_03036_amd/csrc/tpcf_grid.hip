// Neighbour grid: a counting sort of the points by cell (the linked-list
// spatial partition of Sec. 4.1, laid out as contiguous per-cell ranges so
// the pair pass reads neighbour cells with coalesced loads).
//
// Steps: assign (wrap, cell id, histogram) -> scan (cell starts) ->
// scatter (atomic slots) -> order (rank by z, then input index, inside a
// cell, so the layout is deterministic) -> fill (sorted SoA copies).
//
// Crowded cells (long shells in a small box, explicit randoms, the one-cell
// grid) are counted in z slabs: the histogram and the rank then work on a few
// points at a time. With one counter and one quadratic rank per cell, 102,051
// points in one cell took 14.1 ms (order 11.8 ms, the two passes of atomics on
// the one counter 1.15 ms each); with slabs the three kernels take 0.026 ms.
#include "tpcf_cells.h"

namespace tpcf {

namespace {

__device__ inline double wrap_coord(double x, double L) {
    double y = fmod(x, L);
    if (y < 0.0) y += L;
    if (y >= L) y -= L;
    return y;
}

__device__ inline int cell_of(double x, const Grid& g) {
    int c = (int)(x * g.inv_h);
    c = c < 0 ? 0 : c;
    return c >= g.nc ? g.nc - 1 : c;
}

// z slab of a wrapped z inside cell cz: monotone in z (products and floors of
// z are, and the clamp is), so the slabs of a cell follow each other in z and
// points of equal z share one.
__device__ inline int slab_of(double z, int cz, const Grid& g) {
    if (g.zsub == 1) return 0;
    const int s = (int)(z * g.inv_hs) - cz * g.zsub;
    return s < 0 ? 0 : (s >= g.zsub ? g.zsub - 1 : s);
}

__device__ inline int find_cat(const int64_t* off, int ncat, int64_t i) {
    int lo = 0, hi = ncat;  // off[lo] <= i < off[hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

__global__ void k_grid_assign(const double* __restrict__ pos, int64_t n,
                              const int64_t* __restrict__ pt_off, int ncat, Grid g,
                              int* __restrict__ cellid, int* __restrict__ count,
                              int* __restrict__ nonfinite, int* __restrict__ catbad) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
    int c = find_cat(pt_off, ncat, i);
    if (!isfinite(x) || !isfinite(y) || !isfinite(z)) {
        atomicAdd(nonfinite, 1);
        atomicAdd(&catbad[c], 1);
        x = y = z = 0.0;
    }
    x = wrap_coord(x, g.box);
    y = wrap_coord(y, g.box);
    z = wrap_coord(z, g.box);
    const int cz = cell_of(z, g);
    int id = c * g.ncell + (cell_of(x, g) * g.nc + cell_of(y, g)) * g.nc + cz;
    cellid[i] = id;
    atomicAdd(&count[(int64_t)id * g.zsub + slab_of(z, cz, g)], 1);
}

// Exclusive scan of m counts, and of the work items that cells of those counts
// hold, both in one 64-bit sum (counts in the low half: all of them are less
// than 2^31). Blocks of kScanBlock elements: their sums, then each block's scan
// from the sum of the blocks before it, which a block adds up itself: up to
// kScanDirect of them that costs less than a launch for their scan.
// One block takes k_scan_apply alone. Launches bound this stage on small
// grids: with a scan of its own for the items, and a launch for the offsets,
// 41,000 cells took seven launches and 35 us of kernels, now two and 7.5.
constexpr int kScanBlock = 4096;  // 256 threads x 16 elements
constexpr int kScanDirect = 2048;

using ScanSum = unsigned long long;

__device__ __forceinline__ ScanSum scan_value(int n) {
    return (ScanSum)(uint32_t)n | ((ScanSum)(uint32_t)((n + kItemPrims - 1) / kItemPrims) << 32);
}

// Elements [e0, e0 + 16) of the counts (zero past m).
__device__ __forceinline__ void scan_load(const int* __restrict__ count, int64_t e0, int64_t m, int (&v)[16]) {
    if (e0 + 16 <= m) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int4 q = *reinterpret_cast<const int4*>(count + e0 + 4 * k);
            v[4 * k] = q.x, v[4 * k + 1] = q.y, v[4 * k + 2] = q.z, v[4 * k + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = e0 + k < m ? count[e0 + k] : 0;
    }
}

__device__ __forceinline__ ScanSum wave_sum(ScanSum v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ ScanSum wave_scan(ScanSum v) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const ScanSum u = __shfl_up(v, o);
        if (lane_id() >= o) v += u;
    }
    return v;
}

__global__ void __launch_bounds__(256) k_scan_sums(const int* __restrict__ count, int64_t m,
                                                   ScanSum* __restrict__ sums) {
    __shared__ ScanSum part[4];
    int v[16];
    scan_load(count, (int64_t)blockIdx.x * kScanBlock + 16 * threadIdx.x, m, v);
    ScanSum s = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += scan_value(v[k]);
    s = wave_sum(s);
    if (lane_id() == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// One workgroup, a segment of the sums per thread.
__global__ void __launch_bounds__(1024) k_scan_offsets(const ScanSum* __restrict__ sums, int64_t nb,
                                                       ScanSum* __restrict__ offs) {
    __shared__ ScanSum part[16];
    const int t = threadIdx.x;
    const int64_t seg = (nb + 1023) / 1024;
    const int64_t a = t * seg < nb ? t * seg : nb;
    const int64_t b = a + seg < nb ? a + seg : nb;
    ScanSum s = 0;
    for (int64_t i = a; i < b; ++i) s += sums[i];
    const ScanSum incl = wave_scan(s);
    if (lane_id() == 63) part[t >> 6] = incl;
    __syncthreads();
    ScanSum run = incl - s;
    for (int w = 0; w < t >> 6; ++w) run += part[w];
    for (int64_t i = a; i < b; ++i) {
        offs[i] = run;
        run += sums[i];
    }
}

// The offset of a block: offs, or with none the sums of the blocks before it.
__global__ void __launch_bounds__(256) k_scan_apply(const int* __restrict__ count, int64_t m,
                                                    const ScanSum* __restrict__ sums,
                                                    const ScanSum* __restrict__ offs, int* __restrict__ start,
                                                    int* __restrict__ istart) {
    __shared__ ScanSum part[4], pre[4];
    const int t = threadIdx.x, wave = t >> 6;
    const int64_t e0 = (int64_t)blockIdx.x * kScanBlock + 16 * t;
    int v[16];
    scan_load(count, e0, m, v);
    ScanSum s = 0, before = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += scan_value(v[k]);
    if (offs == nullptr)
        for (int i = t; i < (int)blockIdx.x; i += 256) before += sums[i];
    else if (t == 0)
        before = offs[blockIdx.x];
    before = wave_sum(before);
    const ScanSum incl = wave_scan(s);
    if (lane_id() == 63) {
        part[wave] = incl;
        pre[wave] = before;
    }
    __syncthreads();
    ScanSum run = pre[0] + pre[1] + pre[2] + pre[3] + incl - s;
    for (int w = 0; w < wave; ++w) run += part[w];
    int o[17], q[17];
#pragma unroll
    for (int k = 0; k < 17; ++k) {
        o[k] = (int)(uint32_t)run;
        q[k] = (int)(uint32_t)(run >> 32);
        if (k < 16) run += scan_value(v[k]);
    }
    if (e0 + 16 <= m) {
#pragma unroll
        for (int k = 0; k < 16; k += 4) {
            *reinterpret_cast<int4*>(start + e0 + k) = make_int4(o[k], o[k + 1], o[k + 2], o[k + 3]);
            if (istart) *reinterpret_cast<int4*>(istart + e0 + k) = make_int4(q[k], q[k + 1], q[k + 2], q[k + 3]);
        }
    }
#pragma unroll
    for (int k = 0; k < 17; ++k) {
        // the ragged end, and the total past the last element
        if (e0 + 16 <= m ? k == 16 && e0 + 16 == m : e0 + k <= m && (k > 0 || e0 < m)) {
            start[e0 + k] = o[k];
            if (istart) istart[e0 + k] = q[k];
        }
    }
}

__global__ void k_grid_scatter(const int* __restrict__ cellid, int64_t n, Grid g,
                               const int* __restrict__ start, int* __restrict__ cursor,
                               const double* __restrict__ pos,
                               int* __restrict__ tmp_idx, double* __restrict__ tmp_key) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    // the order key: the wrapped z the fill stores (0 for a non-finite point)
    const double x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
    const bool fin = isfinite(x) && isfinite(y) && isfinite(z);
    const double key = wrap_coord(fin ? z : 0.0, g.box);
    const int id = cellid[i];
    const int64_t c = (int64_t)id * g.zsub + slab_of(key, id % g.nc, g);
    const int at = start[c] + atomicAdd(&cursor[c], 1);
    tmp_idx[at] = (int)i;
    tmp_key[at] = key;
}

// Placement inside a cell by z, ties by input index: a point's rank is the
// number of points of its z slab that come before it in that order. Along
// every run of cells consecutive in z the points are then in increasing z,
// which lets the pair pass cut a run to the z range a work item can reach.
// The layout is deterministic.
__global__ void k_grid_order(const int* __restrict__ cellid, int64_t n, Grid g,
                             const int* __restrict__ start, const int* __restrict__ tmp_idx,
                             const double* __restrict__ tmp_key, int* __restrict__ orig) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int i = tmp_idx[s];
    const double zi = tmp_key[s];
    const int id = cellid[i];
    const int64_t c = (int64_t)id * g.zsub + slab_of(zi, id % g.nc, g);
    const int a = start[c], b = start[c + 1];
    int rank = 0;
    for (int t = a; t < b; ++t) {
        const double zt = tmp_key[t];
        rank += zt < zi || (zt == zi && tmp_idx[t] < i);
    }
    orig[a + rank] = i;
}

__global__ void k_grid_fill(const double* __restrict__ pos, const double* __restrict__ w,
                            int64_t n, const int* __restrict__ orig,
                            const int* __restrict__ cellid, Grid g, float4* __restrict__ pf,
                            float* __restrict__ pw, float4* __restrict__ pa, double4* __restrict__ pd,
                            int* __restrict__ perm, int* __restrict__ catid,
                            const int* __restrict__ cell_start, const int* __restrict__ item_start,
                            int* __restrict__ item_cell) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    int i = orig[s];
    double x = pos[3 * (int64_t)i], y = pos[3 * (int64_t)i + 1], z = pos[3 * (int64_t)i + 2];
    if (!isfinite(x) || !isfinite(y) || !isfinite(z)) x = y = z = 0.0;
    x = wrap_coord(x, g.box);
    y = wrap_coord(y, g.box);
    z = wrap_coord(z, g.box);
    double wi = w ? w[i] : 1.0;
    int id = cellid[i];
    int cat = id / g.ncell;
    int loc = id - cat * g.ncell;
    int cz = loc % g.nc;
    int cy = (loc / g.nc) % g.nc;
    int cx = loc / (g.nc * g.nc);
    // Offsets from the cell's lower corner; exact in FP64, rounded once to FP32.
    float4 q;
    q.x = (float)(x - cx * g.h);
    q.y = (float)(y - cy * g.h);
    q.z = (float)(z - cz * g.h);
    q.w = (float)cz;
    pf[s] = q;
    pw[s] = (float)wi;
    pa[s] = make_float4(q.x, q.y, q.z, (float)wi);
    pd[s] = make_double4(x, y, z, wi);
    perm[i] = (int)s;
    catid[s] = cat;
    // the first point of each work item names its cell (a thread per cell,
    // writing all its items, took 0.17 ms for 102,051 points in one cell)
    const int at = (int)s - cell_start[id];
    if (at % kItemPrims == 0) item_cell[item_start[id] + at / kItemPrims] = id;
}

// Zeroes several buffers in one launch (a launch of its own costs each small
// one 3 us of a call that takes 200).
__global__ void k_clear(ClearRanges r) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kClearRanges; ++k) {
        if (i >= 0 && i < r.n[k]) r.p[k][i] = 0;
        i -= r.n[k];
    }
}
// A small table, out of the launch's own arguments.
__global__ void k_put(uint32_t* __restrict__ dst, int n, PutWords w) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = w.v[i];
}
__global__ void k_publish(const int* __restrict__ src, int n, int* __restrict__ host) {
    if ((int)threadIdx.x < n) host[threadIdx.x] = src[threadIdx.x];
}
__global__ void k_fill_u64(unsigned long long* p, int64_t n, unsigned long long v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_grid_cells(const int* __restrict__ slab_start, int64_t m, int zsub, int* __restrict__ cell_start) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c <= m) cell_start[c] = slab_start[c * zsub];
}

// Work items of the binning pass: cell c holds ceil(count / kItemPrims) items.
__global__ void k_items_count(const int* __restrict__ cell_start, int64_t m, int* __restrict__ nitems) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= m) return;
    const int n = cell_start[c + 1] - cell_start[c];
    nitems[c] = (n + kItemPrims - 1) / kItemPrims;
}

// What the host reads of a grid, written to its (pinned) memory: the count of
// non-finite positions, and the first work item of every catalogue.
__global__ void k_items_cat(const int* __restrict__ item_start, int ncat, int ncell,
                            const int* __restrict__ nonfinite, int* __restrict__ host) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c == 0) host[0] = *nonfinite;
    if (c <= ncat) host[1 + c] = item_start[(int64_t)c * ncell];
}

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_items_count(const int* cell_start, int64_t m, int* nitems, hipStream_t s) {
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_items_count, dim3(nblk(m, 256)), dim3(256), 0, s, cell_start, m, nitems);
    return hipGetLastError();
}

hipError_t launch_items_cat(const int* item_start, int ncat, int ncell, const int* nonfinite, int* host,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_items_cat, dim3(nblk(ncat + 1, 256)), dim3(256), 0, s, item_start, ncat, ncell,
                       nonfinite, host);
    return hipGetLastError();
}

hipError_t launch_grid_assign(const double* pos, const double*, int64_t n, const int64_t* pt_off,
                              int ncat, Grid g, int* cellid, int* count, int* nonfinite, int* catbad,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_grid_assign, dim3(nblk(n, 256)), dim3(256), 0, s, pos, n, pt_off, ncat, g,
                       cellid, count, nonfinite, catbad);
    return hipGetLastError();
}

hipError_t launch_grid_scan(const int* count, int64_t m, int* start, int* istart, int* work, hipStream_t s) {
    const int64_t nb = (m + kScanBlock - 1) / kScanBlock;
    ScanSum* sums = reinterpret_cast<ScanSum*>(work);
    ScanSum* offs = nb > kScanDirect ? sums + nb : nullptr;
    if (nb > 1) hipLaunchKernelGGL(k_scan_sums, dim3((unsigned)nb), dim3(256), 0, s, count, m, sums);
    if (offs) hipLaunchKernelGGL(k_scan_offsets, dim3(1), dim3(1024), 0, s, sums, nb, offs);
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(256), 0, s, count, m, sums, offs, start, istart);
    return hipGetLastError();
}

int64_t grid_scan_work_ints(int64_t m) { return 4 * ((m + kScanBlock - 1) / kScanBlock); }

hipError_t launch_grid_scatter(const int* cellid, int64_t n, Grid g, const int* start, int* cursor,
                               const double* pos, int* tmp_idx, double* tmp_key, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_grid_scatter, dim3(nblk(n, 256)), dim3(256), 0, s, cellid, n, g, start,
                       cursor, pos, tmp_idx, tmp_key);
    return hipGetLastError();
}

hipError_t launch_grid_order(const int* cellid, int64_t n, Grid g, const int* start, const int* tmp_idx,
                             const double* tmp_key, int* orig, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_grid_order, dim3(nblk(n, 256)), dim3(256), 0, s, cellid, n, g, start,
                       tmp_idx, tmp_key, orig);
    return hipGetLastError();
}

hipError_t launch_grid_cells(const int* slab_start, int64_t m, int zsub, int* cell_start, hipStream_t s) {
    hipLaunchKernelGGL(k_grid_cells, dim3(nblk(m + 1, 256)), dim3(256), 0, s, slab_start, m, zsub, cell_start);
    return hipGetLastError();
}

hipError_t launch_grid_fill(const double* pos, const double* w, int64_t n, const int* orig,
                            const int* cellid, Grid g, float4* pf, float* pw, float4* pa, double4* pd,
                            int* perm, int* catid, const int* cell_start, const int* item_start, int* item_cell,
                            hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_grid_fill, dim3(nblk(n, 256)), dim3(256), 0, s, pos, w, n, orig, cellid,
                       g, pf, pw, pa, pd, perm, catid, cell_start, item_start, item_cell);
    return hipGetLastError();
}

hipError_t launch_clear(const ClearRanges& r, hipStream_t s) {
    int64_t n = 0;
    for (int k = 0; k < kClearRanges; ++k) n += r.n[k];
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_clear, dim3(nblk(n, 256)), dim3(256), 0, s, r);
    return hipGetLastError();
}

hipError_t launch_put(uint32_t* dst, int n, const PutWords& w, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_put, dim3(1), dim3(256), 0, s, dst, n, w);
    return hipGetLastError();
}

hipError_t launch_publish(const int* src, int n, int* host, hipStream_t s) {
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, src, n, host);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long* p, int64_t n, unsigned long long v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3(nblk(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

}  // namespace tpcf
