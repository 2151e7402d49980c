// Covariance of measurements over a suite of mock catalogues (arXiv:2408.03036,
// Sec. 4.3):
//   C_ij = 1/(N_m - 1) sum_k (d_i^k - dbar_i)(d_j^k - dbar_j)          eq. (covariance)
//   C^-1 = (N_m - N_d - 2)/(N_m - 1) C_hat^-1                           eq. (Hartlap)
//
//  k_cov_gather   X[k][i] = src[k * stride + offset[i]] (the data vector of mock
//                 k) and the sums of every chunk of 64 mocks, in mock order
//  k_cov_center   mean (the chunks in order), then X -= mean
//  k_cov_syrk     X^T X on FP64 16x16x4 MFMA, one wavefront per (upper-
//                 triangle 16x16 tile, slice of the mocks)
//  k_cov_reduce   sum of the slices in a fixed order, / (N_m - 1), mirrored
//  k_inv_step     inverse of a symmetric positive definite matrix by block
//                 Gauss-Jordan (32 x 32 pivot blocks, no pivoting), one launch
//                 per pivot block, ping-pong between two buffers; the last
//                 one applies the Hartlap factor. A non-positive pivot sets a
//                 flag.
#include <algorithm>
#include <mutex>

#include "tpcf_internal.h"

namespace tpcf {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Chunks of kMeanChunk mocks, one thread per (chunk, entry): the mocks of a
// chunk are read kMeanUnroll at a time and added in order (one load at a time
// the sums alone took 18 us for 3000 x 336, most of it latency; gather and
// sums together now take 10 us). An offset outside a row (possible only for offsets
// given in device memory, which the host cannot check) reads the row's first
// entry, drops it and gives NaN.
constexpr int kMeanChunk = 64;
constexpr int kMeanUnroll = 16;

__global__ void __launch_bounds__(64) k_cov_gather(const double* __restrict__ src, int64_t stride,
                                                   const int64_t* __restrict__ off, int nm, int nd,
                                                   double* __restrict__ X, double* __restrict__ psum) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nd) return;
    const int k0 = blockIdx.y * kMeanChunk, k1 = min(nm, k0 + kMeanChunk);
    const int64_t o = off ? off[i] : (int64_t)i;
    const bool in = o >= 0 && o < stride;
    const double* col = src + (in ? o : 0);
    double s = 0.0;
    for (int k = k0; k < k1; k += kMeanUnroll) {
        double v[kMeanUnroll];
#pragma unroll
        for (int u = 0; u < kMeanUnroll; ++u) v[u] = col[(int64_t)min(k + u, k1 - 1) * stride];
#pragma unroll
        for (int u = 0; u < kMeanUnroll; ++u)
            if (k + u < k1) {
                const double x = in ? v[u] : __builtin_nan("");
                s += x;
                X[(int64_t)(k + u) * nd + i] = x;
            }
    }
    psum[(int64_t)blockIdx.y * nd + i] = s;
}

// Mean of every entry (the chunks in order) and the centring of kCenterRows
// mocks; the workgroups of the first mocks write the mean. (The sums start the
// buffer that the products overwrite later, so nothing after this reads them.)
constexpr int kCenterRows = 64;
constexpr int kCenterSums = 64;  // chunk sums staged in LDS at a time

// The chunks added up in their order, once, where they are many: every workgroup
// of the centring doing it for itself makes the work quadratic in the mocks
// (48 entries: 16,000 mocks 44 us without this launch and 48 with it, 40,000
// mocks 76 and 70; 10^6 mocks of 16 entries 10.0 and 0.84 ms).
constexpr int kTotalChunks = 320;

__global__ void __launch_bounds__(64) k_cov_total(const double* __restrict__ psum, int nchunk, int nd,
                                                  double* __restrict__ total) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nd) return;
    double s = 0.0;
#pragma unroll 16
    for (int c = 0; c < nchunk; ++c) s += psum[(int64_t)c * nd + i];
    total[i] = s;
}

__global__ void __launch_bounds__(256) k_cov_center(double* __restrict__ X, const double* __restrict__ psum,
                                                    int nchunk, int nm, int nd, double* __restrict__ mean) {
    __shared__ double sums[kCenterSums][64];
    const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;
    double s = 0.0;
    for (int c0 = 0; c0 < nchunk; c0 += kCenterSums) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kCenterSums; u += 4) {
            const int c = min(c0 + u + sub, nchunk - 1);
            sums[u + sub][lane] = psum[(int64_t)c * nd + min(i, nd - 1)];
        }
        __syncthreads();
        const int top = min(kCenterSums, nchunk - c0);
        for (int c = 0; c < top; ++c) s += sums[c][lane];
    }
    if (i >= nd) return;
    const double mu = s / nm;
    if (mean && blockIdx.y == 0 && threadIdx.x < 64) mean[i] = mu;
    const int k1 = min(nm, (int)(blockIdx.y + 1) * kCenterRows);
#pragma unroll 4
    for (int k = blockIdx.y * kCenterRows + (threadIdx.x >> 6); k < k1; k += 4) X[(int64_t)k * nd + i] -= mu;
}

constexpr int kCovWaves = 4;
constexpr int kSyrkUnroll = 8;

// One wavefront per (upper-triangle 16x16 tile, slice of the mocks): the
// slice's sum of products goes to its own partial, summed over the slices in
// a fixed order by k_cov_reduce.
__global__ void __launch_bounds__(64 * kCovWaves) k_cov_syrk(const double* __restrict__ X, int nm, int nd,
                                                               int kslice, double* __restrict__ part) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nt = (nd + 15) / 16;
    int t = blockIdx.x * kCovWaves + wave;
    if (t >= nt * (nt + 1) / 2) return;
    int ti = 0;
    while (t >= nt - ti) {  // t-th upper-triangle tile, row-major
        t -= nt - ti;
        ++ti;
    }
    const int tj = ti + t;
    const int i = lane & 15, g = lane >> 4;
    const int ca = 16 * ti + i, cb = 16 * tj + i;
    const int k_lo = blockIdx.y * kslice, k_hi = min(nm, k_lo + kslice);
    f64x4 acc = (f64x4)0.0;
    // kSyrkUnroll steps' loads in flight at a time, then the remainder, masked
    // (one step at a time: 26 us for 3000 x 336; now 19 us). The columns past nd
    // repeat the last one and are not stored.
    int k0 = k_lo;
    const double* xa = X + min(ca, nd - 1);
    const double* xb = X + min(cb, nd - 1);
    for (; k0 + 4 * kSyrkUnroll <= k_hi; k0 += 4 * kSyrkUnroll) {
        double a[kSyrkUnroll], b[kSyrkUnroll];
#pragma unroll
        for (int u = 0; u < kSyrkUnroll; ++u) {
            a[u] = xa[(int64_t)(k0 + 4 * u + g) * nd];
            b[u] = xb[(int64_t)(k0 + 4 * u + g) * nd];
        }
#pragma unroll
        for (int u = 0; u < kSyrkUnroll; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
    }
    if (k0 < k_hi) {
        double a[kSyrkUnroll], b[kSyrkUnroll];
#pragma unroll
        for (int u = 0; u < kSyrkUnroll; ++u) {
            const int k = k0 + 4 * u + g;
            const int64_t at = (int64_t)min(k, k_hi - 1) * nd;
            a[u] = xa[at];
            b[u] = xb[at];
            if (k >= k_hi) a[u] = b[u] = 0.0;
        }
#pragma unroll
        for (int u = 0; u < kSyrkUnroll; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
    }
    double* P = part + (int64_t)blockIdx.y * nd * nd;
    const int j = 16 * tj + (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * ti + (lane >> 4) + 4 * r;
        if (row < nd && j < nd && row <= j) P[(int64_t)row * nd + j] = acc[r];
    }
}

// C[i][j] = C[j][i] = (sum over slices, in order) / (N_m - 1), i <= j
__global__ void k_cov_reduce(const double* __restrict__ part, int nslice, int nd, int nm, double* __restrict__ C) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)nd * nd) return;
    const int i = (int)(e / nd), j = (int)(e % nd);
    if (i > j) return;
    double s = 0.0;
    for (int q = 0; q < nslice; ++q) s += part[(int64_t)q * nd * nd + e];
    s /= (double)(nm - 1);
    C[e] = s;
    C[(int64_t)j * nd + i] = s;
}

// Block Gauss-Jordan. With the pivot block D = A_kk^-1, one step takes A to
//   B_ij = A_ij - A_ik D A_kj  (i, j != k),  B_kj = D A_kj,
//   B_ik = -A_ik D,  B_kk = D,
// and after every block the matrix holds the inverse (no pivoting: the pivots
// of a positive definite matrix stay positive). A workgroup forms one 32 x 32
// tile, its four wavefronts a 16 x 16 quarter each, both products on FP64 MFMA.
// The workgroup that forms the next pivot tile inverts it at once and stores
// the inverse in its place (the tile itself is not needed again), so a step is
// one launch; in the first step every workgroup inverts the first pivot block.
// Past n the tiles are padded with the identity.
// Bound: the launches, one after the other, each as long as the inversion of a
// tile (32 pivots in turn). One launch per pivot over the
// whole matrix took 1004 us for n = 336 and 130 us for n = 48; a step per 32
// pivots takes 161 us and 31 us.
constexpr int kIB = 32;
constexpr int kIS = kIB + 1;

// 1 / x to within an ulp or so: the hardware's estimate and two Newton steps
// (a division is on the critical path of every pivot). Where the estimate or a
// step would leave the normal numbers, and for an infinite variance (the
// precision is then 0), it is the division.
__device__ __forceinline__ double fast_inverse(double x) {
    if (!(x > 0x1p-1000 && x < 0x1p1000)) return 1.0 / x;
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

struct PivotLds { double row[2][kIB], col[2][kIB]; };

// Inverts the tile S (row stride kIS) in place by Gauss-Jordan pivots; true
// when every pivot is positive. The whole workgroup calls it: thread (r, g)
// holds columns 4 g .. 4 g + 3 of row r, and the owners of the next pivot row and
// column publish them in LDS, one barrier per pivot. (One wavefront with 16
// columns a lane, every pivot unrolled, took 12 to 25 us per tile, much of it
// fetching the code; this takes about 8 us.)
__device__ __forceinline__ bool invert_tile(double* S, PivotLds& L) {
    const int r = threadIdx.x >> 3, g = threadIdx.x & 7;
    double v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = S[r * kIS + 4 * g + c];
    if (r == 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) L.row[0][4 * g + c] = v[c];
    }
    if (g == 0) L.col[0][r] = v[0];
    bool ok = true;
    for (int p4 = 0; p4 < kIB / 4; ++p4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int p = 4 * p4 + e;
            __syncthreads();
            const double piv = L.row[e & 1][p], f = L.col[e & 1][r];
            double w[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) w[c] = L.row[e & 1][4 * g + c];
            ok &= piv > 0.0;
            const double ip = fast_inverse(piv), t = f * ip;
            const bool mine = r == p;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = mine ? v[c] * ip : fma(-t, w[c], v[c]);
            if (g == p4) v[e] = mine ? ip : -t;
            if (r == p + 1) {
#pragma unroll
                for (int c = 0; c < 4; ++c) L.row[(e + 1) & 1][4 * g + c] = v[c];
            }
            if (g == (e == 3 ? p4 + 1 : p4)) L.col[(e + 1) & 1][r] = v[(e + 1) & 3];
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) S[r * kIS + 4 * g + c] = v[c];
    __syncthreads();
    return ok;
}

template <bool FIRST>
__global__ void __launch_bounds__(256) k_inv_step(const double* __restrict__ A, double* __restrict__ B, int n, int k,
                                                  double scale, int* __restrict__ bad) {
    __shared__ double Ds[kIB * kIS], Rs[kIB * kIS], Ws[kIB * kIS];
    __shared__ PivotLds piv;
    const int ti = blockIdx.y, tj = blockIdx.x;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool ik = ti == k, jk = tj == k, last = (k + 1) * kIB >= n;
    const double out_scale = last ? scale : 1.0;
    auto load = [&](double* S, int bi, int bj) {
        for (int e = threadIdx.x; e < kIB * kIB; e += 256) {
            const int r = e / kIB, c = e % kIB, i = bi * kIB + r, j = bj * kIB + c;
            S[r * kIS + c] = i < n && j < n ? A[(int64_t)i * n + j] : (i == j ? 1.0 : 0.0);
        }
    };
    load(Ds, k, k);
    if (!ik) load(Ws, ti, k);
    if (!jk) load(Rs, k, tj);
    __syncthreads();
    if constexpr (FIRST) {
        const bool ok = invert_tile(Ds, piv);
        if (ik && jk && threadIdx.x == 0 && !ok) atomicOr(bad, 1);
    }
    const int li = lane & 15, lg = lane >> 4;
    const int r0 = 16 * (wave >> 1), c0 = 16 * (wave & 1);  // this wavefront's quarter
    auto product = [&](const double* P, const double* Q, f64x4 acc) {
#pragma unroll
        for (int s = 0; s < kIB; s += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(P[(r0 + li) * kIS + s + lg], Q[(s + lg) * kIS + c0 + li], acc, 0,
                                                       0, 0);
        return acc;
    };
    f64x4 out;
    if (ik && jk) {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = Ds[(r0 + lg + 4 * e) * kIS + c0 + li];
    } else if (ik) {
        out = product(Ds, Rs, (f64x4)0.0);
    } else {
        f64x4 w = product(Ws, Ds, (f64x4)0.0);  // A_ik D
        if (jk) {
            out = -w;
        } else {
            f64x4 c;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = ti * kIB + r0 + lg + 4 * e, j = tj * kIB + c0 + li;
                c[e] = i < n && j < n ? A[(int64_t)i * n + j] : (i == j ? 1.0 : 0.0);
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 4; ++e) Ws[(r0 + lg + 4 * e) * kIS + c0 + li] = -w[e];
            __syncthreads();
            out = product(Ws, Rs, c);
        }
    }
    if (!last && ti == k + 1 && tj == k + 1) {
        // the next pivot tile: its inverse takes its place
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) Ds[(r0 + lg + 4 * e) * kIS + c0 + li] = out[e];
        __syncthreads();
        const bool ok = invert_tile(Ds, piv);
        if (threadIdx.x == 0 && !ok) atomicOr(bad, 1);
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = Ds[(r0 + lg + 4 * e) * kIS + c0 + li];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = ti * kIB + r0 + lg + 4 * e, j = tj * kIB + c0 + li;
        if (i < n && j < n) B[(int64_t)i * n + j] = out[e] * out_scale;
    }
}

}  // namespace

// Scratch of the allocation-free covariance (tpcf_covariance_noalloc): the
// gathered data vectors and the partial products, kCovScratchBytes on every
// device the library runs on, held until the process ends. Host code never
// passes the array's name to a kernel or a copy: it is a host-side stand-in
// there. It uses the device address that cov_scratch_init looks up once per
// device.
__device__ __align__(256) static unsigned char scratch[kCovScratchBytes];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices] = {};
}  // namespace

hipError_t cov_scratch_init(int device, void** out) {
    *out = nullptr;
    if (device < 0 || device >= kScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        // the caller has made `device` current
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

int64_t cov_scratch_need(int nm, int nd) {
    return (int64_t)sizeof(double) * ((int64_t)nm * nd + cov_part_doubles(nm, nd));
}

int64_t cov_part_doubles(int nm, int nd) {
    const int64_t prod = (int64_t)cov_slices(nm, nd) * nd * nd;
    const int64_t sums = ((int64_t)(nm + kMeanChunk - 1) / kMeanChunk + 1) * nd;
    return std::max(prod, sums);
}

int cov_slices(int nm, int nd) {
    // enough (tile, slice) wavefronts to fill the chip, slices of at least 64 mocks
    const int nt = (nd + 15) / 16;
    const int ntiles = nt * (nt + 1) / 2;
    int ns = (4096 + ntiles - 1) / ntiles;
    ns = std::min(ns, std::max(1, nm / 64));
    return std::max(1, std::min(ns, 64));
}

hipError_t launch_cov(const double* src, int64_t stride, const int64_t* off, int nm, int nd, double* X,
                      double* part, double* mean, double* C, hipStream_t s) {
    const int64_t ne = (int64_t)nm * nd;
    if (ne <= 0) return hipSuccess;
    // the chunk sums use the start of `part` (nchunk + 1 rows of nd) before the products
    int nchunk = (nm + kMeanChunk - 1) / kMeanChunk;
    const double* sums = part;
    const int nbx = (nd + 63) / 64;
    hipLaunchKernelGGL(k_cov_gather, dim3(nbx, nchunk), dim3(64), 0, s, src, stride, off, nm, nd, X, part);
    if (nchunk > kTotalChunks) {
        double* total = part + (int64_t)nchunk * nd;
        hipLaunchKernelGGL(k_cov_total, dim3(nbx), dim3(64), 0, s, part, nchunk, nd, total);
        sums = total;
        nchunk = 1;
    }
    hipLaunchKernelGGL(k_cov_center, dim3(nbx, (nm + kCenterRows - 1) / kCenterRows), dim3(256), 0, s, X, sums, nchunk,
                       nm, nd, mean);
    const int nt = (nd + 15) / 16;
    const int ntiles = nt * (nt + 1) / 2;
    const int ns = cov_slices(nm, nd);
    const int kslice = (nm + ns - 1) / ns;
    hipLaunchKernelGGL(k_cov_syrk, dim3((ntiles + kCovWaves - 1) / kCovWaves, ns), dim3(64 * kCovWaves), 0, s, X,
                       nm, nd, kslice, part);
    const int64_t nn = (int64_t)nd * nd;
    hipLaunchKernelGGL(k_cov_reduce, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, part, ns, nd, nm, C);
    return hipGetLastError();
}

hipError_t launch_cov_invert(const double* C, double* A, double* W, int n, double scale, int* bad, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int nk = (n + kIB - 1) / kIB;
    const dim3 grid(nk, nk);
    // step q writes A when nk - q is odd, W otherwise: the last one writes A.
    // The first reads C, which must not be what it writes.
    const double* src = C;
    if (nk % 2 == 1 && C == A) {
        const hipError_t e = hipMemcpyAsync(W, C, sizeof(double) * (size_t)n * n, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
        src = W;
    }
    for (int k = 0; k < nk; ++k) {
        double* dst = (nk - k) % 2 == 1 ? A : W;
        if (k == 0) hipLaunchKernelGGL(k_inv_step<true>, grid, dim3(256), 0, s, src, dst, n, k, scale, bad);
        else hipLaunchKernelGGL(k_inv_step<false>, grid, dim3(256), 0, s, src, dst, n, k, scale, bad);
        src = dst;
    }
    return hipGetLastError();
}

}  // namespace tpcf
