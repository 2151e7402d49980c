// Contraction of the per-primary harmonic coefficients into the global
// moments (arXiv:2408.03036, eq. (measured_mult) averaged over positions, with
// m = m' for the common line of sight):
//
//   G_m[(b1,l1),(b2,l2)] = sum_p w_p Re(A_l1m(p,b1) conj(A_l2m(p,b2)))
//                        = sum over rows (p, re|im) of w_p X[row][c1] X[row][c2]
//
// i.e. a symmetric rank-K update (K = primaries, two rows per primary for
// m >= 1) of a K_m x K_m matrix, K_m = nbins (lmax - m + 1). It runs on MFMA:
//   mode 0: FP64 16x16x4 (plain double path)
//   mode 1: FP32 32x32x2
//   mode 2: split-BF16: x = hi + lo with hi = bf16(x), lo = bf16(x - hi);
//           G ~ hi hi' + hi lo' + lo hi' on 32x32x16 BF16 MFMA, FP32 accumulate.
//   mode 3: x = hi + mid + lo (three BF16 pieces) and the six products whose
//           size is above 2^-24 |x y|: FP32-level accuracy.
// A workgroup owns one subchunk of primaries (a fixed slice of one catalogue)
// and a group of upper-triangle output tiles; it writes its partial sums, and
// the partials are reduced per catalogue in a fixed order in FP64, so the
// result does not depend on scheduling.
//
// The same file holds the isotropic schedule (the l1 = l2 blocks only), the
// degenerate-triangle moments, the fixed-order partial reduction, the final
// conversion to the tripolar multipoles (eq. (slep2sugy)) and the edge
// correction of isotropic multipoles by explicit random triplet counts.
#include <algorithm>
#include <type_traits>

#include "tpcf_internal.h"

namespace tpcf {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- FP64 and FP32
// Work split of the FP64 and FP32 contractions. A workgroup covers one
// (subchunk, m) and up to kWaves * TPW upper-triangle tiles. The operand is
// staged in units: kUnit consecutive primaries of one part (re or im) of every
// column. A step stages as many consecutive units as the threads' registers
// hold (`units`, set per m from the column count, so that the narrow high-m
// operands take few steps), into one of two LDS buffers: the loads of step
// s + 1 are issued before the MFMAs of step s and stored after them. All loads
// are unconditional and in bounds (the operand ends with 8 elements of
// padding; an idle item, or one past the subchunk, reads the start of its row
// or of the buffer), elements that are not the unit's primaries are zeroed
// when stored. The MFMA loop has no branch (a wave's tile count is a template
// parameter). Columns are l-major, and a batched run forms only the tiles
// its multipoles couple, as in the split-BF16 kernel below.
constexpr int kUnit = 32;
constexpr int kGroup = 4;                 // primaries of a staged item
constexpr int kUnitItems = kUnit / kGroup;

// Tiles of the upper triangle (TS columns each, l-major: column c holds
// l - m = c / nb of bin c % nb) whose columns couple some l1, l2 with
// |l1 - l2| <= lcouple, in row-major order: a wave takes the (first + stride q)-th
// of them, q < N; returns how many it has (they come first), and all[0] the
// number of needed tiles. Along a row of tiles the smallest l distance only
// grows, so a row ends at its first tile past the limit.
template <int TS, int N>
__device__ __forceinline__ int pick_tiles(int K, int nb, int lcouple, int first, int stride, int (&ti)[N],
                                          int (&tj)[N], int& all) {
    const int nt = (K + TS - 1) / TS;
    int mine = 0;
    all = 0;
#pragma unroll
    for (int q = 0; q < N; ++q) ti[q] = tj[q] = 0;
    for (int r = 0; r < nt; ++r) {
        const int lhi = (min(K, r * TS + TS) - 1) / nb;
        for (int c = r; c < nt; ++c) {
            if (c * TS / nb - lhi > lcouple) break;
#pragma unroll
            for (int q = 0; q < N; ++q)
                if (all == first + stride * q) {
                    ti[q] = r;
                    tj[q] = c;
                    mine = q + 1;
                }
            ++all;
        }
    }
    return mine;
}

// Writes entry (ci, cj) of an upper-triangle tile (ti, tj) once per unordered
// column pair, at its upper-triangle position in the l-major order
// (l - m) nbins + b that the reduction, finalize and export read: a tile of
// l-major columns goes out in whole rows. (In the bin-major order, with every
// value in a cache line of its own, 36,000 subchunks of 256 primaries, lmax 10
// and 10 bins, took 22.3 ms instead of 19.6 in split BF16.)
template <bool LMAJOR = true>
__device__ __forceinline__ void put_entry(double* G, int K, int nb, int nl, int ti, int tj, int ci, int cj,
                                          double v) {
    if (ci < K && cj < K && (ti < tj || ci <= cj)) {
        if constexpr (LMAJOR) {
            G[(int64_t)ci * K + cj] = v;
        } else {
            const int oi = (ci % nl) * nb + ci / nl, oj = (cj % nl) * nb + cj / nl;
            G[(int64_t)min(oi, oj) * K + max(oi, oj)] = v;
        }
    }
}

// The thread's staged items: flat column it / kUnitItems of the step (unit by
// unit, ncol columns each), primaries k4 .. k4 + 3 of its unit.
template <int IPT, bool LMAJOR = true>
struct Items {
    int row[IPT];   // operand row of part 0, or -1: a column past K
    int unit[IPT];  // unit of the step, or -1: no item
    int col[IPT];
    int k4;
    __device__ __forceinline__ Items(int tid, int threads, int units, int ncol, int K, int nb, int NV, int voff) {
        k4 = (tid % kUnitItems) * kGroup;
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            const int fc = tid / kUnitItems + u * (threads / kUnitItems);
            unit[u] = fc < units * ncol ? fc / ncol : -1;
            col[u] = fc % ncol;
            const int nl = K / nb;
            const int b = LMAJOR ? col[u] % nb : col[u] / nl, lp = LMAJOR ? col[u] / nb : col[u] % nl;
            row[u] = unit[u] >= 0 && col[u] < K ? b * NV + voff + lp : -1;
        }
    }
};

// Units of a step: as many as fill cols flat columns, at most 8.
__host__ __device__ inline int step_units(int ncol, int cols) { return min(8, max(1, cols / ncol)); }

// FP64: 16x16x4 MFMA, eight wavefronts with up to four tiles each. A lane
// group takes eight consecutive primaries of a unit (the order of the sum is
// free), so an operand fragment is one 16-byte LDS read for two MFMAs; a row
// stride of 34 doubles keeps those reads free of bank conflicts.
// Bound: the operand's bytes (1.14 GB for 1e5 primaries at lmax 10, 10 bins:
// 0.24 ms) and, close to it, the MFMAs (0.16 ms); it takes 0.38 ms, 0.63 ms
// with subchunks of 4096. Eight tiles a wave, a branch per tile in the MFMA
// loop, 8-byte LDS reads, one unit per step and subchunks of 4096 took 1.15 ms.
constexpr int kF64Waves = 8, kF64TPW = 4, kF64Stride = kUnit + 2;

__host__ __device__ constexpr size_t f64_lds(int flat_cols, int units, int nbuf) {
    return (size_t)nbuf * ((size_t)flat_cols * kF64Stride + (size_t)units * kUnit) * sizeof(double);
}

template <bool W, int IPT>
__global__ void __launch_bounds__(64 * kF64Waves) k_contract_f64(ContractArgs a, int cols, int nbuf) {
    constexpr int TS = 16, TPW = kF64TPW, KSP = kF64Stride;
    extern __shared__ unsigned char smem[];
    const int s = blockIdx.x, m = blockIdx.y;
    const int nb = a.nb, nl = a.lmax - m + 1, K = nb * nl;
    const int ncol = (K + TS - 1) / TS * TS;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int ti[TPW], tj[TPW], all;
    const int t0 = blockIdx.z * kF64Waves * TPW;
    const int nq = pick_tiles<TS>(K, nb, a.lcouple, t0 + wave, kF64Waves, ti, tj, all);
    if (t0 >= all) return;
    const int parts = m == 0 ? 1 : 2;
    const int units = step_units(ncol, cols);
    const int64_t pa = a.sub_start[s], pb = a.sub_start[s + 1];
    const int total = (int)((pb - pa + kUnit - 1) / kUnit) * parts;  // units of the subchunk
    const int nsteps = (total + units - 1) / units;
    const Items<IPT> it(threadIdx.x, 64 * kF64Waves, units, ncol, K, nb, n_values(a.lmax), value_offset(a.lmax, m));
    const double* A = reinterpret_cast<const double*>(a.A);
    double* lds = reinterpret_cast<double*>(smem);
    const int bufsz = units * (ncol * KSP + kUnit);

    struct Stage {
        double2 x[IPT][2];
        double w;
    };
    auto load = [&](int st, Stage& R) {
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            const int g = st * units + max(it.unit[u], 0);
            const int64_t p0 = pa + (int64_t)(g / parts) * kUnit;
            const bool in = it.row[u] >= 0 && g < total;
            const double* src =
                A + (in ? (int64_t)(it.row[u] + (g % parts) * nl) * a.ldA + p0 + (p0 + it.k4 < pb ? it.k4 : 0) : 0);
            __builtin_memcpy(&R.x[u][0], src, 16);
            __builtin_memcpy(&R.x[u][1], src + 2, 16);
        }
        if constexpr (W) {
            // thread t stages the weight of primary t % kUnit of unit t / kUnit
            const int64_t p = pa + (int64_t)((st * units + (int)threadIdx.x / kUnit) / parts) * kUnit + threadIdx.x % kUnit;
            R.w = a.pd[a.p_begin + (p < pb ? p : pa)].w;
        }
    };
    auto store = [&](int st, int buf, const Stage& R) {
        double* base = lds + buf * bufsz;
        if constexpr (W) {
            if ((int)threadIdx.x < units * kUnit) base[units * ncol * KSP + threadIdx.x] = R.w;
        }
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            if (it.unit[u] < 0) continue;
            const int g = st * units + it.unit[u];
            const int kv = it.row[u] >= 0 && g < total
                               ? (int)min((int64_t)kUnit, pb - pa - (int64_t)(g / parts) * kUnit) - it.k4 : 0;
            double2 v0 = R.x[u][0], v1 = R.x[u][1];
            v0.x = kv > 0 ? v0.x : 0.0;
            v0.y = kv > 1 ? v0.y : 0.0;
            v1.x = kv > 2 ? v1.x : 0.0;
            v1.y = kv > 3 ? v1.y : 0.0;
            double2* dst = reinterpret_cast<double2*>(base + (it.unit[u] * ncol + it.col[u]) * KSP + it.k4);
            dst[0] = v0;
            dst[1] = v1;
        }
    };
    f64x4 acc[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) acc[q] = (f64x4)0.0;
    const int i = lane & 15, kg = lane >> 4;
    auto mma = [&](auto nqc, int buf) {
        constexpr int NQ = decltype(nqc)::value;
        const double* base = lds + buf * bufsz;
        for (int u = 0; u < units; ++u) {
            const double* X = base + u * ncol * KSP + 8 * kg;
            const double* wt = base + units * ncol * KSP + u * kUnit + 8 * kg;
#pragma unroll
            for (int k = 0; k < 8; k += 2) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    double2 av = *reinterpret_cast<const double2*>(X + (ti[q] * TS + i) * KSP + k);
                    const double2 bv = *reinterpret_cast<const double2*>(X + (tj[q] * TS + i) * KSP + k);
                    if constexpr (W) {
                        av.x *= wt[k];
                        av.y *= wt[k + 1];
                    }
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, bv.x, acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.y, bv.y, acc[q], 0, 0, 0);
                }
            }
        }
    };
    auto compute = [&](int buf) {
        switch (nq) {
            case 1: mma(std::integral_constant<int, 1>{}, buf); break;
            case 2: mma(std::integral_constant<int, 2>{}, buf); break;
            case 3: mma(std::integral_constant<int, 3>{}, buf); break;
            case 4: mma(std::integral_constant<int, 4>{}, buf); break;
            default: break;
        }
    };
    Stage R;
    load(0, R);
    store(0, 0, R);
    __syncthreads();
    for (int st = 0; st < nsteps; ++st) {
        if (st + 1 < nsteps) load(st + 1, R);
        compute(nbuf == 2 ? st & 1 : 0);
        if (nbuf == 1) __syncthreads();
        if (st + 1 < nsteps) store(st + 1, nbuf == 2 ? (st + 1) & 1 : 0, R);
        __syncthreads();
    }
    double* G = a.part + (int64_t)s * a.gsize + a.goff[m];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        if (q >= nq) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            put_entry(G, K, nb, nl, ti[q], tj[q], ti[q] * TS + (lane >> 4) + 4 * r, tj[q] * TS + (lane & 15),
                      acc[q][r]);
    }
}

// FP32: 32x32x2 MFMA, eight wavefronts with up to two tiles each. The FP32
// accumulators are emptied into FP64 registers after every kUnit primaries
// (both parts), so single precision only ever sums a few dozen products.
// An MFMA sums primaries k and k + 1, one per lane half, in the order of
// k; a unit's row in LDS holds its even primaries, then its odd ones, so that
// a lane reads four MFMAs' operands at once (row stride 36 floats: no bank
// conflicts). With weights the columns stay bin-major and every tile is
// formed: the weight multiplies the first column of a pair, and the rounding
// of w x depends on which that is.
// 9e6 primaries in subchunks of 256, lmax 4 and 12 bins: 8.8 ms (1.7 TB/s of
// operand); 30,011 at lmax 13 and 7 bins: 126 us. One buffer, a branch per tile
// in the MFMA loop and subchunks of 4096 took 57.8 ms and 370 us.
constexpr int kF32Waves = 8, kF32TPW = 2, kF32Stride = kUnit + 4;

__host__ __device__ constexpr size_t f32_lds(int flat_cols, int units, int nbuf) {
    return (size_t)nbuf * ((size_t)flat_cols * kF32Stride + (size_t)units * kUnit) * sizeof(float);
}

template <bool W, int IPT>
__global__ void __launch_bounds__(64 * kF32Waves) k_contract_f32(ContractArgs a, int cols) {
    constexpr int TS = 32, TPW = kF32TPW, KSP = kF32Stride;
    extern __shared__ unsigned char smem[];
    const int s = blockIdx.x, m = blockIdx.y;
    const int nb = a.nb, nl = a.lmax - m + 1, K = nb * nl;
    const int ncol = (K + TS - 1) / TS * TS;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int ti[TPW], tj[TPW], all;
    const int t0 = blockIdx.z * kF32Waves * TPW;
    const int nq = pick_tiles<TS>(K, nb, W ? a.lmax : a.lcouple, t0 + wave, kF32Waves, ti, tj, all);
    if (t0 >= all) return;
    const int parts = m == 0 ? 1 : 2;
    const int units = step_units(ncol, cols);
    const int64_t pa = a.sub_start[s], pb = a.sub_start[s + 1];
    const int total = (int)((pb - pa + kUnit - 1) / kUnit) * parts;
    const int nsteps = (total + units - 1) / units;
    const Items<IPT, !W> it(threadIdx.x, 64 * kF32Waves, units, ncol, K, nb, n_values(a.lmax), value_offset(a.lmax, m));
    const float* A = reinterpret_cast<const float*>(a.A);
    float* lds = reinterpret_cast<float*>(smem);
    const int bufsz = units * (ncol * KSP + kUnit);

    struct Stage {
        float4 x[IPT];
        float w;
    };
    auto load = [&](int st, Stage& R) {
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            const int g = st * units + max(it.unit[u], 0);
            const int64_t p0 = pa + (int64_t)(g / parts) * kUnit;
            const bool in = it.row[u] >= 0 && g < total;
            const float* src =
                A + (in ? (int64_t)(it.row[u] + (g % parts) * nl) * a.ldA + p0 + (p0 + it.k4 < pb ? it.k4 : 0) : 0);
            __builtin_memcpy(&R.x[u], src, 16);
        }
        if constexpr (W) {
            const int64_t p = pa + (int64_t)((st * units + (int)threadIdx.x / kUnit) / parts) * kUnit + threadIdx.x % kUnit;
            R.w = a.pw[a.p_begin + (p < pb ? p : pa)];
        }
    };
    // position of primary k inside a unit's row: the even ones first
    auto store = [&](int st, int buf, const Stage& R) {
        float* base = lds + buf * bufsz;
        if constexpr (W) {
            const int t = threadIdx.x, k = t % kUnit;
            if (t < units * kUnit) base[units * ncol * KSP + (t - k) + (k & 1) * (kUnit / 2) + k / 2] = R.w;
        }
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            if (it.unit[u] < 0) continue;
            const int g = st * units + it.unit[u];
            const int kv = it.row[u] >= 0 && g < total
                               ? (int)min((int64_t)kUnit, pb - pa - (int64_t)(g / parts) * kUnit) - it.k4 : 0;
            const float2 ev = make_float2(kv > 0 ? R.x[u].x : 0.f, kv > 2 ? R.x[u].z : 0.f);
            const float2 od = make_float2(kv > 1 ? R.x[u].y : 0.f, kv > 3 ? R.x[u].w : 0.f);
            float* dst = base + (it.unit[u] * ncol + it.col[u]) * KSP + it.k4 / 2;
            *reinterpret_cast<float2*>(dst) = ev;
            *reinterpret_cast<float2*>(dst + kUnit / 2) = od;
        }
    };
    f32x16 acc[TPW];
    double accd[TPW][16];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        acc[q] = (f32x16)0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) accd[q][r] = 0.0;
    }
    const int i = lane & 31, kg = lane >> 5;
    auto mma = [&](auto nqc, int st, int buf) {
        constexpr int NQ = decltype(nqc)::value;
        const float* base = lds + buf * bufsz;
        for (int u = 0; u < units; ++u) {
            const float* X = base + u * ncol * KSP + kg * (kUnit / 2);
            const float* wt = base + units * ncol * KSP + u * kUnit + kg * (kUnit / 2);
#pragma unroll
            for (int k = 0; k < kUnit / 2; k += 4) {
                float4 wv = make_float4(1.f, 1.f, 1.f, 1.f);
                if constexpr (W) wv = *reinterpret_cast<const float4*>(wt + k);
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    float4 av = *reinterpret_cast<const float4*>(X + (ti[q] * TS + i) * KSP + k);
                    const float4 bv = *reinterpret_cast<const float4*>(X + (tj[q] * TS + i) * KSP + k);
                    if constexpr (W) {
                        av.x *= wv.x;
                        av.y *= wv.y;
                        av.z *= wv.z;
                        av.w *= wv.w;
                    }
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, bv.x, acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, bv.y, acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, bv.z, acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.w, bv.w, acc[q], 0, 0, 0);
                }
            }
            if ((st * units + u) % parts == parts - 1) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) accd[q][r] += (double)acc[q][r];
                    acc[q] = (f32x16)0.0f;
                }
            }
        }
    };
    Stage R;
    load(0, R);
    store(0, 0, R);
    __syncthreads();
    for (int st = 0; st < nsteps; ++st) {
        if (st + 1 < nsteps) load(st + 1, R);
        if (nq == 2) mma(std::integral_constant<int, 2>{}, st, st & 1);
        else if (nq == 1) mma(std::integral_constant<int, 1>{}, st, st & 1);
        if (st + 1 < nsteps) store(st + 1, (st + 1) & 1, R);
        __syncthreads();
    }
    double* G = a.part + (int64_t)s * a.gsize + a.goff[m];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        if (q >= nq) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            put_entry<!W>(G, K, nb, nl, ti[q], tj[q], ti[q] * TS + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3),
                      tj[q] * TS + (lane & 31), accd[q][r]);
    }
}

// ---------------------------------------------------------------- isotropic schedule
// The isotropic multipoles are the L = 0 case of eq. (slep2sugy) (Sec. 2.3:
// the tripolar basis with L = 0 reduces to Legendre polynomials of the angle
// between r1 and r2), and they read only the l1 = l2 blocks of G_m:
//   G_m[(b1,l),(b2,l)] = sum_p w_p Re(A_lm(p,b1) conj(A_lm(p,b2))).
// One wavefront per (subchunk, (l, m)) forms that nb x nb block on 16x16x4
// MFMA in 16 x 16 tiles over (b1, b2) (up to 32 bins). A step covers 64
// primaries from the subchunk's first: lane (i, g) = (lane % 16, lane / 16)
// loads 16 consecutive values of bin i (vector loads, masked to the subchunk)
// and feeds 16 MFMAs, each summing four primaries, one per lane group. FP64
// operands use FP64 MFMA; FP32 operands use FP32 MFMA, and the FP32 sums of
// one step (16 products per entry and chain) go into FP64 registers.
constexpr int kIsoWaves = 4;

// 16 consecutive values of one row (at any alignment), kept in their storage type
// until used: the next step's values are loaded while the current step's
// MFMAs run.
template <typename TA> struct Raw16;
typedef float fvec4 __attribute__((ext_vector_type(4)));
template <> struct Raw16<float> {
    fvec4 v[4];
    __device__ __forceinline__ void load(const float* src) {
#pragma unroll
        for (int q = 0; q < 4; ++q) __builtin_memcpy(&v[q], src + 4 * q, 16);
    }
    __device__ __forceinline__ double get(int k) const { return (double)v[k >> 2][k & 3]; }
};
template <> struct Raw16<double> {
    double2 v[8];
    __device__ __forceinline__ void load(const double* src) {
#pragma unroll
        for (int q = 0; q < 8; ++q) __builtin_memcpy(&v[q], src + 2 * q, 16);
    }
    __device__ __forceinline__ double get(int k) const { return (k & 1) ? v[k >> 1].y : v[k >> 1].x; }
};

template <typename TA, bool W>
__global__ void __launch_bounds__(64 * kIsoWaves) k_contract_iso(ContractArgs a) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lmax = a.lmax, nb = a.nb;
    int u = blockIdx.y * kIsoWaves + wave;
    const int nlm = (lmax + 1) * (lmax + 2) / 2;
    if (u >= nlm) return;
    int m = 0;
    while (u >= lmax - m + 1) {  // units ordered m-major, l = m..lmax
        u -= lmax - m + 1;
        ++m;
    }
    const int l = m + u;
    const int nl = lmax - m + 1, K = nb * nl;
    const int parts = m == 0 ? 1 : 2;
    const int NV = n_values(lmax);
    const int v0 = value_offset(lmax, m) + (l - m);
    const int s = blockIdx.x;
    const int64_t pa = a.sub_start[s], pb = a.sub_start[s + 1];
    const int i = lane & 15, g = lane >> 4;
    const int nt = (nb + 15) / 16;  // 1 or 2 tiles of bins
    const TA* A = reinterpret_cast<const TA*>(a.A);
    // rows of bins i and 16 + i (clamped in range; their values are zeroed)
    const bool ok0 = i < nb, ok1 = nt > 1 && 16 + i < nb;
    const int64_t row0 = ((int64_t)min(i, nb - 1) * NV + v0) * a.ldA;
    const int64_t row1 = ((int64_t)min(16 + i, nb - 1) * NV + v0) * a.ldA;
    const int64_t pstep = (int64_t)nl * a.ldA;  // re -> im rows
    f64x4 acc[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) acc[q] = (f64x4)0.0;

    // Steps of 64 primaries from the subchunk's first, so that the sums do not
    // depend on where it lies in the chunk; the operand ends with 16 elements of
    // padding, so that every group starting below pb is inside it
    const int nsteps = (int)((pb - pa + 63) / 64);
    const int nit = nsteps * parts;
    auto group = [&](int it) { return pa + (int64_t)(it / parts) * 64 + 16 * g; };
    // FP32 weights of a group are prefetched with its values (the weight
    // buffer ends with 16 floats of padding); FP64 reads them from the points
    constexpr bool F32 = std::is_same<TA, float>::value;
    constexpr bool WPRE = W && F32;
    struct Set {
        Raw16<TA> r0, r1;
        Raw16<float> w;
    };
    // Loads of iteration it into set S: unconditional, a group past the
    // subchunk reads the first group instead (its values are masked), so the
    // loads in flight are the same on every path and the wait before a set is
    // used covers only that set (a two-set ping-pong, no register rotation).
    auto fetch = [&](int it, Set& S) {
        int64_t q0 = group(it);
        if (q0 >= pb) q0 = pa;
        const int64_t off = (it % parts) * pstep + q0;
        S.r0.load(A + row0 + off);
        if (nt > 1) S.r1.load(A + row1 + off);
        if constexpr (WPRE) {
            // not 16-byte aligned in general
            const float* wsrc = a.pw + a.p_begin + q0;
#pragma unroll
            for (int q = 0; q < 4; ++q) __builtin_memcpy(&S.w.v[q], wsrc + 4 * q, 16);
        }
    };
    // FP32 operands: FP32 16x16x4 MFMA in two chains, emptied into FP64
    // after every step of 64 primaries (16 products per chain and entry)
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    double accd[3][4];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) accd[q][r] = 0.0;
    auto step = [&](int it, const Set& S) {
        const Raw16<TA>& c0 = S.r0;
        const Raw16<TA>& c1 = S.r1;
        const int64_t q0 = group(it);
        const int hi = (int)max<int64_t>(0, min<int64_t>(pb - q0, 16));
        if constexpr (F32) {
            f32x4 sa[3], sb[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) sa[q] = sb[q] = (f32x4)0.0f;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const bool in = k < hi;
                const float x0 = (in && ok0) ? c0.v[k >> 2][k & 3] : 0.0f;
                const float wk = W ? (in ? S.w.v[k >> 2][k & 3] : 0.0f) : 1.0f;
                const float wa0 = W ? x0 * wk : x0;
                f32x4* acc = (k & 1) ? sb : sa;
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(wa0, x0, acc[0], 0, 0, 0);
                if (nt > 1) {
                    const float x1 = (in && ok1) ? c1.v[k >> 2][k & 3] : 0.0f;
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wa0, x1, acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(W ? x1 * wk : x1, x1, acc[2], 0, 0, 0);
                }
            }
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) accd[q][r] += (double)sa[q][r] + (double)sb[q][r];
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const bool in = k < hi;
                const double x0 = (in && ok0) ? c0.get(k) : 0.0;
                const double wk = W ? (in ? a.pd[a.p_begin + q0 + k].w : 0.0) : 1.0;
                const double wa0 = W ? x0 * wk : x0;
                acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(wa0, x0, acc[0], 0, 0, 0);
                if (nt > 1) {
                    const double x1 = (in && ok1) ? c1.get(k) : 0.0;
                    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(wa0, x1, acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(W ? x1 * wk : x1, x1, acc[2], 0, 0, 0);
                }
            }
        }
    };
    Set sA, sB;
    if (nit > 0) fetch(0, sA);
    for (int it = 0; it < nit; it += 2) {
        fetch(it + 1, sB);
        step(it, sA);
        fetch(it + 2, sA);
        if (it + 1 < nit) step(it + 1, sB);
    }
    // upper triangle of the block: tiles (0,0), (0,1), (1,1)
    const int64_t base = (int64_t)s * a.gsize + a.goff[m];
    const int j = lane & 15;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (q > 0 && nt < 2) break;
        const int ti = q == 2 ? 1 : 0, tj = q == 0 ? 0 : 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // output rows of a 16x16 MFMA: FP64 lane / 16 + 4 r, FP32 4 (lane / 16) + r
            const int c1r = 16 * ti + (F32 ? 4 * (lane >> 4) + r : (lane >> 4) + 4 * r), c2 = 16 * tj + j;
            if (c1r < nb && c2 < nb && c1r <= c2)
                a.part[base + (int64_t)((l - m) * nb + c1r) * K + (l - m) * nb + c2] =
                    F32 ? accd[q][r] : acc[q][r];
        }
    }
}

// ---------------------------------------------------------------- split-BF16 contraction
// One workgroup per (subchunk, m): eight wavefronts, up to two 32x32 output
// tiles each. Per step (KS primaries of one part, KS chosen per m), every
// thread stages 8 consecutive primaries of one column: two vector loads,
// packed round-to-nearest BF16 conversion of the pieces, one 16-byte LDS
// store per plane. Two LDS buffers: the loads of the next step are in flight
// while the MFMAs of the current one run. Columns are l-major, and a batched
// run forms only the tiles its multipoles couple (lcouple).
constexpr int kBfWaves = 8;
constexpr int kBfTPW = 2;
// staged 8-element groups per thread and step: four without weights, two with
// (the weighted staging also holds the weights)
template <bool W> constexpr int bf_ipt() { return W ? 2 : 4; }

// Step length (primaries) of each m, passed by value to the kernel.
struct BfSteps { int ks[kMaxLmax + 1]; };

// Step length of one m: the longest power of two from cap down to 16 whose
// staging fits the threads' registers (ncol * KS / 8 items of 8 primaries,
// ipt per thread) and whose nbuf LDS buffers fit in lds bytes; 0 if none.
// The narrow high-m operands thus take long steps, and their workgroups
// fewer of them: every step waits for its loads and a barrier.
inline int bf_step(int ncol, int nplanes, int ipt, int nbuf, int cap, size_t lds) {
    for (int ks = cap; ks >= 16; ks /= 2) {
        if ((int64_t)ncol * (ks / 8) > (int64_t)64 * kBfWaves * ipt) continue;
        if ((size_t)nbuf * nplanes * ncol * (ks + 8) * sizeof(uint16_t) > lds) continue;
        return ks;
    }
    return 0;
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ inline uint32_t cvt_pk_bf16(float a, float b) {
    bf16x2_t v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}

// Splits 8 floats into NPC BF16 pieces, piece q as 4 packed dwords.
template <int NPC>
__device__ inline void split8(float (&x)[8], uint4 (&out)[NPC]) {
#pragma unroll
    for (int q = 0; q < NPC; ++q) {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w[j] = cvt_pk_bf16(x[2 * j], x[2 * j + 1]);
            if (q + 1 < NPC) {
                x[2 * j] -= __uint_as_float(w[j] << 16);
                x[2 * j + 1] -= __uint_as_float(w[j] & 0xffff0000u);
            }
        }
        out[q] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

template <bool W>
struct BfStage {
    float x[bf_ipt<W>()][8];
    float w[W ? bf_ipt<W>() : 1][8];
};

template <int NPC, bool W>
__global__ void __launch_bounds__(64 * kBfWaves) k_contract_bf16(ContractArgs a, BfSteps steps, int nbuf) {
    constexpr int TS = 32;
    extern __shared__ unsigned char smem[];
    const int s = blockIdx.x;
    const int m = blockIdx.y;
    const int lmax = a.lmax, nb = a.nb;
    const int nl = lmax - m + 1;
    const int K = nb * nl;
    const int nt = (K + TS - 1) / TS;
    const int t0 = blockIdx.z * kBfWaves * kBfTPW;
    const int parts = m == 0 ? 1 : 2;
    const int NV = n_values(lmax);
    const int voff = value_offset(lmax, m);
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t pa = a.sub_start[s], pb = a.sub_start[s + 1];
    const int ncol = nt * TS;
    constexpr bool weighted = W;
    constexpr int IPT = bf_ipt<W>();
    const int nplanes = weighted ? 2 * NPC : NPC;
    const int KS = steps.ks[m];
    const int KSP = KS + 8;
    const int plane = ncol * KSP;                 // elements per plane
    const int bufsz = nplanes * plane;            // elements per buffer
    uint16_t* lds = reinterpret_cast<uint16_t*>(smem);
    const float* A = reinterpret_cast<const float*>(a.A);

    int ti[kBfTPW], tj[kBfTPW], all;
    const int nq = pick_tiles<TS>(K, nb, a.lcouple, t0 + wave, kBfWaves, ti, tj, all);
    if (t0 >= all) return;
    f32x16 acc32[kBfTPW];
    double accd[kBfTPW][16];
#pragma unroll
    for (int q = 0; q < kBfTPW; ++q) {
        acc32[q] = (f32x16)0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) accd[q][r] = 0.0;
    }

    const int groups = KS / 8;
    const int nitems = ncol * groups;
    const int nkst = (int)((pb - pa + KS - 1) / KS);
    const int nsteps = nkst * parts;

    // The thread's staging items do not change from step to step: column c
    // and primaries k8..k8+7 of the step. Their A row (part 0), LDS offset and
    // validity are computed once.
    int64_t irow[IPT];
    int ioff[IPT], ik8[IPT];
    bool iok[IPT], istore[IPT];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        const int it = threadIdx.x + u * 64 * kBfWaves;
        const int c = it / groups, k8 = (it - c * groups) * 8;
        const int lp = c / nb, b = c - lp * nb;
        istore[u] = it < nitems;
        iok[u] = it < nitems && c < K;
        ik8[u] = k8;
        ioff[u] = c * KSP + k8;
        irow[u] = ((int64_t)b * NV + voff + lp) * a.ldA;
    }
    const int64_t part_stride = (int64_t)nl * a.ldA;

    // Loads of step st into registers: two unconditional 16-byte loads per
    // item (and two of weights), all in bounds (the operand and the weight
    // buffers end with 8 elements of padding; an idle item, or one past the
    // step's primaries, reads the start of its row or of the buffer). The
    // elements that are not the step's primaries are zeroed when the step is
    // stored. Unconditional loads keep the count of loads in flight the same
    // on every path, so that waiting for one step never waits for the next.
    auto load = [&](int st, BfStage<W>& R) {
        const int part = st % parts;
        const int64_t p0 = pa + (int64_t)(st / parts) * KS;
        const int kv = (int)min((int64_t)KS, pb - p0);
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            const int kk = ik8[u] < kv ? ik8[u] : 0;
            const float* src = A + (iok[u] ? irow[u] + part * part_stride + p0 + kk : 0);
            float4 v0, v1;
            __builtin_memcpy(&v0, src, 16);
            __builtin_memcpy(&v1, src + 4, 16);
            R.x[u][0] = v0.x; R.x[u][1] = v0.y; R.x[u][2] = v0.z; R.x[u][3] = v0.w;
            R.x[u][4] = v1.x; R.x[u][5] = v1.y; R.x[u][6] = v1.z; R.x[u][7] = v1.w;
            if constexpr (W) {
                const float* wsrc = a.pw + a.p_begin + p0 + kk;
                __builtin_memcpy(&v0, wsrc, 16);
                __builtin_memcpy(&v1, wsrc + 4, 16);
                R.w[u][0] = v0.x; R.w[u][1] = v0.y; R.w[u][2] = v0.z; R.w[u][3] = v0.w;
                R.w[u][4] = v1.x; R.w[u][5] = v1.y; R.w[u][6] = v1.z; R.w[u][7] = v1.w;
            }
        }
    };
    // converts the registers of step st into BF16 planes of buffer `buf`
    auto store = [&](int st, int buf, BfStage<W>& R) {
        uint16_t* base = lds + buf * bufsz;
        const int64_t p0 = pa + (int64_t)(st / parts) * KS;
        const int kv = (int)min((int64_t)KS, pb - p0);
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            if (!istore[u]) continue;
            const int off = ioff[u];
            float x[8], y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool ok = iok[u] && ik8[u] + e < kv;
                x[e] = ok ? R.x[u][e] : 0.f;
                if constexpr (W) y[e] = ok ? R.x[u][e] * R.w[u][e] : 0.f;
            }
            uint4 pc[NPC];
            split8<NPC>(x, pc);
#pragma unroll
            for (int q = 0; q < NPC; ++q) *reinterpret_cast<uint4*>(base + q * plane + off) = pc[q];
            if constexpr (W) {
                split8<NPC>(y, pc);
#pragma unroll
                for (int q = 0; q < NPC; ++q) *reinterpret_cast<uint4*>(base + (NPC + q) * plane + off) = pc[q];
            }
        }
    };

    // FP32 accumulation spans at most 128 primaries of one part, or one step
    // of both parts where a step is shorter: then the sums go to FP64
    auto flush = [&]() {
#pragma unroll
        for (int q = 0; q < kBfTPW; ++q) {
#pragma unroll
            for (int r = 0; r < 16; ++r) accd[q][r] += (double)acc32[q][r];
            acc32[q] = (f32x16)0.0f;
        }
    };
    const int i = lane & 31, kg = lane >> 5;
    // MFMAs of NQ valid tiles over one step: no branch inside, so that the
    // LDS reads of one tile or slice overlap the MFMAs of the previous one
    auto mma = [&](auto nq, const uint16_t* xp, const uint16_t* wp) {
        constexpr int NQ = decltype(nq)::value;
        int ra[NQ], rb[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            ra[q] = (ti[q] * TS + i) * KSP + 8 * kg;
            rb[q] = (tj[q] * TS + i) * KSP + 8 * kg;
        }
        const int kc = KS > 128 ? 128 : KS;
        for (int kb = 0; kb < KS; kb += kc) {
#pragma unroll 2
            for (int k0 = kb; k0 < kb + kc; k0 += 16) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    bf16x8 ap[NPC], bp[NPC];
#pragma unroll
                    for (int u = 0; u < NPC; ++u) {
                        ap[u] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(wp + u * plane + ra[q] + k0));
                        bp[u] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(xp + u * plane + rb[q] + k0));
                    }
                    // products of pieces u, v with u + v <= NPC - 1
#pragma unroll
                    for (int u = 0; u < NPC; ++u)
#pragma unroll
                        for (int v2 = 0; v2 < NPC; ++v2)
                            if (u + v2 <= NPC - 1)
                                acc32[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ap[u], bp[v2], acc32[q], 0, 0, 0);
                }
            }
            if (KS > 128) flush();
        }
    };
    // MFMAs of step st from LDS buffer buf, then the FP64 flushes
    auto compute = [&](int st, int buf) {
        const uint16_t* xp = lds + buf * bufsz;
        const uint16_t* wp = weighted ? xp + NPC * plane : xp;
        if (nq == 2) mma(std::integral_constant<int, 2>{}, xp, wp);
        else if (nq == 1) mma(std::integral_constant<int, 1>{}, xp, wp);
        if (KS <= 128 && st % parts == parts - 1) flush();
    };

    if (nbuf == 2) {
        // two LDS buffers and one register stage: the loads of step st + 1
        // are issued before the MFMAs of step st and converted into the
        // other buffer after them (a second register stage, loading two
        // steps ahead, spilled registers and measured slower)
        BfStage<W> R;
        load(0, R);
        store(0, 0, R);
        __syncthreads();
        for (int st = 0; st < nsteps; ++st) {
            if (st + 1 < nsteps) load(st + 1, R);
            compute(st, st & 1);
            if (st + 1 < nsteps) store(st + 1, (st + 1) & 1, R);
            __syncthreads();
        }
    } else {
        BfStage<W> R;
        load(0, R);
        store(0, 0, R);
        __syncthreads();
        for (int st = 0; st < nsteps; ++st) {
            compute(st, 0);
            if (st + 1 < nsteps) {
                __syncthreads();
                load(st + 1, R);
                store(st + 1, 0, R);
            }
            __syncthreads();
        }
    }
    double* G = a.part + (int64_t)s * a.gsize + a.goff[m];
#pragma unroll
    for (int q = 0; q < kBfTPW; ++q) {
        if (q >= nq) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            put_entry(G, K, nb, nl, ti[q], tj[q], ti[q] * TS + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3),
                      tj[q] * TS + (lane & 31), accd[q][r]);
    }
}

// Degenerate-triangle moments sum_p w_p sum_j w_j^2 R^0_L(z_pj) and pair
// counts per bin. One workgroup per (subchunk, group of kSelfTasks tasks); the
// subchunk's primary weights are staged in LDS once (not with unit weights),
// and every wavefront sums its tasks with four independent FP64 partial sums
// in a fixed order. A row is streamed kSelfUnroll loads per lane at a time, so
// that enough loads are in flight to cover the memory latency. With unit
// weights the pair count of a bin is its L = 0 moment (an exact integer sum),
// written by that task.
constexpr int kSelfTasks = 16;
constexpr int kSelfMaxSub = 4096;  // primaries per subchunk
constexpr int kSelfUnroll = 16;

template <bool UNIT, typename T>
__global__ void __launch_bounds__(256) k_self_moments(SelfArgs a) {
    __shared__ double wsh[UNIT ? 1 : kSelfMaxSub];
    const int s = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nL = 2 * a.lmax + 1;
    const int width = nL + 1;
    const int ntask = a.nb * width;
    const int NV = n_values(a.lmax);
    const int na = n_alm_values(a.lmax);
    const int64_t pa = a.sub_start[s], pb = a.sub_start[s + 1];
    const int n = (int)(pb - pa);
    if constexpr (!UNIT) {
        for (int i = threadIdx.x; i < n; i += 256) wsh[i] = a.pd[a.p_begin + pa + i].w;
        __syncthreads();
    }
    constexpr int kSpan = 64 * kSelfUnroll;
    for (int q = 0; q < kSelfTasks / 4; ++q) {
        const int task = blockIdx.y * kSelfTasks + wave * (kSelfTasks / 4) + q;
        if (task >= ntask) break;
        const int b = task / width, L = task - b * width;
        if (UNIT && L == nL) continue;  // written by the L = 0 task
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        if (a.self_lo && L > a.lmax && L < nL) {
            // not written by the harmonic pass of such a run: the moment is zero
        } else if (L < nL) {
            const T* row = reinterpret_cast<const T*>(a.A) + ((int64_t)b * NV + na + L) * a.ldA + pa;
            auto span = [&](int p0, auto whole) {
                // the last span is masked, its loads clamped into the row, so
                // that they are in flight together too. The values wait in the
                // operand's own type (converted and chosen per load, they
                // cost twice the registers and a branch: 2.33 ms against 0.73
                // for 64 catalogues at lmax 10)
                constexpr bool ALL = decltype(whole)::value;
                T v[kSelfUnroll];
#pragma unroll
                for (int u = 0; u < kSelfUnroll; ++u) {
                    const int p = p0 + 64 * u + lane;
                    v[u] = row[ALL ? p : min(p, n - 1)];
                }
#pragma unroll
                for (int u = 0; u < kSelfUnroll; ++u) {
                    const int p = p0 + 64 * u + lane;
                    if (ALL || p < n) acc[u & 3] += UNIT ? (double)v[u] : wsh[p] * (double)v[u];
                }
            };
            int p0 = 0;
            for (; p0 + kSpan <= n; p0 += kSpan) span(p0, std::true_type{});
            if (p0 < n) span(p0, std::false_type{});
        } else {
            for (int p0 = 0; p0 < n; p0 += 256) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int p = p0 + 64 * u + lane;
                    if (p < n) acc[u] += (double)a.cnt[(pa + p) * a.nb + b];
                }
            }
        }
        double sum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (lane == 0) {
            double* out = a.part + (int64_t)s * a.nb * width;
            out[task] = sum;
            if (UNIT && L == 0) out[b * width + nL] = sum;
        }
    }
}

// Sums of each catalogue's subchunks, those of the contraction and of the self
// moments in one launch. Latency bound: a thread adds one value of a few dozen
// subchunks in their order, eight loads in flight. A catalogue whose subchunks
// come in several launches goes on from the sum so far, so that its sum does
// not depend on how they are cut. Of the blocks only what is formed is read,
// the upper triangle and the coupled orders (36,000 subchunks, lmax 10, 10 bins,
// L = 0: 2.8 ms with all entries, 1.6 without the rest).
__global__ void k_reduce_partials(ReduceArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int c = a.cat_lo + blockIdx.y;
    if (i >= a.width[0] + a.width[1]) return;
    const int k = i >= a.width[0];
    const int64_t width = a.width[k], e = k ? i - a.width[0] : i;
    if (k == 0) {
        int m = 0;
        while (a.goff[m + 1] <= e) ++m;
        const int K = a.nb * (a.lmax - m + 1), r = (int)(e - a.goff[m]), ci = r / K, cj = r - ci * K;
        if (cj < ci || cj / a.nb - ci / a.nb > a.lcouple) return;
    }
    const double* p = a.part[k] + e;
    double* out = a.out[k] + c * width + e;
    const int first = a.cat_sub[c];
    const int q1 = min(a.cat_sub[c + 1], a.sub_hi) - a.sub_lo;
    int q = max(first, a.sub_lo) - a.sub_lo;
    double s = first >= a.sub_lo ? 0.0 : *out;
    for (; q + 8 <= q1; q += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(q + u) * width];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; q < q1; ++q) s += p[q * width];
    *out = s;
}

__global__ void k_finalize(FinalArgs a) {
    const int nb = a.nb;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per = (int64_t)a.n_mult * nb * nb;
    const int c = blockIdx.y;
    if (idx >= per || c >= a.ncat) return;
    const int t = (int)(idx / (nb * nb));
    const int b1 = (int)((idx / nb) % nb), b2 = (int)(idx % nb);
    const int l1 = a.mult[3 * t], l2 = a.mult[3 * t + 1];
    const int mm = min(l1, l2);
    const int nL = 2 * a.lmax + 1;
    const int sw = nb * (nL + 1);
    const double* G = a.G + (int64_t)c * a.gsize;
    // of the self moments only the order L of the multipole has a coefficient
    const int L = a.mult[3 * t + 2];
    const bool self = b1 == b2 && a.subtract_self;
    const double S = self ? a.S[(int64_t)c * sw + b1 * (nL + 1) + L] : 0.0;
    double sum = 0.0;
#pragma unroll 4
    for (int m = 0; m <= mm; ++m) {
        const int nl = a.lmax - m + 1;
        const int K = nb * nl;
        const int ci = (l1 - m) * nb + b1, cj = (l2 - m) * nb + b2;
        const double g = G[a.goff[m] + (int64_t)min(ci, cj) * K + max(ci, cj)];
        sum += a.coefG[t * (a.lmax + 1) + m] * g;
        if (self) sum -= a.coefS[((int64_t)t * (a.lmax + 1) + m) * nL + L] * S;
    }
    const double nd = a.nd[c];
    const double rrr = nd * (nd - 1.0) * (nd - 2.0) * a.vol[b1] * a.vol[b2] * a.inv_box6;
    a.out[(int64_t)c * per + idx] = sum / rrr;
}

// Edge correction of the isotropic multipoles for the Szapudi-Szalay estimator
// with explicit randoms (eq. (ssest)): the triplet counts of the data-minus-
// randoms field and of the randoms are related as functions of the opening
// angle by N = zeta R, which for Legendre coefficients reads
//   N_l = sum_{l'} M_{l l'} zeta_{l'},  M_{l l'} = sum_{l''} T[l][l'][l''] R_{l''},
// with T[l][l'][l''] = (2l+1)/2 int P_l P_l' P_l'' (the relation of Slepian &
// Eisenstein 2015). One thread per (b1, b2) forms M in LDS and solves by
// Gaussian elimination with partial pivoting in FP64; a singular M sets *bad.
__global__ void k_edge_iso(const double* __restrict__ N, const double* __restrict__ R, const double* __restrict__ T,
                           int nl, int nbb, double* __restrict__ out, int* __restrict__ bad) {
    extern __shared__ double esh[];
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nbb) return;
    double* M = esh + (size_t)threadIdx.x * (nl * nl + nl);
    double* x = M + nl * nl;
    for (int l = 0; l < nl; ++l) {
        x[l] = N[(int64_t)l * nbb + q];
        for (int lp = 0; lp < nl; ++lp) {
            double v = 0.0;
            for (int lpp = 0; lpp < nl; ++lpp) v += T[(l * nl + lp) * nl + lpp] * R[(int64_t)lpp * nbb + q];
            M[l * nl + lp] = v;
        }
    }
    for (int c = 0; c < nl; ++c) {
        int piv = c;
        for (int r = c + 1; r < nl; ++r)
            if (fabs(M[r * nl + c]) > fabs(M[piv * nl + c])) piv = r;
        if (!(fabs(M[piv * nl + c]) > 0.0)) {
            atomicOr(bad, 1);
            return;
        }
        if (piv != c) {
            for (int k = 0; k < nl; ++k) {
                const double t = M[c * nl + k];
                M[c * nl + k] = M[piv * nl + k];
                M[piv * nl + k] = t;
            }
            const double t = x[c];
            x[c] = x[piv];
            x[piv] = t;
        }
        const double ip = 1.0 / M[c * nl + c];
        for (int r = c + 1; r < nl; ++r) {
            const double f = M[r * nl + c] * ip;
            for (int k = c; k < nl; ++k) M[r * nl + k] -= f * M[c * nl + k];
            x[r] -= f * x[c];
        }
    }
    for (int c = nl - 1; c >= 0; --c) {
        double v = x[c];
        for (int k = c + 1; k < nl; ++k) v -= M[c * nl + k] * x[k];
        x[c] = v / M[c * nl + c];
    }
    for (int l = 0; l < nl; ++l) out[(int64_t)l * nbb + q] = x[l];
}

__global__ void k_export_nnn(NnnArgs a) {
    const int nb = a.nb, s1 = a.lmax + 1, nL = 2 * a.lmax + 1;
    const int64_t n = (int64_t)s1 * s1 * s1 * nb * nb;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    const int b2 = (int)(idx % nb), b1 = (int)((idx / nb) % nb);
    const int64_t t = idx / ((int64_t)nb * nb);
    const int l2 = (int)(t % s1), l1 = (int)((t / s1) % s1), m = (int)(t / ((int64_t)s1 * s1));
    double v = 0.0;
    if (l1 >= m && l2 >= m && (!a.isotropic || l1 == l2)) {
        const int nl = a.lmax - m + 1, K = nb * nl;
        const int ci = (l1 - m) * nb + b1, cj = (l2 - m) * nb + b2;
        v = a.scale[l1 * s1 + m] * a.scale[l2 * s1 + m] *
            a.G[a.goff[m] + (int64_t)min(ci, cj) * K + max(ci, cj)];
        if (b1 == b2 && a.subtract_self) {
            const double* g = a.gaunt + ((int64_t)(m * s1 + l1) * s1 + l2) * nL;
            const double* S = a.S + b1 * (nL + 1);
            for (int L = 0; L < nL; ++L) v -= g[L] * S[L];
        }
    }
    a.out[idx] = v;
}

__global__ void k_export_alm(AlmExportArgs a) {
    const int nb = a.nb, s1 = a.lmax + 1;
    const int NV = n_values(a.lmax);
    const int64_t n = a.count * nb * s1 * s1;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    const int m = (int)(idx % s1), l = (int)((idx / s1) % s1), b = (int)((idx / (s1 * s1)) % nb);
    const int64_t i = idx / ((int64_t)s1 * s1 * nb);
    double re = 0.0, im = 0.0;
    if (m <= l) {
        const int64_t p = a.perm[a.first + i] - a.p_begin;
        const int nl = a.lmax - m + 1;
        const int v0 = value_offset(a.lmax, m) + (l - m);
        const int64_t r0 = ((int64_t)b * NV + v0) * a.ldA + p;
        if (a.fp64) {
            const double* A = reinterpret_cast<const double*>(a.A);
            re = A[r0];
            if (m > 0) im = A[r0 + (int64_t)nl * a.ldA];
        } else {
            const float* A = reinterpret_cast<const float*>(a.A);
            re = A[r0];
            if (m > 0) im = A[r0 + (int64_t)nl * a.ldA];
        }
        const double f = a.sign_scale[l * s1 + m];
        re *= f;
        im *= f;
    }
    a.out[2 * idx] = re;
    a.out[2 * idx + 1] = im;
}

// Flat columns that a step of the FP64 / FP32 contraction stages: 128 / 256
// (two / four items per thread: every m of up to 128 / 256 columns, the narrow
// ones several units at a time), else all columns of the widest m, with as
// many items per thread as they take.
struct StepPlan { int ncol, cols, nbuf; size_t lds; };
StepPlan step_plan(bool f64, int nb, int lmax) {
    const int TS = f64 ? 16 : 32, base = f64 ? 128 : 256;
    StepPlan p;
    p.ncol = (nb * (lmax + 1) + TS - 1) / TS * TS;
    p.cols = std::max(base, p.ncol);
    // the largest step over the m: whole units within p.cols flat columns, at
    // most 8 units (a unit of the widest m alone where it exceeds p.cols / 2)
    p.nbuf = !f64 || f64_lds(p.cols, 8, 2) <= 160 * 1024 ? 2 : 1;
    p.lds = f64 ? f64_lds(p.cols, 8, p.nbuf) : f32_lds(p.cols, 8, p.nbuf);
    return p;
}

template <bool W>
hipError_t launch_contract_f64(const ContractArgs& a, const StepPlan& p, hipStream_t s) {
    const int nt = p.ncol / 16;
    const dim3 grid(a.nsub, a.lmax + 1, (nt * (nt + 1) / 2 + kF64Waves * kF64TPW - 1) / (kF64Waves * kF64TPW));
    auto run = [&](auto ipt) {
        constexpr int IPT = decltype(ipt)::value;
        const hipError_t e = allow_full_lds((const void*)k_contract_f64<W, IPT>);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_contract_f64<W, IPT>), grid, dim3(64 * kF64Waves), p.lds, s, a, p.cols, p.nbuf);
        return hipGetLastError();
    };
    if (p.cols <= 128) return run(std::integral_constant<int, 2>{});
    if (p.cols <= 256) return run(std::integral_constant<int, 4>{});
    return run(std::integral_constant<int, 9>{});
}

template <bool W>
hipError_t launch_contract_f32(const ContractArgs& a, const StepPlan& p, hipStream_t s) {
    const int nt = p.ncol / 32;
    const dim3 grid(a.nsub, a.lmax + 1, (nt * (nt + 1) / 2 + kF32Waves * kF32TPW - 1) / (kF32Waves * kF32TPW));
    auto run = [&](auto ipt) {
        constexpr int IPT = decltype(ipt)::value;
        const hipError_t e = allow_full_lds((const void*)k_contract_f32<W, IPT>);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_contract_f32<W, IPT>), grid, dim3(64 * kF32Waves), p.lds, s, a, p.cols);
        return hipGetLastError();
    };
    return p.cols <= 256 ? run(std::integral_constant<int, 4>{}) : run(std::integral_constant<int, 9>{});
}

hipError_t launch_contract_plain(const ContractArgs& a, bool f64, hipStream_t s) {
    const StepPlan p = step_plan(f64, a.nb, a.lmax);
    if (f64) return a.unit_weights ? launch_contract_f64<false>(a, p, s) : launch_contract_f64<true>(a, p, s);
    return a.unit_weights ? launch_contract_f32<false>(a, p, s) : launch_contract_f32<true>(a, p, s);
}

}  // namespace

// Step cap and buffer count of the split-BF16 contraction. Every m takes
// its own step (bf_step): the longest up to cap (512, or ks_max when given)
// that fits the registers and LDS for its columns; m = 0, the widest, needs
// at least 16. Double-buffered when every m's buffers fit in LDS. lds is the
// largest need over the m (the allocation of each workgroup).
struct BfPlan { BfSteps steps; int nbuf; size_t lds; };
BfPlan bf_plan(int npc, int nb, int lmax, bool weighted, int ks_max = 0) {
    const int nplanes = weighted ? 2 * npc : npc;
    const int ipt = weighted ? bf_ipt<true>() : bf_ipt<false>();
    const int cap = ks_max >= 16 ? std::min(ks_max, 512) : 512;
    BfPlan pl{};
    for (int nbuf = 2; nbuf >= 1; --nbuf) {
        size_t need = 0;
        bool ok = lmax <= kMaxLmax;
        for (int m = 0; m <= lmax && ok; ++m) {
            const int ncol = (nb * (lmax - m + 1) + 31) / 32 * 32;
            const int ks = bf_step(ncol, nplanes, ipt, nbuf, cap, 160 * 1024);
            ok = ks > 0;
            pl.steps.ks[m] = ks;
            need = std::max(need, (size_t)nbuf * nplanes * ncol * (ks + 8) * sizeof(uint16_t));
        }
        if (ok) {
            pl.nbuf = nbuf;
            pl.lds = need;
            return pl;
        }
    }
    return BfPlan{};
}

template <int NPC, bool W>
hipError_t launch_contract_bf16_w(const ContractArgs& a, hipStream_t s) {
    const int K0 = a.nb * (a.lmax + 1);
    const int nt0 = (K0 + 31) / 32;
    const int ntiles0 = nt0 * (nt0 + 1) / 2;
    const int ngroups = (ntiles0 + kBfWaves * kBfTPW - 1) / (kBfWaves * kBfTPW);
    const BfPlan pl = bf_plan(NPC, a.nb, a.lmax, !a.unit_weights, a.ks_max);
    if (pl.nbuf == 0) return hipErrorInvalidValue;
    const hipError_t e = allow_full_lds((const void*)k_contract_bf16<NPC, W>);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_contract_bf16<NPC, W>), dim3(a.nsub, a.lmax + 1, ngroups), dim3(64 * kBfWaves),
                       pl.lds, s, a, pl.steps, pl.nbuf);
    return hipGetLastError();
}

template <int NPC>
hipError_t launch_contract_bf16(const ContractArgs& a, hipStream_t s) {
    return a.unit_weights ? launch_contract_bf16_w<NPC, false>(a, s) : launch_contract_bf16_w<NPC, true>(a, s);
}

hipError_t launch_contract_iso(const ContractArgs& a, hipStream_t s) {
    if (a.nsub <= 0) return hipSuccess;
    if (a.nb > 32) return hipErrorInvalidValue;
    const int nlm = (a.lmax + 1) * (a.lmax + 2) / 2;
    const dim3 grid(a.nsub, (nlm + kIsoWaves - 1) / kIsoWaves);
    const bool f64 = a.mode == 0;
    if (a.unit_weights) {
        if (f64) hipLaunchKernelGGL((k_contract_iso<double, false>), grid, dim3(64 * kIsoWaves), 0, s, a);
        else hipLaunchKernelGGL((k_contract_iso<float, false>), grid, dim3(64 * kIsoWaves), 0, s, a);
    } else {
        if (f64) hipLaunchKernelGGL((k_contract_iso<double, true>), grid, dim3(64 * kIsoWaves), 0, s, a);
        else hipLaunchKernelGGL((k_contract_iso<float, true>), grid, dim3(64 * kIsoWaves), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_contract(const ContractArgs& a, hipStream_t s) {
    if (a.nsub <= 0) return hipSuccess;
    switch (a.mode) {
        case 0: return launch_contract_plain(a, true, s);
        case 1: return launch_contract_plain(a, false, s);
        case 2:
        case 3: {
            // a split-BF16 step must stage at least 16 primaries of every
            // column in the threads' registers (nbins (lmax + 1) <= 512 with
            // weights); beyond that the FP32 MFMA contraction runs instead
            if (bf_plan(a.mode == 2 ? 2 : 3, a.nb, a.lmax, !a.unit_weights, a.ks_max).nbuf == 0)
                return launch_contract_plain(a, false, s);
            return a.mode == 2 ? launch_contract_bf16<2>(a, s) : launch_contract_bf16<3>(a, s);
        }
        default: return hipErrorInvalidValue;
    }
}

size_t contract_lds_bytes(int mode, int nb, int lmax) {
    if (mode <= 1) return step_plan(mode == 0, nb, lmax).lds;
    const BfPlan pl = bf_plan(mode == 2 ? 2 : 3, nb, lmax, true);
    return pl.nbuf ? pl.lds : step_plan(false, nb, lmax).lds;
}

hipError_t launch_self_moments(const SelfArgs& a, hipStream_t s) {
    if (a.nsub <= 0) return hipSuccess;
    const int ntask = a.nb * (2 * a.lmax + 2);
    const dim3 grid(a.nsub, (ntask + kSelfTasks - 1) / kSelfTasks);
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a); };
    if (a.unit_w) a.fp64 ? run(k_self_moments<true, double>) : run(k_self_moments<true, float>);
    else a.fp64 ? run(k_self_moments<false, double>) : run(k_self_moments<false, float>);
    return hipGetLastError();
}

hipError_t launch_reduce_partials(const ReduceArgs& a, hipStream_t s) {
    const int64_t n = a.width[0] + a.width[1];
    if (a.ncat <= 0 || n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_partials, dim3((unsigned)((n + 255) / 256), a.ncat), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_finalize(const FinalArgs& a, hipStream_t s) {
    const int64_t per = (int64_t)a.n_mult * a.nb * a.nb;
    if (per <= 0 || a.ncat <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_finalize, dim3((unsigned)((per + 255) / 256), a.ncat), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_edge_iso(const double* N, const double* R, const double* T, int nl, int nbb, double* out, int* bad,
                           hipStream_t s) {
    if (nbb <= 0 || nl <= 0) return hipSuccess;
    // one system (nl^2 + nl doubles) per thread in LDS: up to 32 threads, within 160 KiB
    const size_t per = (size_t)(nl * nl + nl) * sizeof(double);
    const int kThreads = (int)std::max<size_t>(1, std::min<size_t>(32, (size_t)160 * 1024 / per));
    const size_t lds = (size_t)kThreads * per;
    if (lds > 64 * 1024) {
        hipError_t e = allow_full_lds((const void*)k_edge_iso);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_edge_iso, dim3((nbb + kThreads - 1) / kThreads), dim3(kThreads), lds, s, N, R, T, nl, nbb,
                       out, bad);
    return hipGetLastError();
}

hipError_t launch_export_nnn(const NnnArgs& a, hipStream_t s) {
    const int64_t n = (int64_t)(a.lmax + 1) * (a.lmax + 1) * (a.lmax + 1) * a.nb * a.nb;
    hipLaunchKernelGGL(k_export_nnn, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_export_alm(const AlmExportArgs& a, hipStream_t s) {
    const int64_t n = a.count * a.nb * (a.lmax + 1) * (a.lmax + 1);
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_export_alm, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace tpcf
