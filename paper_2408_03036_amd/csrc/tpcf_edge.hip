// Edge correction of the anisotropic 3PCF by explicit randoms: the
// Szapudi-Szalay estimator of eq. (ssest), zeta = (D - R)^3 / R^3, read as a
// ratio of two functions of the triangle (arXiv:2408.03036, Sec. 4).
//
// With N and R the data-minus-randoms and random triplet counts of one
// (r1, r2) bin pair, each a real function of the two side directions and
// expanded in the orthonormal basis Y_l1m(r1) conj(Y_l2m(r2)) (the per-m
// coefficients NNN^m of the contraction, normalised by their analytic RRR),
// N = zeta R at every pair of directions gives
//   N^m_{l1 l2} = sum zeta^{m'}_{l1' l2'} R^{m-m'}_{l1'' l2''}
//                 g(l1 m; l1' m'; l1'') g(l2 m; l2' m'; l2''),
// g(l m; l' m'; l'') = integral of conj(Y_lm) Y_l'm' Y_l'',m-m' (real), all
// indices truncated at lmax. The real (reflection-symmetric) sector is solved:
// every coefficient is real and X^{-m} = X^m, so the unknowns are zeta^m for
// m >= 0 and the columns of m' > 0 collect the terms of +m' and -m'.
//
//  k_edge_assemble  the n x n systems (n = number of (l1, l2, m >= 0) with
//                   m <= l1, l2 <= lmax), a lane per system
//  k_edge_solve     one workgroup per system: blocked LU with partial
//                   pivoting in FP64 (MFMA for the trailing update), then back
//                   substitution; writes zeta^m in the export layout
//  k_edge_mult      TripoSH sums of zeta^m for the requested multipoles
#include <algorithm>

#include "tpcf_internal.h"

namespace tpcf {

namespace {

// The systems' matrices: M[q][row][col] = sum over the terms of +m' and -m',
// c1 and c2 of g1 g2 R_c1c2[q]. Every system has the same Gaunt factors, so a
// lane is one system: the factors are uniform over a wavefront, zero terms are
// skipped by scalar branches and the R loads are contiguous. A workgroup does
// kAsmCols columns of one row for kAsmSys systems and turns its tile in LDS,
// so that the matrices are written in 128-byte pieces. (One thread per
// entry, with the systems' R strided over the lanes: 4.5 ms at lmax 10 and
// 10 bins; this form 0.42 ms.)
constexpr int kAsmSys = 64, kAsmCols = 16, kAsmWaves = 4;

__global__ void __launch_bounds__(64 * kAsmWaves) k_edge_assemble(EdgeArgs a) {
    __shared__ double tile[kAsmCols][kAsmSys + 1];
    const int n = a.n, nbb = a.nsys, lmax = a.lmax;
    const int S = lmax + 1, S2 = 2 * lmax + 1;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int row = blockIdx.y, col0 = blockIdx.x * kAsmCols, q0 = blockIdx.z * kAsmSys;
    const int q = min(q0 + lane, nbb - 1);
    const int4 r = a.units[row];  // (l1, l2, m)
    const int l1 = r.x, l2 = r.y, m = r.z;
    const double irr = a.inv_rrr_R[q];
    for (int cc = wave; cc < kAsmCols; cc += kAsmWaves) {
        const int col = col0 + cc;
        if (col >= n) break;
        const int4 c = a.units[col];
        double acc = 0.0;
        for (int s = 0; s < (c.z > 0 ? 2 : 1); ++s) {
            const int mq = s == 0 ? c.z : -c.z;  // m' of this term
            const int mpp = m - mq;
            const int am = mpp < 0 ? -mpp : mpp;
            if (am > lmax) continue;
            // g(l, m; l', m'; l'') at ((((l S + m) S + l') S2 + m' + lmax) S + l''): zero
            // unless |l - l'| <= l'' <= l + l' and l + l' + l'' is even
            const double* g1 = a.gaunt + ((((int64_t)l1 * S + m) * S + c.x) * S2 + mq + lmax) * S;
            const double* g2 = a.gaunt + ((((int64_t)l2 * S + m) * S + c.y) * S2 + mq + lmax) * S;
            const double* Rm = a.R + (int64_t)am * S * S * nbb + q;
            auto first = [&](int l, int lp) {
                int lo = max(abs(l - lp), am);
                return lo + ((l + lp + lo) & 1);
            };
            const int top1 = min(l1 + c.x, lmax), top2 = min(l2 + c.y, lmax), lo2 = first(l2, c.y);
            for (int c1 = first(l1, c.x); c1 <= top1; c1 += 2) {
                double t = 0.0;
                for (int c2 = lo2; c2 <= top2; c2 += 2) t = fma(g2[c2], Rm[((int64_t)c1 * S + c2) * nbb], t);
                acc = fma(g1[c1], t, acc);
            }
        }
        tile[cc][lane] = acc * irr;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kAsmCols * kAsmSys; e += 64 * kAsmWaves) {
        const int cc = e % kAsmCols, qq = e / kAsmCols;
        if (col0 + cc < n && q0 + qq < nbb) a.M[((int64_t)(q0 + qq) * n + row) * n + col0 + cc] = tile[cc][qq];
    }
    if (blockIdx.x == 0 && wave == 0 && q0 + lane < nbb)
        a.rhs[(int64_t)q * n + row] = a.N[(((int64_t)m * S + l1) * S + l2) * nbb + q] * a.inv_rrr_N[q];
}

// ---------------------------------------------------------------- the solve
// Blocked right-looking LU with partial pivoting, one workgroup per system.
// A panel is kPB columns: thread t holds row t of the panel in registers, so
// a column step is a wavefront maximum, one barrier and kPB fused
// multiply-adds; rows are not exchanged inside the panel, the pivots only
// marked. The panel's L goes to LDS in its final row order, a thread per
// column to the right takes the pivot rows through the unit lower triangle
// (moving the rows they displace), and the trailing update runs on 16x16x4
// FP64 MFMA with L from LDS. The right-hand side is column n.
//
// One workgroup fills one CU, so the time is that of one system: at n = 506
// the update's MFMAs are 0.31 ms of it at the CU's peak, and 506 column steps
// of about 0.4 us the next. Eliminating one pivot at a time on the whole
// matrix in memory took 79.6 ms for 100 systems (lmax 10, 10 bins); this
// takes 2.0 ms.
constexpr int kPB = 32;
constexpr int kLP = kPB + 1;  // LDS row stride of the panel
constexpr int kSolveMaxThreads = 512;
static_assert(kMaxEdgeUnknowns <= kSolveMaxThreads, "one thread per row");

typedef double f64x4 __attribute__((ext_vector_type(4)));

struct SolveLds {
    double prow[2][kSolveMaxThreads / 64][kPB];  // each wavefront's candidate pivot row
    double pinv[2][kSolveMaxThreads / 64];
    unsigned long long key[2][kSolveMaxThreads / 64];
    double xb[kPB];
    int row[2][kSolveMaxThreads / 64];
    int piv[kPB], disp[kPB], vac[kPB];
    int ndisp;
};

size_t solve_lds_bytes(int n) {
    return (sizeof(SolveLds) + 15) / 16 * 16 + sizeof(double) * (size_t)std::max((n + 15) / 16 * 16, kPB) * kLP;
}

template <int CTRL, int RMASK>
__device__ __forceinline__ unsigned long long dpp_max(unsigned long long v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, RMASK, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, RMASK, 0xf, false);
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;
    return o > v ? o : v;
}
// Maximum over the wavefront (of unsigned values; lanes out of a shift's
// range give 0), in every lane.
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
    v = dpp_max<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8
    v = dpp_max<0x112, 0xf>(v);
    v = dpp_max<0x114, 0xf>(v);
    v = dpp_max<0x118, 0xf>(v);
    v = dpp_max<0x142, 0xa>(v);  // row_bcast 15, 31
    v = dpp_max<0x143, 0xc>(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
    return ((unsigned long long)hi << 32) | lo;
}

__global__ void __launch_bounds__(kSolveMaxThreads) k_edge_solve(EdgeArgs a) {
    extern __shared__ unsigned char esmem[];
    SolveLds& W = *reinterpret_cast<SolveLds*>(esmem);
    double* Lp = reinterpret_cast<double*>(esmem + (sizeof(SolveLds) + 15) / 16 * 16);
    const int q = blockIdx.x;
    const int n = a.n, T = blockDim.x, nw = T >> 6;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double* M = a.M + (int64_t)q * n * n;
    double* x = a.rhs + (int64_t)q * n;
    // column j of the augmented system: the matrix, then the right-hand side
    auto column = [&](int j, int& stride) {
        stride = j < n ? n : 1;
        return j < n ? M + j : x;
    };
    for (int k0 = 0; k0 < n; k0 += kPB) {
        const int pw = min(kPB, n - k0), m = n - k0;  // panel width, rows left
        for (int e = tid; e < m * kPB; e += T) {
            const int r = e / kPB, c = e % kPB;
            Lp[r * kLP + c] = c < pw ? M[(int64_t)(k0 + r) * n + k0 + c] : 0.0;
        }
        __syncthreads();
        double r[kPB];
#pragma unroll
        for (int c = 0; c < kPB; ++c) r[c] = tid < m ? Lp[tid * kLP + c] : 0.0;
        bool active = tid < m;
        int mypos = -1;  // the pivot this row became
#pragma unroll
        for (int c = 0; c < kPB; ++c) {
            if (c < pw) {
                // largest |r[c]| of the rows left: non-negative doubles order as
                // their bits; NaN and rows already taken count as 0
                const double v = fabs(r[c]);
                const unsigned long long key =
                    active && v >= 0.0 ? (unsigned long long)__double_as_longlong(v) : 0ull;
                const unsigned long long best = wave_max(key);
                const int win = __ffsll((long long)__ballot(key == best)) - 1;
                if (lane == win) {
                    W.key[c & 1][wave] = best;
                    W.row[c & 1][wave] = tid;
                    W.pinv[c & 1][wave] = 1.0 / r[c];
#pragma unroll
                    for (int j = c + 1; j < kPB; ++j) W.prow[c & 1][wave][j] = r[j];
                }
                __syncthreads();
                unsigned long long top = W.key[c & 1][0];
                int bw = 0;
                for (int w = 1; w < nw; ++w) {
                    const unsigned long long o = W.key[c & 1][w];
                    if (o > top) {
                        top = o;
                        bw = w;
                    }
                }
                if (top == 0ull) {
                    if (tid == 0) atomicOr(a.bad, 1);
                    return;  // uniform: every thread read the same keys
                }
                if (tid == W.row[c & 1][bw]) {
                    active = false;
                    mypos = c;
                } else if (active) {
                    const double f = r[c] * W.pinv[c & 1][bw];
                    r[c] = f;
                    const double* pr = W.prow[c & 1][bw];
#pragma unroll
                    for (int j = c + 1; j < kPB; ++j) r[j] = fma(-f, pr[j], r[j]);
                }
            }
        }
        // final rows: pivot c at panel row c; a row it displaced goes to a row
        // that a pivot left (the panel's first pw rows are all in wavefront 0)
        if (mypos >= 0) W.piv[mypos] = tid;
        const unsigned long long below = (1ull << lane) - 1ull;
        int rank = -1;
        if (wave == 0) {
            const bool moved = lane < pw && mypos < 0;
            const unsigned long long mv = __ballot(moved);
            if (moved) {
                rank = __popcll(mv & below);
                W.disp[rank] = lane;
            }
            if (lane == 0) W.ndisp = __popcll(mv);
        }
        __syncthreads();
        if (wave == 0) {
            const int p = lane < pw ? W.piv[lane] : 0;
            const unsigned long long left = __ballot(lane < pw && p >= pw);
            if (lane < pw && p >= pw) W.vac[__popcll(left & below)] = p;
        }
        __syncthreads();
        if (tid < m) {
            const int at = mypos >= 0 ? mypos : (rank >= 0 ? W.vac[rank] : tid);
#pragma unroll
            for (int c = 0; c < kPB; ++c) Lp[at * kLP + c] = -r[c];
            if (mypos >= 0) {
                double* u = M + (int64_t)(k0 + mypos) * n + k0;
#pragma unroll
                for (int c = 0; c < kPB; ++c)
                    if (c >= mypos && c < pw) u[c] = r[c];
            }
        }
        __syncthreads();
        // columns to the right: pivot rows through the unit lower triangle
        for (int j = k0 + pw + tid; j <= n; j += T) {
            int st;
            double* col = column(j, st) ;
            double u[kPB];
#pragma unroll
            for (int c = 0; c < kPB; ++c) u[c] = c < pw ? col[(int64_t)(k0 + W.piv[c]) * st] : 0.0;
            const int nd = W.ndisp;
            for (int i = 0; i < nd; ++i) col[(int64_t)(k0 + W.vac[i]) * st] = col[(int64_t)(k0 + W.disp[i]) * st];
#pragma unroll
            for (int c = 1; c < kPB; ++c)
                if (c < pw) {
#pragma unroll
                    for (int d = 0; d < c; ++d) u[c] = fma(Lp[c * kLP + d], u[d], u[c]);
                }
#pragma unroll
            for (int c = 0; c < kPB; ++c)
                if (c < pw) col[(int64_t)(k0 + c) * st] = u[c];
        }
        __syncthreads();
        // trailing update C -= L U: a wavefront takes strips of 16 columns
        const int b = k0 + pw, mt = n - b;
        if (mt > 0) {
            const int li = lane & 15, lg = lane >> 4;
            for (int j0 = b + 16 * wave; j0 <= n; j0 += 16 * nw) {
                const int j = min(j0 + li, n);
                const bool jv = j0 + li <= n;
                int st;
                double* col = column(j, st);
                double u[kPB / 4];
#pragma unroll
                for (int kk = 0; kk < kPB / 4; ++kk) u[kk] = col[(int64_t)(k0 + 4 * kk + lg) * st];
                auto fetch = [&](int i0, f64x4& c) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) c[e] = col[(int64_t)min(b + i0 + lg + 4 * e, n - 1) * st];
                };
                f64x4 next;
                fetch(0, next);
                for (int i0 = 0; i0 < mt; i0 += 16) {
                    f64x4 c = next;
                    if (i0 + 16 < mt) fetch(i0 + 16, next);
                    const double* L = Lp + (pw + i0 + li) * kLP + lg;
#pragma unroll
                    for (int kk = 0; kk < kPB / 4; ++kk)
                        c = __builtin_amdgcn_mfma_f64_16x16x4f64(L[4 * kk], u[kk], c, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = b + i0 + lg + 4 * e;
                        if (jv && i < n) col[(int64_t)i * st] = c[e];
                    }
                }
            }
        }
        __syncthreads();
    }
    // back substitution by blocks of kPB unknowns: one wavefront solves the
    // triangle (lane i holds unknown i), then all subtract the block's columns
    // from the rows above (32 lanes to a row)
    for (int k0 = (n - 1) / kPB * kPB; k0 >= 0; k0 -= kPB) {
        const int pw = min(kPB, n - k0);
        for (int e = tid; e < kPB * kPB; e += T) {
            const int i = e / kPB, c = e % kPB;
            if (i < pw && c < pw) Lp[i * kLP + c] = M[(int64_t)(k0 + i) * n + k0 + c];
        }
        __syncthreads();
        if (wave == 0) {
            const int i = min(lane, pw - 1);
            double xi = x[k0 + i];
            const double inv = 1.0 / Lp[i * kLP + i];
#pragma unroll
            for (int c = kPB - 1; c >= 0; --c) {
                if (c < pw) {
                    const double xc = __shfl(xi * inv, c, 64);
                    if (i == c) xi = xc;
                    else if (i < c) xi = fma(-Lp[i * kLP + c], xc, xi);
                }
            }
            if (lane < pw) {
                W.xb[lane] = xi;
                x[k0 + lane] = xi;
            }
        }
        __syncthreads();
        const int c = lane & 31;
        const double xc = c < pw ? W.xb[c] : 0.0;
        for (int i = 2 * wave + (lane >> 5); i < k0; i += 2 * nw) {
            double v = c < pw ? M[(int64_t)i * n + k0 + c] * xc : 0.0;
            for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if (c == 0) x[i] -= v;
        }
        __syncthreads();
    }
    const int S = a.lmax + 1;
    for (int u = tid; u < n; u += T) {
        const int4 r = a.units[u];
        a.zeta[(((int64_t)r.z * S + r.x) * S + r.y) * a.nsys + q] = x[u];
    }
}

__global__ void k_edge_mult(EdgeArgs a) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)a.n_mult * a.nsys) return;
    const int tm = (int)(t / a.nsys), q = (int)(t % a.nsys);
    const int S = a.lmax + 1;
    const int l1 = a.mult[3 * tm], l2 = a.mult[3 * tm + 1];
    const int mm = l1 < l2 ? l1 : l2;
    double v = 0.0;
    for (int m = 0; m <= mm; ++m)
        v += a.coef[(int64_t)tm * S + m] * a.zeta[(((int64_t)m * S + l1) * S + l2) * a.nsys + q];
    a.out[t] = v;
}

}  // namespace

hipError_t launch_edge_aniso(const EdgeArgs& a, hipStream_t s) {
    if (a.n < 1 || a.n > kMaxEdgeUnknowns || a.nsys < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_edge_assemble,
                       dim3((a.n + kAsmCols - 1) / kAsmCols, a.n, (a.nsys + kAsmSys - 1) / kAsmSys),
                       dim3(64 * kAsmWaves), 0, s, a);
    // a thread per row, in whole wavefronts
    const hipError_t e = allow_full_lds((const void*)k_edge_solve);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_edge_solve, dim3((unsigned)a.nsys), dim3((a.n + 63) / 64 * 64), solve_lds_bytes(a.n), s, a);
    const int64_t nm = (int64_t)a.n_mult * a.nsys;
    if (nm > 0) hipLaunchKernelGGL(k_edge_mult, dim3((unsigned)((nm + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace tpcf
