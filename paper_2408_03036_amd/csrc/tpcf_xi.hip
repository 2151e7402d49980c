// Pair counts of the anisotropic 2PCF (arXiv:2408.03036, Sec. 4.1): DD(r, mu)
// over ordered pairs, r the minimum-image separation and mu = dz / r the
// cosine to the line of sight z, and the Legendre multipoles of the natural
// estimator DD / RR - 1 with analytic periodic RR (eq. (xi_natest),
// (xi_meas_leg)).
//
//  k_xi_count     persistent workgroups over the work items of the neighbour
//                 grid (up to 16 primaries of one cell). Every unordered pair
//                 is tested once: the stencil is halved (cell offsets that are
//                 positive in (x, y, z) order, plus the home cell), and a pair
//                 with its neighbour outside the home cell adds both ordered
//                 pairs, (p, j) at mu and (j, p) at -mu, whose separation is
//                 exactly the negated one. Home-cell pairs are seen from both
//                 ends and add one each. The half stencil is staged in LDS in
//                 the home cell's frame, cut to the reach of the item's
//                 primaries, and tested against them; each hit increments
//                 uint32 counters of a workgroup histogram in LDS, flushed to
//                 the 64-bit global counts once at the end (or earlier when a
//                 counter could overflow). Bound by the instructions of the
//                 tests (81 % of the vector issue slots). 720,000 points, 30 x
//                 200 bins: 2.75 ms, 7.9e11 ordered pairs/s. It was 5.14 ms:
//                 the near-edge pairs evaluated after each tile cost 1.1 ms of
//                 that, a second t and a square root besides the reciprocal
//                 0.9, tiles of 128 uncut candidates 0.4. Items are taken from eight queues, one per
//                 contiguous eighth of the cells, so that the workgroups of
//                 one XCD share neighbours in that XCD's L2; a workgroup
//                 whose queue is empty moves on to the next one. In
//                 single-cell mode (small boxes) the stencil is the whole box
//                 and every ordered pair is tested.
//  k_xi_finalize  xi_l(r_b) = sum_k c_lk (DD(b, k) / RR_b - 1).
//
// Bin decisions equal those of an exact double-precision evaluation:
// r^2 = dx*dx + dy*dy + dz*dz against the squared edges, and
// k = floor((dz / sqrt(r^2) + 1) * nmu / 2) clamped to [0, nmu - 1], every
// operation rounded in double. The FP32 test sends every pair within a
// rounding-error bound of an r or mu edge to that exact evaluation.
#include <algorithm>

#include "tpcf_cells.h"

namespace tpcf {

namespace {

constexpr int kXW = 4;                     // wavefronts per workgroup
constexpr int kXG = kItemPrims / kXW;      // primaries per wavefront
constexpr int kXLoad = 256;                // candidates staged at a time (one per thread)
constexpr int kXTile = kXLoad + 64;        // room of a tile: what staging keeps, after up to 63 carried over
constexpr int kXUT = kXTile / 64;          // tile candidates per lane
constexpr int kXQueue = 96;                // near-edge pairs an item can defer
constexpr int kQueues = 8;
constexpr int kQueueStride = 32;           // ints between queue cursors (128 bytes)
static_assert(kXG * kXW == kItemPrims, "item size");

// Exact bin indices b * nmu + k of the pair (p, j) and of the reversed pair
// (j, p), or -1 (outside the shells, or zero separation). The reversed pair's
// separation is exactly the negated one (rounding and rint are odd), so its
// mu is exactly -mu. Periodic shifts come from the stencil code (equal to the
// minimum image inside the shells) or, in single-cell mode, from rint.
template <bool SINGLE>
__device__ __forceinline__ int2 exact_xi_t(const double4 P, const double4 Q, int wbits, double box, int nb,
                                        const double* e2, int nmu, double hmu) {
#pragma clang fp contract(off)
    double dx = Q.x - P.x, dy = Q.y - P.y, dz = Q.z - P.z;
    if constexpr (SINGLE) {
        dx -= box * rint(dx / box);
        dy -= box * rint(dy / box);
        dz -= box * rint(dz / box);
    } else {
        dx += wrap_shift(wbits, 0, box);
        dy += wrap_shift(wbits, 1, box);
        dz += wrap_shift(wbits, 2, box);
    }
    double r2 = dx * dx;
    r2 += dy * dy;
    r2 += dz * dz;
    if (r2 == 0.0 || r2 < e2[0] || r2 >= e2[nb]) return make_int2(-1, -1);
    int b = 0;
    while (b + 1 < nb && r2 >= e2[b + 1]) ++b;
    const double r = sqrt(r2);
    const double mu = dz / r;
    auto kbin = [&](double m) {
        const int k = (int)floor((m + 1.0) * hmu);
        return k < 0 ? 0 : (k > nmu - 1 ? nmu - 1 : k);
    };
    return make_int2(b * nmu + kbin(mu), b * nmu + kbin(-mu));
}

// Inlined, and evaluated after a tile's tests for the pairs they marked: as
// a call inside the test loop it would cost the kernel the callee-saved
// registers and make every tile wait for its pending loads.
template <bool SINGLE>
__device__ __forceinline__ int2 exact_xi_pair(const double4* pd, int64_t p, uint32_t entry, uint32_t mask,
                                           int cshift, int cx, int cy, int cz, int k, int nc, double box,
                                           int nb, const double* e2, int nmu, double hmu) {
    const int64_t j = (int64_t)(entry & mask);
    const int wb = SINGLE ? 0 : wrap_bits_of((int)(entry >> cshift), cx, cy, cz, k, nc);
    return exact_xi_t<SINGLE>(pd[p], pd[j], wb, box, nb, e2, nmu, hmu);
}

// One candidate being staged: its point, its piece's shift and its index.
struct XStaged {
    int r;
    float4 q;
    float sx, sy, zo;
    int code;
    uint32_t j;
    bool ok;
};

__device__ __forceinline__ void xstage_load(XStaged& st, const Pieces& S, int total, int g, const float4* pf) {
    st.ok = g < total;
    if (st.ok) {
        int r = st.r;
        while (S.pref[r + 1] <= g) ++r;
        st.r = r;
        const float4 rc = S.rec[r];
        st.j = (uint32_t)(g + __float_as_int(rc.x));
        st.sx = rc.y;
        st.sy = rc.z;
        st.zo = rc.w;
        st.code = S.code[r] & 0xffff;
        st.q = pf[st.j];
    }
}

// A staged candidate in the home cell's frame, its list entry (index | stencil
// code << cshift) in w.
template <bool SINGLE>
__device__ __forceinline__ float4 xstage_point(const XStaged& st, int cshift, float hf) {
    if constexpr (SINGLE) {
        return make_float4(st.q.x, st.q.y, st.q.z, __uint_as_float(st.j));
    } else {
        const int oz = (int)(st.q.w + st.zo);
        return make_float4(st.q.x + st.sx, st.q.y + st.sy, fmaf((float)oz, hf, st.q.z),
                           __uint_as_float(st.j | ((uint32_t)(st.code + oz) << cshift)));
    }
}

struct XiLds {
    double e2[kMaxBins + 1];
    float e2f[kMaxBins + 1];
    float guard[kMaxBins + 1];
    ItemBox box;   // of the item's primaries
    int kept[3];   // candidates that staging added to a tile, in rotation
    int item;
    int nq;        // near-edge pairs of the item: list entry and primary
    uint32_t qentry[kXQueue];
    uint8_t qprim[kXQueue];
};

__host__ __device__ inline size_t xi_hist_offset() { return (sizeof(XiLds) + 15) / 16 * 16; }

template <bool SINGLE, bool UNIFORM>
__global__ void __launch_bounds__(64 * kXW) k_xi_count(XiArgs a) {
    extern __shared__ unsigned char smem[];
    XiLds& X = *reinterpret_cast<XiLds*>(smem);
    const int nh = a.nb * a.nmu;
    size_t off = xi_hist_offset();
    uint32_t* hist = reinterpret_cast<uint32_t*>(smem + off);
    off += ((size_t)nh * sizeof(uint32_t) + 15) / 16 * 16;
    float4* tiles = reinterpret_cast<float4*>(smem + off);
    off += sizeof(float4) * 2 * kXTile;
    Pieces S = pieces_view(smem + off, a.npmax);

    for (int i = threadIdx.x; i <= a.nb; i += blockDim.x) {
        X.e2[i] = a.e2[i];
        X.e2f[i] = a.e2f[i];
        X.guard[i] = a.guard[i];
    }
    for (int i = threadIdx.x; i < nh; i += blockDim.x) hist[i] = 0u;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id();
    const int cshift = 32 - a.g.code_bits;
    const uint32_t mask = a.g.idx_mask;
    const uint32_t home_code = (uint32_t)a.home_code;
    const unsigned nbu = (unsigned)a.nb;
    const float ne0 = -a.e0f * a.inv_dr, half_nb = 0.5f * (float)a.nb;
    const int top = a.nmu - 1;
    const int64_t per = (a.nitems + kQueues - 1) / kQueues;
    int qi = 0;                       // queues visited (thread 0)
    const int home = blockIdx.x % kQueues;
    unsigned long long bound = 0;     // upper bound of the hits since the last flush

    auto flush = [&]() {
        for (int i = threadIdx.x; i < nh; i += blockDim.x) {
            const uint32_t v = hist[i];
            if (v) {
                atomicAdd(a.counts + i, (unsigned long long)v);
                hist[i] = 0u;
            }
        }
    };

    for (;;) {
        if (threadIdx.x == 0) {
            int item = -1;
            while (qi < kQueues) {
                const int q = (home + qi) % kQueues;
                const int64_t lo = (int64_t)q * per, hi = min(lo + per, a.nitems);
                if (lo < hi) {
                    const int v = atomicAdd(a.queue + q * kQueueStride, 1);
                    if (lo + v < hi) {
                        item = (int)(lo + v);
                        break;
                    }
                }
                ++qi;
            }
            X.item = item;
        }
        __syncthreads();
        const int item = X.item;
        if (item < 0) break;

        const int gc = a.item_cell[item];
        const int64_t first = (int64_t)a.cell_start[gc] + (int64_t)(item - a.item_start[gc]) * kItemPrims;
        const int64_t last = min(first + kItemPrims, (int64_t)a.cell_start[gc + 1]);
        const int cz = gc % a.g.nc, cy = (gc / a.g.nc) % a.g.nc, cx = gc / (a.g.nc * a.g.nc);
        if (wave == 0) {
            // candidates cut to the reach of the item's primaries, as in the
            // 3PCF binning (a pair within the outer edge keeps its candidate)
            if constexpr (SINGLE) {
                build_pieces(S, a, 0, 0, 0, 0);
            } else {
                const ItemBox box = item_box(a.pf, first, last, a.reach2);
                build_pieces<true>(S, a, 0, cx, cy, cz, box);
                if (lane == 0) X.box = box;
            }
            if (lane < 3) X.kept[lane] = 0;
            if (lane == 0) X.nq = 0;
        }
        __syncthreads();
        const int total = __builtin_amdgcn_readfirstlane(S.pref[*S.n]);
        const int rem = (int)(last - first);
        const int ng = rem > wave ? (rem - wave + kXW - 1) / kXW : 0;

        // a counter may reach at most twice the tests of the items since the last flush
        bound += 2ull * (unsigned long long)rem * (unsigned long long)total;
        if (bound > 0x7fffffffull) {
            flush();
            __syncthreads();
            bound = 2ull * (unsigned long long)rem * (unsigned long long)total;
        }

        float px[kXG], py[kXG], pz[kXG];
#pragma unroll
        for (int g = 0; g < kXG; ++g) {
            px[g] = py[g] = pz[g] = 0.f;
            if (g < ng) {
                // uniform over the wavefront: scalar registers
                const float4 P = a.pf[first + wave + kXW * g];
                px[g] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(P.x)));
                py[g] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(P.y)));
                pz[g] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(P.z)));
            }
        }

        // The first kXLoad / 64 wavefronts stage, a candidate per thread: its
        // load is issued before a tile's tests, and after them it joins the
        // next tile if it lies within reach of the box of the item's primaries.
        // The pieces are cut column by column, so about a quarter of their
        // candidates do not: dropping those here, once, saves testing each
        // against every primary. A tile's tests take whole wavefronts of
        // candidates; the rest of the tile moves to the next one, but after
        // the last.
        XStaged st;
        st.r = 0;
        const bool stager = wave < kXLoad / 64;
        auto join = [&](float4* tile, int* kept, int carried) {
            const float4 v = xstage_point<SINGLE>(st, cshift, a.g.hf);
            bool keep = st.ok;
            if constexpr (!SINGLE) {
                const ItemBox& B = X.box;
                const float gx = fmaxf(0.f, fmaxf(v.x - B.xhi, B.xlo - v.x));
                const float gy = fmaxf(0.f, fmaxf(v.y - B.yhi, B.ylo - v.y));
                const float gz = fmaxf(0.f, fmaxf(v.z - B.zhi, B.zlo - v.z));
                keep = keep && fmaf(gx, gx, fmaf(gy, gy, gz * gz)) <= a.reach2;
            }
            const unsigned long long kb = __ballot(keep);
            int at = 0;
            if (lane == 0) at = atomicAdd(kept, __popcll(kb));
            at = __builtin_amdgcn_readfirstlane(at);
            if (keep) tile[carried + at + __popcll(kb & ((1ull << lane) - 1ull))] = v;
        };
        // an exact pair (rare)
        auto exact = [&](int64_t p, uint32_t entry) {
            const bool both = !SINGLE && (entry >> cshift) != home_code;
            const int2 idx = exact_xi_pair<SINGLE>(a.pd, p, entry, mask, cshift, cx, cy, cz, a.g.k, a.g.nc, a.g.box,
                                                   a.nb, X.e2, a.nmu, a.hmu);
            if (idx.x >= 0) {
                atomicAdd(hist + idx.x, 1u);
                if (both) atomicAdd(hist + idx.y, 1u);
            }
        };
        int next = 0;  // candidates staged
        if (stager) {
            xstage_load(st, S, total, (int)threadIdx.x, a.pf);
            join(tiles, X.kept, 0);
        }
        next = kXLoad;
        __syncthreads();
        int buf = 0, rot = 0, carried = 0;
        for (;;) {
            const float4* cur = tiles + buf * kXTile;
            const int have = carried + __builtin_amdgcn_readfirstlane(X.kept[rot]);
            const bool more = next < total;
            // whole wavefronts of candidates, or all of them after the last load
            const int nt = more ? have & ~63 : have;
            if (more && stager) xstage_load(st, S, total, next + (int)threadIdx.x, a.pf);
            if (threadIdx.x == 0) X.kept[rot == 0 ? 2 : rot - 1] = 0;  // read by all before the last barrier
            uint32_t nearbits = 0;
            static_assert(kXUT * kXG <= 32, "near-edge marks");
#pragma unroll
            for (int u = 0; u < kXUT; ++u) {
                const int i = u * 64 + lane;
                if (i >= nt) break;
                const float4 q = cur[i];
                const uint32_t entry = __float_as_uint(q.w);
                // neighbours outside the home cell stand for both ordered pairs
                const bool both = !SINGLE && (entry >> cshift) != home_code;
                // the separations of the wavefront's primaries, then their tests
                float r2v[kXG], dzv[kXG];
#pragma unroll
                for (int g = 0; g < kXG; ++g) {
                    float dx = q.x - px[g], dy = q.y - py[g], dz = q.z - pz[g];
                    if constexpr (SINGLE) {
                        dx -= a.g.boxf * rintf(dx * a.inv_boxf);
                        dy -= a.g.boxf * rintf(dy * a.inv_boxf);
                        dz -= a.g.boxf * rintf(dz * a.inv_boxf);
                    }
                    r2v[g] = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                    dzv[g] = dz;
                }
                // bins of unequal width: every edge, read once, against all the
                // primaries; then only the two edges of the bin can be near,
                // since the one in between is nearer than any other, and a
                // separation clear of its own edges is on the right side of
                // all of them (with the guard of every edge tested in the
                // loop, 20,011 points in 17 log bins took 138 us, now 109)
                int bbv[kXG];
                if constexpr (!UNIFORM) {
#pragma unroll
                    for (int g = 0; g < kXG; ++g) bbv[g] = -1;
                    for (int e = 0; e <= a.nb; ++e) {
                        const float ef = X.e2f[e];
#pragma unroll
                        for (int g = 0; g < kXG; ++g) bbv[g] += r2v[g] >= ef;
                    }
                }
#pragma unroll
                for (int g = 0; g < kXG; ++g) {
                    if (g >= ng) break;
                    // 1 / r, of at least the smallest normal r^2: with r = 0 the
                    // guard bands send the pair to the exact path
                    const float rinv = __builtin_amdgcn_rsqf(fmaxf(r2v[g], 1.17549435e-38f));
                    int bb;
                    bool near;
                    if constexpr (UNIFORM) {
                        // the shells in bin units, widened by a guard band that
                        // lies inside the one of the near test (a separation
                        // whose square overflows has u = NaN, and is outside)
                        const float uu = fmaf(r2v[g] * rinv, a.inv_dr, ne0);
                        if (!(fabsf(uu - half_nb) <= a.reach_u)) continue;
                        near = fabsf(__builtin_amdgcn_fractf(uu) - 0.5f) > 0.5f - a.delta;
                        bb = (int)uu;
                    } else {
                        bb = bbv[g];
                        const int lo = max(bb, 0), hi = min(bb + 1, a.nb);
                        near = fabsf(r2v[g] - X.e2f[lo]) < X.guard[lo] || fabsf(r2v[g] - X.e2f[hi]) < X.guard[hi];
                        if (!near && (unsigned)bb >= nbu) continue;
                    }
                    // t = (mu + 1) nmu / 2 in FP32 with its error bound. The
                    // reversed pair's t is nmu minus this one, so a t clear of
                    // the integers puts it in the mirrored bin.
                    const float tt = fmaf(dzv[g] * rinv, a.hmu_f, a.hmu_f);
                    const float gt = fmaf(a.gmu_a, rinv, a.gmu_b);
                    near |= fabsf(__builtin_amdgcn_fractf(tt) - 0.5f) + gt > 0.5f;
                    // A pair near an edge is put on the item's list here, or
                    // marked when that is full.
                    if (near) {
                        const int at = atomicAdd(&X.nq, 1);
                        if (at < kXQueue) {
                            X.qentry[at] = entry;
                            X.qprim[at] = (uint8_t)(wave + kXW * g);
                        } else {
                            nearbits |= 1u << (u * kXG + g);
                        }
                    } else {
                        const int row = bb * a.nmu, k = min(max((int)tt, 0), top);
                        atomicAdd(hist + row + k, 1u);
                        if (both) atomicAdd(hist + row + (top - k), 1u);
                    }
                }
            }
            if (more) {
                const int left = have - nt;
                float4* nxt = tiles + (buf ^ 1) * kXTile;
                if (wave == kXW - 1 && lane < left) nxt[lane] = cur[nt + lane];
                if (stager) join(nxt, X.kept + (rot == 2 ? 0 : rot + 1), left);
            }
            // the marked pairs (more than an item can list: lattices), exactly
            if (__ballot(nearbits != 0u) != 0ull) {
#pragma unroll
                for (int g = 0; g < kXG; ++g) {
                    uint32_t m = nearbits & (0x11111111u << g);  // bits u kXG + g
                    while (m != 0u) {
                        const int bit = __builtin_ctz(m);
                        m &= m - 1u;
                        exact(first + wave + kXW * g, __float_as_uint(cur[(bit / kXG) * 64 + lane].w));
                    }
                }
            }
            __syncthreads();
            if (!more) break;
            carried = have - nt;
            next += kXLoad;
            buf ^= 1;
            rot = rot == 2 ? 0 : rot + 1;
        }
        // The item's near-edge pairs, exactly, a lane each. (Evaluated tile by
        // tile, one or two lanes at a time, their FP64 arithmetic and their
        // gathers stalled a third of the tiles.)
        const int nq = min(X.nq, kXQueue);
        for (int t = threadIdx.x; t < nq; t += 64 * kXW) exact(first + X.qprim[t], X.qentry[t]);
    }
    flush();
}

// A wavefront per (l, b), its lanes over the mu bins, then a butterfly (one
// thread per sum waited for 200 loads in turn: 23 us at nmu 200).
__global__ void __launch_bounds__(64) k_xi_finalize(XiFinalArgs a) {
    const int t = blockIdx.x, lane = lane_id();
    const int i = t / a.nb, b = t % a.nb;
    const double inv = 1.0 / a.rr[b];
    double s = 0.0;
#pragma unroll 4
    for (int k = lane; k < a.nmu; k += 64) {
        const double xi = (double)a.counts[(size_t)b * a.nmu + k] * inv - 1.0;
        s = fma(a.coef[(size_t)i * a.nmu + k], xi, s);
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) a.out[t] = s;
}

template <bool SINGLE, bool UNIFORM>
hipError_t launch_xi_variant(const XiArgs& a, hipStream_t s) {
    const size_t lds = xi_lds_bytes(a.nb, a.nmu, a.npmax);
    if (lds > 64 * 1024) {
        hipError_t e = allow_full_lds((const void*)k_xi_count<SINGLE, UNIFORM>);
        if (e != hipSuccess) return e;
    }
    int dev = 0, ncu = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_xi_count<SINGLE, UNIFORM>, 64 * kXW,
                                                          lds)) != hipSuccess)
        return e;
    int64_t grid = (int64_t)std::max(per_cu, 1) * std::max(ncu, 1);
    grid = std::min<int64_t>(grid, (a.nitems + 1) / 2 * 2);
    grid = std::max<int64_t>((grid + kQueues - 1) / kQueues * kQueues, kQueues);
    hipLaunchKernelGGL((k_xi_count<SINGLE, UNIFORM>), dim3((unsigned)grid), dim3(64 * kXW), lds, s, a);
    return hipGetLastError();
}

}  // namespace

size_t xi_lds_bytes(int nb, int nmu, int npmax) {
    return xi_hist_offset() + ((size_t)nb * nmu * sizeof(uint32_t) + 15) / 16 * 16 +
           sizeof(float4) * 2 * kXTile + pieces_lds_bytes(npmax);
}

hipError_t launch_xi_count(const XiArgs& a, hipStream_t s) {
    if (a.nitems <= 0) return hipSuccess;
    if (a.g.single) return a.uniform ? launch_xi_variant<true, true>(a, s) : launch_xi_variant<true, false>(a, s);
    return a.uniform ? launch_xi_variant<false, true>(a, s) : launch_xi_variant<false, false>(a, s);
}

hipError_t launch_xi_finalize(const XiFinalArgs& a, hipStream_t s) {
    const int n = a.n_ell * a.nb;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_xi_finalize, dim3(n), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace tpcf
