// Gaussian-smoothed RDF (forward) and its adjoint: an extension of the
// paper's rectangular-transfer-function RDF (Methods: "Descriptive,
// two-point spatial statistics") that is differentiable in the positions
// and in a scale factor of the z axis.
//
// Bin b of a pair at distance D receives w_b(D) = Phi((e_{b+1}-D)/sigma) -
// Phi((e_b-D)/sigma), evaluated through the tail of the normal distribution
// that does not cancel; only bins meeting (D - 6 sigma, D + 6 sigma) and
// pairs with D < r_max + 6 sigma count.  dw_b/dD = -(phi(t_{b+1}) -
// phi(t_b)) / sigma.
//
// Both kernels assign ions to wavefronts statically and sum in a fixed
// order, so results are reproducible bit for bit:
//  * forward: one wavefront per target; its pairs are collected, then the
//    Gaussian tail at each (pair, bin edge) is computed on its own lane, and
//    the bin terms (differences of adjacent edges) are added pair by pair to
//    the wavefront's FP64 LDS histograms; a reduction kernel sums the
//    per-wavefront rows in a fixed order;
//  * adjoint: pair lists are recomputed, not stored.  Every ion that takes
//    part in a pair (target or neighbour) gathers the derivative of L with
//    respect to its own position over its pairs in both roles, so no two
//    wavefronts write the same output and no atomics are needed.
#include "apt_pairdev.hpp"
#include "apt_smooth.hpp"

#pragma clang fp contract(off)

namespace apt {

// Dynamic LDS of a workgroup: the terms of a flush, the buffered pairs and,
// with the tables (smooth_table), the bin edges with (forward) two copies of
// the histogram or (adjoint) dL/dh; without, one copy of the histogram.
size_t smooth_lds_bytes(bool fwd, bool table, int n_bins, int n_terms) {
    size_t b = (size_t)n_terms * 8u + (size_t)kWave * (fwd ? 8u : 5u * 8u + 4u);
    if (fwd) b += (size_t)n_bins * (table ? 16u : 8u);
    else if (table) b += (size_t)n_bins * 8u;
    if (table) b += ((size_t)n_bins + 1u) * 8u;
    return b;
}

// Edge b of the bins, in FP64.
__device__ __forceinline__ double smooth_edge(double r_max, int n_bins, int b) {
    return ((double)b * r_max) / (double)n_bins;
}

__global__ void k_smooth_edges(double* E, float r_max, int n_bins) {
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b <= n_bins; b += gridDim.x * blockDim.x)
        E[b] = smooth_edge((double)r_max, n_bins, b);
}

__global__ void k_fill_f32(float* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0f;
}

// Coefficients of the tail below: (1 + 2x) exp(x^2) erfc(x) as a polynomial
// in y = (x - 3.75) / (x + 3.75), from the function's Chebyshev expansion on
// y in [-1, 1] in 80-digit arithmetic (its next coefficients are below 1e-16),
// after M. M. Shepherd and J. G. Laframboise, Math. Comp. 36 (1981) 249.
constexpr int kTailTerms = 23;
static_assert(kTailTerms % 2 == 1, "pairs of an odd and an even power beside the constant");
__device__ constexpr double kTail[kTailTerms] = {
    1.2375126308378275, -0.14024059858554525, 0.0035854154854790257, 0.08227673848999506,
    -0.10880393014244462, 0.09230432116428125, -0.05869339857664934, 0.028362277372111139,
    -0.0097465796832652621, 0.0017556261651970652, 0.00029371437804495801, -0.00029015535246077655,
    5.1646529741774162e-05, 2.2387565714911816e-05, -1.1438048033346894e-05, -9.7926257073035231e-07,
    1.7419821586224816e-06, -5.0844653786873023e-08, -2.4857126248016745e-07, 1.8790823223700481e-08,
    3.1979266716668042e-08, -1.9551358868985616e-09, -2.6231073471334759e-09};

// The tail of the normal distribution beyond |t|: 0.5 erfc(|t| / sqrt 2),
// within 7e-16 of its value for all t (exp(-t^2/2) takes the rounding of
// t^2/2 into account).  One path for all lanes, about 80 FP64 instructions;
// erfc() has several, and the lanes of a wavefront, at the edges of one
// pair's window, took all of them; through |t| / sqrt 2 it was off by up to
// 4e-14 in the far tail.
__device__ __forceinline__ double smooth_tail(double t) {
    const double x = fabs(t) * M_SQRT1_2;
    const double y = (x - 3.75) / (x + 3.75);
    // (even and odd powers in chains of their own, half as long as one; the
    // constant term, the largest, comes last, so that their roundings are a
    // tenth of its)
    const double y2 = y * y;
    double odd = kTail[kTailTerms - 2], even = kTail[kTailTerms - 1];
#pragma unroll
    for (int q = kTailTerms - 4; q >= 1; q -= 2) {
        odd = fma(odd, y2, kTail[q]);
        even = fma(even, y2, kTail[q + 1]);
    }
    const double p = fma(fma(even, y, odd), y, kTail[0]);
    const double h = 0.5 * t, z = h * t, ze = fma(h, t, -z);
    // (p over its factor, by the reciprocal that does not wait for p and a
    // correction of the quotient)
    const double d = fma(2.0, x, 1.0), r = 1.0 / d, q0 = p * r, q = fma(fma(-q0, d, p), r, q0);
    const double e = 0.5 * exp(-z) * q;
    return fma(-e, ze, e);
}

// Bins [b0, b1] that meet (D - 6 sigma, D + 6 sigma); D < r_max + 6 sigma
// guarantees that the range is not empty.
template <class EDGE>
__device__ __forceinline__ void smooth_window(const SmoothArgs& a, EDGE&& edge, double D, int* b0, int* b1) {
    const int nb = a.n_bins;
    const double lo = D - a.w6, hi = D + a.w6;
    int g = (int)floor(lo * a.inv_width);
    g = g < 0 ? 0 : (g > nb - 1 ? nb - 1 : g);
    while (g > 0 && edge(g) > lo) --g;
    while (g < nb - 1 && !(edge(g + 1) > lo)) ++g;
    int h = (int)floor(hi * a.inv_width);
    h = h < 0 ? 0 : (h > nb - 1 ? nb - 1 : h);
    while (h < nb - 1 && edge(h + 1) < hi) ++h;
    while (h > 0 && !(edge(h) < hi)) --h;
    *b0 = g;
    *b1 = h;
}

// Bin mass from the signed tails at its edges (negative below D): both edges
// above D, both below, or D inside the bin (an edge exactly at D falls to the
// last case with the same value).
__device__ __forceinline__ double smooth_mass(double slo, double shi) {
    const double vlo = fabs(slo), vhi = fabs(shi);
    return slo > 0.0 ? vlo - vhi : (shi < 0.0 ? vhi - vlo : (1.0 - vhi) - vlo);
}

__device__ __forceinline__ bool smooth_is_target(const SmoothArgs& a, uint32_t i) {
    const uint8_t l = a.lab[i];
    return (a.A == APT_ANY || l == a.A) && (a.d_bnd == nullptr || a.d_bnd[i] >= a.d_srf);
}
__device__ __forceinline__ bool smooth_is_nbr(const SmoothArgs& a, uint32_t i) {
    return a.B == APT_ANY || a.lab[i] == a.B;
}

// Bound by latency: a chain of dependent steps per ion and flush, and few
// wavefronts per SIMD beside it, limited by LDS.  So the edges (TABLE) and
// dL/dh are read from LDS, not memory, the forward keeps only what it needs
// of a pair, and where windows have at most 32 edges (`narrow`) each half of
// the wavefront takes a pair of its own, its terms never leave the registers
// and its bins go to a histogram of the half's own: 64 pairs per flush instead
// of 34, no search for a term's pair, and no pair waits for the one before.
// 1e6 ions, 200 bins, sigma 0.02 nm: 216 -> 127 us forward, 135 -> 110 us
// adjoint.
template <bool BWD, bool TABLE>
__device__ __forceinline__ void smooth_body(const SmoothArgs& a) {
    constexpr bool PAIRS2 = !BWD && TABLE;
    extern __shared__ __align__(16) uint8_t smem[];
    double* s_term = reinterpret_cast<double*>(smem);   // [n_terms] per-(pair, edge) terms
    double* s_D = s_term + a.n_terms;                   // [64] buffered pairs: distance,
    double* s_dx = s_D + kWave;                         //   adjoint: scaled displacement (candidate - ion),
    double* s_dy = s_dx + kWave;
    double* s_dz = s_dy + kWave;
    double* s_zz = s_dz + kWave;                        //   unscaled z difference,
    int* s_mul = reinterpret_cast<int*>(s_zz + kWave);  //   roles: count | (ion is the target) << 8
    // forward: histogram, [2][n_bins] with TABLE; adjoint with TABLE: dL/dh
    double* s_hist = BWD ? reinterpret_cast<double*>(s_mul + kWave) : s_D + kWave;
    double* s_E = s_hist + (size_t)a.n_bins * (PAIRS2 ? 2 : 1);
    auto edge = [&](int b) { return TABLE ? s_E[b] : a.E[b]; };

    const GridPlan P = *a.plan;
    const int l = lane_id();
    const double s = a.zscale ? *a.zscale : 1.0;
    const float rp = a.r_pre + P.eps;
    const float rp2 = rp * rp;
    if (blockIdx.x >= P.nT) return;      // (k_smooth_reduce reads the rows of the first nT)
    if (!BWD)
        for (int b = l; b < a.n_bins * (PAIRS2 ? 2 : 1); b += kWave) s_hist[b] = 0.0;
    if (TABLE) {
        for (int b = l; b <= a.n_bins; b += kWave) s_E[b] = smooth_edge(a.r_max, a.n_bins, b);
        if (BWD)
            for (int b = l; b < a.n_bins; b += kWave) s_hist[b] = a.grad_h[b];
    }
    wave_sync();
    double gs = 0.0;   // adjoint: this lane's share of dL/ds

    for (uint32_t t = blockIdx.x; t < P.nT; t += (uint32_t)a.W) {
        const uint32_t m = a.t_id[t];
        const float xm = a.xyz[3 * (size_t)m], ym = a.xyz[3 * (size_t)m + 1], zm = a.xyz[3 * (size_t)m + 2];
        const double Xm = (double)xm, Ym = (double)ym, Zm = s * (double)zm;
        const float pz = (float)Zm;
        const bool mT = BWD ? smooth_is_target(a, m) : true;
        const bool mB = BWD ? smooth_is_nbr(a, m) : false;
        double gx = 0.0, gy = 0.0, gz = 0.0;
        int nh = 0;   // buffered pairs (wave-uniform)

        auto flush = [&]() {
            wave_sync();
            // per pair: its window's bins b0 .. b0 + mh - 1 and their mh + 1
            // edges; the Gaussian tail (forward) or density (adjoint) is
            // evaluated once per edge, on its own lane, and shared by the
            // two bins that meet there
            int b0 = 0, mh = 0, me = 0;
            if (l < nh) {
                int b1;
                smooth_window(a, edge, s_D[l], &b0, &b1);
                mh = b1 - b0 + 1;
                me = mh + 1;
            }
            // the adjoint's share of pair l, given its dL/dD
            auto gather = [&](double g) {
                const double D = s_D[l];
                if (D != 0.0) {
                    const int mul = s_mul[l];
                    const double cnt = (double)(mul & 0xff);
                    gx -= cnt * (g * (s_dx[l] / D));
                    gy -= cnt * (g * (s_dy[l] / D));
                    gz -= cnt * ((g * (s_dz[l] / D)) * s);
                    if (mul >> 8) {
                        const double zz = s_zz[l];
                        gs += g * s * zz * zz / D;
                    }
                }
            };
            if (TABLE && a.narrow) {
                // every window has at most 32 edges: half h of the wavefront
                // takes the edges of one pair, two pairs each per step.
                // Forward: its bins go to the half's own histogram (a
                // wavefront's LDS accesses happen in program order); adjoint:
                // their sum is the pair's dL/dD
                const int half = l >> 5, ln = l & 31;
                double* hist = s_hist + (BWD ? 0 : (size_t)half * (size_t)a.n_bins);
                for (int h0 = 0; h0 < nh; h0 += 4) {
                    double u[2];
                    int bin[2], cnt[2];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int h = h0 + 2 * k + half, hc = h < nh ? h : 0;
                        bin[k] = __shfl(b0, hc, kWave) + ln;
                        const int edges = __shfl(me, hc, kWave);
                        cnt[k] = h < nh ? edges - 1 : 0;      // bins of the window
                        const double t = (edge(ln < edges ? bin[k] : bin[k] - ln) - s_D[hc]) / a.sigma;
                        if (BWD) {
                            u[k] = exp(-0.5 * t * t) / sqrt(2.0 * M_PI);
                        } else {
                            const double v = smooth_tail(t);
                            u[k] = t >= 0.0 ? v : -v;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const double next = __shfl_down(u[k], 1, kWave);   // the bin's upper edge
                        if (!BWD) {
                            if (ln < cnt[k]) hist[bin[k]] += smooth_mass(u[k], next);
                        } else {
                            double g = ln < cnt[k] ? hist[bin[k]] * (-(next - u[k]) / a.sigma) : 0.0;
#pragma unroll
                            for (int d = 16; d >= 1; d >>= 1) g += __shfl_xor(g, d, kWave);
                            if (ln == 0 && cnt[k] > 0) s_term[h0 + 2 * k + half] = g;
                        }
                    }
                }
                wave_sync();
                if (BWD && l < nh) gather(s_term[l]);
                wave_sync();
                nh = 0;
                return;
            }
            const uint32_t inc = wave_incl_scan((uint32_t)me);
            const uint32_t tot = readlane(inc, kWave - 1);
            const uint32_t off = inc - (uint32_t)me;
            for (uint32_t c0 = 0; c0 < tot; c0 += kWave) {
                const uint32_t v = c0 + (uint32_t)l;
                int h = -1, ev = 0;
                const int r0 = __popcll(__ballot(inc <= c0));   // first pair ending after c0
                for (int rr = r0; rr < nh; ++rr) {
                    const uint32_t o = readlane(off, rr);
                    if (o >= c0 + kWave) break;
                    const uint32_t ln = (uint32_t)readlane(me, rr);
                    if (v >= o && v < o + ln) {
                        h = rr;
                        ev = readlane(b0, rr) + (int)(v - o);
                    }
                }
                if (h >= 0) {
                    const double t = (edge(ev) - s_D[h]) / a.sigma;
                    if (!BWD) {
                        // the tail beyond |t|, negated when t < 0
                        const double u = smooth_tail(t);
                        s_term[v] = t >= 0.0 ? u : -u;
                    } else {
                        s_term[v] = exp(-0.5 * t * t) / sqrt(2.0 * M_PI);
                    }
                }
            }
            wave_sync();
            if (!BWD) {
                auto mass = [&](uint32_t o) { return smooth_mass(s_term[o], s_term[o + 1]); };
                if (PAIRS2) {
                    // two pairs at a time, pair by pair within a half (the
                    // wavefront's LDS accesses happen in program order)
                    const int half = l >> 5, ln32 = l & 31;
                    double* hist = s_hist + (size_t)half * (size_t)a.n_bins;
                    for (int h0 = 0; h0 < nh; h0 += 2) {
                        const int h = h0 + half < nh ? h0 + half : h0;
                        const uint32_t o = (uint32_t)__shfl((int)off, h, kWave);
                        const int bb = __shfl(b0, h, kWave);
                        const int ln = h0 + half < nh ? __shfl(mh, h, kWave) : 0;
                        for (int q = ln32; q < ln; q += 32) hist[bb + q] += mass(o + (uint32_t)q);
                    }
                } else {
                    // pair by pair (windows of different pairs overlap)
                    for (int h = 0; h < nh; ++h) {
                        const uint32_t o = readlane(off, h);
                        const int ln = readlane(mh, h), bb = readlane(b0, h);
                        for (int q = l; q < ln; q += kWave) s_hist[bb + q] += mass(o + (uint32_t)q);
                        wave_sync();
                    }
                }
            } else if (l < nh) {
                double g = 0.0;
                for (int q = 0; q < mh; ++q) {
                    const double plo = s_term[off + (uint32_t)q], phi = s_term[off + (uint32_t)q + 1];
                    g += (TABLE ? s_hist[b0 + q] : a.grad_h[b0 + q]) * (-(phi - plo) / a.sigma);
                }
                gather(g);
            }
            wave_sync();
            nh = 0;
        };

        enumerate(P, a.cell_start, a.bpos, xm, ym, pz, a.r_pre, [&](bool valid, float4 c) {
            const uint32_t o = __builtin_bit_cast(uint32_t, c.w);
            bool hit = false;
            double D = 0.0, dX = 0.0, dY = 0.0, dZ = 0.0, zz = 0.0;
            int mul = 0;
            if (valid && o != m) {
                const float fx = c.x - xm, fy = c.y - ym, fz = c.z - pz;
                if (fx * fx + fy * fy + fz * fz < rp2) {
                    int t1 = 1, t2 = 0;
                    if (BWD) {
                        t1 = (mT && smooth_is_nbr(a, o)) ? 1 : 0;
                        t2 = (mB && smooth_is_target(a, o)) ? 1 : 0;
                    }
                    if (t1 + t2 > 0) {
                        const float zo = a.xyz[3 * (size_t)o + 2];
                        dX = (double)c.x - Xm;
                        dY = (double)c.y - Ym;
                        dZ = s * (double)zo - Zm;
                        D = sqrt((dX * dX + dY * dY) + dZ * dZ);
                        hit = D < a.cut;
                        mul = (t1 + t2) | (t1 << 8);
                        zz = (double)zo - (double)zm;
                    }
                }
            }
            uint64_t bal = __ballot(hit);
            while (bal) {
                const int room = a.hcap - nh;
                const bool mine = (bal >> l) & 1ull;
                const int rank = __popcll(bal & lanemask_lt());
                const uint64_t take = __ballot(mine && rank < room);
                if ((take >> l) & 1ull) {
                    const int slot = nh + rank;
                    s_D[slot] = D;
                    if (BWD) {
                        s_dx[slot] = dX;
                        s_dy[slot] = dY;
                        s_dz[slot] = dZ;
                        s_zz[slot] = zz;
                        s_mul[slot] = mul;
                    }
                }
                nh += __popcll(take);
                bal &= ~take;
                if (nh == a.hcap) flush();
            }
        });
        if (nh > 0) flush();

        if (BWD) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                gx += __shfl_xor(gx, d, kWave);
                gy += __shfl_xor(gy, d, kWave);
                gz += __shfl_xor(gz, d, kWave);
            }
            if (l == 0) {
                a.grad_xyz[3 * (size_t)m] = (float)gx;
                a.grad_xyz[3 * (size_t)m + 1] = (float)gy;
                a.grad_xyz[3 * (size_t)m + 2] = (float)gz;
            }
        }
    }

    if (!BWD) {
        wave_sync();
        double* row = a.part + (size_t)blockIdx.x * (size_t)a.n_bins;
        for (int b = l; b < a.n_bins; b += kWave) row[b] = PAIRS2 ? s_hist[b] + s_hist[a.n_bins + b] : s_hist[b];
    } else {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) gs += __shfl_xor(gs, d, kWave);
        if (l == 0) a.part[blockIdx.x] = gs;
    }
}

// (three wavefronts per SIMD without spills are faster than four: 129 / 137 us)
template <bool TABLE>
__global__ __launch_bounds__(kWave, 3) void k_smooth_fwd(SmoothArgs a) {
    smooth_body<false, TABLE>(a);
}
template <bool TABLE>
__global__ __launch_bounds__(kWave, 4) void k_smooth_bwd(SmoothArgs a) {
    smooth_body<true, TABLE>(a);
}
template __global__ void k_smooth_fwd<false>(SmoothArgs);
template __global__ void k_smooth_fwd<true>(SmoothArgs);
template __global__ void k_smooth_bwd<false>(SmoothArgs);
template __global__ void k_smooth_bwd<true>(SmoothArgs);

// out[b] = sum over the first min(W, nT) per-wavefront rows of part[w][b], in
// a fixed order (the same result on every run): kReduceGroups consecutive row
// ranges, each summed in row order, then the range sums pairwise.  Workgroup:
// BINS bins x as many ranges as make kReduceBlock threads.  Few bins: 4, so that
// 200 of them fill 50 workgroups of 256 ranges each (64 bins x 16 ranges were four,
// 62 us); many, whose rows are few: 64, a row's as a whole line (4000 bins, 524
// rows: 7.0 us, 4 bins a workgroup 14.0).
template <int BINS>
__global__ __launch_bounds__(kReduceBlock) void k_smooth_reduce(SmoothReduceArgs a) {
    constexpr int kReduceBins = BINS, kReduceGroups = kReduceBlock / BINS;
    __shared__ double s_p[kReduceGroups][kReduceBins];
    const int tb = threadIdx.x % kReduceBins, g = threadIdx.x / kReduceBins;
    const int b = blockIdx.x * kReduceBins + tb;
    const uint32_t nT = a.plan->nT;
    const int64_t W = nT < (uint32_t)a.W ? (int64_t)nT : (int64_t)a.W;
    const int w0 = (int)(W * g / kReduceGroups), w1 = (int)(W * (g + 1) / kReduceGroups);
    double acc = 0.0;
    if (b < a.n_bins) {
        const double* col = a.part + (size_t)b;
        int w = w0;
        for (; w + 8 <= w1; w += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = col[(size_t)(w + u) * (size_t)a.n_bins];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += v[u];
        }
        for (; w < w1; ++w) acc += col[(size_t)w * (size_t)a.n_bins];
    }
    s_p[g][tb] = acc;
    for (int step = 1; step < kReduceGroups; step *= 2) {
        __syncthreads();
        if (g % (2 * step) == 0) s_p[g][tb] += s_p[g + step][tb];
    }
    if (g == 0 && b < a.n_bins) a.out[b] = s_p[0][tb];
}

template __global__ void k_smooth_reduce<4>(SmoothReduceArgs);
template __global__ void k_smooth_reduce<64>(SmoothReduceArgs);

}  // namespace apt
