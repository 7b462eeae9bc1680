// Ion-to-edge distancing (paper, Methods: "Ion-to-edge distancing";
// Supplementary: "Triangle filtering methods for ion-to-edge distancing").
//
// The paper filters the candidate triangles of each ion with a coarse
// distance map and an R-tree.  Here every triangle is covered by pieces (a
// large triangle is cut into slices parallel to its shortest edge, each
// slice into parts about as wide as it is high) that are binned once by
// their centroid into a uniform grid over the ions' bounding box.  A piece
// lies within its radius of its centroid, and the distance is always taken
// to the whole triangle; the pieces keep long slivers (a hull's cap fans)
// from widening every search.
//
// Ions are taken in the cell order of their own binning, 64 consecutive ones
// per wavefront, cut at the end of a cell row so that they are one compact
// group.  The search is the group's, not each ion's: the rows of the
// triangle grid that the group's box grown by the reach meets (one pair of
// offsets per row tells whether it holds anything, so a group deep inside the
// specimen ends after a few loads), the piece nearest to the box's centre,
// and from it the reach that certainly holds the nearest triangle of every
// ion of the group.  The pieces within that reach go through an LDS list,
// and every lane tests each of them against its own ion with an FP32 lower
// bound (below); the few that survive get the exact distance, FP64 on the
// stored FP32 values: the plane distance when the perpendicular's foot lies
// inside the triangle (all three barycentric weights of the foot, in
// dot-product form, non-negative), else the nearest of the three edges.
#include "apt_edge.hpp"

namespace apt {

// the accumulators of the triangle sizes
__global__ void k_edge_zero(EdgeArgs a) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    a.tp->rmax_bits = 0u;
    a.tp->cmax_bits = 0u;
    a.tp->n_valid = 0u;
    a.tp->r_sum = 0.0;
    for (int j = 0; j < kPieceSizes; ++j) a.tp->pieces_at[j] = 0ull;
    a.tp->piece_ctr = 0u;
    a.tp->piece_rmax_bits = 0u;
    a.tp->piece_cap = a.piece_cap;
}

// FP32 centroid and radius of N points, the radius about the centroid as
// stored and widened for its own rounding (a convex piece is its corners'
// hull, so it lies within it)
template <int N>
__device__ __forceinline__ float4 centroid_radius(const float* q) {
    float cx = q[0], cy = q[1], cz = q[2];
#pragma unroll
    for (int k = 1; k < N; ++k) {
        cx += q[3 * k];
        cy += q[3 * k + 1];
        cz += q[3 * k + 2];
    }
    cx /= (float)N;
    cy /= (float)N;
    cz /= (float)N;
    float r2 = 0.0f;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const float dx = q[3 * k] - cx, dy = q[3 * k + 1] - cy, dz = q[3 * k + 2] - cz;
        r2 = fmaxf(r2, dx * dx + dy * dy + dz * dz);
    }
    return make_float4(cx, cy, cz, sqrtf(r2) * 1.00001f + 1e-6f);
}

// (few, large workgroups, each with one atomic per sum: a wavefront's own
// atomics on these few addresses ran one after the other, 59 us for 1e5
// triangles in 1600 wavefronts)
__global__ __launch_bounds__(kEdgePrepBlock) void k_edge_prep(EdgeArgs a) {
    __shared__ uint32_t s_nv, s_rm, s_cm;
    __shared__ double s_rs[kEdgePrepBlock / kWave];
    if (threadIdx.x == 0) s_nv = s_rm = s_cm = 0u;
    __syncthreads();
    uint32_t nv = 0;
    float rm = 0.0f, cm = 0.0f;
    double rs = 0.0;
    for (uint32_t t = blockIdx.x * kEdgePrepBlock + threadIdx.x; t < a.n_tri; t += gridDim.x * kEdgePrepBlock) {
        const float* T = a.tri + 9 * (size_t)t;
        float v[9], m = 0.0f;
        bool ok = true;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            v[k] = T[k];
            ok = ok && isfinite(v[k]);
            m = fmaxf(m, fabsf(v[k]));
        }
        if (!ok) {
            a.tc[t] = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
            atomicOr(a.status, APT_STATUS_NONFINITE);
            continue;
        }
        const float4 c = centroid_radius<3>(v);
        a.tc[t] = c;
        ++nv;
        rm = fmaxf(rm, c.w);
        cm = fmaxf(cm, m);
        rs += (double)c.w;
    }
    nv = wave_sum(nv);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        rm = fmaxf(rm, __shfl_xor(rm, d, kWave));
        cm = fmaxf(cm, __shfl_xor(cm, d, kWave));
        rs += __shfl_xor(rs, d, kWave);
    }
    if (lane_id() == 0) {
        s_rs[threadIdx.x / kWave] = rs;
        if (nv) {
            atomicAdd(&s_nv, nv);
            atomicMax(&s_rm, __float_as_uint(rm));
            atomicMax(&s_cm, __float_as_uint(cm));
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_nv) {
        for (int v = 1; v < kEdgePrepBlock / kWave; ++v) s_rs[0] += s_rs[v];
        atomicAdd(&a.tp->n_valid, s_nv);
        atomicMax(&a.tp->rmax_bits, s_rm);
        atomicMax(&a.tp->cmax_bits, s_cm);
        atomicAdd(&a.tp->r_sum, s_rs[0]);
    }
}

// the triangle grid: over the ions' bounding box, cells about twice the
// mean triangle radius (and at least a third of the probe distance, so that
// a probe needs few rings), at most kTriCells of them
__global__ void k_edge_plan(EdgeArgs a) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    const GridPlan P = *a.plan;
    TriPlan& T = *a.tp;
    T.r_max = __uint_as_float(T.rmax_bits);
    double ext[3], vol = 1.0, amax = 0.0;
    for (int c = 0; c < 3; ++c) {
        const float l = P.nB > 0 ? P.lo[c] : 0.0f, hh = P.nB > 0 ? P.hi[c] : 0.0f;
        T.lo[c] = l;
        ext[c] = (double)hh - (double)l;
        vol *= fmax(ext[c], 1e-3);
        amax = fmax(amax, fmax(fabs((double)l), fabs((double)hh)));
    }
    double h = T.n_valid ? 2.0 * T.r_sum / (double)T.n_valid : 1.0;
    if (isfinite(a.d_prb)) h = fmax(h, (double)a.d_prb / 3.0);
    h = fmax(h, cbrt(vol / (double)kTriCells) * 1.0001);
    h = fmax(h, 1e-3);
    for (;;) {
        double cells = 1.0;
        for (int c = 0; c < 3; ++c) cells *= floor(ext[c] / h) + 1.0;
        if (cells <= (double)kTriCells) break;
        h *= 1.1;
    }
    uint32_t nc = 1;
    for (int c = 0; c < 3; ++c) {
        T.dim[c] = (int32_t)floor(ext[c] / h) + 1;
        nc *= (uint32_t)T.dim[c];
    }
    T.n_cells = nc;
    T.h = (float)h;
    T.inv_h = (float)(1.0 / h);
    T.rho = (float)(0.75 * h);                   // one and a half times the mean radius: most triangles stay whole
    // cell indices, centroids and piece vertices are FP32: each may sit a
    // few roundings away from the exact value (of the ions' coordinates, and
    // of the triangles', which may lie farther out)
    const double cmax = (double)__uint_as_float(T.cmax_bits);
    T.slack = (float)(1e-5 * (amax + h) + 1e-6 + 1e-6 * cmax);
    // (FP32 squared distances between such coordinates may overflow: no bound
    // excludes a piece)
    if (!(fmax(amax, cmax) < 5e18)) T.slack = INFINITY;
}

__device__ __forceinline__ float piece_rho(const TriPlan& T, int j) {
    return j < kPieceSizes - 1 ? T.rho * (float)(1u << j) : T.r_max;
}
// How a triangle of radius r (vertices v) is cut for the piece radius rho:
// one piece if it is no larger, else m1 slices from the vertex opposite the
// shortest edge to that edge, each in m2 parts.  (Sub-triangles of a
// barycentric m x m subdivision cut a sliver as often across as along: a
// cap fan's 25 nm x 0.6 nm slivers took 1700 pieces each, now 30.)
struct Cut {
    uint32_t m1, m2;
    int apex;
};
__device__ __forceinline__ Cut cut_of(const float* v, float r, float rho) {
    Cut c{1u, 1u, 0};
    if (r <= rho) return c;
    float e2[3];   // squared edges opposite vertices 0, 1, 2
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int p = (k + 1) % 3, q = (k + 2) % 3;
        const float dx = v[3 * p] - v[3 * q], dy = v[3 * p + 1] - v[3 * q + 1], dz = v[3 * p + 2] - v[3 * q + 2];
        e2[k] = dx * dx + dy * dy + dz * dz;
    }
    c.apex = e2[0] <= e2[1] ? (e2[0] <= e2[2] ? 0 : 2) : (e2[1] <= e2[2] ? 1 : 2);
    const float base = sqrtf(fminf(e2[0], fminf(e2[1], e2[2])));
    const float side = sqrtf(fmaxf(e2[0], fmaxf(e2[1], e2[2])));
    const float step = 1.2f * rho;   // a square part of this edge has radius 0.85 rho
    auto parts = [&](float len) {
        const float m = ceilf(len / step);
        return !(m > 1.0f) ? 1u : (m > 4096.0f ? 4096u : (uint32_t)m);
    };
    c.m1 = parts(side);
    c.m2 = parts(base);
    return c;
}

// pieces the triangles would take for each candidate piece radius (few, large
// workgroups as for k_edge_prep: 231 -> 9 us), and the clearing of the
// triangle grid's counts
__global__ __launch_bounds__(kEdgePrepBlock) void k_edge_measure(EdgeArgs a) {
    __shared__ unsigned long long s_acc[kPieceSizes];
    const TriPlan T = *a.tp;
    for (uint32_t c = blockIdx.x * kEdgePrepBlock + threadIdx.x; c < T.n_cells; c += gridDim.x * kEdgePrepBlock)
        a.tcnt[c] = 0u;
    if (threadIdx.x < kPieceSizes) s_acc[threadIdx.x] = 0ull;
    __syncthreads();
    unsigned long long acc[kPieceSizes];
#pragma unroll
    for (int j = 0; j < kPieceSizes; ++j) acc[j] = 0ull;
    for (uint32_t t = blockIdx.x * kEdgePrepBlock + threadIdx.x; t < a.n_tri; t += gridDim.x * kEdgePrepBlock) {
        const float r = a.tc[t].w;
        if (r < 0.0f) continue;
        float v[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) v[k] = a.tri[9 * (size_t)t + k];
#pragma unroll
        for (int j = 0; j < kPieceSizes; ++j) {
            const Cut c = cut_of(v, r, piece_rho(T, j));
            acc[j] += (unsigned long long)c.m1 * c.m2;
        }
    }
#pragma unroll
    for (int j = 0; j < kPieceSizes; ++j) {
        unsigned long long v = acc[j];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, d, kWave);
            const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), d, kWave);
            v += ((unsigned long long)hi << 32) | lo;
        }
        if (lane_id() == 0 && v) atomicAdd(&s_acc[j], v);
    }
    __syncthreads();
    if (threadIdx.x < kPieceSizes && s_acc[threadIdx.x])
        atomicAdd(&a.tp->pieces_at[threadIdx.x], s_acc[threadIdx.x]);
}

// the smallest piece radius whose pieces fit the workspace (the last
// candidate, one piece per triangle, always does)
__global__ void k_edge_plan_pieces(EdgeArgs a) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    TriPlan& T = *a.tp;
    int j = 0;
    while (j < kPieceSizes - 1 && T.pieces_at[j] > (unsigned long long)T.piece_cap) ++j;
    T.rho = piece_rho(T, j);
}

// The pieces of 64 triangles per wavefront, dealt to its lanes one by one
// whatever triangle they belong to (a sliver's pieces by its own lane kept
// the launch waiting for that lane), and in the place of the triangle's
// centroid its unit normal (zero where the vertices do not fix one to FP32).
__global__ __launch_bounds__(kBlock) void k_edge_pieces(EdgeArgs a) {
    const TriPlan T = *a.tp;
    const int l = lane_id();
    float rmax = 0.0f;
    const uint32_t n_waves = gridDim.x * (kBlock / kWave);
    for (uint32_t t0 = (blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave) * kWave; t0 < a.n_tri;
         t0 += n_waves * kWave) {
        const uint32_t t = t0 + (uint32_t)l;
        float4 tc = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
        Cut cut{0u, 0u, 0};
        if (t < a.n_tri) tc = a.tc[t];
        if (tc.w >= 0.0f) {
            float v[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) v[k] = a.tri[9 * (size_t)t + k];
            cut = cut_of(v, tc.w, T.rho);
            const double e1x = (double)v[3] - v[0], e1y = (double)v[4] - v[1], e1z = (double)v[5] - v[2];
            const double e2x = (double)v[6] - v[0], e2y = (double)v[7] - v[1], e2z = (double)v[8] - v[2];
            const double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
            const double nn = nx * nx + ny * ny + nz * nz;
            const double ee = (e1x * e1x + e1y * e1y + e1z * e1z) * (e2x * e2x + e2y * e2y + e2z * e2z);
            // |n| / (|e1| |e2|) = sin of the angle at vertex 0: below 1e-7 the
            // FP64 products no longer give the direction to 1e-8
            const double inv = nn > 1e-14 * ee && nn > 1e-280 ? 1.0 / sqrt(nn) : 0.0;
            a.tc[t] = make_float4((float)(nx * inv), (float)(ny * inv), (float)(nz * inv), 0.0f);
        }
        const uint32_t cnt = cut.m1 * cut.m2;
        const uint32_t inc = wave_incl_scan(cnt);
        const uint32_t tot = readlane(inc, kWave - 1);
        uint32_t base = 0;
        if (l == 0 && tot) base = atomicAdd(&a.tp->piece_ctr, tot);
        base = readlane(base, 0);
        const uint32_t off = inc - cnt;
        for (uint32_t p0 = 0; p0 < tot; p0 += kWave) {
            const uint32_t p = p0 + (uint32_t)l;
            int own = 0;   // the last lane whose pieces start at or before p and that has any
#pragma unroll
            for (int step = 32; step > 0; step >>= 1) {
                const uint32_t o = (uint32_t)__shfl((int)off, own + step, kWave);
                if (o <= p) own += step;
            }
            const uint32_t o = (uint32_t)__shfl((int)off, own, kWave);
            const uint32_t m1 = (uint32_t)__shfl((int)cut.m1, own, kWave);
            const uint32_t m2 = (uint32_t)__shfl((int)cut.m2, own, kWave);
            const int apex = __shfl(cut.apex, own, kWave);
            float4 c;
            c.x = __shfl(tc.x, own, kWave);
            c.y = __shfl(tc.y, own, kWave);
            c.z = __shfl(tc.z, own, kWave);
            c.w = __shfl(tc.w, own, kWave);
            if (p >= tot || base + p >= a.piece_cap) continue;
            const uint32_t tt = t0 + (uint32_t)own;
            if (m1 * m2 > 1u) {
                const float* v = a.tri + 9 * (size_t)tt;
                const float* A = v + 3 * apex;
                const float* B = v + 3 * ((apex + 1) % 3);
                const float* C = v + 3 * ((apex + 2) % 3);
                const uint32_t e = p - o, s = e / m2, u = e - s * m2;
                float q[12];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float f = (float)(s + (k >> 1)) / (float)m1, w = (float)(u + (k & 1)) / (float)m2;
#pragma unroll
                    for (int x = 0; x < 3; ++x) q[3 * k + x] = A[x] + f * ((B[x] - A[x]) + w * (C[x] - B[x]));
                }
                c = centroid_radius<4>(q);
                c.w += T.slack;
            }
            a.pc[base + p] = c;
            a.ptri[base + p] = tt;
            rmax = fmaxf(rmax, c.w);
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) rmax = fmaxf(rmax, __shfl_xor(rmax, d, kWave));
    if (l == 0 && rmax > 0.0f) atomicMax(&a.tp->piece_rmax_bits, __float_as_uint(rmax));
}

// pieces in the workspace's arrays (k_edge_pieces cuts with the radius that
// k_edge_measure counted them for, so that all fit: at most pieces_at of it)
__device__ __forceinline__ uint32_t n_pieces(const TriPlan& T) {
    return T.piece_ctr < T.piece_cap ? T.piece_ctr : T.piece_cap;
}

__device__ __forceinline__ int edge_axis(const TriPlan& T, int c, float x) {
    const float f = floorf((x - T.lo[c]) * T.inv_h);
    if (!(f >= 0.0f)) return 0;
    const int m = (int)fminf(f, (float)(T.dim[c] - 1));
    return m;
}

__global__ __launch_bounds__(kBlock) void k_edge_count(EdgeArgs a) {
    const TriPlan T = *a.tp;
    for (uint32_t p = blockIdx.x * kBlock + threadIdx.x; p < n_pieces(T); p += gridDim.x * kBlock) {
        const float4 c = a.pc[p];
        const uint32_t cell = ((uint32_t)edge_axis(T, 2, c.z) * (uint32_t)T.dim[1] + (uint32_t)edge_axis(T, 1, c.y)) *
                                  (uint32_t)T.dim[0] + (uint32_t)edge_axis(T, 0, c.x);
        a.pcell[p] = cell;
        atomicAdd(a.tcnt + cell, 1u);
    }
}

// exclusive offsets of the cell counts: each block scans its tile of
// kTriScanTile cells and leaves the tile's sum; the second kernel adds the
// sums of the tiles before it
__global__ __launch_bounds__(kBlock) void k_edge_scan_blocks(EdgeArgs a) {
    const uint32_t nc = a.tp->n_cells;
    const uint32_t base = blockIdx.x * (uint32_t)kTriScanTile;
    if (base >= nc) return;
    __shared__ uint32_t s_w[kWavesPerBlock];
    constexpr int per = kTriScanTile / kBlock;   // 16 consecutive cells per thread
    const uint32_t c0 = base + threadIdx.x * per;
    uint32_t v[per], sum = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        v[k] = c0 + k < nc ? a.tcnt[c0 + k] : 0u;
        sum += v[k];
    }
    const uint32_t inc = wave_incl_scan(sum);
    const int w = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) s_w[w] = inc;
    __syncthreads();
    uint32_t run = inc - sum;
    for (int u = 0; u < w; ++u) run += s_w[u];
#pragma unroll
    for (int k = 0; k < per; ++k) {
        if (c0 + k < nc) a.tstart[c0 + k] = run;
        run += v[k];
    }
    if (threadIdx.x == kBlock - 1) a.tblk[blockIdx.x] = run;
}

__global__ __launch_bounds__(kBlock) void k_edge_scan_add(EdgeArgs a) {
    const uint32_t nc = a.tp->n_cells;
    const uint32_t base = blockIdx.x * (uint32_t)kTriScanTile;
    if (base >= nc) return;
    __shared__ uint32_t s_off;
    if (threadIdx.x < kWave) {
        uint32_t s = 0;
        for (uint32_t b = lane_id(); b < blockIdx.x; b += kWave) s += a.tblk[b];
        s = wave_sum(s);
        if (lane_id() == 0) s_off = s;
    }
    __syncthreads();
    const uint32_t off = s_off;
    const uint32_t end = base + kTriScanTile < nc ? base + kTriScanTile : nc;
    for (uint32_t c = base + threadIdx.x; c < end; c += kBlock) a.tstart[c] += off;
    if (end == nc && threadIdx.x == 0) a.tstart[nc] = off + a.tblk[blockIdx.x];
}

__global__ __launch_bounds__(kBlock) void k_edge_fill(EdgeArgs a) {
    const uint32_t np = n_pieces(*a.tp);
    for (uint32_t p = blockIdx.x * kBlock + threadIdx.x; p < np; p += gridDim.x * kBlock) {
        const uint32_t cell = a.pcell[p];
        const uint32_t pos = a.tstart[cell] + atomicSub(a.tcnt + cell, 1u) - 1u;
        a.torder[pos] = a.ptri[p];
        a.tsorted[pos] = a.pc[p];
    }
}

// squared distance of p to the segment [u, u + e] (FP64)
__device__ __forceinline__ double seg_dist2(double px, double py, double pz, double ux, double uy, double uz,
                                            double ex, double ey, double ez) {
#pragma clang fp contract(off)
    const double wx = px - ux, wy = py - uy, wz = pz - uz;
    const double ee = ex * ex + ey * ey + ez * ez;
    double t = ee > 0.0 ? (wx * ex + wy * ey + wz * ez) / ee : 0.0;
    t = fmin(fmax(t, 0.0), 1.0);
    const double qx = wx - t * ex, qy = wy - t * ey, qz = wz - t * ez;
    return qx * qx + qy * qy + qz * qz;
}

// squared distance of p to the closed triangle T (FP64 on the FP32 vertices)
__device__ __forceinline__ double tri_dist2(double px, double py, double pz, const float* __restrict__ T) {
#pragma clang fp contract(off)
    const double ax = T[0], ay = T[1], az = T[2];
    const double bx = T[3], by = T[4], bz = T[5];
    const double cx = T[6], cy = T[7], cz = T[8];
    const double e1x = bx - ax, e1y = by - ay, e1z = bz - az;   // b - a
    const double e2x = cx - ax, e2y = cy - ay, e2z = cz - az;   // c - a
    const double nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
    const double nn = nx * nx + ny * ny + nz * nz;
    const double wx = px - ax, wy = py - ay, wz = pz - az;
    if (nn > 0.0) {
        // barycentric weights of the foot of the perpendicular, scaled by nn
        const double d1 = e1x * wx + e1y * wy + e1z * wz, d2 = e2x * wx + e2y * wy + e2z * wz;
        const double bpx = px - bx, bpy = py - by, bpz = pz - bz;
        const double d3 = e1x * bpx + e1y * bpy + e1z * bpz, d4 = e2x * bpx + e2y * bpy + e2z * bpz;
        const double cpx = px - cx, cpy = py - cy, cpz = pz - cz;
        const double d5 = e1x * cpx + e1y * cpy + e1z * cpz, d6 = e2x * cpx + e2y * cpy + e2z * cpz;
        const double wa = d3 * d6 - d5 * d4, wb = d5 * d2 - d1 * d6, wc = d1 * d4 - d3 * d2;
        if (wa >= 0.0 && wb >= 0.0 && wc >= 0.0) {
            const double hgt = wx * nx + wy * ny + wz * nz;
            return hgt * hgt / nn;
        }
    }
    double d = seg_dist2(px, py, pz, ax, ay, az, e1x, e1y, e1z);
    d = fmin(d, seg_dist2(px, py, pz, bx, by, bz, cx - bx, cy - by, cz - bz));
    d = fmin(d, seg_dist2(px, py, pz, ax, ay, az, e2x, e2y, e2z));
    return d;
}

// FP32 gap (nm) between [p0, p1] and cell m's interval on axis c
__device__ __forceinline__ float axis_gap(const TriPlan& T, int c, float p0, float p1, int m) {
    const float l = T.lo[c] + (float)m * T.h, u = l + T.h;
    return fmaxf(fmaxf(l - p1, p0 - u), 0.0f);
}

// The pieces in the rows of the triangle grid within S of the box: f(valid,
// k), k a slot of the sorted arrays, is called by all 64 lanes per step.
// (Pieces outside the grid are registered in its outermost cells, nearer to
// the box than they are: the gaps stay lower bounds.)  Returns whether the
// box grown by S covers the grid (cells at its corners may still be beyond S).
template <class F>
__device__ __forceinline__ bool edge_rows(const TriPlan& T, const uint32_t* __restrict__ tstart, float x0, float y0,
                                          float z0, float x1, float y1, float z1, float S, F&& f) {
    const int l = lane_id();
    const int cy0 = edge_axis(T, 1, y0 - S), cy1 = edge_axis(T, 1, y1 + S);
    const int cz0 = edge_axis(T, 2, z0 - S), cz1 = edge_axis(T, 2, z1 + S);
    const int ny = cy1 - cy0 + 1, nrows = ny * (cz1 - cz0 + 1);
    for (int rb = 0; rb < nrows; rb += kWave) {
        const int r = rb + l;
        uint32_t st = 0, len = 0;
        if (r < nrows) {
            const int cz = cz0 + r / ny, cy = cy0 + r % ny;
            const float gy = axis_gap(T, 1, y0, y1, cy), gz = axis_gap(T, 2, z0, z1, cz);
            const float rest = S * S - (gy * gy + gz * gz);
            if (!(rest < 0.0f)) {
                const float ex = rest < INFINITY ? sqrtf(rest) : INFINITY;   // (squares that overflowed: the whole row)
                const uint32_t row = ((uint32_t)cz * (uint32_t)T.dim[1] + (uint32_t)cy) * (uint32_t)T.dim[0];
                st = tstart[row + (uint32_t)edge_axis(T, 0, x0 - ex)];
                len = tstart[row + (uint32_t)edge_axis(T, 0, x1 + ex) + 1u] - st;
            }
        }
        const uint32_t inc = wave_incl_scan(len);
        const uint32_t tot = readlane(inc, kWave - 1);
        const uint32_t off = inc - len;
        for (uint32_t b0 = 0; b0 < tot; b0 += kWave) {
            const uint32_t v = b0 + (uint32_t)l;
            int row = 0;   // the last row starting at or before v
#pragma unroll
            for (int step = 32; step > 0; step >>= 1) {
                const uint32_t o = (uint32_t)__shfl((int)off, row + step, kWave);
                if (o <= v) row += step;
            }
            const uint32_t k = (uint32_t)__shfl((int)(st - off), row, kWave) + v;
            f(v < tot, v < tot ? k : 0u);
        }
    }
    return edge_axis(T, 0, x0 - S) == 0 && edge_axis(T, 0, x1 + S) == T.dim[0] - 1 && cy0 == 0 &&
           cy1 == T.dim[1] - 1 && cz0 == 0 && cz1 == T.dim[2] - 1;
}

// 64 ions per wavefront, one wavefront per workgroup (7.7e6 ions, a
// 102 912-triangle hull, d_prb 2.5 nm: 13.4 -> 2.05 ms).  The whole group is
// tested against the grid first, which ends most of a specimen's groups; near
// the edge it is taken 16 ions at a time, four lanes to an ion, each with a
// quarter of the pieces: the reach that must hold every ion's triangle grows
// with the group's box, and with it the pieces (180 for 16 ions 2 nm deep,
// about 400 for 64 at once).  The pieces that the lower bound cannot exclude
// are queued as (piece's triangle, ion) and their FP64 distances taken 64 at a
// time, so that no lane waits while another evaluates (one triangle for all
// lanes at once, as the bound passed it: 5.4 ms).  Wavefronts near a cap's
// centre take a hundred times as long as the others, hence no second wavefront
// waits beside them for the workgroup's registers.  One ion per lane with a
// search of its own, as before, had every lane of a wavefront walk hundreds of
// cells at its own pace.
//
// The lower bound: the piece lies in its triangle's plane and within w of its
// centroid c, so with h = |(p - c) . n| the distance of p to the plane and
// t = sqrt(|p - c|^2 - h^2) the distance within it, no point of the piece is
// closer than sqrt(h^2 + max(0, t - w)^2).  On a flat stretch of hull that
// leaves the few triangles under the ion, where |p - c| - w left a disc of
// them.  The FP32 roundings of n and of the dot product move h by at most
// 1e-6 |p - c|, those of |p - c|^2 - h^2 move it by at most 6e-6 |p - c|^2;
// c lies within T.slack of the plane.
__global__ __launch_bounds__(kWave, 4) void k_edge_dist(EdgeArgs a) {
    constexpr int kSub = 16, kPer = kWave / kSub;   // ions of a subgroup; lanes of an ion, subgroups of a chunk
    __shared__ float4 lc[kEdgeList], ln[kEdgeList];
    __shared__ uint2 queue[2 * kWave];
    __shared__ float4 pos[kWave];
    __shared__ unsigned long long best[kWave];      // squared distances (FP64 bits; non-negative)
    const GridPlan P = *a.plan;
    const TriPlan T = *a.tp;
    const int l = (int)threadIdx.x;
    const bool any = n_pieces(T) > 0;
    const float skip = __uint_as_float(T.piece_rmax_bits) + T.slack;   // a cell's pieces reach this far out
    const uint32_t n_chunks = (P.nB + kWave - 1) / kWave;
    // small clouds: a wavefront for each of a chunk's subgroups (20 000 ions
    // inside a hull of 113 000 triangles, 313 chunks: the call 8.3 -> 2.8 ms)
    const uint32_t per = n_chunks <= (1u << 15) ? (uint32_t)kPer : 1u;
    for (uint32_t it = blockIdx.x; it < n_chunks * per; it += gridDim.x) {
        const uint32_t ch = it / per;
        const int sub0 = (int)(it - ch * per), sub1 = per == 1u ? kPer : sub0 + 1;
        const uint32_t j = ch * (uint32_t)kWave + (uint32_t)l;
        const bool valid = j < P.nB;
        const float4 rec = a.bpos[valid ? j : P.nB - 1u];
        const uint32_t idx = __builtin_bit_cast(uint32_t, rec.w);
        const bool fin = valid && isfinite(rec.x) && isfinite(rec.y) && isfinite(rec.z);
        wave_sync();
        pos[l] = rec;
        best[l] = __builtin_bit_cast(unsigned long long, (double)INFINITY);
        wave_sync();
        const uint32_t crow = fin ? (uint32_t)cell_axis(P, 2, rec.z) * (uint32_t)P.dim[1] +
                                        (uint32_t)cell_axis(P, 1, rec.y)
                                  : 0xFFFFFFFFu;
        uint64_t todo = any ? __ballot(fin) : 0ull;
        while (todo) {
            const bool part = fin && crow == readlane(crow, __builtin_ctzll(todo));
            const uint64_t pm = __ballot(part);
            todo &= ~pm;
            float x0 = wave_min_f(part ? rec.x : INFINITY), x1 = wave_max_f(part ? rec.x : -INFINITY);
            float y0 = wave_min_f(part ? rec.y : INFINITY), y1 = wave_max_f(part ? rec.y : -INFINITY);
            float z0 = wave_min_f(part ? rec.z : INFINITY), z1 = wave_max_f(part ? rec.z : -INFINITY);
            float cx, cy, cz, hd, near2;
            auto centre = [&]() {
                cx = 0.5f * (x0 + x1);
                cy = 0.5f * (y0 + y1);
                cz = 0.5f * (z0 + z1);
                const float bx = x1 - x0, by = y1 - y0, bz = z1 - z0;
                hd = 0.5f * sqrtf(bx * bx + by * by + bz * bz) * 1.00001f + T.slack;
                near2 = INFINITY;
            };
            // the centroid nearest to the box's centre, of the rows within R
            // of the box; true if the box grown by R covers the grid
            auto nearest = [&](float R) {
                const bool whole = edge_rows(T, a.tstart, x0, y0, z0, x1, y1, z1, (R + skip) * 1.00001f + T.slack,
                                             [&](bool ok, uint32_t k) {
                                                 const float4 c = a.tsorted[k];
                                                 const float dx = c.x - cx, dy = c.y - cy, dz = c.z - cz;
                                                 if (ok) near2 = fminf(near2, fminf(dx * dx + dy * dy + dz * dz, 3e38f));
                                             });
                near2 = wave_min_f(near2);
                return whole;
            };
            // the whole part first, within a reach that doubles until there is
            // a piece or the probe's reach is passed.  Once the reach spans the
            // grid along every axis, only the corners are left out (their rows
            // lie beyond it diagonally): the rest of the probe's reach at once
            centre();
            for (float R = fminf(2.0f * T.h, a.d_prb);;) {
                const bool whole = nearest(R);
                if (near2 < INFINITY || R >= a.d_prb) break;
                R = whole ? a.d_prb : fminf(2.0f * R, a.d_prb);
            }
            if (!(near2 < INFINITY)) continue;       // nothing within reach of the group
            const float gx = cx, gy = cy, gz = cz, gnear = sqrtf(near2) * 1.00001f + T.slack;

            for (int sub = sub0; sub < sub1; ++sub) {
                if (((pm >> (sub * kSub)) & ((1ull << kSub) - 1ull)) == 0ull) continue;
                const int slot = sub * kSub + l / kPer, q = l % kPer;   // this lane's ion and quarter
                const bool mine = (pm >> slot) & 1ull;
                const float4 r = pos[slot];
                x0 = wave_min_f(mine ? r.x : INFINITY);
                x1 = wave_max_f(mine ? r.x : -INFINITY);
                y0 = wave_min_f(mine ? r.y : INFINITY);
                y1 = wave_max_f(mine ? r.y : -INFINITY);
                z0 = wave_min_f(mine ? r.z : INFINITY);
                z1 = wave_max_f(mine ? r.z : -INFINITY);
                centre();
                // the piece nearest to the part's centre bounds the distance
                // of this box's centre; its own nearest lies within that
                const float mx = cx - gx, my = cy - gy, mz = cz - gz;
                const float bound = gnear + sqrtf(mx * mx + my * my + mz * mz) * 1.00001f + T.slack;
                (void)nearest(fminf(bound, a.d_prb));
                const float near = fminf(bound, sqrtf(near2) * 1.00001f + T.slack);
                const float B = fminf(a.d_prb, near + hd);           // no ion of the box needs more

                const float ex = r.x - cx, ey = r.y - cy, ez = r.z - cz;
                const float own = near + sqrtf(ex * ex + ey * ey + ez * ez) * 1.00001f + T.slack;
                float cull2 = -1.0f;                                  // squared: pieces beyond it are skipped
                if (mine) {
                    const float c = fminf(own, a.d_prb * 1.00001f);
                    cull2 = c * c * 1.00001f;
                }
                // the roundings of h (|p - c| is at most B + 2 hd + w)
                const float margin = T.slack + 1e-6f * (B + 2.0f * hd + skip);
                int cnt = 0, qn = 0;
                // the first `m` <= 64 queued distances
                auto evaluate = [&](int m) {
                    wave_sync();
                    if (l < m) {
                        const uint2 e = queue[l];
                        const float4 p = pos[e.y];
                        const double d = tri_dist2(p.x, p.y, p.z, a.tri + 9 * (size_t)e.x);
                        if (d >= 0.0) atomicMin(&best[e.y], __builtin_bit_cast(unsigned long long, d));
                    }
                    wave_sync();
                    const uint2 rest = queue[kWave + l];
                    wave_sync();
                    if (l < qn - m) queue[l] = rest;
                    qn -= m;
                    wave_sync();
                    if (mine) cull2 = fminf(cull2, (float)__builtin_bit_cast(double, best[slot]) * 1.00001f + 1e-30f);
                };
                auto run = [&]() {
                    wave_sync();
                    float u2 = INFINITY;
                    for (int t = q; t < cnt; t += kPer) {
                        const float4 c = lc[t];
                        const float dx = r.x - c.x, dy = r.y - c.y, dz = r.z - c.z;
                        u2 = fminf(u2, fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
                    }
#pragma unroll
                    for (int d = kPer / 2; d >= 1; d >>= 1) u2 = fminf(u2, __shfl_xor(u2, d, kWave));
                    if (mine) {
                        const float c = sqrtf(u2) * 1.00001f + T.slack;
                        cull2 = fminf(cull2, c * c * 1.00001f);
                    }
                    for (int t0 = 0; t0 < cnt; t0 += kPer) {
                        const int t = t0 + q < cnt ? t0 + q : t0;
                        const float4 c = lc[t], n = ln[t];
                        const float dx = r.x - c.x, dy = r.y - c.y, dz = r.z - c.z;
                        const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                        const float h = fabsf(fmaf(dz, n.z, fmaf(dy, n.y, dx * n.x)));
                        const float hs = fmaxf(0.0f, h - margin);
                        const float ts = fmaxf(0.0f, sqrtf(fmaxf(0.0f, fmaf(d2, 1.0f - 6e-6f, -h * h))) - c.w);
                        const bool pass = t0 + q < cnt && fmaf(hs, hs, ts * ts) * 0.99999f <= cull2;
                        const uint64_t m = __ballot(pass);
                        if (m) {
                            if (pass)
                                queue[qn + __popcll(m & lanemask_lt())] =
                                    make_uint2(__builtin_bit_cast(uint32_t, n.w), (uint32_t)slot);
                            qn += __popcll(m);
                            if (qn >= kWave) evaluate(kWave);
                        }
                    }
                    wave_sync();
                    cnt = 0;
                };
                (void)edge_rows(T, a.tstart, x0, y0, z0, x1, y1, z1, (B + skip) * 1.00001f + T.slack,
                                [&](bool ok, uint32_t k) {
                                    const float4 c = a.tsorted[k];
                                    const float dx = c.x - cx, dy = c.y - cy, dz = c.z - cz;
                                    const float lb = sqrtf(dx * dx + dy * dy + dz * dz) * 0.99999f - c.w - T.slack - hd;
                                    const bool keep = ok && !(lb > B);
                                    const uint64_t m = __ballot(keep);
                                    if (keep) {
                                        const uint32_t t = a.torder[k];
                                        const float4 n = a.tc[t];
                                        const int at = cnt + __popcll(m & lanemask_lt());
                                        lc[at] = make_float4(c.x, c.y, c.z, c.w + T.slack);
                                        ln[at] = make_float4(n.x, n.y, n.z, __builtin_bit_cast(float, t));
                                    }
                                    cnt += __popcll(m);
                                    if (cnt > kEdgeList - kWave) run();
                                });
                if (cnt > 0) run();
                if (qn > 0) evaluate(qn);
            }
        }
        wave_sync();
        if (valid && l / kSub >= sub0 && l / kSub < sub1) {
            const double d = sqrt(__builtin_bit_cast(double, best[l]));
            a.d_out[idx] = !fin ? __builtin_nanf("") : (d < (double)a.d_prb) ? (float)d : __builtin_inff();
        }
    }
}

}  // namespace apt
