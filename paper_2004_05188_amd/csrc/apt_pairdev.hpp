// Device-side building blocks of the target-neighbour pair loop, shared by
// the plain kernel (apt_pair.hip) and the batched-replicate kernel
// (apt_batched.hip): the stencil enumeration, the exact kNN key sort and
// the per-target work (RDF counts and k nearest neighbours of one target).
#pragma once
#include "apt_pair.hpp"

namespace apt {

__device__ __forceinline__ uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }

// The next batch of a wavefront's work: items [*i0, *i1) of queue *x, which
// holds 2^lg items for each of [n x / kXcd, n (x + 1) / kXcd).  A wavefront
// takes from its own XCD's queue (consecutive items: a compact region, whose
// records its L2 keeps) and, once that is empty, from the others', starting
// with `x` = its XCD and `empty` = 0; false when all are empty.  The XCDs'
// eighths are equal in number, not in work: without the second part the
// first XCDs to finish waited for a third of the dense-target tile kernel's
// time (7.7e6-ion needle).  (Another queue is read before its counter is
// added to: every wavefront passes every queue at the end, and atomics on one
// address take about 16 ns each.)
__device__ __forceinline__ bool next_batch(uint32_t* queue, uint32_t n, uint32_t lg, uint32_t batch, int& x,
                                           int& empty, uint32_t* i0, uint32_t* i1) {
    for (; empty < kXcd; ++empty, x = x + 1 < kXcd ? x + 1 : 0) {
        const uint32_t first = (uint32_t)((uint64_t)n * (uint64_t)x / kXcd);
        const uint32_t own = ((uint32_t)((uint64_t)n * (uint64_t)(x + 1) / kXcd) - first) << lg;
        uint32_t* q = queue + x * kWorkStride;
        uint32_t c = 0;
        if (lane_id() == 0) {
            if (empty == 0 || __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < own)
                c = atomicAdd(q, batch);
            else
                c = own;
        }
        c = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
        if (c < own) {
            *i0 = c;
            *i1 = own - c > batch ? c + batch : own;
            return true;
        }
    }
    return false;
}

// Ascending sort of buf[0..c) by one wavefront; c <= kKnnCap.  Up to 64
// keys: each lane takes one key and counts the smaller ones (equal ones by
// position), broadcast lane by lane (no LDS round trips); beyond: a bitonic
// network over buf padded to a power of two with all-ones keys.
__device__ inline void wave_sort_keys(uint64_t* buf, int c) {
    const int l = lane_id();
    if (c <= kWave) {
        wave_sync();
        const uint64_t mine = l < c ? buf[l] : ~0ull;
        const uint32_t lo = (uint32_t)mine, hi = (uint32_t)(mine >> 32);
        int rank = 0;
        for (int j = 0; j < c; ++j) {
            const uint64_t kj = ((uint64_t)readlane(hi, j) << 32) | (uint64_t)readlane(lo, j);
            rank += (kj < mine || (kj == mine && j < l)) ? 1 : 0;
        }
        wave_sync();
        if (l < c) buf[rank] = mine;
        wave_sync();
        return;
    }
    int N = kWave;
    while (N < c) N <<= 1;
    for (int i = c + l; i < N; i += kWave) buf[i] = ~0ull;
    wave_sync();
    for (int size = 2; size <= N; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int p = l; p < (N >> 1); p += kWave) {
                const int i = ((p & ~(stride - 1)) << 1) | (p & (stride - 1));
                const int j = i + stride;
                const bool asc = (i & size) == 0;
                const uint64_t x = buf[i], y = buf[j];
                if ((x > y) == asc) {
                    buf[i] = y;
                    buf[j] = x;
                }
            }
            wave_sync();
        }
    }
}

// Visit the neighbours in the cell rows that a sphere of radius R around
// (px, py, pz) meets.  f(idx, x, y, z) is called by all 64 lanes per step,
// idx == kNone on lanes without a candidate.  kUnroll batches of 64
// candidates are located and their positions loaded before any is visited,
// so that several memory round trips overlap.
constexpr int kUnroll = 4;

// The i-th of L rows centre-out (middle of the range first, then
// alternately below and above; a permutation of [0, L)): enumerations that
// feed a k-smallest list visit rows in this order, so that the list fills
// with the nearest candidates early and later, farther candidates seldom
// change it; others keep raster order, which walks memory in sequence (the
// visiting order never changes a result).
__device__ __forceinline__ int centre_out(int i, int L) {
    return L / 2 + ((i & 1) ? -((i + 1) >> 1) : (i >> 1));
}

// Records [st, st + len) of the cell row (cy, cz) that can lie within R of
// the box [x0,x1] x [y0,y1] x [z0,z1] (R2 = (R + eps)^2): the row's cells
// trimmed to the x-range the sphere reaches at the row's distance from the
// box; len = 0 for a row beyond R.
__device__ __forceinline__ void row_span(const GridPlan& P, const uint32_t* __restrict__ cell_start, int cy, int cz,
                                         float x0, float y0, float z0, float x1, float y1, float z1, float R2,
                                         uint32_t& st, uint32_t& len) {
    const float ya = P.lo[1] + (float)cy * P.h - P.eps, yb = P.lo[1] + (float)(cy + 1) * P.h + P.eps;
    const float za = P.lo[2] + (float)cz * P.h - P.eps, zb = P.lo[2] + (float)(cz + 1) * P.h + P.eps;
    const float dy = fmaxf(0.0f, fmaxf(ya - y1, y0 - yb));
    const float dz = fmaxf(0.0f, fmaxf(za - z1, z0 - zb));
    const float d2 = dy * dy + dz * dz;
    st = 0;
    len = 0;
    if (d2 <= R2) {
        const float ex = sqrtf(R2 - d2) + P.eps;
        const int cx0 = cell_axis(P, 0, x0 - ex), cx1 = cell_axis(P, 0, x1 + ex);
        const uint32_t base = ((uint32_t)cz * (uint32_t)P.dim[1] + (uint32_t)cy) * (uint32_t)P.dim[0];
        st = cell_start[base + (uint32_t)cx0];
        len = cell_start[base + (uint32_t)cx1 + 1u] - st;
    }
}

struct NoStep {
    __device__ __forceinline__ void operator()() const {}
};

// after_step() is called by all lanes after each kUnroll batches (work that
// would cost registers in every unrolled copy of f).
template <class F, class G = NoStep>
__device__ __forceinline__ void enumerate_box(const GridPlan& P, const uint32_t* __restrict__ cell_start,
                                              const float4* __restrict__ bpos, float x0, float y0, float z0,
                                              float x1, float y1, float z1, float R, F&& f, bool centre = false,
                                              G&& after_step = G{}) {
    // neighbours within R of the box [x0,x1] x [y0,y1] x [z0,z1]
    const int l = lane_id();
    const float Re = R + P.eps;
    const float R2 = Re * Re;
    const int cy0 = cell_axis(P, 1, y0 - Re), cy1 = cell_axis(P, 1, y1 + Re);
    const int cz0 = cell_axis(P, 2, z0 - Re), cz1 = cell_axis(P, 2, z1 + Re);
    const int ny = cy1 - cy0 + 1, nz = cz1 - cz0 + 1;
    const int nrows = ny * nz;
    for (int rb = 0; rb < nrows; rb += kWave) {
        const int r = rb + l;
        uint32_t st = 0, len = 0;
        if (r < nrows) {
            const int iz = r / ny, iy = r % ny;
            const int cz = cz0 + (centre ? centre_out(iz, nz) : iz), cy = cy0 + (centre ? centre_out(iy, ny) : iy);
            row_span(P, cell_start, cy, cz, x0, y0, z0, x1, y1, z1, R2, st, len);
        }
        const uint32_t inc = wave_incl_scan(len);
        const uint32_t tot = readlane(inc, kWave - 1);
        const uint32_t off = inc - len;
        for (uint32_t b0 = 0; b0 < tot; b0 += kWave * kUnroll) {
            uint32_t idx[kUnroll];
            float4 c[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const uint32_t b = b0 + (uint32_t)(kWave * u);
                const uint32_t v = b + (uint32_t)l;
                idx[u] = kNone;
                if (b < tot) {
                    const int r0 = __popcll(__ballot(inc <= b));   // first row ending after b
                    const uint32_t e0 = readlane(inc, r0);
                    if (e0 >= b + kWave) {
                        // the whole step lies in row r0
                        idx[u] = readlane(st, r0) + (v - (e0 - readlane(len, r0)));
                    } else {
                        // rows r0..r1 start before the step's end: each lane finds
                        // the last of them starting at or before its slot (binary
                        // lifting over the ascending row offsets, lane shuffles)
                        const uint32_t lim = b + kWave < tot ? b + kWave : tot;
                        const int r1 = __popcll(__ballot(off < lim)) - 1;
                        int row = r0;
                        for (int step = 32; step > 0; step >>= 1) {
                            if (step > r1 - r0) continue;            // uniform
                            const int c = row + step;
                            const uint32_t oc = (uint32_t)__shfl((int)off, c < kWave ? c : kWave - 1, kWave);
                            if (c <= r1 && oc <= v) row = c;
                        }
                        const uint32_t base = (uint32_t)__shfl((int)(st - off), row, kWave);
                        if (v < tot) idx[u] = base + v;
                    }
                }
            }
            // lanes without a candidate read record 0 (always present when tot > 0)
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) c[u] = bpos[idx[u] == kNone ? 0u : idx[u]];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (b0 + (uint32_t)(kWave * u) < tot) f(idx[u] != kNone, c[u]);
            after_step();
        }
    }
}


template <class F, class G = NoStep>
__device__ __forceinline__ void enumerate(const GridPlan& P, const uint32_t* __restrict__ cell_start,
                                          const float4* __restrict__ bpos, float px, float py, float pz,
                                          float R, F&& f, bool centre = false, G&& after_step = G{}) {
    enumerate_box(P, cell_start, bpos, px, py, pz, px, py, pz, R, f, centre, after_step);
}

// Everything one target needs besides its position and index.
struct PairTask {
    const float4* bpos;          // neighbour records, cell order
    const uint32_t* cell_start;  // [n_cells + 1] into bpos
    // RDF
    int n_bins;
    float r_enum, thr2, inv_w, half_band;
    double inv_w64;
    const double* E2;
    uint32_t* hist_l;            // per-wavefront LDS histogram (LDS variant)
    uint64_t* hist_g;            // global histogram (global variant)
    // kNN
    int k;
    float rk0, rknn, rknn2;
    uint64_t* kbuf;              // per-wavefront LDS key buffer [kKnnCap]
};

// One pair's RDF count, at FP32 squared distance d2 < thr2: the FP32 bin, or
// near an edge the FP64 one.  With an LDS histogram thr2 is so near r_max^2
// that a position past the last bin is always near its edge: only those pairs
// test whether the bin exists.  Nothing is kept of how many were counted
// (callers bound it by the candidates scanned).
template <bool LDS_HIST>
__device__ __forceinline__ void rdf_count(const PairTask& T, float px, float py, float pz, float4 c, float d2) {
    const float t = __builtin_amdgcn_sqrtf(d2) * T.inv_w;
    int b = (int)t;
    bool in = LDS_HIST || b < T.n_bins;
    if (__builtin_expect(fabsf(__builtin_amdgcn_fractf(t) - 0.5f) > T.half_band, 0)) {
        b = exact_bin(exact_D2(px, py, pz, c.x, c.y, c.z), T.E2, T.n_bins, T.inv_w64);
        in = b < T.n_bins;
    }
    if (in) {
        if (LDS_HIST) atomicAdd(&T.hist_l[b], 1u);
        else atomicAdd((unsigned long long*)&T.hist_g[b], 1ull);
    }
}

// RDF counts and kNN keys of one target.  Leaves the sorted keys in kbuf and
// returns how many of the k nearest were found; adds the RDF's steps of 64
// candidates to `steps`.
template <int FLAGS, bool KNN>
__device__ __forceinline__ int run_target(const GridPlan& P, const PairTask& T, float px, float py, float pz,
                                          uint32_t i, uint32_t& steps, bool rdf_on = true) {
    constexpr bool RDF_T = (FLAGS & (kRdfLds | kRdfGlobal)) != 0;
    const bool RDF = RDF_T && rdf_on;
    constexpr bool LDS_HIST = (FLAGS & kRdfLds) != 0;
    constexpr bool SELF = (FLAGS & kSelf) != 0;
    const int l = lane_id();
    const bool finite = isfinite(px) && isfinite(py) && isfinite(pz);
    auto dist2 = [&](float4 c) {
        const float dx = c.x - px, dy = c.y - py, dz = c.z - pz;
        return fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    };
    auto cid = [](float4 c) { return __builtin_bit_cast(uint32_t, c.w); };

    auto rdf_one = [&](bool valid, float4 c, float d2) {
        bool ok = valid && d2 < T.thr2;
        if (SELF) ok = ok && !(d2 == 0.0f && cid(c) == i);     // the target itself
        if (ok) rdf_count<LDS_HIST>(T, px, py, pz, c, d2);
        ++steps;
    };

    // ---- kNN: keys of candidates in (rk2_prev, rk2] into the LDS buffer
    int cnt = 0;                        // keys in kbuf
    uint64_t thr_key = ~0ull;           // keys must be below this once the buffer was cut
    float rk = KNN ? fminf(T.rk0, T.rknn) : 0.0f;
    float rk2 = (KNN && rk >= T.rknn) ? T.rknn2 : rk * rk;
    float rk2_prev = -1.0f;
    auto knn_one = [&](bool valid, float4 c, float d2) {
        const uint32_t j = cid(c);
        bool q = valid && d2 <= rk2 && d2 > rk2_prev;
        if (SELF) q = q && j != i;
        const uint64_t key = ((uint64_t)f2u(d2) << 32) | (uint64_t)j;
        q = q && key < thr_key;
        uint64_t m = __ballot(q);
        if (m) {
            int nn = __popcll(m);
            // for small k the buffer is cut at 64 keys (once it holds k),
            // so that cuts and the final sort stay within one wavefront's
            // rank sort and later candidates meet the raised bar sooner
            if (cnt + nn > (T.k <= 32 ? kWave : kKnnCap) && cnt >= T.k) {
                // keep the k smallest keys, raise the bar to the k-th
                wave_sort_keys(T.kbuf, cnt);
                cnt = T.k;
                thr_key = T.kbuf[T.k - 1];
                q = q && key < thr_key;
                m = __ballot(q);
                nn = __popcll(m);
            }
            if (q) T.kbuf[cnt + __popcll(m & lanemask_lt())] = key;
            cnt += nn;
            wave_sync();
        }
    };

    if (finite) {
        if (RDF && (!KNN || rk * 1.000001f < T.r_enum)) {
            enumerate(P, T.cell_start, T.bpos, px, py, pz, T.r_enum,
                      [&](bool v, float4 c) { rdf_one(v, c, dist2(c)); });
            if (KNN)
                enumerate(P, T.cell_start, T.bpos, px, py, pz, rk * 1.000001f,
                          [&](bool v, float4 c) { knn_one(v, c, dist2(c)); }, true);
        } else if (RDF) {
            // the first kNN radius covers r_max: one enumeration for both
            enumerate(P, T.cell_start, T.bpos, px, py, pz, rk * 1.000001f, [&](bool v, float4 c) {
                const float d2 = dist2(c);
                rdf_one(v, c, d2);
                knn_one(v, c, d2);
            }, true);
        } else if (KNN) {
            enumerate(P, T.cell_start, T.bpos, px, py, pz, rk * 1.000001f,
                      [&](bool v, float4 c) { knn_one(v, c, dist2(c)); }, true);
        }
        if (KNN) {
            // grow the radius until k keys are certain (or everything was seen)
            while (cnt < T.k && rk < T.rknn && rk < P.r_all) {
                float g = cbrtf((float)(T.k + 1) / (float)(cnt + 1)) * 1.1f;
                g = fminf(fmaxf(g, 1.25f), 4.0f);
                rk2_prev = rk2;
                rk = fminf(rk * g, fminf(T.rknn, P.r_all));
                rk2 = rk >= T.rknn ? T.rknn2 : rk * rk;
                enumerate(P, T.cell_start, T.bpos, px, py, pz, rk * 1.000001f,
                          [&](bool v, float4 c) { knn_one(v, c, dist2(c)); }, true);
            }
        }
    }
    if (!KNN) return 0;
    wave_sort_keys(T.kbuf, cnt);
    (void)l;
    return cnt < T.k ? cnt : T.k;
}

// ---------------------------------------------------------------- tiles --
// Bin of a k-th squared distance as far as FP32 decides it (the band of
// key_bin, below): -1 where the FP64 distance has to.
__device__ __forceinline__ int kth_bin_fp32(float d2, int kb_nbins, double kb_inv_w64) {
    const float t = __builtin_amdgcn_sqrtf(d2) * (float)kb_inv_w64;
    if (!(t < (float)kb_nbins + 2.0f)) return kb_nbins;
    const float band = (float)fmin(0.25, fmax(1e-6 * kb_inv_w64, 4e-6 * (double)kb_nbins));
    const int bf = (int)t;
    const float fr = t - (float)bf;
    if (fr > band && fr < 1.0f - band) return bf < kb_nbins ? bf : kb_nbins;
    return -1;
}

// 64 targets per wavefront, one per lane: the neighbour records within R of
// the targets' bounding box are staged through LDS in chunks, and every lane
// scans them for its own target.  Used when targets are dense, so that the
// 64 targets of a tile are close together.
constexpr int kStage = 512;   // records per staging chunk (16 B each)

// Whether a record can lie within R of the box (R2 = (R + eps)^2).  The rows
// that enumerate_box trims end at whole cells, a third or more of whose records
// lie farther: tested once per record of a tile, by one lane, they are never
// scanned by 64 (7.5e6 dense targets, k = 10: the kernel 1.55 -> 1.32 ms; eight
// replicates of six pairs 13.7 -> 10.9).
__device__ __forceinline__ bool box_near(float4 c, float x0, float y0, float z0, float x1, float y1, float z1, float R2) {
    const float ex = fmaxf(0.0f, fmaxf(x0 - c.x, c.x - x1));
    const float ey = fmaxf(0.0f, fmaxf(y0 - c.y, c.y - y1));
    const float ez = fmaxf(0.0f, fmaxf(z0 - c.z, c.z - z1));
    return ex * ex + ey * ey + ez * ez <= R2;
}

template <int KMAX>
struct TopK {
    uint64_t key[KMAX > 0 ? KMAX : 1];
};

// RDF only, with any number of records; counted(bound) after each scan.
template <int FLAGS, class C>
__device__ __forceinline__ void run_tile(const GridPlan& P, const PairTask& T, bool valid, float px, float py, float pz,
                                         uint32_t i, float4* stage, C&& counted) {
    constexpr bool LDS_HIST = (FLAGS & kRdfLds) != 0;
    constexpr bool SELF = (FLAGS & kSelf) != 0;
    const bool fin = valid && isfinite(px) && isfinite(py) && isfinite(pz);
    if (!__any(fin)) return;
    const float x0 = wave_min_f(fin ? px : INFINITY), x1 = wave_max_f(fin ? px : -INFINITY);
    const float y0 = wave_min_f(fin ? py : INFINITY), y1 = wave_max_f(fin ? py : -INFINITY);
    const float z0 = wave_min_f(fin ? pz : INFINITY), z1 = wave_max_f(fin ? pz : -INFINITY);
    auto scan = [&](int m) {
        wave_sync();
        for (int j = 0; j < m; ++j) {
            const float4 c = stage[j];
            const float dx = c.x - px, dy = c.y - py, dz = c.z - pz;
            const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            if (fin && (!SELF || __builtin_bit_cast(uint32_t, c.w) != i) && d2 < T.thr2)
                rdf_count<LDS_HIST>(T, px, py, pz, c, d2);
        }
        wave_sync();
        counted((uint32_t)m * kWave);
    };
    int m = 0;   // staged records
    const float Re = T.r_enum + P.eps, Re2 = Re * Re;
    enumerate_box(P, T.cell_start, T.bpos, x0, y0, z0, x1, y1, z1, T.r_enum, [&](bool v, float4 c) {
        v = v && box_near(c, x0, y0, z0, x1, y1, z1, Re2);
        const uint64_t bal = __ballot(v);
        const int nn = __popcll(bal);
        if (m + nn > kStage) {
            scan(m);
            m = 0;
        }
        if (v) stage[m + __popcll(bal & lanemask_lt())] = c;
        m += nn;
    });
    if (m > 0) scan(m);
}

// RDF and kNN keys, with the records of a tile in the stage at once:
// the scan keeps KMAX + 2 values per lane, each the squared distance's bits
// with the lowest kSlotBits replaced by the record's place in the stage, as
// floats in ascending order (one median per place); afterwards the KMAX + 2
// records are read back, their exact keys sorted, and the rows are certain
// unless a record left out could tie: its value, so its distance rounded
// down, is at least the last one kept.  Keeping the 64-bit keys themselves in
// order cost a 64-bit comparison and four selects per place and candidate
// (7.5e6 dense targets, k = 10: 2.64 ms against 1.56).
// Returns false, with nothing counted, when the stage cannot hold the tile's
// records (the caller leaves its targets to the one-by-one pass); *unsure:
// this lane's rows may miss a tie and have to be searched again.
constexpr int kSlotBits = 9;
static_assert((1 << kSlotBits) == kStage, "a stage place per slot");

template <int FLAGS, int KMAX>
__device__ __forceinline__ bool run_tile_packed(const GridPlan& P, const PairTask& T, bool valid, float px, float py,
                                                float pz, uint32_t i, float Rk, int k, float4* stage, TopK<KMAX>& top,
                                                bool* unsure) {
    constexpr bool RDF = (FLAGS & (kRdfLds | kRdfGlobal)) != 0;
    constexpr bool LDS_HIST = (FLAGS & kRdfLds) != 0;
    constexpr bool SELF = (FLAGS & kSelf) != 0;
    constexpr int S = KMAX + 2;
    constexpr uint32_t kSlot = (1u << kSlotBits) - 1u;
    *unsure = false;
#pragma unroll
    for (int q = 0; q < KMAX; ++q) top.key[q] = ~0ull;
    const float rk2 = Rk * Rk;
    if (!(rk2 < 1e38f)) return false;   // squared distances below stay finite values
    const bool fin = valid && isfinite(px) && isfinite(py) && isfinite(pz);
    if (!__any(fin)) return true;
    const float x0 = wave_min_f(fin ? px : INFINITY), x1 = wave_max_f(fin ? px : -INFINITY);
    const float y0 = wave_min_f(fin ? py : INFINITY), y1 = wave_max_f(fin ? py : -INFINITY);
    const float z0 = wave_min_f(fin ? pz : INFINITY), z1 = wave_max_f(fin ? pz : -INFINITY);
    const float R = RDF ? fmaxf(T.r_enum, Rk * 1.000001f) : Rk * 1.000001f;
    int m = 0;
    const float Re = R + P.eps, Re2 = Re * Re;
    enumerate_box(P, T.cell_start, T.bpos, x0, y0, z0, x1, y1, z1, R, [&](bool v, float4 c) {
        v = v && box_near(c, x0, y0, z0, x1, y1, z1, Re2);
        const uint64_t bal = __ballot(v);
        const int nn = __popcll(bal);
        if (v && m + nn <= kStage) stage[m + __popcll(bal & lanemask_lt())] = c;
        m += nn;
    }, true);
    wave_sync();
    if (m > kStage) return false;

    // (the largest finite value: no record within Rk)
    const float none = u2f(0x7F7FFFFFu);
    float kept[S];
#pragma unroll
    for (int q = 0; q < S; ++q) kept[q] = none;
    float4 next = stage[0];
    for (int j = 0; j < m; ++j) {
        const float4 c = next;
        next = stage[j + 1 < m ? j + 1 : j];
        const float dx = c.x - px, dy = c.y - py, dz = c.z - pz;
        const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        const bool me = fin && (!SELF || __builtin_bit_cast(uint32_t, c.w) != i);
        if (RDF && me && d2 < T.thr2) rdf_count<LDS_HIST>(T, px, py, pz, c, d2);
        const float x = me && d2 <= rk2 ? u2f((f2u(d2) & ~kSlot) | (uint32_t)j) : none;
        if (__any(x < kept[S - 1])) {
#pragma unroll
            for (int q = S - 1; q > 0; --q) kept[q] = __builtin_amdgcn_fmed3f(kept[q - 1], x, kept[q]);
            kept[0] = fminf(kept[0], x);
        }
    }
    // exact keys, sorted (they are nearly so: only equal leading bits can be
    // out of order, so a few passes of neighbours suffice and one without an
    // exchange ends them)
    uint64_t key[S];
#pragma unroll
    for (int q = 0; q < S; ++q) {
        key[q] = ~0ull;
        if (kept[q] < none) {
            const float4 c = stage[f2u(kept[q]) & kSlot];
            const float dx = c.x - px, dy = c.y - py, dz = c.z - pz;
            const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            key[q] = ((uint64_t)f2u(d2) << 32) | (uint64_t)__builtin_bit_cast(uint32_t, c.w);
        }
    }
    for (int pass = 0; pass < S; ++pass) {
        bool moved = false;
#pragma unroll
        for (int q = 0; q + 1 < S; ++q) {
            const uint64_t a = key[q], b = key[q + 1];
            const bool sw = b < a;
            key[q] = sw ? b : a;
            key[q + 1] = sw ? a : b;
            moved = moved || sw;
        }
        if (!__any(moved)) break;
    }
    uint64_t kth = key[0];
#pragma unroll
    for (int q = 1; q < KMAX; ++q)
        if (q == k - 1) kth = key[q];
    // a record not kept has at least the last value's leading bits
    if (kept[S - 1] < none) *unsure = (uint32_t)(kth >> 32) >= (f2u(kept[S - 1]) & ~kSlot);
#pragma unroll
    for (int q = 0; q < KMAX; ++q) top.key[q] = key[q];
    wave_sync();
    return true;
}

// One target per lane: each lane walks the cell rows within R of its own
// target (rows trimmed to the x-range the sphere reaches, as in
// enumerate_box) and reads the records one by one, kLaneU of them in flight;
// no staging, and no lane waits on a shared candidate list.  Same results as
// run_tile (same candidate set, order-free updates).  Without an RDF only
// the kNN keys within Rk are taken (a small radius when the neighbours are
// dense: a few dozen records per lane).  Adds this lane's RDF counts to `hits`.
// Eight records in flight per lane
// (2e9-ion needle, 1.0 nm cells: 23.4 ms with four, 22.4 with eight, 34
// with two; sixteen spill).
constexpr int kLaneU = 8;

template <int FLAGS, int KMAX>
__device__ __forceinline__ void run_lane(const GridPlan& P, const PairTask& T, bool valid, float px, float py,
                                         float pz, uint32_t i, float Rk, TopK<KMAX>& top, uint32_t& hits) {
    constexpr bool RDF = (FLAGS & (kRdfLds | kRdfGlobal)) != 0;
    constexpr bool LDS_HIST = (FLAGS & kRdfLds) != 0;
    constexpr bool SELF = (FLAGS & kSelf) != 0;
#pragma unroll
    for (int m = 0; m < (KMAX > 0 ? KMAX : 1); ++m) top.key[m] = ~0ull;
    const bool fin = valid && isfinite(px) && isfinite(py) && isfinite(pz);
    const float rk2 = Rk * Rk;
    float R = 0.0f;
    if (RDF) R = T.r_enum;
    if (KMAX > 0) R = fmaxf(R, Rk * 1.000001f);
    const float Re = R + P.eps;
    const float R2 = Re * Re;
    const int cy0 = cell_axis(P, 1, py - Re), cy1 = cell_axis(P, 1, py + Re);
    const int cz0 = cell_axis(P, 2, pz - Re), cz1 = cell_axis(P, 2, pz + Re);
    const int ny = cy1 - cy0 + 1, nz = cz1 - cz0 + 1;
    const int nrows = fin ? ny * nz : 0;
    int r = 0;                     // next row of this lane
    uint32_t j = 0, j1 = 0;        // records left in the current row
    for (;;) {
        // advance to the next row with records (rows beyond R are empty)
        while (j >= j1 && r < nrows) {
            const int cz = cz0 + centre_out(r / ny, nz), cy = cy0 + centre_out(r % ny, ny);
            ++r;
            uint32_t st, len;
            row_span(P, T.cell_start, cy, cz, px, py, pz, px, py, pz, R2, st, len);
            if (len) {
                j = st;
                j1 = st + len;
            }
        }
        if (j >= j1) break;
        float4 c[kLaneU];
#pragma unroll
        for (int u = 0; u < kLaneU; ++u) c[u] = T.bpos[j + (uint32_t)u < j1 ? j + (uint32_t)u : j];
        // (all of them issued before the first is waited for: with the last two
        // after it the 4e8-ion needle's Sc targets took 5.1 ms, now 4.4)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kLaneU; ++u) {
            if (j + (uint32_t)u >= j1) break;
            const float dx = c[u].x - px, dy = c[u].y - py, dz = c[u].z - pz;
            const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            const uint32_t cj = __builtin_bit_cast(uint32_t, c[u].w);
            const bool me = !SELF || cj != i;
            if (RDF && me && d2 < T.thr2) {
                rdf_count<LDS_HIST>(T, px, py, pz, c[u], d2);
                ++hits;
            }
            if (KMAX > 0) {
                const uint64_t key = ((uint64_t)__builtin_bit_cast(uint32_t, d2) << 32) | (uint64_t)cj;
                if (me && d2 <= rk2 && key < top.key[KMAX - 1]) {
                    // (from the last place down: one comparison per place, none
                    // waiting for another)
                    bool here = true;   // key < top.key[q]
#pragma unroll
                    for (int q = KMAX - 1; q > 0; --q) {
                        const bool before = key < top.key[q - 1];
                        top.key[q] = before ? top.key[q - 1] : here ? key : top.key[q];
                        here = before;
                    }
                    top.key[0] = here ? key : top.key[0];
                }
            }
        }
        j += kLaneU;
    }
}

// The k-th key of each lane's target only (with the RDF counts), for the
// k-th distance histogram: the scan keeps the k smallest squared distances,
// ascending, with one median per place (place q takes the middle of its left
// neighbour, the newcomer and itself), and no indices.  An index is needed only
// where FP32 leaves the k-th distance's bin open, about one target in 25: the
// wavefront then looks through the staged records for it together.  (A second
// enumeration and scan for all lanes' indices, and a minimum and a maximum per
// place, took the 7.7e6-ion needle's dense pairs 2.8 ms per replicate
// instead of 2.0.)  Tiles with more candidates than the stage holds
// enumerate twice.  kb_nbins <= 0: no histogram, no index needed.  Returns the
// k-th key (FP32 d2 bits << 32 | index), or ~0 when it is not settled here:
// fewer than k neighbours within Rk, or an index needed at a distance that
// several of the k nearest share (the caller finishes those targets exactly).
template <int FLAGS, int KMAX, class C>
__device__ __forceinline__ uint64_t run_tile_kth(const GridPlan& P, const PairTask& T, bool valid, float px,
                                                 float py, float pz, uint32_t i, float Rk, int k, float4* stage,
                                                 C&& counted, int kb_nbins, double kb_inv_w64) {
    constexpr bool RDF = (FLAGS & (kRdfLds | kRdfGlobal)) != 0;
    constexpr bool LDS_HIST = (FLAGS & kRdfLds) != 0;
    constexpr bool SELF = (FLAGS & kSelf) != 0;
    static_assert(KMAX > 0, "k-th key needs KMAX > 0");
    const int l = lane_id();
    const bool fin = valid && isfinite(px) && isfinite(py) && isfinite(pz);
    if (!__any(fin)) return ~0ull;
    const float x0 = wave_min_f(fin ? px : INFINITY), x1 = wave_max_f(fin ? px : -INFINITY);
    const float y0 = wave_min_f(fin ? py : INFINITY), y1 = wave_max_f(fin ? py : -INFINITY);
    const float z0 = wave_min_f(fin ? pz : INFINITY), z1 = wave_max_f(fin ? pz : -INFINITY);
    const float rk2 = Rk * Rk;
    const float R = RDF ? fmaxf(T.r_enum, Rk * 1.000001f) : Rk * 1.000001f;
    float top[KMAX];
#pragma unroll
    for (int q = 0; q < KMAX; ++q) top[q] = INFINITY;

    auto scan = [&](int m) {
        wave_sync();
        float4 next = stage[0];
        for (int j = 0; j < m; ++j) {
            const float4 c = next;
            next = stage[j + 1 < m ? j + 1 : j];
            const float dx = c.x - px, dy = c.y - py, dz = c.z - pz;
            const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            const uint32_t cj = __builtin_bit_cast(uint32_t, c.w);
            const bool me = fin && (!SELF || cj != i);
            if (RDF && me && d2 < T.thr2) rdf_count<LDS_HIST>(T, px, py, pz, c, d2);
            const bool in = me && d2 <= rk2;
            if (__ballot(in && d2 < top[KMAX - 1])) {
                const float x = in ? d2 : INFINITY;
#pragma unroll
                for (int q = KMAX - 1; q > 0; --q) top[q] = __builtin_amdgcn_fmed3f(top[q - 1], x, top[q]);
                top[0] = fminf(top[0], x);
            }
        }
        wave_sync();
        if (RDF) counted((uint32_t)m * kWave);
    };
    int m = 0;              // records in the stage
    bool once = true;       // it holds all of the tile's
    auto stage_one = [&](auto&& sc, float Rs) {
        const float Re = Rs + P.eps, Re2 = Re * Re;
        return [&, sc, Re2](bool v, float4 c) {
            v = v && box_near(c, x0, y0, z0, x1, y1, z1, Re2);
            const uint64_t bal = __ballot(v);
            const int nn = __popcll(bal);
            if (m + nn > kStage) {
                sc(m);
                m = 0;
                once = false;
            }
            if (v) stage[m + __popcll(bal & lanemask_lt())] = c;
            m += nn;
        };
    };
    enumerate_box(P, T.cell_start, T.bpos, x0, y0, z0, x1, y1, z1, R, stage_one(scan, R), true);
    if (m > 0) scan(m);

    // the k-th distance and how many of the k nearest lie strictly nearer
    float tau = top[0];
#pragma unroll
    for (int q = 1; q < KMAX; ++q)
        if (q == k - 1) tau = top[q];
    int nearer = 0;
#pragma unroll
    for (int q = 0; q < KMAX; ++q) nearer += (q < k && top[q] < tau);
    // the smallest index at exactly the k-th distance, for the lanes that need
    // it (others keep an index that nothing reads, and may share the distance)
    const bool within = fin && tau <= rk2;
    const bool needs = within && kb_nbins > 0 && kth_bin_fp32(tau, kb_nbins, kb_inv_w64) < 0;
    const bool open = needs && nearer == k - 1;
    bool settled = within && (open || !needs);
    uint32_t jk = open ? 0xFFFFFFFFu : 0u;
    if (once) {
        for (uint64_t todo = __ballot(open); todo; todo &= todo - 1) {
            const int ln = __builtin_ctzll(todo);
            const uint32_t ti = readlane(i, ln);
            const float tx = readlane(px, ln), ty = readlane(py, ln), tz = readlane(pz, ln), tt = readlane(tau, ln);
            uint32_t best = 0xFFFFFFFFu;
            for (int j0 = 0; j0 < m; j0 += kWave) {
                const float4 c = stage[j0 + l < m ? j0 + l : j0];
                const float dx = c.x - tx, dy = c.y - ty, dz = c.z - tz;
                const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                const uint32_t cj = __builtin_bit_cast(uint32_t, c.w);
                for (uint64_t hit = __ballot(j0 + l < m && d2 == tt && (!SELF || cj != ti)); hit; hit &= hit - 1) {
                    const uint32_t cand = readlane(cj, __builtin_ctzll(hit));
                    best = cand < best ? cand : best;
                }
            }
            if (l == ln) jk = best;
        }
    } else if (__any(open)) {
        const float tmax = wave_max_f(open ? tau : 0.0f);
        auto scan2 = [&](int mm) {
            wave_sync();
            for (int j = 0; j < mm; ++j) {
                const float4 c = stage[j];
                const float dx = c.x - px, dy = c.y - py, dz = c.z - pz;
                const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                const uint32_t cj = __builtin_bit_cast(uint32_t, c.w);
                const bool me = open && (!SELF || cj != i);
                if (me && d2 == tau && cj < jk) jk = cj;
            }
            wave_sync();
        };
        m = 0;
        const float Rt = sqrtf(tmax) * 1.000001f;
        enumerate_box(P, T.cell_start, T.bpos, x0, y0, z0, x1, y1, z1, Rt, stage_one(scan2, Rt));
        if (m > 0) scan2(m);
    }
    settled = settled && jk != 0xFFFFFFFFu;
    return settled ? (((uint64_t)__builtin_bit_cast(uint32_t, tau) << 32) | (uint64_t)jk) : ~0ull;
}

// RDF counts of one target after `steps` steps of 64 candidates, at most: the
// candidates of full steps, and never more than the nB neighbours (a step that
// ends a group of 64 rows may be nearly empty, one for each group that holds a
// record).
__device__ __forceinline__ uint32_t counts_of(uint32_t steps, uint32_t nB) {
    return steps < nB / (uint32_t)kWave ? steps * (uint32_t)kWave : nB;
}
// The counts from which a wavefront's u32 LDS counters are flushed before
// another target: below it, that target's nB at most still fit.
__device__ __forceinline__ uint32_t flush_limit(uint32_t nB) { return 0xFFFFFFFFu - nB; }

// Flush a per-wavefront u32 LDS histogram into a global u64 histogram.
__device__ __forceinline__ void flush_hist(uint32_t* hist_l, uint64_t* hist_g, int n_bins) {
    for (int b = lane_id(); b < n_bins; b += kWave) {
        const uint32_t v = hist_l[b];
        if (v) atomicAdd((unsigned long long*)&hist_g[b], (unsigned long long)v);
        hist_l[b] = 0;
    }
    wave_sync();
}

// The last flush of a kernel: a workgroup's wavefronts' histograms (`stride`
// counters apart) summed before one global atomic per bin.  All wavefronts of
// a launch end together and add to the same few bins, and atomics on one
// address take about 16 ns each: 6144 wavefronts' own flushes were 0.1 ms on
// every bin.  Every thread of the workgroup calls it.
__device__ __forceinline__ void flush_hist_block(const uint32_t* hist_l, int stride, uint64_t* hist_g, int n_bins) {
    __syncthreads();
    for (int b = (int)threadIdx.x; b < n_bins; b += kBlock) {
        unsigned long long v = 0;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) v += hist_l[w * stride + b];
        if (v) atomicAdd((unsigned long long*)&hist_g[b], v);
    }
}

// Bin of the distance of a kNN key (bits(d2f) << 32 | index) in the k-th
// distance histogram: the FP32 bin of the key's squared distance, exact
// away from the edges (the same band as the RDF's fast path: the FP32
// squared distance, root and scaling err by a few ulps); inside the band,
// the FP64 distance of the stored positions decides.
__device__ __forceinline__ int key_bin(uint64_t key, const float* xyz, float px, float py, float pz,
                                       const double* KE2, int kb_nbins, double kb_inv_w64) {
    const int bf = kth_bin_fp32(u2f((uint32_t)(key >> 32)), kb_nbins, kb_inv_w64);
    if (bf >= 0) return bf;
    const uint32_t j = (uint32_t)key;
    return exact_bin(exact_D2(px, py, pz, xyz[3 * (size_t)j], xyz[3 * (size_t)j + 1], xyz[3 * (size_t)j + 2]),
                     KE2, kb_nbins, kb_inv_w64);
}

// Bin of the k-th neighbour's distance (kb_nbins when missing).
__device__ __forceinline__ int kth_bin(int found, int k, const uint64_t* kbuf, const float* xyz, float px,
                                       float py, float pz, const double* KE2, int kb_nbins, double kb_inv_w64) {
    if (found < k) return kb_nbins;
    return key_bin(kbuf[k - 1], xyz, px, py, pz, KE2, kb_nbins, kb_inv_w64);
}

}  // namespace apt
