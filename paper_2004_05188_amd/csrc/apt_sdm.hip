// Two-point statistic: for every eligible target (one per wavefront), the
// neighbours within R found by the same row enumeration as the RDF, each
// pair's displacement vector p_j - p_i counted in a cubic voxel of [-R, R)^3.
//
// RDF and kNN integrate this statistic over directions (paper, Methods:
// "Descriptive, two-point spatial statistics, and clustering"; its sections
// through the target's plane are the spatial distribution maps, and the
// paper's SDMs take R = 2 nm with voxels of 0.025 nm, Results: "Strong
// scaling efficiency for hybrid execution").
//
// Exactness as for the RDF: the pair test and the voxel of each component
// are decided from the FP32 difference, and re-decided in FP64 (differences
// of the stored FP32 coordinates, the faces' FP64 table) inside a band
// around R and around every face that covers the FP32 rounding.
//
// Counts: 160^3 voxels are 33 MB, no copy of which fits LDS, and one global
// u64 atomic per pair ran at 2.4e10 pairs/s whatever else the kernel did.  So
// a wavefront buffers its pairs' voxel numbers in LDS, sorts a full buffer by
// run of 2^16 voxels (63 runs: one per lane) and appends each run's 16-bit
// numbers (fewer voxels make shorter runs) to that run's list, with one atomic per run and
// buffer; k_sdm_merge then counts a quarter of a run per workgroup in LDS and
// adds it to the histogram (7.7e6 ions, Sc against Al, 6.8e7 pairs: k_sdm 2.8
// ms; k_sdm_list 0.55 and k_sdm_merge 0.11 ms).  Pairs that no longer fit their list (the lists
// take the sort's freed arrays, 48 B per ion) are counted directly, and so are
// all pairs of calls with few of them or with more than 2^22 voxels.
#include "apt_sdm.hpp"
#include "apt_pairdev.hpp"

namespace apt {

// voxel of one displacement component: FP32 coordinate, FP64 near a face
__device__ __forceinline__ int sdm_axis(const SdmArgs& a, float v32, float pi, float pj) {
    const float t = (v32 + a.R) * a.inv_w;
    int m = (int)t;
    const float fr = t - (float)m;
    if (__builtin_expect(fr < a.band || fr > 1.0f - a.band || !(t >= 0.0f), 0)) {
#pragma clang fp contract(off)
        const double v = (double)pj - (double)pi;
        int q = (int)floor((v + (double)a.R) * ((double)a.n_vox / (2.0 * (double)a.R)));
        q = q < 0 ? 0 : (q > a.n_vox - 1 ? a.n_vox - 1 : q);
        while (q > 0 && v < a.F[q]) --q;
        while (q < a.n_vox - 1 && v >= a.F[q + 1]) ++q;
        return q;
    }
    return m < 0 ? 0 : (m > a.n_vox - 1 ? a.n_vox - 1 : m);
}

// A wavefront's buffered pairs.
struct SdmBuf {
    uint32_t v[kWave * kSdmItems];   // flat voxel numbers
    uint32_t first[kSdmRuns];        // count, then first place in the sorted buffer, of each run
    unsigned long long at[kSdmRuns]; // first place in each run's list
};

// The first cnt buffered pairs, sorted by run, to their lists.
__device__ __forceinline__ void sdm_flush(const SdmArgs& a, SdmBuf& B, int cnt, int xcd) {
    const int l = lane_id();
    uint32_t v[kSdmItems], rank[kSdmItems];
    wave_sync();
    B.first[l] = 0u;
    wave_sync();
#pragma unroll
    for (int u = 0; u < kSdmItems; ++u) {
        const int i = u * kWave + l;
        v[u] = i < cnt ? B.v[i] : 0u;
        rank[u] = i < cnt ? atomicAdd(&B.first[v[u] >> a.lg_run], 1u) : 0u;
    }
    wave_sync();
    const uint32_t n = B.first[l];
    const uint32_t first = wave_incl_scan(n) - n;
    B.first[l] = first;
    B.at[l] = n ? atomicAdd(a.used + xcd * kSdmRuns + l, (unsigned long long)n) : 0ull;
    wave_sync();
#pragma unroll
    for (int u = 0; u < kSdmItems; ++u)
        if (u * kWave + l < cnt) B.v[B.first[v[u] >> a.lg_run] + rank[u]] = v[u];
    wave_sync();
    for (int i = l; i < cnt; i += kWave) {
        const uint32_t w = B.v[i], r = w >> a.lg_run;
        const unsigned long long at = B.at[r] + (uint32_t)(i - (int)B.first[r]);
        if (at < a.cap) a.list[(size_t)(xcd * kSdmRuns + (int)r) * a.cap + at] = (uint16_t)(w & ((1u << a.lg_run) - 1u));
        else atomicAdd((unsigned long long*)&a.hist[w], 1ull);
    }
    wave_sync();
}

// LIST: through the lists.  Six wavefronts per SIMD without them; the
// buffers' LDS leaves five.
template <bool LIST>
__device__ __forceinline__ void sdm_targets(const SdmArgs& a, SdmBuf* B) {
    const GridPlan P = *a.plan;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const bool self = a.self_possible != 0;
    // XCD-aware deal of the targets in cell order (the grid is a multiple of kXcd)
    const int xcd = blockIdx.x % kXcd;
    const int per_xcd = gridDim.x / kXcd;
    const uint32_t wx = (uint32_t)(blockIdx.x / kXcd) * kWavesPerBlock + (uint32_t)w;
    const uint32_t wstride = (uint32_t)per_xcd * kWavesPerBlock;
    const uint32_t t0 = (uint32_t)((uint64_t)P.nT * (uint64_t)xcd / kXcd);
    const uint32_t t1 = (uint32_t)((uint64_t)P.nT * (uint64_t)(xcd + 1) / kXcd);
    const uint32_t nv = (uint32_t)a.n_vox;
    int cnt = 0;
    // the next target is loaded while this one's pairs are counted (not with the
    // lists, whose kernel has no registers left for it)
    uint32_t next_i = 0;
    float next_x = 0.0f, next_y = 0.0f, next_z = 0.0f;
    auto load = [&](uint32_t s) {
        if (s >= t1) return;
        next_i = a.t_id[s];
        next_x = a.tx[s];
        next_y = a.ty[s];
        next_z = a.tz[s];
    };
    if (!LIST) load(t0 + wx);
    for (uint32_t s = t0 + wx; s < t1; s += wstride) {
        if (LIST) load(s);
        const uint32_t i = __builtin_amdgcn_readfirstlane(next_i);
        const float px = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, next_x)));
        const float py = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, next_y)));
        const float pz = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, next_z)));
        if (!LIST) load(s + wstride);
        if (!(isfinite(px) && isfinite(py) && isfinite(pz))) continue;
        enumerate(P, a.cell_start, a.bpos, px, py, pz, a.r_enum, [&](bool valid, float4 c) {
            const float dx = c.x - px, dy = c.y - py, dz = c.z - pz;
            const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            bool ok = valid && d2 < a.out2;
            if (self) ok = ok && __builtin_bit_cast(uint32_t, c.w) != i;
            if (ok && __builtin_expect(!(d2 < a.in2), 0))
                ok = exact_D2(px, py, pz, c.x, c.y, c.z) < a.R2;   // near the sphere: FP64 decides
            uint32_t v = 0;
            if (ok) {
                const uint32_t mx = (uint32_t)sdm_axis(a, dx, px, c.x);
                const uint32_t my = (uint32_t)sdm_axis(a, dy, py, c.y);
                const uint32_t mz = (uint32_t)sdm_axis(a, dz, pz, c.z);
                v = (mz * nv + my) * nv + mx;                       // below 2^27
                if (!LIST) atomicAdd((unsigned long long*)&a.hist[v], 1ull);
            }
            if (LIST) {
                const uint64_t m = __ballot(ok);
                if (ok) B->v[cnt + __popcll(m & lanemask_lt())] = v;
                cnt += __popcll(m);
            }
        }, false, [&]() {
            // (a step adds at most kUnroll wavefronts of pairs)
            if (LIST && cnt > kWave * (kSdmItems - kUnroll)) {
                sdm_flush(a, *B, cnt, xcd);
                cnt = 0;
            }
        });
    }
    if (LIST && cnt > 0) sdm_flush(a, *B, cnt, xcd);
}

// Lists pay from about a million pairs (below, the merge's pass over the
// histogram costs more than the atomics it saves) and where a target has
// many: with ten neighbours each, the buffer's ballots and its LDS cost the
// enumeration more than the atomics (7.5e6 Al against Sc, 9 pairs each: 7.8
// against 5.4 ms; 77 000 Sc against Sc, 42 each: 0.27 / 0.26; against Al, 890
// each: 1.1 / 3.3).  The counts are expected ones at the mean density of the
// bounding box, which a needle fills by half.  Both kernels below see the same
// plan, so exactly one of the two works.
__device__ __forceinline__ bool sdm_by_list(const SdmArgs& a) {
    if (!a.list) return false;
    const GridPlan& P = *a.plan;
    double vol = 1.0;
    for (int c = 0; c < 3; ++c) vol *= fmax((double)P.hi[c] - (double)P.lo[c], (double)a.R);
    const double each = (double)P.nB * (4.1888 * (double)a.R * (double)a.R * (double)a.R) / vol;
    return each >= 32.0 && (double)P.nT * each >= 1.0e6;
}

__global__ __launch_bounds__(kBlock, 6) void k_sdm(SdmArgs a) {
    if (sdm_by_list(a)) return;
    sdm_targets<false>(a, nullptr);
}

__global__ __launch_bounds__(kBlock, 5) void k_sdm_list(SdmArgs a) {
    __shared__ SdmBuf B[kWavesPerBlock];
    if (!sdm_by_list(a)) return;
    sdm_targets<true>(a, &B[threadIdx.x / kWave]);
}

// Workgroup (q, r) counts quarter q of run r over the XCDs' lists.
__global__ __launch_bounds__(kSdmMergeBlock) void k_sdm_merge(SdmArgs a) {
    __shared__ uint32_t s_n[kSdmPart];
    const uint32_t q = blockIdx.x, r = blockIdx.y, lg_part = a.lg_run - 2u, part = 1u << lg_part;
    uint64_t any = 0;
    for (int x = 0; x < kXcd; ++x) any |= a.used[x * kSdmRuns + r];
    if (!any) return;
    for (uint32_t i = threadIdx.x; i < part; i += kSdmMergeBlock) s_n[i] = 0u;
    __syncthreads();
    for (int x = 0; x < kXcd; ++x) {
        const unsigned long long used = a.used[x * kSdmRuns + r];
        const uint32_t n = used < a.cap ? (uint32_t)used : a.cap;
        const uint16_t* __restrict__ L = a.list + (size_t)(x * kSdmRuns + (int)r) * a.cap;
        auto take = [&](uint32_t v) {
            if (v >> lg_part == q) atomicAdd(&s_n[v & (part - 1u)], 1u);
        };
        // eight numbers per load, four loads in flight (cap, and with it every
        // list, is a multiple of 64 entries from a 256-byte boundary)
        constexpr uint32_t kStep = kSdmMergeBlock * 8u, kLoads = 4;
        for (uint32_t i0 = threadIdx.x * 8u; i0 < n; i0 += kStep * kLoads) {
            uint4 v[kLoads];
#pragma unroll
            for (uint32_t u = 0; u < kLoads; ++u) {
                const uint32_t i = i0 + u * kStep;
                v[u] = *reinterpret_cast<const uint4*>(L + (i < n ? i : i0));
            }
#pragma unroll
            for (uint32_t u = 0; u < kLoads; ++u) {
                const uint32_t i = i0 + u * kStep;
                const uint32_t e[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (uint32_t k = 0; k < 8; ++k)
                    if (i + k < n) take((e[k / 2] >> (16 * (k % 2))) & 0xFFFFu);
            }
        }
    }
    __syncthreads();
    const uint32_t nv = (uint32_t)a.n_vox, total = nv * nv * nv, base = (r << a.lg_run) + q * part;
    for (uint32_t i = threadIdx.x; i < part; i += kSdmMergeBlock)
        if (s_n[i] && base + i < total) a.hist[base + i] += s_n[i];   // (this workgroup's voxels alone)
}

}  // namespace apt
