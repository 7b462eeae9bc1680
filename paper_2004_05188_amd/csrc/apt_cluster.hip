// Maximum-separation clustering (paper, Methods: "Descriptive, two-point
// spatial statistics, and clustering": the MS method, a DBScan variant with
// the parameters d_max and N_min; Supplementary, "Efficient batch processing
// of spatial statistics": clusters with ions at the dataset edge are
// flagged as truncated).
//
// The ions of the species are binned as targets and neighbours of one query;
// every target visits its neighbours within d_max (the RDF's row
// enumeration, one target per wavefront) and links each pair once, from its
// lower index, in a union-find forest over ion indices.  A link hooks the
// larger of the two roots under the smaller (compare-and-swap on the root),
// so the root of every tree is its smallest ion index: the cluster's name
// does not depend on the order of the links.  Finds halve the path with
// plain stores: a pointer only ever moves to an ancestor, and a vertex that
// is not a root never becomes one again, so every interleaving leaves a
// valid forest.  The pair test is the FP32 squared distance, re-decided in
// FP64 (differences of the stored FP32 coordinates) near d_max.
#include "apt_cluster.hpp"
#include "apt_pairdev.hpp"

namespace apt {

__device__ __forceinline__ uint32_t uf_load(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void uf_store(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t uf_find(uint32_t* parent, uint32_t x) {
    for (;;) {
        const uint32_t p = uf_load(parent + x);
        if (p == x) return x;
        const uint32_t g = uf_load(parent + p);
        if (g == p) return p;
        uf_store(parent + x, g);      // halving: x now points at its grandparent
        x = g;
    }
}

__device__ __forceinline__ void uf_union(uint32_t* parent, uint32_t a, uint32_t b) {
    for (;;) {
        a = uf_find(parent, a);
        b = uf_find(parent, b);
        if (a == b) return;
        if (a > b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        // hook the larger root under the smaller; if b stopped being a root
        // meanwhile, start again from where it went
        const uint32_t old = atomicCAS(parent + b, b, a);
        if (old == b) return;
        b = old;
    }
}

// The forest of the species' ions only (`tid`: their indices, ascending): the
// other ions' entries are never read, and writing all of them was 8 B an ion
// of a cloud whose species may be a hundredth of it.
__global__ __launch_bounds__(kBlock) void k_ms_init(ClusterOutArgs a) {
    const uint32_t nT = a.plan->nT;
    for (uint32_t t = blockIdx.x * kBlock + threadIdx.x; t < nT; t += gridDim.x * kBlock) {
        const uint32_t i = a.tid[t];
        a.parent[i] = i;
        a.size[i] = 0u;
    }
}

__global__ __launch_bounds__(kBlock) void k_ms_link(ClusterLinkArgs a) {
    const GridPlan P = *a.plan;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // XCD-aware deal of the targets in cell order (the grid is a multiple of kXcd)
    const int xcd = blockIdx.x % kXcd;
    const int per_xcd = gridDim.x / kXcd;
    const uint32_t wx = (uint32_t)(blockIdx.x / kXcd) * kWavesPerBlock + (uint32_t)w;
    const uint32_t wstride = (uint32_t)per_xcd * kWavesPerBlock;
    const uint32_t t0 = (uint32_t)((uint64_t)P.nT * (uint64_t)xcd / kXcd);
    const uint32_t t1 = (uint32_t)((uint64_t)P.nT * (uint64_t)(xcd + 1) / kXcd);
    for (uint32_t s = t0 + wx; s < t1; s += wstride) {
        const float4 own = a.t_id ? make_float4(a.tx[s], a.ty[s], a.tz[s], __builtin_bit_cast(float, a.t_id[s])) : a.bpos[s];
        const uint32_t i = __builtin_amdgcn_readfirstlane(__builtin_bit_cast(uint32_t, own.w));
        const float px = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, own.x)));
        const float py = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, own.y)));
        const float pz = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, own.z)));
        if (!(isfinite(px) && isfinite(py) && isfinite(pz))) continue;
        enumerate(P, a.cell_start, a.bpos, px, py, pz, a.r_enum, [&](bool valid, float4 c) {
            const uint32_t j = __builtin_bit_cast(uint32_t, c.w);
            if (!valid || j <= i) return;          // each pair once, from its lower index
            const float dx = c.x - px, dy = c.y - py, dz = c.z - pz;
            const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            if (!(d2 <= a.out2)) return;           // (NaN too: an ion without a finite position has no links)
            if (d2 > a.in2 && !(exact_D2(px, py, pz, c.x, c.y, c.z) <= a.lim2)) return;
            uf_union(a.parent, i, j);
        });
    }
}

__device__ __forceinline__ bool ms_species(uint8_t l, int A) { return A == APT_ANY || (int)l == A; }

// Every ion of the species finds its root (its cluster's smallest index) and
// counts itself there; an ion at the edge marks its root as truncated.
__global__ __launch_bounds__(kBlock) void k_ms_roots(ClusterOutArgs a) {
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < a.n; i += gridDim.x * kBlock) {
        if (!ms_species(a.lab[i], a.A)) {
            a.label[i] = -1;
            continue;
        }
        const uint32_t r = uf_find(a.parent, i);
        a.label[i] = (int64_t)r;
        atomicAdd(a.size + r, 1u);
        if (a.d_bnd && !(a.d_bnd[i] >= a.d_srf)) atomicOr(a.size + r, 0x80000000u);
    }
}

__device__ __forceinline__ unsigned long long wave_sum64(unsigned long long v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, d, kWave);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), d, kWave);
        v += ((unsigned long long)hi << 32) | lo;
    }
    return v;
}

// Labels of clusters below n_min become -1; every root adds its cluster to
// the size histogram and, when kept, to the counts.  Bound by the atomics:
// most clusters of a sparse species are single ions, so nearly every root
// adds to the same counter, and global atomics on one address run one after
// the other (about 12 ns each).  Sizes below kMsLdsSizes are therefore
// counted in LDS and merged once per workgroup, and the kernel runs over the
// species' ions instead of the whole cloud (7.7e6 ions, 77 000 of the
// species in 41 000 clusters: 503 -> 7 us).
__global__ __launch_bounds__(kBlock) void k_ms_final(ClusterOutArgs a) {
    __shared__ uint32_t s_size[kMsLdsSizes];
    __shared__ unsigned long long s_cnt[3];
    const uint32_t nT = a.plan->nT;
    // counters of the histogram that have an LDS copy (the last one counts
    // every size from n_size_bins on)
    const uint32_t n_lds = a.size_hist ? min((uint32_t)a.n_size_bins, (uint32_t)kMsLdsSizes) : 0u;
    for (uint32_t b = threadIdx.x; b < n_lds; b += kBlock) s_size[b] = 0u;
    if (threadIdx.x < 3) s_cnt[threadIdx.x] = 0ull;
    __syncthreads();
    uint32_t kept = 0, trunc = 0;
    unsigned long long ions = 0;
    for (uint32_t t = blockIdx.x * kBlock + threadIdx.x; t < nT; t += gridDim.x * kBlock) {
        const uint32_t i = a.tid[t];
        const uint32_t r = (uint32_t)a.label[i];
        const uint32_t sz = a.size[r];
        const uint32_t s = sz & 0x7FFFFFFFu;
        if ((int64_t)s < (int64_t)a.n_min) a.label[i] = -1;
        if (r != i) continue;                      // one visit per cluster: its root
        if (a.size_hist) {
            const uint32_t b = (s < (uint32_t)a.n_size_bins ? s : (uint32_t)a.n_size_bins) - 1u;
            if (b < n_lds) atomicAdd(&s_size[b], 1u);
            else atomicAdd((unsigned long long*)(a.size_hist + b), 1ull);
        }
        if ((int64_t)s >= (int64_t)a.n_min) {
            ++kept;
            trunc += sz >> 31;
            ions += s;
        }
    }
    // (every lane leaves the loop before the sums)
    kept = wave_sum(kept);
    trunc = wave_sum(trunc);
    ions = wave_sum64(ions);
    if (lane_id() == 0 && kept) {
        atomicAdd(&s_cnt[0], (unsigned long long)kept);
        atomicAdd(&s_cnt[1], (unsigned long long)trunc);
        atomicAdd(&s_cnt[2], ions);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < n_lds; b += kBlock)
        if (s_size[b]) atomicAdd((unsigned long long*)(a.size_hist + b), (unsigned long long)s_size[b]);
    if (threadIdx.x < 3 && s_cnt[threadIdx.x]) atomicAdd(a.counts + threadIdx.x, s_cnt[threadIdx.x]);
}

}  // namespace apt
