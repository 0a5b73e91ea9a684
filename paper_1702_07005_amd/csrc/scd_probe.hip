// scd_probe.hip -- set-up statistics for gfx950: how often each shared-vector entry is used (hits),
// the threshold that selects the most used entries, and the coupling probe.
//
// All of them scatter: one add per stored entry (hits) or nine (the probe's vectors).  Device-scope
// atomic adds run at 20-25 G requests/s of up to 64 bytes, and far slower where many hit one address
// (click-log data: the commonest values of a field are in a fifth of all rows).  So the adds of the
// most used entries are summed in LDS, a copy per workgroup, and only the sums go to memory; the
// others go there directly, a row of eight probes' sums as one request.  scd_create with an atomic per add, with
// slots, and with rows as one request too: 5 M click rows (195 M entries) 295, 37 and 18 ms, 50 M rows 2.5, 0.38 and
// 0.17 s, 350,000 text rows (1.3 B entries, a third of which have slots) 0.97, 0.50 and 0.20 s, 5 M entries spread evenly
// (no slots) 3.3, 2.9 and 1.05 ms.
#include <algorithm>

#include "scd_device.h"

namespace scd {

// ----------------------------------------------------------------------------------------
// hits[i] = number of stored entries with index i.  Each workgroup keeps a table of kCountSlots
// (index, count) pairs; the first index that reaches a slot holds it to the end, so an entry that is
// used often is nearly always counted in LDS.  Every entry is added exactly once, to its slot or to
// hits.  195 M click entries (39 fields, the commonest value 1.1 M times): 22.3 ms with one atomic per
// entry; 64 KB of table, two workgroups a CU.
// ----------------------------------------------------------------------------------------
constexpr int kCountThreads = 1024;
constexpr int kCountSlotBits = 13;
constexpr int kCountSlots = 1 << kCountSlotBits;
constexpr int kCountUnroll = 4;

__global__ __launch_bounds__(kCountThreads) void k_count_hits(const int32_t* __restrict__ idx, int64_t nnz,
                                                              unsigned* __restrict__ hits) {
    __shared__ unsigned tag[kCountSlots];  // index + 1, 0 = free
    __shared__ unsigned cnt[kCountSlots];
    for (int i = threadIdx.x; i < kCountSlots; i += kCountThreads) tag[i] = cnt[i] = 0u;
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * kCountThreads;
    for (int64_t b = (int64_t)blockIdx.x * kCountThreads + threadIdx.x; b < nnz; b += step * kCountUnroll) {
        unsigned ix[kCountUnroll];
#pragma unroll
        for (int r = 0; r < kCountUnroll; ++r) ix[r] = b + r * step < nnz ? (unsigned)idx[b + r * step] : 0xFFFFFFFFu;
#pragma unroll
        for (int r = 0; r < kCountUnroll; ++r) {
            if (ix[r] == 0xFFFFFFFFu) continue;  // past the end (indices are below 2^31)
            const unsigned slot = (ix[r] * 0x9E3779B1u) >> (32 - kCountSlotBits), mine = ix[r] + 1u;
            unsigned t = tag[slot];
            if (t == 0u) {
                t = atomicCAS(tag + slot, 0u, mine);
                if (t == 0u) t = mine;
            }
            if (t == mine)
                atomicAdd(cnt + slot, 1u);
            else
                atomicAdd(hits + ix[r], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kCountSlots; i += kCountThreads)
        if (cnt[i]) atomicAdd(hits + (tag[i] - 1u), cnt[i]);
}

__global__ __launch_bounds__(256) void k_max_u32(const unsigned* __restrict__ v, int64_t n, unsigned* __restrict__ out) {
    __shared__ unsigned red[4];
    unsigned best = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) best = max(best, v[i]);
    for (int o = 32; o > 0; o >>= 1) best = max(best, (unsigned)__shfl_xor((int)best, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        best = max(max(red[0], red[1]), max(red[2], red[3]));
        if (best) atomicMax(out, best);
    }
}

// bins[b] += entries v of hits with lo + b * width <= v < lo + (b + 1) * width and v < hi.
__global__ __launch_bounds__(256) void k_hits_histogram(const unsigned* __restrict__ hits, int64_t L, unsigned lo,
                                                        unsigned hi, unsigned width, unsigned* __restrict__ bins) {
    __shared__ unsigned h[kHitBins];
    for (int i = threadIdx.x; i < kHitBins; i += 256) h[i] = 0u;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < L; i += (int64_t)gridDim.x * 256) {
        const unsigned v = hits[i];
        if (v >= lo && v < hi) atomicAdd(h + (v - lo) / width, 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kHitBins; i += 256)
        if (h[i]) atomicAdd(bins + i, h[i]);
}

static unsigned stat_grid(int64_t n) { return (unsigned)std::min<int64_t>(1024, std::max<int64_t>(1, (n + 255) / 256)); }

hipError_t launch_count_hits(const int32_t* idx, int64_t nnz, unsigned* hits, hipStream_t s) {
    if (nnz <= 0) return hipSuccess;
    const int64_t per = (int64_t)kCountThreads * kCountUnroll;
    hipLaunchKernelGGL(k_count_hits, dim3((unsigned)std::min<int64_t>(512, (nnz + per - 1) / per)), dim3(kCountThreads), 0, s,
                       idx, nnz, hits);
    return hipGetLastError();
}

hipError_t launch_max_hits(const unsigned* hits, int64_t L, unsigned* out, hipStream_t s) {
    hipLaunchKernelGGL(k_max_u32, dim3(stat_grid(L)), dim3(256), 0, s, hits, L, out);
    return hipGetLastError();
}

hipError_t launch_hits_histogram(const unsigned* hits, int64_t L, unsigned lo, unsigned hi, unsigned width,
                                 unsigned* bins, hipStream_t s) {
    if (width < 1 || (hi - lo + width - 1) / width > (unsigned)kHitBins) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_hits_histogram, dim3(stat_grid(L)), dim3(256), 0, s, hits, L, lo, hi, width, bins);
    return hipGetLastError();
}

// Distinct keys that the workgroup's threads insert (open addressing in LDS; at most kLineEntries of them in twice as
// many places).  True for the one insertion of each key.
__device__ __forceinline__ bool line_insert(uint32_t* table, uint32_t key) {
    constexpr uint32_t places = 2 * kLineEntries;
    uint32_t at = (key * 0x9E3779B1u) % places;
    for (;;) {
        const uint32_t was = atomicCAS(table + at, 0xFFFFFFFFu, key);
        if (was == 0xFFFFFFFFu) return true;
        if (was == key) return false;
        at = (at + 1u) % places;
    }
}

// One workgroup per segment of the sample.  Exact for the entries it takes, in whatever order they are stored.
__global__ __launch_bounds__(256) void k_lines(const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx, uint32_t C,
                                               uint32_t* __restrict__ out) {
    __shared__ uint32_t table[2 * kLineEntries];
    const uint32_t c = (uint32_t)((uint64_t)blockIdx.x * C / gridDim.x);
    const int64_t s0 = ptr[c], len = ptr[c + 1] - s0;
    const uint32_t n = len < (int64_t)kLineEntries ? (uint32_t)len : kLineEntries;
    if (threadIdx.x == 0 && n) atomicAdd(out, n);
    for (int shift = 4; shift >= 3; --shift) {  // 16 fp32 or 8 fp64 entries a line
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < 2 * kLineEntries; i += 256) table[i] = 0xFFFFFFFFu;
        __syncthreads();
        uint32_t lines = 0;
        for (uint32_t i = threadIdx.x; i < n; i += 256) lines += line_insert(table, (uint32_t)idx[s0 + i] >> shift) ? 1u : 0u;
        for (int o = 32; o > 0; o >>= 1) lines += __shfl_xor(lines, o, 64);
        if ((threadIdx.x & 63) == 0 && lines) atomicAdd(out + (5 - shift), lines);
    }
}

hipError_t launch_lines(const int64_t* ptr, const int32_t* idx, uint32_t C, uint32_t* out, hipStream_t s) {
    if (const hipError_t e = launch_fill_zero(reinterpret_cast<uint64_t*>(out), kLineWords, s); e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lines, dim3(std::min(C, kLineSegments)), dim3(256), 0, s, ptr, idx, C, out);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------------
// Coupling probe.  With a~_c = sigma_c a_c / sqrt(|a_c|^2 + mu) (sigma_c = the label for the SVM, 1
// otherwise; mu = lambda N for the ridge steps, 0 for the SVM step), G = A~^T A~ holds the
// step-normalised couplings between coordinates.  A probe with Rademacher signs z_c scatters
// T = A~ z; the gather pass forms (A~^T T)_c - G_cc z_c, the off-diagonal part of (G z)_c, whose square
// has expectation kappa_c = sum_{j != c} G_cj^2 (Hutchinson), accumulated per coordinate.  z = 1
// (probe 0) gives the coherent sum |A~ 1|^2 instead.
//
// NP probes run in one pass over the matrix: T holds a row of NP values per shared-vector entry, so
// that the gather pass reads one 32-byte row per stored entry instead of eight entries of eight
// vectors, and the matrix is read twice instead of 17 times.  NP = 8 adds probe 0 into T0 in the same
// scatter; NP = 1 (no memory for the rows) runs probe 0 like the others.
//
// The scatter is bound by its atomics: the n_hot entries with slots in LDS (kProbeSlots at most, chosen
// where they have at least kProbeMinHits, several per workgroup) leave 20-60% of the entries on click
// and text data to go to memory.  One workgroup of 16 waves per CU when there are slots.
// ----------------------------------------------------------------------------------------
__device__ __forceinline__ float probe_sign(uint32_t c, uint32_t probe) {
    if (probe == 0) return 1.0f;
    return (murmur_fmix32(c ^ (probe * 0x9E3779B9u)) & 1u) ? 1.0f : -1.0f;
}

constexpr int kProbeUnroll = 4;  // entries per lane in flight

template <int G, int NP>
__global__ __launch_bounds__(1024) void k_probe_scatter(ProbeArgs a) {
    constexpr int W = NP > 1 ? NP + 1 : 1;  // sums per slot: the NP probes, and probe 0 beside eight
    extern __shared__ float acc[];
    const uint32_t n_acc = a.n_hot * W;
    for (uint32_t i = threadIdx.x; i < n_acc; i += blockDim.x) acc[i] = 0.0f;
    __syncthreads();
    const int lane = threadIdx.x & (G - 1), wlane = threadIdx.x & 63;
    const uint32_t ngroups = gridDim.x * (blockDim.x / G);
    const uint32_t c_wave = (blockIdx.x * blockDim.x + (threadIdx.x & ~63u)) / G;  // the wave's first group
    for (uint32_t cw = c_wave; cw < a.C; cw += ngroups) {  // the wave stays together: its lanes exchange entries below
        const uint32_t c = cw + (uint32_t)(wlane / G);
        const float sc = c < a.C ? a.norms[c] : 0.0f;
        const bool on = sc > 0.0f;
        const float coef = on ? (a.sign ? a.sign[c] : 1.0f) * rsqrtf(sc + a.mu) : 0.0f;
        uint32_t minus = 0;  // bit p: the sign of probe first + p is negative
#pragma unroll
        for (int p = 0; p < NP; ++p) minus |= (probe_sign(c, a.first + p) < 0.0f ? 1u : 0u) << p;
        const int64_t s0 = on ? a.ptr[c] : 0, s1 = on ? a.ptr[c + 1] : 0;
        for (int64_t b = s0 + lane; __any(b < s1); b += (int64_t)G * kProbeUnroll) {
            int ix[kProbeUnroll];
            float v[kProbeUnroll];
            uint32_t slot[kProbeUnroll];
#pragma unroll
            for (int r = 0; r < kProbeUnroll; ++r) {
                const int64_t k = b + (int64_t)r * G;
                ix[r] = -1;
                v[r] = 0.0f;
                if (k < s1) {
                    ix[r] = a.idx[k];
                    v[r] = coef * a.val[k];
                }
            }
#pragma unroll
            for (int r = 0; r < kProbeUnroll; ++r) slot[r] = a.n_hot && ix[r] >= 0 ? a.slot_of[ix[r]] : (uint32_t)kHotCold;
#pragma unroll
            for (int r = 0; r < kProbeUnroll; ++r) {
                if (slot[r] != kHotCold) {
                    float* q = acc + slot[r] * W;
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        __hip_atomic_fetch_add(q + p, (minus >> p) & 1u ? -v[r] : v[r], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                    if constexpr (NP > 1)
                        __hip_atomic_fetch_add(q + NP, v[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    ix[r] = -1;
                }
                if constexpr (NP == 1) {
                    if (ix[r] >= 0) atomic_add_u(a.T + ix[r], minus & 1u ? -v[r] : v[r]);
                } else {
                    static_assert(NP == 8, "eight lanes per row");
                    if (ix[r] >= 0) atomic_add_u(a.T0 + ix[r], v[r]);
                    // Eight entries at a time, a lane per probe: a row's eight adds are one 32-byte request, and rows
                    // that follow one another share lines.  With a lane per entry they were eight requests to as many
                    // lines as there are entries, which took segments of neighbouring entries longer than one pass
                    // per probe does (8,000 x 1,000 dense, scd_create: 1.76 ms with passes, 2.88, now 0.88; 5 M click
                    // rows 37.3 -> 19.2).
                    const int p = wlane & 7;
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int from = j * 8 + (wlane >> 3);
                        const int row = __shfl(ix[r], from);
                        const float x = __shfl(v[r], from);
                        const uint32_t m = (uint32_t)__shfl((int)minus, from);
                        if (row >= 0) atomic_add_u(a.T + (size_t)row * NP + p, (m >> p) & 1u ? -x : x);
                    }
                }
            }
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_acc; i += blockDim.x) {
        const float x = acc[i];
        if (x == 0.0f) continue;
        const uint32_t id = (uint32_t)a.hot_ids[i / W], p = i % W;
        if (NP > 1 && p == (uint32_t)NP)
            atomic_add_u(a.T0 + id, x);
        else
            atomic_add_u(a.T + (size_t)id * NP + p, x);
    }
}

// kappa sums of probes first .. first + NP - 1.  K (NP = 1) accumulates over calls; max_bits receives
// the largest per-coordinate mean over `probes` probes (non-negative floats order like their bit
// patterns) in the last call, null before.
template <int G, int NP>
__global__ __launch_bounds__(256) void k_probe_gather(ProbeArgs a) {
    constexpr int R = NP > 1 ? 2 : 8;
    __shared__ float red[4];
    const int lane = threadIdx.x & (G - 1);
    const uint32_t ngroups = gridDim.x * (256u / G);
    float best = 0.0f;
    for (uint32_t c = (blockIdx.x * 256u + threadIdx.x) / G; c < a.C; c += ngroups) {
        const float sc = a.norms[c];
        if (!(sc > 0.0f)) continue;
        double d[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) d[p] = 0.0;
        const int64_t s0 = a.ptr[c], s1 = a.ptr[c + 1];
        for (int64_t b = s0 + lane; b < s1; b += (int64_t)G * R) {
            int ix[R];
            float v[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                // Stands in with an entry of the same segment: T is finite (its entries are sums of entries of unit vectors).
                const bool in = b + (int64_t)r * G < s1;
                const int64_t k = in ? b + (int64_t)r * G : b;
                ix[r] = a.idx[k];
                v[r] = in ? a.val[k] : 0.0f;
            }
            float t[R][NP];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (NP == 8) {
                    const float4* row = reinterpret_cast<const float4*>(a.T + (size_t)ix[r] * NP);
                    const float4 x = row[0], y = row[1];
                    t[r][0] = x.x, t[r][1] = x.y, t[r][2] = x.z, t[r][3] = x.w;
                    t[r][4] = y.x, t[r][5] = y.y, t[r][6] = y.z, t[r][7] = y.w;
                } else {
                    t[r][0] = a.T[ix[r]];
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int p = 0; p < NP; ++p) d[p] += (double)v[r] * (double)t[r][p];
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) d[p] = group_sum_f64<G>(d[p]);
        if (lane == 0) {
            const double scale = (a.sign ? (double)a.sign[c] : 1.0) / sqrt((double)sc + (double)a.mu);
            const double diag = (double)sc / ((double)sc + (double)a.mu);
            float K = a.K ? a.K[c] : 0.0f;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                // Off-diagonal part of (G z)_c: its square has expectation sum_{j != c} G_cj^2.
                const double g = d[p] * scale - diag * (double)probe_sign(c, a.first + p);
                K += (float)(g * g);
            }
            if (a.K) a.K[c] = K;
            best = fmaxf(best, K * a.inv_probes);
        }
    }
    if (!a.max_bits) return;
    for (int o = 32; o > 0; o >>= 1) best = fmaxf(best, __shfl_xor(best, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        best = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
        if (best > 0.0f) atomicMax(a.max_bits, __float_as_uint(best));
    }
}

// Per workgroup: sum of T0^2 (|A~ 1|^2), sum of G_cc, non-empty coordinates.
__global__ __launch_bounds__(256) void k_probe_totals(const float* __restrict__ T0, int64_t L,
                                                      const float* __restrict__ norms, uint32_t C, float mu,
                                                      double* __restrict__ partials) {
    __shared__ double red[3][4];
    double t[3] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < L; i += (int64_t)gridDim.x * 256) {
        const double x = T0[i];
        t[0] += x * x;
    }
    for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < C; c += (int64_t)gridDim.x * 256) {
        const float sc = norms[c];
        if (!(sc > 0.0f)) continue;
        t[1] += (double)sc / ((double)sc + (double)mu);
        t[2] += 1.0;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double x = group_sum_f64<64>(t[k]);
        if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = x;
    }
    __syncthreads();
    if (threadIdx.x < 3)
        partials[(size_t)blockIdx.x * 3 + threadIdx.x] =
            ((red[threadIdx.x][0] + red[threadIdx.x][1]) + red[threadIdx.x][2]) + red[threadIdx.x][3];
}

template <int G, int NP>
static hipError_t probe_scatter_typed(const ProbeArgs& a, int cus, hipStream_t s) {
    const size_t lds = sizeof(float) * (size_t)a.n_hot * (NP > 1 ? NP + 1 : 1);
    if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_probe_scatter<G, NP>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // Sixteen waves share a workgroup's slots; without slots small workgroups spread few segments over more
    // CUs (600 columns of 4,000: 38 CUs and 150).
    const int threads = a.n_hot ? 1024 : 256, per_cu = a.n_hot ? 1 : 8;
    const int64_t want = ((int64_t)a.C * G + threads - 1) / threads;
    const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(want, (int64_t)cus * per_cu));
    hipLaunchKernelGGL((k_probe_scatter<G, NP>), dim3(blocks), dim3(threads), lds, s, a);
    return hipGetLastError();
}

template <int G, int NP>
static hipError_t probe_gather_typed(const ProbeArgs& a, int blocks, hipStream_t s) {
    hipLaunchKernelGGL((k_probe_gather<G, NP>), dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

#define SCD_PROBE_BY_G(CALL)              \
    switch (G) {                          \
        case 4: return CALL(4);           \
        case 8: return CALL(8);           \
        case 16: return CALL(16);         \
        case 32: return CALL(32);         \
        default: return CALL(64);         \
    }

hipError_t launch_probe_scatter(const ProbeArgs& a, int np, int G, int cus, hipStream_t s) {
#define SCD_CALL(GW) (np > 1 ? probe_scatter_typed<GW, kProbeRow>(a, cus, s) : probe_scatter_typed<GW, 1>(a, cus, s))
    SCD_PROBE_BY_G(SCD_CALL)
#undef SCD_CALL
}

hipError_t launch_probe_gather(const ProbeArgs& a, int np, int G, int blocks, hipStream_t s) {
#define SCD_CALL(GW) (np > 1 ? probe_gather_typed<GW, kProbeRow>(a, blocks, s) : probe_gather_typed<GW, 1>(a, blocks, s))
    SCD_PROBE_BY_G(SCD_CALL)
#undef SCD_CALL
}
#undef SCD_PROBE_BY_G

hipError_t launch_probe_totals(const float* T0, int64_t L, const float* norms, uint32_t C, float mu, int blocks,
                               double* partials, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_probe_totals, dim3(blocks), dim3(256), 0, s, T0, L, norms, C, mu, partials);
    return launch_sum_partials(partials, blocks, 3, out, s);
}

}  // namespace scd
