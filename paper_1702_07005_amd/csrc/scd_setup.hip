// scd_setup.hip -- set-up and evaluation kernels for gfx950: the permutation array, the frozen
// gather-dot, squared norms (and <y, a_c>), input validation, the objective / duality-gap
// reductions and precision conversions.
#include <algorithm>

#include "scd_device.h"

namespace scd {

__global__ void k_perm_fill(PermKeys p, int32_t* __restrict__ out) {
    uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < p.n) out[j] = (int32_t)perm_at(j, p);
}

// ----------------------------------------------------------------------------------------
// Gathers of the frozen passes (gather-dot, objectives).  Scattered loads bound them: 130-140 G/s on
// click rows, whose stored values would stream in a third of that time.  With HOT, the solver's hot set
// (the most used entries, most of them in every wave's rows) is copied into LDS by each workgroup and
// read there; `key` stands in for idx (-1 - slot, or the index), and only the cold entries' loads
// leave the CU (hot lanes use an out-of-range offset of the raw buffer: no access).
// ----------------------------------------------------------------------------------------
constexpr int kHotPassThreads = 1024;  // two workgroups of 16 waves a CU share the copies

template <typename U>
__device__ __forceinline__ void hot_fill(U* cells, const HotCells& hc, const U* u) {
    for (uint32_t i = threadIdx.x; i < hc.n; i += blockDim.x) cells[i] = u[hc.ids[i]];
    __syncthreads();
}

template <typename U>
__device__ __forceinline__ U hot_or_load(const __amdgpu_buffer_rsrc_t& r, const U* cells, int key) {
    const U h = cells[key < 0 ? -1 - key : 0];
    const int off = key < 0 ? (int)0x7FFFFFF8 : (int)((uint32_t)key * (uint32_t)sizeof(U));
    if constexpr (sizeof(U) == 4) {
        const float g = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
        return key < 0 ? h : g;
    } else {
        const double g = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
        return key < 0 ? h : g;
    }
}

// ----------------------------------------------------------------------------------------
// Frozen gather-dot: out[c] = <a_c, u> with the epoch kernel's arithmetic (fp32 FMA per
// lane, group butterfly), for every coordinate in index order.  Blocks of G * R entries: all index
// and value loads, then all gathers; a lane past the end re-reads entry s0 with weight 0.  Where u is infinite
// there, that product is NaN although the lane has no entry: a sum that comes out NaN is formed again from the
// entries alone (masking every gathered value instead, 5 M click rows: 0.732 -> 0.747-0.753 ms).
// 5 M click rows (195 M entries): 1.40 ms one entry at a time, 0.75 in blocks with the hot set in LDS (the
// objectives 1.34 and 0.86); 16.6 M columns of 1 to 350,000 entries, no hot set: 18.1 and 8.6 ms.
// ----------------------------------------------------------------------------------------
template <int G, int R, bool HOT>
__global__ __launch_bounds__(HOT ? kHotPassThreads : 256) void k_gather_dots(
    const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx, const float* __restrict__ val,
    const float* __restrict__ u, uint32_t C, HotCells hc, uint32_t u_bytes, float* __restrict__ out) {
    extern __shared__ __align__(16) unsigned char pass_lds[];
    float* const cells = reinterpret_cast<float*>(pass_lds);
    if constexpr (HOT) hot_fill(cells, hc, u);
    const __amdgpu_buffer_rsrc_t ur = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(u), (short)0, (int)u_bytes, 0x00020000);
    const int lane = threadIdx.x & (G - 1);
    const uint32_t ngroups = gridDim.x * (blockDim.x / G);
    for (uint32_t c = (blockIdx.x * blockDim.x + threadIdx.x) / G; c < C; c += ngroups) {
        const int64_t s0 = ptr[c], s1 = ptr[c + 1];
        float acc = 0.0f;
        if constexpr (!HOT && (G <= 8 || G == 64)) {
            // One entry at a time where blocks do not pay: short segments (3.3 M click entries, all in cache:
            // 13.8 us, 14.6 in blocks) and whole waves (9,000 text rows of 1,000: 38.5 us, 41.8 in blocks).
            for (int64_t k = s0 + lane; k < s1; k += G) acc = fmaf(val[k], u[idx[k]], acc);
        } else
        for (int64_t b = s0; b < s1; b += (int64_t)G * R) {
            int ix[R];
            float vx[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t k = b + lane + (int64_t)r * G;
                const bool in = k < s1;
                const int64_t kk = in ? k : s0;
                ix[r] = HOT ? hc.key[kk] : idx[kk];
                const float v = val[kk];
                vx[r] = in ? v : 0.0f;
            }
            float g[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (HOT) g[r] = hot_or_load<float>(ur, cells, ix[r]);
                else g[r] = u[ix[r]];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) acc = fmaf(vx[r], g[r], acc);
        }
        acc = group_sum<G>(acc);
        if (acc != acc) {  // the same in every lane of the group
            acc = 0.0f;
            for (int64_t k = s0 + lane; k < s1; k += G) acc = fmaf(val[k], u[idx[k]], acc);
            acc = group_sum<G>(acc);
        }
        if (lane == 0) out[c] = acc;
    }
}

// ----------------------------------------------------------------------------------------
// Set-up: squared segment norms and, when y is given (ridge primal), cy_c = <y, a_c>
// (fp64 accumulation, fp32 results); input validation.
// ----------------------------------------------------------------------------------------
template <int G>
__global__ __launch_bounds__(256) void k_norms(const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx,
                                               const float* __restrict__ val, const float* __restrict__ y,
                                               uint32_t C, float* __restrict__ out, float* __restrict__ cy,
                                               double* __restrict__ cyd) {
    const int lane = threadIdx.x & (G - 1);
    const uint32_t ngroups = gridDim.x * (256u / G);
    for (uint32_t c = (blockIdx.x * 256u + threadIdx.x) / G; c < C; c += ngroups) {
        double acc = 0.0, dy = 0.0;
        for (int64_t k = ptr[c] + lane; k < ptr[c + 1]; k += G) {
            acc += (double)val[k] * (double)val[k];
            if (y) dy += (double)val[k] * (double)y[idx[k]];
        }
        acc = group_sum_f64<G>(acc);
        if (y) dy = group_sum_f64<G>(dy);
        if (lane == 0) {
            out[c] = (float)acc;
            if (y) {
                cy[c] = (float)dy;
                cyd[c] = dy;
            }
        }
    }
}

// flags bits: 1 ptr not monotone / wrong ends, 2 index out of range, 4 non-finite value,
// 8 non-finite label, 16 label not +-1.
// flags[1] (as unsigned long long) receives the longest segment.
__global__ __launch_bounds__(256) void k_validate_ptr(const int64_t* __restrict__ ptr, uint32_t S, int64_t nnz, int* flags) {
    __shared__ unsigned long long red[4];
    if (blockIdx.x == 0 && threadIdx.x == 0 && (ptr[0] != 0 || ptr[S] != nnz)) atomicOr(flags, 1);
    unsigned long long longest = 0;
    for (uint64_t c = (uint64_t)blockIdx.x * 256u + threadIdx.x; c < S; c += (uint64_t)gridDim.x * 256u) {
        const int64_t len = ptr[c + 1] - ptr[c];
        if (len < 0) atomicOr(flags, 1);
        else longest = max(longest, (unsigned long long)len);
    }
    // One atomic per workgroup: one per segment, all on one address, took 0.9 ms for 5 M segments.
    for (int o = 32; o > 0; o >>= 1) longest = max(longest, (unsigned long long)__shfl_xor(longest, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = longest;
    __syncthreads();
    if (threadIdx.x == 0) {
        longest = max(max(red[0], red[1]), max(red[2], red[3]));
        if (longest) atomicMax(reinterpret_cast<unsigned long long*>(flags) + 1, longest);
    }
}

__global__ void k_validate_entries(const int32_t* __restrict__ idx, const float* __restrict__ val, int64_t nnz,
                                   int64_t bound, int* flags) {
    int f = 0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * blockDim.x) {
        const int32_t i = idx[k];
        if (i < 0 || (int64_t)i >= bound) f |= 2;
        if (!isfinite(val[k])) f |= 4;
    }
    if (f) atomicOr(flags, f);
}

__global__ void k_validate_labels(const float* __restrict__ y, int64_t n, int pm1, int* flags) {
    int f = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float v = y[i];
        if (!isfinite(v)) f |= 8;
        else if (pm1 && v != 1.0f && v != -1.0f) f |= 16;
    }
    if (f) atomicOr(flags, f);
}

// ----------------------------------------------------------------------------------------
// Objective / duality-gap reductions (fp64).  Every workgroup sums, over the coordinates it owns,
// the fp64 dot d_c and up to three terms, and over its slice of the shared vector two more, and
// stores its five partial sums; one workgroup then adds the partials in workgroup order
// (deterministic; no cross-workgroup fences inside the pass).
//   ridge primal (u = w, r = y - w, d = <a_c, r> = <a_c, y> - <a_c, w>):
//                                  S0 += d^2,  S1 += beta^2          | V0 += r^2, V1 += r*y
//   svm dual     (u = w):          S0 += max(0, 1 - y d), S1 += alpha | V0 += w^2
//   ridge dual   (u = wbar):       S0 += (d/lambda - y)^2, S1 += alpha^2, S2 += alpha*y | V0 += wbar^2
// ----------------------------------------------------------------------------------------
template <int NS>
__device__ __forceinline__ void block_reduce_store(double (&v)[NS], double* out) {
    __shared__ double red[NS][kHotPassThreads / 64];
    const int tid = threadIdx.x;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        double x = v[s];
        x = group_sum_f64<64>(x);
        if ((tid & 63) == 0) red[s][tid >> 6] = x;
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            double x = 0.0;
            for (uint32_t w = 0; w < blockDim.x / 64; ++w) x += red[s][w];
            out[s] = x;
        }
    }
}

// Entries per lane per block of the objective's gather-dot.  Narrow groups take one block per segment
// of the lengths that choose them, so that few lanes re-read entry s0.
constexpr int obj_slices(int G) { return G <= 8 ? slice_depth(G) : 8; }

// DIRECT (ridge primal only): <a_c, y - w> is gathered from y and w in fp64 instead of taken as
// <y, a_c> (o.cyd, computed at set-up) minus <a_c, w>; for callers that hold no set-up data.
template <int FORM, int G, typename U, bool DIRECT, bool HOT>
__global__ __launch_bounds__(HOT ? kHotPassThreads : 256) void k_objective(ObjArgs o, double* __restrict__ partials) {
    static_assert(!(DIRECT && HOT), "callers without set-up data hold no hot set");
    constexpr int NS = 5, kObjSlices = obj_slices(G);
    extern __shared__ __align__(16) unsigned char pass_lds[];
    const U* __restrict__ u = static_cast<const U*>(o.u);
    U* const cells = reinterpret_cast<U*>(pass_lds);
    if constexpr (HOT) hot_fill(cells, o.hot, u);
    const __amdgpu_buffer_rsrc_t ur =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(o.u), (short)0, HOT ? (int)(o.L * (int64_t)sizeof(U)) : 0, 0x00020000);
    const int lane = threadIdx.x & (G - 1);
    const uint32_t ngroups = gridDim.x * (blockDim.x / G);
    double t[NS] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (uint32_t c = (blockIdx.x * blockDim.x + threadIdx.x) / G; c < o.C; c += ngroups) {
        // Blocks of G * kObjSlices entries: all index and value loads of a block, then all its
        // gathers, so that a block costs two memory round trips instead of two per entry.  Lanes
        // past the end re-read entry s0 with weight 0.
        const int64_t s0 = o.ptr[c], s1 = o.ptr[c + 1];
        double d = 0.0;
        for (int64_t b = s0; b < s1; b += (int64_t)G * kObjSlices) {
            int ix[kObjSlices];
            float vx[kObjSlices];
#pragma unroll
            for (int r = 0; r < kObjSlices; ++r) {
                const int64_t k = b + lane + (int64_t)r * G;
                const bool in = k < s1;
                const int64_t kk = in ? k : s0;
                ix[r] = HOT ? o.hot.key[kk] : o.idx[kk];
                const float v = o.val[kk];
                vx[r] = in ? v : 0.0f;
            }
            U g[kObjSlices];
#pragma unroll
            for (int r = 0; r < kObjSlices; ++r) {
                if constexpr (HOT) g[r] = hot_or_load<U>(ur, cells, ix[r]);
                else g[r] = u[ix[r]];
            }
            if constexpr (DIRECT) {
                float yy[kObjSlices];
#pragma unroll
                for (int r = 0; r < kObjSlices; ++r) yy[r] = o.yv[ix[r]];
#pragma unroll
                for (int r = 0; r < kObjSlices; ++r) d += (double)vx[r] * ((double)yy[r] - (double)g[r]);
            } else {
#pragma unroll
                for (int r = 0; r < kObjSlices; ++r) d += (double)vx[r] * (double)g[r];
            }
        }
        d = group_sum_f64<G>(d);
        if (lane == 0) {
            const double mo = o.model[c];
            if constexpr (FORM == FORM_RIDGE_PRIMAL) {
                const double r = DIRECT ? d : o.cyd[c] - d;
                t[0] += r * r;
                t[1] += mo * mo;
            } else if constexpr (FORM == FORM_SVM_DUAL) {
                const double l = 1.0 - (double)o.y[c] * d;
                t[0] += l > 0.0 ? l : 0.0;
                t[1] += mo;
            } else {
                const double e = d / o.lam - (double)o.y[c];
                t[0] += e * e;
                t[1] += mo * mo;
                t[2] += mo * (double)o.y[c];
            }
        }
    }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < o.L; i += (int64_t)gridDim.x * blockDim.x) {
        if constexpr (FORM == FORM_RIDGE_PRIMAL) {
            const double r = (double)o.yv[i] - (double)u[i];
            t[3] += r * r;
            t[4] += r * (double)o.yv[i];
        } else {
            const double x = (double)u[i];
            t[3] += x * x;
        }
    }
    block_reduce_store<NS>(t, partials + (size_t)blockIdx.x * NS);
}

// Sums `width` (at most kSumWidthMax) columns of `partials` [nparts][width] in one workgroup, in an
// order fixed by nparts alone (so the result does not depend on timing): thread t adds rows t,
// t + 256, ... in turn, each wave combines its lanes by an xor butterfly, and thread 0 adds the
// four wave sums in wave order.
constexpr int kSumWidthMax = 8;

__global__ __launch_bounds__(256) void k_sum_partials(const double* __restrict__ partials, int nparts, int width,
                                                      double* __restrict__ out) {
    __shared__ double sh[4][kSumWidthMax];
    double x[kSumWidthMax];
#pragma unroll
    for (int w = 0; w < kSumWidthMax; ++w) x[w] = 0.0;
    for (int p = threadIdx.x; p < nparts; p += 256) {
#pragma unroll
        for (int w = 0; w < kSumWidthMax; ++w)
            if (w < width) x[w] += partials[(size_t)p * width + w];
    }
#pragma unroll
    for (int w = 0; w < kSumWidthMax; ++w)
        for (int o = 32; o > 0; o >>= 1) x[w] += __shfl_xor(x[w], o, 64);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int w = 0; w < kSumWidthMax; ++w) sh[wave][w] = x[w];
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 0; w < width; ++w) out[w] = ((sh[0][w] + sh[1][w]) + sh[2][w]) + sh[3][w];
}

// Packed shared vector <-> its spread copy (entry i at byte offset i << kSpreadShift of the copy; the
// bytes between entries are never read).
template <typename U>
__global__ __launch_bounds__(256) void k_spread(U* __restrict__ packed, U* __restrict__ spread, int64_t L,
                                                bool to_spread) {
    constexpr uint32_t step = (1u << kSpreadShift) / sizeof(U);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < L; i += (int64_t)gridDim.x * 256) {
        if (to_spread)
            spread[i * step] = packed[i];
        else
            packed[i] = spread[i * step];
    }
}

hipError_t launch_sum_partials(const double* partials, int nparts, int width, double* out, hipStream_t s) {
    if (width > kSumWidthMax) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, s, partials, nparts, width, out);
    return hipGetLastError();
}

hipError_t launch_spread(void* packed, void* spread, int64_t L, bool wide, bool to_spread, hipStream_t s) {
    if (wide)
        hipLaunchKernelGGL(k_spread<double>, dim3(grid_for(L)), dim3(256), 0, s, static_cast<double*>(packed),
                           static_cast<double*>(spread), L, to_spread);
    else
        hipLaunchKernelGGL(k_spread<float>, dim3(grid_for(L)), dim3(256), 0, s, static_cast<float*>(packed),
                           static_cast<float*>(spread), L, to_spread);
    return hipGetLastError();
}

hipError_t launch_perm_fill(const PermKeys& p, int32_t* out, hipStream_t s) {
    const uint32_t blocks = (p.n + 255) / 256;
    hipLaunchKernelGGL(k_perm_fill, dim3(blocks), dim3(256), 0, s, p, out);
    return hipGetLastError();
}

// The hot passes' launch: dynamic LDS for the cells, and two workgroups per CU at most.
static hipError_t hot_pass_lds(const void* f, size_t lds) {
    return lds > 65536 ? hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) : hipSuccess;
}

static unsigned hot_pass_blocks(int64_t C, int G, int cus) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(2 * (int64_t)cus, (C * G + kHotPassThreads - 1) / kHotPassThreads));
}

template <int G>
static hipError_t gather_typed(const int64_t* ptr, const int32_t* idx, const float* val, const float* u, uint32_t C,
                               int64_t L, const HotCells& hc, int blocks, int cus, float* out, hipStream_t s) {
    constexpr int R = slice_depth(G);
    if (hc.n) {
        const size_t lds = sizeof(float) * hc.n;
        const hipError_t e = hot_pass_lds(reinterpret_cast<const void*>(&k_gather_dots<G, R, true>), lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_gather_dots<G, R, true>), dim3(hot_pass_blocks(C, G, cus)), dim3(kHotPassThreads), lds, s, ptr,
                           idx, val, u, C, hc, (uint32_t)(L * 4), out);
    } else {
        hipLaunchKernelGGL((k_gather_dots<G, R, false>), dim3(blocks), dim3(256), 0, s, ptr, idx, val, u, C, hc, 0u, out);
    }
    return hipGetLastError();
}

hipError_t launch_gather_dots(const int64_t* ptr, const int32_t* idx, const float* val, const float* u, uint32_t C,
                              int64_t L, const HotCells& hc, int G, int blocks, int cus, float* out, hipStream_t s) {
    switch (G) {
        case 4: return gather_typed<4>(ptr, idx, val, u, C, L, hc, blocks, cus, out, s);
        case 8: return gather_typed<8>(ptr, idx, val, u, C, L, hc, blocks, cus, out, s);
        case 16: return gather_typed<16>(ptr, idx, val, u, C, L, hc, blocks, cus, out, s);
        case 32: return gather_typed<32>(ptr, idx, val, u, C, L, hc, blocks, cus, out, s);
        default: return gather_typed<64>(ptr, idx, val, u, C, L, hc, blocks, cus, out, s);
    }
}

hipError_t launch_norms(const int64_t* ptr, const int32_t* idx, const float* val, const float* y, uint32_t C, int G,
                        int blocks, float* out, float* cy, double* cyd, hipStream_t s) {
    switch (G) {
        case 4: hipLaunchKernelGGL(k_norms<4>, dim3(blocks), dim3(256), 0, s, ptr, idx, val, y, C, out, cy, cyd); break;
        case 8: hipLaunchKernelGGL(k_norms<8>, dim3(blocks), dim3(256), 0, s, ptr, idx, val, y, C, out, cy, cyd); break;
        case 16: hipLaunchKernelGGL(k_norms<16>, dim3(blocks), dim3(256), 0, s, ptr, idx, val, y, C, out, cy, cyd); break;
        case 32: hipLaunchKernelGGL(k_norms<32>, dim3(blocks), dim3(256), 0, s, ptr, idx, val, y, C, out, cy, cyd); break;
        default: hipLaunchKernelGGL(k_norms<64>, dim3(blocks), dim3(256), 0, s, ptr, idx, val, y, C, out, cy, cyd); break;
    }
    return hipGetLastError();
}

hipError_t launch_validate(const int64_t* ptr, uint32_t S, const int32_t* idx, const float* val, int64_t nnz,
                           int64_t bound, const float* y, int64_t ny, int pm1, int* flags, hipStream_t s) {
    hipLaunchKernelGGL(k_validate_ptr, dim3(std::min<uint32_t>(1024, (S + 255u) / 256u)), dim3(256), 0, s, ptr, S, nnz, flags);
    if (nnz > 0) {
        int64_t b = (nnz + 255) / 256;
        if (b > 8192) b = 8192;
        hipLaunchKernelGGL(k_validate_entries, dim3((unsigned)b), dim3(256), 0, s, idx, val, nnz, bound, flags);
    }
    int64_t b = (ny + 255) / 256;
    if (b > 4096) b = 4096;
    if (b < 1) b = 1;
    hipLaunchKernelGGL(k_validate_labels, dim3((unsigned)b), dim3(256), 0, s, y, ny, pm1, flags);
    return hipGetLastError();
}

template <int FORM, int G, typename U, bool DIRECT>
static hipError_t objective_launch(const ObjArgs& o, int* blocks, int cus, double* partials, hipStream_t s) {
    if constexpr (!DIRECT) {
        if (o.hot.n) {
            const size_t lds = sizeof(U) * o.hot.n;
            const hipError_t e = hot_pass_lds(reinterpret_cast<const void*>(&k_objective<FORM, G, U, false, true>), lds);
            if (e != hipSuccess) return e;
            *blocks = (int)hot_pass_blocks(o.C, G, cus);
            hipLaunchKernelGGL((k_objective<FORM, G, U, false, true>), dim3(*blocks), dim3(kHotPassThreads), lds, s, o, partials);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_objective<FORM, G, U, DIRECT, false>), dim3(*blocks), dim3(256), 0, s, o, partials);
    return hipGetLastError();
}

template <int FORM, typename U, bool DIRECT>
static hipError_t objective_typed(const ObjArgs& o, int G, int* blocks, int cus, double* partials, hipStream_t s) {
    switch (G) {
        case 4: return objective_launch<FORM, 4, U, DIRECT>(o, blocks, cus, partials, s);
        case 8: return objective_launch<FORM, 8, U, DIRECT>(o, blocks, cus, partials, s);
        case 16: return objective_launch<FORM, 16, U, DIRECT>(o, blocks, cus, partials, s);
        case 32: return objective_launch<FORM, 32, U, DIRECT>(o, blocks, cus, partials, s);
        default: return objective_launch<FORM, 64, U, DIRECT>(o, blocks, cus, partials, s);
    }
}

template <int FORM>
static hipError_t objective_form(const ObjArgs& o, int G, int* blocks, int cus, double* partials, hipStream_t s) {
    // The ridge primal without <y, a_c> from set-up gathers y beside w.
    if constexpr (FORM == FORM_RIDGE_PRIMAL) {
        if (!o.cyd)
            return o.wide ? objective_typed<FORM, double, true>(o, G, blocks, cus, partials, s)
                          : objective_typed<FORM, float, true>(o, G, blocks, cus, partials, s);
    }
    return o.wide ? objective_typed<FORM, double, false>(o, G, blocks, cus, partials, s)
                  : objective_typed<FORM, float, false>(o, G, blocks, cus, partials, s);
}

__global__ __launch_bounds__(256) void k_fill_zero(uint64_t* __restrict__ p, uint32_t n) {
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) p[i] = 0ull;
}

hipError_t launch_fill_zero(uint64_t* p, uint32_t n_words, hipStream_t s) {
    if (n_words == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_zero, dim3((n_words + 255) / 256 > 64 ? 64 : (n_words + 255) / 256), dim3(256), 0, s, p,
                       n_words);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_reset_waits(int* __restrict__ err, uint64_t* __restrict__ slots) {
    if (err && threadIdx.x == 0) *err = 0;
    if (slots)
        for (int i = threadIdx.x; i <= kLockSlotWords; i += 256) slots[i] = i == kLockSlotWords ? 1ull : 0ull;
}

hipError_t launch_reset_waits(int* err, uint64_t* slots, hipStream_t s) {
    hipLaunchKernelGGL(k_reset_waits, dim3(1), dim3(256), 0, s, err, slots);
    return hipGetLastError();
}

// sums[0..2] = coordinate sums, sums[3..4] = vector sums.
hipError_t launch_objective(int form, const ObjArgs& o, int G, int blocks, int cus, double* partials, double* sums,
                            hipStream_t s) {
    hipError_t e = hipErrorInvalidValue;
    switch (form) {
        case FORM_RIDGE_PRIMAL: e = objective_form<FORM_RIDGE_PRIMAL>(o, G, &blocks, cus, partials, s); break;
        case FORM_SVM_DUAL: e = objective_form<FORM_SVM_DUAL>(o, G, &blocks, cus, partials, s); break;
        case FORM_RIDGE_DUAL: e = objective_form<FORM_RIDGE_DUAL>(o, G, &blocks, cus, partials, s); break;
        default: break;
    }
    if (e != hipSuccess) return e;
    return launch_sum_partials(partials, blocks, 5, sums, s);
}

// ----------------------------------------------------------------------------------------
// Storage-width conversions of the shared vector.
// ----------------------------------------------------------------------------------------
template <typename A, typename B>
__global__ __launch_bounds__(256) void k_convert(const A* __restrict__ in, int64_t n, B* __restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) out[i] = (B)in[i];
}

hipError_t launch_convert_f32_to_f64(const float* in, int64_t n, double* out, hipStream_t s) {
    hipLaunchKernelGGL((k_convert<float, double>), dim3(grid_for(n)), dim3(256), 0, s, in, n, out);
    return hipGetLastError();
}

hipError_t launch_convert_f64_to_f32(const double* in, int64_t n, float* out, hipStream_t s) {
    hipLaunchKernelGGL((k_convert<double, float>), dim3(grid_for(n)), dim3(256), 0, s, in, n, out);
    return hipGetLastError();
}

}  // namespace scd
