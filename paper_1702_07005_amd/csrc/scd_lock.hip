// scd_lock.hip -- lockstep epoch kernel: few coordinates in flight, long segments, and a shared vector
// that fits the LDS of a few CUs.
//
// With a handful of coordinates in flight an epoch is a chain of steps, and in the pipelined kernel each
// step is two trips to memory: the gathers, and the atomics that must land before the next gathers (about
// 2 us for eight columns of 2,000 entries or rows of 370).  Here the shared vector stays in LDS for the
// epoch, as fp64 cells (LDS fp32 adds are eight times slower and more), cut into index ranges over K
// workgroups of one XCD, and the only trip left is the exchange of the partial inner products (0.7 us
// between eight workgroups):
//
//   Round r takes the W coordinates at positions r W .. r W + W - 1, one per wave: wave w of each of the K
//   workgroups (the members) handles position r W + w, on the entries of its member's range.
//   1. gather from the member's LDS and reduce in the wave (DPP);
//   2. publish the partial in a 64-bit slot (fp32 bits + round tag) and poll the K slots of this wave until
//      all carry the tag; the K partials are added in member order, so all members take the same step;
//   3. step, and add coef * a_m into the member's LDS;
//   4. a workgroup barrier, after which every wave of the member gathers the next round.
//
// A coordinate misses the updates of the W - 1 others of its round at most, and of those only the ones
// before it in the visiting order are ones the sequential algorithm would have seen, so W is the automatic window
// itself.  (The steps of a round are taken from one state: not for coordinates that mostly pull the same way, see
// the plan's rule.)
//
// Slots: (tag mod 2, wave, member).  A wave overwrites its slot of round g at round g + 2, after it has seen
// every member's partial of round g + 1, which each publishes only after it has read all of round g.  Each
// slot is one location, written and read whole at device scope.  Every poll is bounded; a wave that gives up
// sets *err and its round's flag in LDS (one of two, so that no wave of the round reads it early), and its
// workgroup leaves in the next round, as do the others in turn.
//
// Tags grow by one per round and on from launch to launch: the first one is kept in device memory behind the
// slots, read by every member when it starts and advanced by member 0 when it ends, so a launch replayed from a
// captured graph gets new tags too.  In a launch whose waits all end, round 0 has been exchanged by then and every
// member has read it.  Member 0 may also give up in round 0 and advance it before another member starts, which
// then reads the next launch's first tag and publishes under it.  Such a launch has set *err, and the state is
// invalid until scd_set_state, which clears the slots and starts the tags again (launch_reset_waits, on the same
// stream, so after that launch): no later launch sees those partials.
//
// Placement: workgroup b runs on XCD b mod 8; the members are those of one XCD (correct on any, slower
// across).  K is at most 8, so that the four kernels a process runs at once by default all fit one XCD's 32
// CUs, one member each, and none waits for members that cannot start; handles use the XCDs in turn.  Beside the
// other kernels with waits between workgroups: a team epoch has at most 32 workgroups per XCD, of which a CU takes four
// (and keeps none from a member with less than all its LDS), so it is resident whole beside any members and ends
// without them; a staged epoch claims its batches, so any one of its stagers lets it end.  Members that could not start
// do so then, well within the wait limit.  (More than four kernels at once, GPU_MAX_HW_QUEUES above its default, may
// hold five lockstep epochs of one XCD, 40 CUs: their waits end with an error.)
//
// Measured, pipelined at its share of the automatic window W and this kernel at W, per epoch: 2,000 x 200 dense
// (7 and 9 in flight) 55 and 46 us; 500 x 60 dense (2 and 3) 49 and 31 us; text rows of 370 entries on 166,000
// columns (6 and 8) 1.22 and 0.68 ms; of 809 on 127,000 (4 and 6) 2.16 and 0.69 ms.  A round takes 1.5-2 us: the
// exchange, the loads that its wait covers, and the LDS reads and adds of up to four slices a wave.
//
// S slices of 64 entries of a part stay in registers; what is beyond is streamed twice, loads and LDS in turn.
// Four take parts of 256 entries, eight of 512, at 10% more time where the parts are short (2,000 x 200 dense 42.5
// and 47.4 us an epoch, text rows of 370 0.583 and 0.647 ms) and less where they are long (4,000 x 100 dense, parts of
// 500, 53.0 and 45.1 us; 1,000 rows of 450 with 370 in one range 0.564 and 0.466 ms); scd_create chooses by the parts.
#include <algorithm>

#include "scd_device.h"
#include "scd_kernels.h"

namespace scd {
namespace {

struct LockMeta {
    int64_t base;
    uint32_t o0, o1, m;
    float m_old, sn, ylab;
};

// Metadata of position j (a stand-in past the end: never used).  The zero in a vector register keeps the
// loaded values there: as provably equal in all lanes they would be moved to scalar registers, by a wait, as
// soon as they are loaded.
__device__ __forceinline__ LockMeta lock_meta(const LockArgs& t, uint64_t j, uint32_t k) {
    uint32_t zero = 0u;
    asm volatile("" : "+v"(zero));
    LockMeta c;
    c.m = perm_at(j < t.e.perm.n ? (uint32_t)j : 0u, t.e.perm) + zero;
    c.base = t.e.ptr[c.m];
    const uint32_t* o = t.off + (size_t)c.m * (t.K + 1) + k;
    c.o0 = o[0];
    c.o1 = o[1];
    c.m_old = t.e.model[c.m];
    c.sn = t.e.norms[c.m];
    c.ylab = t.e.y[c.m];
    return c;
}

// The first 64 S entries of the part; lanes past its end hold `none`, a cell of value 0 behind the
// member's own (any of those may hold an infinity, which would make the sums of other coordinates NaN).
template <int S>
__device__ __forceinline__ void lock_load(const LockArgs& t, const LockMeta& c, uint32_t lane, uint32_t none,
                                          uint32_t (&ci)[S], float (&cv)[S]) {
    const uint32_t len = c.o1 - c.o0;
#pragma unroll
    for (int r = 0; r < S; ++r) {
        const uint32_t i = lane + 64u * (uint32_t)r;
        ci[r] = none;
        cv[r] = 0.0f;
        if (i < len) {
            ci[r] = t.idx[c.base + c.o0 + i];
            cv[r] = t.val[c.base + c.o0 + i];
        }
    }
}

template <int FORM, typename U, int S>
__global__ __launch_bounds__(64 * kLockMaxWindow) void k_epoch_lock(LockArgs t) {
    extern __shared__ __align__(16) unsigned char lock_lds[];
    __shared__ int gave_up[2];
    if (blockIdx.x % kTeamXcds != t.xcd) return;
    const uint32_t k = blockIdx.x / kTeamXcds;
    if (k >= t.K) return;
    const EpochArgs& a = t.e;
    double* const cells = reinterpret_cast<double*>(lock_lds);
    const uint32_t cell0 = t.cell0[k], n_cells = t.cell0[k + 1] - cell0;
    U* const u = static_cast<U*>(a.u);
    for (uint32_t i = threadIdx.x; i < n_cells; i += blockDim.x) cells[i] = (double)u[t.ids[cell0 + i]];
    if (threadIdx.x == 0) cells[n_cells] = 0.0;
    if (threadIdx.x < 2) gave_up[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t n = a.perm.n, W = t.W, rounds = (n + W - 1) / W;
    // In round r: cur and ci/cv are its metadata and part, nxt round r + 1's metadata, all there.  Round
    // r + 1's part and round r + 2's metadata are loaded between this round's partial sum and its poll,
    // whose wait covers them (a wave's loads return in order).  Loaded before the partial is published they
    // hold it up, and the waves that poll for it hold up each other: 0.68 -> 2.1 ms an epoch on the text
    // rows, 46 -> 137 us on the dense columns.
    LockMeta cur = lock_meta(t, wave, k), nxt = lock_meta(t, (uint64_t)wave + W, k);
    uint32_t ci[S];
    float cv[S];
    lock_load(t, cur, lane, n_cells, ci, cv);
    uint64_t* const base_tag = t.slots + kLockSlotWords;
    const uint32_t tag0 = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)__hip_atomic_load(base_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the loop's waits need not allow for these loads
    uint32_t tag = tag0;
    for (uint32_t r = 0; r < rounds; ++r, ++tag) {
        const uint32_t j = r * W + wave;
        // Of the last round: the same for every wave.
        const int left = __hip_atomic_load(gave_up + ((r + 1u) & 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const uint32_t len = (uint32_t)__builtin_amdgcn_readfirstlane((int)(cur.o1 - cur.o0));
        const int64_t at = cur.base + cur.o0;
        float acc = 0.0f;
#pragma unroll
        for (int q = 0; q < S; ++q)
            if (64u * (uint32_t)q < len) acc = fmaf(cv[q], (float)cells[ci[q]], acc);
        for (uint32_t i = 64u * S + lane; i < len; i += 64u) acc = fmaf(t.val[at + i], (float)cells[t.idx[at + i]], acc);
        if (left) break;
        // (Past the last position, in the last round, a wave goes through the motions on its stand-in.)
        const float p = group_sum<64>(acc);
        uint64_t* const slot = t.slots + ((size_t)(tag & 1u) * kLockMaxWindow + wave) * kLockMaxMembers;
        if (lane == 0)
            __hip_atomic_store(slot + k, ((uint64_t)tag << 32) | (uint64_t)__float_as_uint(p), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_sched_barrier(0);
        uint32_t ni[S];
        float nv[S];
        lock_load(t, nxt, lane, n_cells, ni, nv);
        const LockMeta nn = lock_meta(t, (uint64_t)j + 2ull * W, k);
        __builtin_amdgcn_sched_barrier(0);
        uint32_t pv = 0;
        for (uint32_t spins = 0;; ++spins) {
            // lanes past the last member re-read its slot
            const uint64_t v = __hip_atomic_load(slot + (lane < t.K ? lane : t.K - 1u), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
            pv = (uint32_t)v;
            if (__all((uint32_t)(v >> 32) == tag)) break;
            if (spins >= t.spin_limit) {
                if (lane == 0) {
                    __hip_atomic_fetch_or(t.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(gave_up + (r & 1u), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                break;
            }
            if (spins > 64) __builtin_amdgcn_s_sleep(1);
        }
        float g = 0.0f;
#pragma unroll
        for (int q = 0; q < kLockMaxMembers; ++q)
            if ((uint32_t)q < t.K) g += __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)pv, q));
        float coef;
        const float m_new = coord_step<FORM>(g, cur.sn, cur.m_old, cur.ylab, a.k, &coef);
        if (j < n && coef != 0.0f) {
#pragma unroll
            for (int q = 0; q < S; ++q)
                if (64u * (uint32_t)q < len && lane + 64u * (uint32_t)q < len) atomicAdd(cells + ci[q], (double)(coef * cv[q]));
            for (uint32_t i = 64u * S + lane; i < len; i += 64u)
                atomicAdd(cells + t.idx[at + i], (double)(coef * t.val[at + i]));
        }
        if (lane == 0 && j < n && j % t.K == k) a.model[cur.m] = m_new;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            ci[q] = ni[q];
            cv[q] = nv[q];
        }
        cur = nxt;
        nxt = nn;
        // This wave's LDS adds have completed, then every wave's.
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
    __syncthreads();
    if (k == 0 && threadIdx.x == 0)
        __hip_atomic_store(base_tag, (uint64_t)(uint32_t)(tag0 + rounds + 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (uint32_t i = threadIdx.x; i < n_cells; i += blockDim.x) u[t.ids[cell0 + i]] = (U)cells[i];
}

template <int FORM, typename U, int S>
hipError_t launch_lock_typed(const LockArgs& t, hipStream_t s) {
    const size_t lds = lock_lds_bytes(t.max_cells);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_epoch_lock<FORM, U, S>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_epoch_lock<FORM, U, S>), dim3(t.K * kTeamXcds), dim3(64 * t.W), lds, s, t);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------------
// The members' ranges and cells (set-up).  On the host this was a copy of the hits and two loops over L: 0.6 ms of
// scd_create's 2.6 for 3,500 text rows on 166,000 columns.
// ----------------------------------------------------------------------------------------
constexpr int kRangeThreads = kHotAssignBlock / 4;  // four consecutive indices a thread

__device__ __forceinline__ void range_load(const unsigned* hits, int64_t L, int64_t i0, unsigned (&v)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = i0 + r < L ? hits[i0 + r] : 0u;
}

// Exclusive sums over the workgroup (N threads) of a and b.
template <int N>
__device__ __forceinline__ void block_scan(uint64_t& a, uint32_t& b) {
    __shared__ uint64_t sa[N];
    __shared__ uint32_t sb[N];
    const uint64_t a0 = a;
    const uint32_t b0 = b;
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int o = 1; o < N; o <<= 1) {  // inclusive Hillis-Steele scan
        const bool in = threadIdx.x >= (unsigned)o;
        const uint64_t xa = in ? sa[threadIdx.x - o] : 0ull;
        const uint32_t xb = in ? sb[threadIdx.x - o] : 0u;
        __syncthreads();
        sa[threadIdx.x] += xa;
        sb[threadIdx.x] += xb;
        __syncthreads();
    }
    a = sa[threadIdx.x] - a0;
    b = sb[threadIdx.x] - b0;
}

__global__ __launch_bounds__(kRangeThreads) void k_lock_block_sums(const unsigned* __restrict__ hits, int64_t L,
                                                                  LockBlock* __restrict__ blocks) {
    unsigned v[4];
    range_load(hits, L, (int64_t)blockIdx.x * kHotAssignBlock + 4 * threadIdx.x, v);
    uint64_t entries = (uint64_t)v[0] + v[1] + v[2] + v[3];
    uint32_t used = (v[0] != 0u) + (v[1] != 0u) + (v[2] != 0u) + (v[3] != 0u);
    const uint64_t e0 = entries;
    const uint32_t u0 = used;
    block_scan<kRangeThreads>(entries, used);
    if (threadIdx.x == kRangeThreads - 1) blocks[blockIdx.x] = LockBlock{entries + e0, used + u0, 0u};
}

// blocks[b] becomes the sums of the blocks before b; the cuts' defaults; r->cell0[K] = used indices.
__global__ __launch_bounds__(1024) void k_lock_block_scan(LockBlock* __restrict__ blocks, uint32_t n, uint32_t K, uint32_t L,
                                                          LockRanges* __restrict__ r) {
    const LockBlock own = threadIdx.x < n ? blocks[threadIdx.x] : LockBlock{0ull, 0u, 0u};
    uint64_t entries = own.entries;
    uint32_t used = own.used;
    block_scan<1024>(entries, used);
    if (threadIdx.x < n) blocks[threadIdx.x] = LockBlock{entries, used, 0u};
    if (threadIdx.x == 1023) {
        const uint32_t all = used + own.used;
        r->cell0[K] = all;
        for (int c = 0; c < 2; ++c)
            for (uint32_t q = 0; q <= K; ++q) {
                r->cut_bound[c][q] = q ? L : 0u;
                r->cut_cell[c][q] = q ? all : 0u;
            }
    }
}

// Cut q of K, by entries and by cells: after the index at which the running sum reaches q / K of the total.
__global__ __launch_bounds__(kRangeThreads) void k_lock_cuts(const unsigned* __restrict__ hits, int64_t L, uint64_t nnz, uint32_t K,
                                                            const LockBlock* __restrict__ blocks, LockRanges* __restrict__ r) {
    const int64_t i0 = (int64_t)blockIdx.x * kHotAssignBlock + 4 * threadIdx.x;
    unsigned v[4];
    range_load(hits, L, i0, v);
    uint64_t entries = (uint64_t)v[0] + v[1] + v[2] + v[3];
    uint32_t used = (v[0] != 0u) + (v[1] != 0u) + (v[2] != 0u) + (v[3] != 0u);
    block_scan<kRangeThreads>(entries, used);
    entries += blocks[blockIdx.x].entries;
    used += blocks[blockIdx.x].used;
    const uint64_t cells = r->cell0[K];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (!v[j]) continue;
        for (uint32_t q = 1; q < K; ++q) {
            const uint64_t te = (q * nnz + K - 1) / K, tc = (q * cells + K - 1) / K;
            if (entries < te && entries + v[j] >= te) {
                r->cut_bound[0][q] = (uint32_t)(i0 + j) + 1u;
                r->cut_cell[0][q] = used + 1u;
            }
            if (used < tc && used + 1u >= tc) {
                r->cut_bound[1][q] = (uint32_t)(i0 + j) + 1u;
                r->cut_cell[1][q] = used + 1u;
            }
        }
        entries += v[j];
        ++used;
    }
}

__global__ __launch_bounds__(kRangeThreads) void k_lock_assign(const unsigned* __restrict__ hits, int64_t L, uint32_t K, uint32_t cap,
                                                              const LockBlock* __restrict__ blocks, LockRanges* __restrict__ r,
                                                              uint16_t* __restrict__ cell_of, int32_t* __restrict__ ids) {
    if (r->cell0[K] > K * cap) return;
    uint32_t most = 0;
    for (uint32_t k = 0; k < K; ++k) most = max(most, r->cut_cell[0][k + 1] - r->cut_cell[0][k]);
    const int by = most > cap ? 1 : 0;
    if (blockIdx.x == 0 && threadIdx.x <= K) {
        r->bound[threadIdx.x] = r->cut_bound[by][threadIdx.x];
        r->cell0[threadIdx.x] = r->cut_cell[by][threadIdx.x];  // cell0[K] keeps its value
    }
    const int64_t i0 = (int64_t)blockIdx.x * kHotAssignBlock + 4 * threadIdx.x;
    unsigned v[4];
    range_load(hits, L, i0, v);
    uint64_t entries = 0;
    uint32_t used = (v[0] != 0u) + (v[1] != 0u) + (v[2] != 0u) + (v[3] != 0u);
    block_scan<kRangeThreads>(entries, used);
    used += blocks[blockIdx.x].used;
    for (int j = 0; j < 4; ++j) {
        if (i0 + j >= L) break;
        uint32_t first = 0;
        for (uint32_t k = 1; k < K; ++k)
            if ((uint32_t)(i0 + j) >= r->cut_bound[by][k]) first = r->cut_cell[by][k];
        cell_of[i0 + j] = v[j] ? (uint16_t)(used - first) : (uint16_t)0;
        if (v[j]) ids[used++] = (int32_t)(i0 + j);
    }
}

__global__ __launch_bounds__(256) void k_lock_excess(const uint32_t* __restrict__ off, uint32_t C, uint32_t K, uint32_t base0,
                                                     uint32_t base1, LockExcess* __restrict__ excess) {
    __shared__ uint32_t h[2 * kLockExcessBins];
    uint32_t* const out = excess->n[0];
    if (threadIdx.x < 2 * kLockExcessBins) h[threadIdx.x] = 0u;
    __syncthreads();
    for (uint64_t c = blockIdx.x * 256u + threadIdx.x; c < C; c += (uint64_t)gridDim.x * 256u) {
        const uint32_t* o = off + c * (K + 1);
        uint32_t most = 0;
        for (uint32_t k = 0; k < K; ++k) most = max(most, o[k + 1] - o[k]);
        const uint32_t slices = most / 64u + (most % 64u != 0u);
        if (slices > base0) atomicAdd(h + (31 - __clz((int)(slices - base0))), 1u);
        if (slices > base1) atomicAdd(h + kLockExcessBins + (31 - __clz((int)(slices - base1))), 1u);
    }
    __syncthreads();
    if (threadIdx.x < 2 * kLockExcessBins && h[threadIdx.x]) atomicAdd(out + threadIdx.x, h[threadIdx.x]);
}

// Cell of every stored entry of the grouped copy: cell_of[index] within its range.
__global__ __launch_bounds__(256) void k_lock_cells(const int32_t* __restrict__ idx, int64_t nnz,
                                                    const uint16_t* __restrict__ cell_of, uint16_t* __restrict__ out) {
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * 256)
        out[e] = cell_of[idx[e]];
}

}  // namespace

template <int FORM>
static hipError_t launch_lock_form(bool wide, const LockArgs& t, hipStream_t s) {
    if (t.slices == (uint32_t)kLockSlicesLong)
        return wide ? launch_lock_typed<FORM, double, kLockSlicesLong>(t, s) : launch_lock_typed<FORM, float, kLockSlicesLong>(t, s);
    return wide ? launch_lock_typed<FORM, double, kLockSlices>(t, s) : launch_lock_typed<FORM, float, kLockSlices>(t, s);
}

hipError_t launch_epoch_lock(int form, bool wide, const LockArgs& t, hipStream_t s) {
    if (t.K < 1 || t.K > (uint32_t)kLockMaxMembers || t.W < 1 || t.W > (uint32_t)kLockMaxWindow || t.xcd >= kTeamXcds ||
        (t.slices != (uint32_t)kLockSlices && t.slices != (uint32_t)kLockSlicesLong))
        return hipErrorInvalidValue;
    switch (form) {
        case FORM_RIDGE_PRIMAL: return launch_lock_form<FORM_RIDGE_PRIMAL>(wide, t, s);
        case FORM_SVM_DUAL: return launch_lock_form<FORM_SVM_DUAL>(wide, t, s);
        case FORM_RIDGE_DUAL: return launch_lock_form<FORM_RIDGE_DUAL>(wide, t, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_lock_ranges(const unsigned* hits, int64_t L, int64_t nnz, uint32_t K, uint32_t cap, LockBlock* blocks,
                              LockRanges* r, uint16_t* cell_of, int32_t* ids, hipStream_t s) {
    const int64_t nb = lock_blocks(L);
    if (nb < 1 || nb > 1024 || nnz < 1 || K < 1 || K > (uint32_t)kLockMaxMembers) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nb), threads(kRangeThreads);
    hipLaunchKernelGGL(k_lock_block_sums, grid, threads, 0, s, hits, L, blocks);
    hipLaunchKernelGGL(k_lock_block_scan, dim3(1), dim3(1024), 0, s, blocks, (uint32_t)nb, K, (uint32_t)L, r);
    hipLaunchKernelGGL(k_lock_cuts, grid, threads, 0, s, hits, L, (uint64_t)nnz, K, blocks, r);
    hipLaunchKernelGGL(k_lock_assign, grid, threads, 0, s, hits, L, K, cap, blocks, r, cell_of, ids);
    return hipGetLastError();
}

hipError_t launch_lock_excess(const uint32_t* off, uint32_t C, uint32_t K, const uint32_t (&base)[2], LockExcess* excess,
                              hipStream_t s) {
    static_assert(sizeof(LockExcess) == 8 * kLockExcessBins, "whole 64-bit words");
    if (const hipError_t e = launch_fill_zero(reinterpret_cast<uint64_t*>(excess), kLockExcessBins, s); e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lock_excess, dim3(std::min(grid_for(C), 256u)), dim3(256), 0, s, off, C, K, base[0], base[1], excess);
    return hipGetLastError();
}

hipError_t launch_lock_cells(const int32_t* idx, int64_t nnz, const uint16_t* cell_of, uint16_t* out, hipStream_t s) {
    if (nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_lock_cells, dim3(grid_for(nnz)), dim3(256), 0, s, idx, nnz, cell_of, out);
    return hipGetLastError();
}

}  // namespace scd
