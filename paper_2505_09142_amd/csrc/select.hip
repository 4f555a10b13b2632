// ISRTF batch selection on the device (Sec. 4.1: the batch is formed from the
// jobs with the fewest predicted remaining tokens; ties go to the earlier
// arrival, then the lower index).
//
// Each job gets a total-order key (orderable-u32(pred), arrival, index):
//   * the float is mapped to an unsigned integer whose order is the float
//     order, with -0 folded onto +0 and every NaN mapped to the maximum (after
//     +inf), so the comparison is exact integer work with no rounding;
//   * n <= 8192, and up to 12288 where k is a large part of n: every work-group
//     ranks a few jobs by counting the keys below theirs (all keys in LDS), and
//     the job of rank r < k lands in out_idx[r];
//   * larger n (k <= 8192), where the smallest jobs of some groups bound the number of
//     candidates (see "group minima"): three launches;
//   * else radix selection over the whole device, most
//     significant digit first. Three counting passes over the float keys
//     (11, 11, 10 bits) fix the key P of the k-th job: in every pass each
//     work-group histograms its own contiguous chunk of jobs (those matching
//     the prefix fixed so far) and stores the counts; 32 small work-groups
//     total the buckets and the last of them picks the bucket holding the
//     k-th job. A scatter pass then lists, per chunk and in index order, the
//     jobs with key < P and the ties (key == P). Nothing in these passes is a
//     same-address global atomic (those serialise at tens of ns apiece across
//     the XCDs). A single work-group takes the needed number of
//     ties by (arrival, index) - an LDS sort when there are at most 8192 of
//     them, otherwise a radix selection of its own over the 96-bit
//     (arrival, index) keys - and lists the k chosen jobs, which the ranking
//     kernel puts in order. The pred array is read four times (16 bytes per
//     job); arrivals are read for ties only.
#include <limits.h>

#include <mutex>

#include "kernels.h"
#include "kth_range.h"

namespace elis {

namespace {

constexpr int kThreads = 1024;
constexpr int kRankMaxN = 12288;  // most jobs of one ranking launch
constexpr int kSortMaxN = 8192;   // most jobs of one LDS sort, and most that are always ranked directly

__device__ __forceinline__ uint32_t order_key(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0xffffffffu;  // NaN, any sign / payload
    if (u == 0x80000000u) u = 0u;                               // -0 -> +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ bool key_less(uint32_t ka, int64_t aa, int ia, uint32_t kb, int64_t ab, int ib) {
    if (ka != kb) return ka < kb;
    if (aa != ab) return aa < ab;
    return ia < ib;
}

// Where the ranking kernel gets job i's key and arrival from, and what it writes for a chosen job.
struct PlainJobs {
    const float* pred;
    const int64_t* arrival;
    const int32_t* slots;  // null: write the index, else slots[index]
    __device__ float key(int i) const { return pred[i]; }
    __device__ int64_t arrived(int i) const { return arrival[i]; }
    __device__ bool before(int i, int j) const { return i < j; }  // the lower index, between equal arrivals
    __device__ int32_t chosen(int i) const { return slots ? slots[i] : i; }
    __device__ void check(int) const {}
};

// The jobs of a table, their keys aged when wait is given (jobs_key in kernels.h).
struct TableJobs {
    JobTable t;
    const int32_t* slots;
    const float* wait;
    float aging;
    __device__ bool ok(int32_t s) const { return s >= 0 && s < t.max_jobs; }
    __device__ float key(int i) const {
        const int32_t s = slots[i];
        return ok(s) ? jobs_key(t.pred[s], wait, aging, i) : __int_as_float(0x7fc00000);
    }
    __device__ int64_t arrived(int i) const {
        const int32_t s = slots[i];
        return ok(s) ? t.arrival[s] : 0;
    }
    __device__ bool before(int i, int j) const { return i < j; }
    __device__ int32_t chosen(int i) const { return slots[i]; }
    __device__ void check(int i) const {
        if (!ok(slots[i])) atomicOr(t.status, ELIS_DEV_BAD_SLOT);
    }
};

// Ranks a work-group's J jobs among all n <= 1024 PER and writes those of rank below k. Every
// work-group holds all n float keys in LDS; a thread counts, for one of the J jobs, the smaller
// keys of its slice of them (16 bytes per LDS read, two instructions per key). Only a job with
// fewer than k smaller keys can be chosen: a wave looks through the keys equal to its own and
// ranks those by (arrival, index). n * n / 64 lane steps, spread over up to 256 CUs.
// Bound by launch and load latency up to about 2,000 jobs, then by the counting. It replaces one
// work-group that ranked up to 1,024 jobs by full comparisons and sorted up to 8,192 in LDS:
// 256 jobs 12 -> 3.8 us, 1,024 jobs 64 -> 4, 4,096 jobs 74 -> 5.5, 8,192 jobs 151 -> 11 (k = 64).
// PER: keys a thread loads, all in flight together.
template <int J, int PER, class Jobs>
__global__ __launch_bounds__(kThreads) void select_rank_kernel(Jobs jobs, int n, int k, int32_t* __restrict__ out_idx,
                                                               int32_t* __restrict__ out_count,
                                                               uint32_t* __restrict__ status) {
    __shared__ __attribute__((aligned(16))) uint32_t sk[kThreads * PER];
    __shared__ int part[kThreads / kWave][J];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int n4 = (n + 3) / 4, i0 = blockIdx.x * J;
    float f[PER];
#pragma unroll
    for (int c = 0; c < PER; ++c) f[c] = tid + c * kThreads < n ? jobs.key(tid + c * kThreads) : 0.f;
#pragma unroll
    for (int c = 0; c < PER; ++c) {
        const int i = tid + c * kThreads;
        if (i < 4 * n4) sk[i] = i < n ? order_key(f[c]) : 0xffffffffu;  // padding is below nothing
    }
    __syncthreads();
    const uint4* s4 = reinterpret_cast<const uint4*>(sk);
    {
        const int i = i0 + (tid & (J - 1));
        const uint32_t ki = sk[i < n ? i : 0];
        int below = 0;
#pragma unroll 4
        for (int q = tid / J; q < n4; q += kThreads / J) {
            const uint4 v = s4[q];
            below += static_cast<int>(v.x < ki) + static_cast<int>(v.y < ki) + static_cast<int>(v.z < ki) +
                     static_cast<int>(v.w < ki);
        }
#pragma unroll
        for (int o = J; o < kWave; o <<= 1) below += __shfl_xor(below, o, kWave);
        if (lane < J) part[wid][lane] = below;
    }
    __syncthreads();
    for (int r = wid; r < J; r += kThreads / kWave) {  // one wave per job; all but the tie count is uniform over it
        const int i = i0 + r;
        if (i >= n) break;
        if (lane == 0) jobs.check(i);
        int rank = 0;
#pragma unroll
        for (int w = 0; w < kThreads / kWave; ++w) rank += part[w][r];
        if (rank >= k) continue;
        const uint32_t ki = sk[i];
        int ties = 0;
#pragma unroll 4
        for (int q = lane; q < n4; q += kWave) {
            const uint4 v = s4[q];
            const uint32_t e[4] = {v.x, v.y, v.z, v.w};
            if ((v.x == ki) | (v.y == ki) | (v.z == ki) | (v.w == ki)) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int j = 4 * q + c;
                    if (e[c] == ki && j != i && j < n) {
                        const int64_t ai = jobs.arrived(i), aj = jobs.arrived(j);
                        ties += static_cast<int>(aj != ai ? aj < ai : jobs.before(j, i));
                    }
                }
            }
        }
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) ties += __shfl_xor(ties, o, kWave);
        rank += ties;
        if (lane == 0 && rank < k) out_idx[rank] = jobs.chosen(i);
    }
    if (blockIdx.x == 0 && tid == 0) {
        *out_count = k < n ? k : n;
        if (status) *status = 0u;
    }
}

// Ranks up to 64 jobs. Every wave holds all of them, one per lane, and takes four in turn: the jobs before
// one are the set bits of one comparison over the wave. No LDS and no barrier, so that what remains is the
// launch and one load: 2 to 32 jobs 1.8 us, 64 jobs 2.0, whatever ties (the counting kernel above 2.4 to 2.75 with
// distinct keys and up to 3.5 with equal ones, the loop over LDS before it 1.8 for 2 jobs, 2.8 for 32).
constexpr int kFewMaxN = kWave, kFewPerWave = 4;
template <class Jobs>
__global__ __launch_bounds__(kFewMaxN / kFewPerWave* kWave) void select_few_kernel(Jobs jobs, int n, int k,
                                                                                   int32_t* __restrict__ out_idx,
                                                                                   int32_t* __restrict__ out_count,
                                                                                   uint32_t* __restrict__ status) {
    const int j = threadIdx.x & (kWave - 1), first = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) * kFewPerWave;
    uint32_t kj = 0u;
    int64_t aj = 0;
    int32_t cj = 0;
    if (j < n) {
        cj = jobs.chosen(j);
        aj = jobs.arrived(j);
        kj = order_key(jobs.key(j));
        if (first == 0) jobs.check(j);
    }
    const int lo = static_cast<int>(aj), hi = static_cast<int>(aj >> 32);
    int mine = INT_MAX;  // rank of this lane's job, where this wave ranks it
#pragma unroll
    for (int r = 0; r < kFewPerWave; ++r) {
        const int i = first + r;
        const uint32_t ki = __builtin_amdgcn_readlane(kj, i);
        const int64_t ai = static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(hi, i))) << 32 |
                                                static_cast<uint32_t>(__builtin_amdgcn_readlane(lo, i)));
        const bool before = (j < n) & ((kj < ki) | ((kj == ki) & ((aj < ai) | ((aj == ai) & (j < i)))));
        const int rank = __builtin_popcountll(__builtin_amdgcn_ballot_w64(before));
        mine = j == i ? rank : mine;
    }
    if (j < n && mine < k) out_idx[mine] = cj;
    if (threadIdx.x == 0) {
        *out_count = k < n ? k : n;
        if (status) *status = 0u;
    }
}

template <class Jobs>
hipError_t launch_rank(const Jobs& jobs, int n, int k, int32_t* out_idx, int32_t* out_count, uint32_t* status,
                       hipStream_t st) {
    // 16 jobs per work-group keep all 256 CUs busy up to 4,096 jobs; above, 32 halve the keys read per job.
    auto go = [&](auto kernel, int j) {
        return launch_kernel(kernel, dim3((n + j - 1) / j), dim3(kThreads), 0, st, jobs, n, k, out_idx, out_count, status);
    };
    if (n <= kFewMaxN)
        return launch_kernel(select_few_kernel<Jobs>, dim3(1), dim3((n + kFewPerWave - 1) / kFewPerWave * kWave), 0, st, jobs, n, k,
                             out_idx, out_count, status);
    if (n <= 4096) return go(select_rank_kernel<16, 4, Jobs>, 16);
    if (n <= 8192) return go(select_rank_kernel<32, 8, Jobs>, 32);
    return go(select_rank_kernel<32, kRankMaxN / kThreads, Jobs>, 32);
}

// ------------------------------------------------------------------------------ large n
constexpr int kLargeMaxN = 1 << 28;
constexpr int kBins = 2048;        // 11-bit digits
constexpr int kBlock = 1024;       // threads of the counting / scatter work-groups
constexpr int kMaxGroups = 256;    // work-groups of a counting / scatter pass (one chunk each)
constexpr int kReduceBlocks = kBins / 64;  // 64 bins per reducing work-group

// Device state of one large selection (workspace, written by select_init_kernel).
struct SelState {
    uint32_t need;      // jobs still to choose inside the current prefix
    uint32_t level;     // leading key bits fixed so far (0, 11, 22, 32)
    uint32_t prefix;    // their value
    uint32_t resolved;  // the bucket of the current prefix is taken whole
    uint32_t ticket;    // reduce work-groups done with the current pass
    uint32_t pad[3];
};

struct LargeWs {
    uint32_t* status;
    SelState* state;
    uint32_t* totals;   // [kBins] bucket counts of the current pass
    uint32_t* partial;  // [groups][kBins] per-work-group counts of the current pass
    uint32_t* counts;   // [groups][2] jobs chosen / tied, per work-group
    int32_t* chosen;    // [groups][kSortMaxN] chosen indices, per work-group
    int32_t* ties;      // [n] tied indices, each work-group at the start of its own chunk
    int32_t* picked;    // [kSortMaxN] ties taken by (arrival, index), then the other chosen jobs
    int chunk;          // jobs per work-group
    int groups;
};

__device__ __forceinline__ uint32_t ld_relaxed(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Four consecutive predictions i .. i+3 (16-byte load when aligned and in range); lanes past
// hi read nothing and get 0.
__device__ __forceinline__ void load4(const float* __restrict__ pred, int i, int hi, bool vec, float (&v)[4]) {
    if (vec && i + 3 < hi) {
        const f32x4 f = *reinterpret_cast<const f32x4*>(pred + i);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = f[c];
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = (i + c < hi) ? pred[i + c] : 0.f;
    }
}

// Exclusive prefix over the wave of a per-lane count below 8, and the wave total.
__device__ __forceinline__ uint32_t wave_prefix8(uint32_t c, uint32_t& total) {
    uint32_t ex = 0;
    total = 0;
#pragma unroll
    for (int bit = 0; bit < 3; ++bit) {
        const uint64_t m = __builtin_amdgcn_ballot_w64((c >> bit) & 1u);
        ex += __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)) << bit;
        total += static_cast<uint32_t>(__builtin_popcountll(m)) << bit;
    }
    return ex;
}

__global__ __launch_bounds__(256) void select_init_kernel(LargeWs ws, int k, int32_t* __restrict__ out_count) {
    if (threadIdx.x == 0) {
        SelState s{};
        s.need = static_cast<uint32_t>(k);
        *ws.state = s;
        *ws.status = 0u;
        *out_count = k;
    }
}

// Counting pass over one chunk: histogram of digit (key >> SHIFT) & (2^BITS - 1) of the jobs
// whose leading key bits equal the current prefix, stored (not added) to partial[group].
template <int SHIFT, int BITS>
__global__ __launch_bounds__(kBlock) void select_count_kernel(const float* __restrict__ pred, int n, LargeWs ws) {
    __shared__ uint32_t lh[kBins];
    const SelState* st = ws.state;
    if (st->resolved) return;
    const uint32_t level = st->level, prefix = st->prefix;
    for (int b = threadIdx.x; b < kBins; b += kBlock) lh[b] = 0u;
    __syncthreads();
    const int lo = blockIdx.x * ws.chunk;
    const int hi = lo + ws.chunk < n ? lo + ws.chunk : n;
    const bool vec = (reinterpret_cast<uintptr_t>(pred) & 15u) == 0;
    for (int base = lo; base < hi; base += 4 * kBlock) {
        float v[4];
        load4(pred, base + 4 * threadIdx.x, hi, vec, v);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool in = base + 4 * static_cast<int>(threadIdx.x) + c < hi;
            const uint32_t key = order_key(v[c]);
            const bool take = in && (level == 0 || (key >> (32 - level)) == prefix);
            const uint32_t d = (key >> SHIFT) & ((1u << BITS) - 1u);
            // Plain per-lane LDS atomics: measured faster than aggregating equal digits of a
            // wave first, even for the few leading digits of real predictions.
            if (take) atomicAdd(&lh[d], 1u);
        }
    }
    __syncthreads();
    uint32_t* out = ws.partial + static_cast<size_t>(blockIdx.x) * kBins;
    for (int b = threadIdx.x; b < kBins; b += kBlock) out[b] = lh[b];
}

// Bucket totals over the work-groups: each of kReduceBlocks work-groups owns 64 bins, its
// threads split the chunks 16 ways; the last work-group to finish picks the bucket holding
// the need-th job and advances the state.
template <int BITS>
__global__ __launch_bounds__(1024) void select_reduce_kernel(LargeWs ws) {
    __shared__ uint32_t part[16][64];
    __shared__ uint32_t scan[256];
    __shared__ bool last;
    const SelState* st = ws.state;
    if (st->resolved) return;
    const int b = threadIdx.x & 63, slice = threadIdx.x >> 6;
    const int bin = blockIdx.x * 64 + b;
    uint32_t t = 0;
    const int groups = ws.groups;
#pragma unroll 16
    for (int g = slice; g < groups; g += 16) t += ws.partial[static_cast<size_t>(g) * kBins + bin];
    part[slice][b] = t;
    __syncthreads();
    if (threadIdx.x < 64) {
        uint32_t s2 = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) s2 += part[q][threadIdx.x];
        ws.totals[blockIdx.x * 64 + threadIdx.x] = s2;
    }
    // One release fence after the barrier covers the work-group's stores (fences are costly
    // here: an agent-scope fence writes back and invalidates the XCD's L2).
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        last = atomicAdd(&ws.state->ticket, 1u) == kReduceBlocks - 1;
        if (last) __threadfence();
    }
    __syncthreads();
    if (!last) return;  // uniform over the work-group
    // The first 256 threads scan 8 bins each; all 1024 take part in the barriers.
    constexpr int PER = kBins / 256;
    const bool act = threadIdx.x < 256;
    uint32_t h[PER], sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        h[j] = act ? ld_relaxed(&ws.totals[threadIdx.x * PER + j]) : 0u;
        sum += h[j];
    }
    if (act) scan[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint32_t v = (act && threadIdx.x >= off) ? scan[threadIdx.x - off] : 0u;
        __syncthreads();
        if (act) scan[threadIdx.x] += v;
        __syncthreads();
    }
    if (!act) return;
    const uint32_t need = st->need, level = st->level, prefix = st->prefix;
    uint32_t below = scan[threadIdx.x] - sum;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (below < need && need <= below + h[j]) {
            SelState* w = ws.state;
            w->prefix = (prefix << BITS) | static_cast<uint32_t>(threadIdx.x * PER + j);
            w->level = level + BITS;
            w->need = need - below;
            w->resolved = (h[j] == need - below) ? 1u : 0u;
            w->ticket = 0u;
        }
        below += h[j];
    }
}

// Scatter over one chunk, in index order: key < prefix (or == prefix when resolved) ->
// chosen[group]; key == prefix otherwise -> this chunk's part of the tie list.
__global__ __launch_bounds__(kBlock) void select_scatter_kernel(const float* __restrict__ pred, int n, LargeWs ws) {
    __shared__ uint32_t wsum[2][kBlock / kWave];
    const SelState* st = ws.state;
    const uint32_t level = st->level, prefix = st->prefix;
    const bool resolved = st->resolved != 0u;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int lo = blockIdx.x * ws.chunk;
    const int hi = lo + ws.chunk < n ? lo + ws.chunk : n;
    int32_t* chosen = ws.chosen + static_cast<size_t>(blockIdx.x) * kSortMaxN;
    int32_t* ties = ws.ties + lo;
    const bool vec = (reinterpret_cast<uintptr_t>(pred) & 15u) == 0;
    uint32_t nc = 0, nt = 0;  // running counts of this work-group (uniform)
    for (int base = lo; base < hi; base += 4 * kBlock) {
        const int i0 = base + 4 * threadIdx.x;
        float v[4];
        load4(pred, i0, hi, vec, v);
        bool c[4], t[4];
        uint32_t cc = 0, ct = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t top = order_key(v[q]) >> (32 - level);
            const bool in = i0 + q < hi;
            c[q] = in && (top < prefix || (top == prefix && resolved));
            t[q] = in && top == prefix && !resolved;
            cc += c[q] ? 1u : 0u;
            ct += t[q] ? 1u : 0u;
        }
        uint32_t wc, wt;
        const uint32_t rc = wave_prefix8(cc, wc), rt = wave_prefix8(ct, wt);
        if (lane == 0) {
            wsum[0][wv] = wc;
            wsum[1][wv] = wt;
        }
        __syncthreads();
        uint32_t oc = nc, ot = nt, tc = 0, tt = 0;
        for (int w = 0; w < kBlock / kWave; ++w) {
            if (w < wv) {
                oc += wsum[0][w];
                ot += wsum[1][w];
            }
            tc += wsum[0][w];
            tt += wsum[1][w];
        }
        oc += rc;
        ot += rt;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (c[q]) chosen[oc++] = i0 + q;
            if (t[q]) ties[ot++] = i0 + q;
        }
        nc += tc;
        nt += tt;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        ws.counts[2 * blockIdx.x] = nc;
        ws.counts[2 * blockIdx.x + 1] = nt;
    }
}

// 96-bit tie key (arrival made unsigned-orderable, then index): bits [lo, lo + w).
__device__ __forceinline__ uint32_t tie_digit(uint64_t a, uint32_t idx, int lo, int w) {
    const uint64_t mask = (1ull << w) - 1ull;
    if (lo >= 32) return static_cast<uint32_t>((a >> (lo - 32)) & mask);
    if (lo + w <= 32) return static_cast<uint32_t>((idx >> lo) & mask);
    return static_cast<uint32_t>((((a << (32 - lo)) | (idx >> lo))) & mask);
}

__device__ __forceinline__ uint64_t arrival_key(int64_t a) { return static_cast<uint64_t>(a) ^ 0x8000000000000000ull; }

// One work-group: bitonic sort of P (power of two) entries in LDS by (key, arrival, index).
__device__ void block_bitonic(uint32_t* sk, int64_t* sa, int32_t* si, int P) {
    for (int size = 2; size <= P; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = threadIdx.x; t < (P >> 1); t += kThreads) {
                const int lo = 2 * t - (t & (stride - 1));
                const int hi = lo + stride;
                const bool up = (lo & size) == 0;
                const bool hi_first = key_less(sk[hi], sa[hi], si[hi], sk[lo], sa[lo], si[lo]);
                if (hi_first == up) {
                    const uint32_t tk = sk[lo];
                    sk[lo] = sk[hi];
                    sk[hi] = tk;
                    const int64_t ta = sa[lo];
                    sa[lo] = sa[hi];
                    sa[hi] = ta;
                    const int32_t ti = si[lo];
                    si[lo] = si[hi];
                    si[hi] = ti;
                }
            }
            __syncthreads();
        }
    }
}

__device__ __forceinline__ int pow2_at_least(int n) {
    int P = 1;
    while (P < n) P <<= 1;
    return P;
}

// Exclusive scan of per-work-group counts (groups <= kThreads) into offs[g]; returns the total.
__device__ uint32_t block_offsets(const uint32_t* counts, int which, int groups, uint32_t* offs, uint32_t* scan) {
    const uint32_t v = threadIdx.x < groups ? counts[2 * threadIdx.x + which] : 0u;
    scan[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < kThreads; off <<= 1) {
        const uint32_t u = threadIdx.x >= off ? scan[threadIdx.x - off] : 0u;
        __syncthreads();
        scan[threadIdx.x] += u;
        __syncthreads();
    }
    if (threadIdx.x < groups) offs[threadIdx.x] = scan[threadIdx.x] - v;
    const uint32_t total = scan[kThreads - 1];
    __syncthreads();
    return total;
}

// Index r (< total) of a list split over work-groups: which group holds it (binary search
// over the exclusive offsets) and at which position.
__device__ __forceinline__ int find_group(const uint32_t* offs, int groups, uint32_t r) {
    int lo = 0, hi = groups - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (offs[mid] <= r) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// One work-group: choose the needed ties by (arrival, index), then list the k chosen jobs.
__global__ __launch_bounds__(kThreads) void select_ties_kernel(const int64_t* __restrict__ arrival, LargeWs ws) {
    __shared__ uint32_t sk[kSortMaxN];
    __shared__ int64_t sa[kSortMaxN];
    __shared__ int32_t si[kSortMaxN];
    __shared__ uint32_t offc[kMaxGroups], offt[kMaxGroups];
    __shared__ uint32_t scan[kThreads];
    __shared__ uint32_t hist[kBins];
    __shared__ uint32_t sh_bucket, sh_below, sh_cnt;
    const int groups = ws.groups;
    const uint32_t nchosen = block_offsets(ws.counts, 0, groups, offc, scan);
    uint32_t ntie = block_offsets(ws.counts, 1, groups, offt, scan);
    const uint32_t need0 = ws.state->resolved ? 0u : ws.state->need;
    uint32_t npicked = 0;
    if (need0 > 0 && ntie <= static_cast<uint32_t>(kSortMaxN)) {
        // All ties share the float key: sort them by (arrival, index), take the first need0.
        const int P = pow2_at_least(static_cast<int>(ntie));
        for (int r = threadIdx.x; r < P; r += kThreads) {
            if (r < static_cast<int>(ntie)) {
                const int g = find_group(offt, groups, static_cast<uint32_t>(r));
                const int32_t j = ws.ties[static_cast<size_t>(g) * ws.chunk + (r - static_cast<int>(offt[g]))];
                sk[r] = 0u;
                sa[r] = arrival[j];
                si[r] = j;
            } else {
                sk[r] = 0xffffffffu;
                sa[r] = LLONG_MAX;
                si[r] = INT_MAX;
            }
        }
        __syncthreads();
        block_bitonic(sk, sa, si, P);
        for (int r = threadIdx.x; r < static_cast<int>(need0); r += kThreads) ws.picked[r] = si[r];
        npicked = need0;
        __syncthreads();
    } else if (need0 > 0) {
        // Many ties: make the tie list contiguous (in place, moving forward), then a radix
        // selection over the 96-bit (arrival, index) key by this work-group, compacting the
        // list after every digit.
        for (int g = 0; g < groups; ++g) {
            const uint32_t cnt = ws.counts[2 * g + 1];
            // offt[g] <= g * chunk: every sweep reads its sources before any is overwritten.
            for (uint32_t base = 0; base < cnt; base += kThreads) {
                const uint32_t r = base + threadIdx.x;
                int32_t j = 0;
                if (r < cnt) j = ws.ties[static_cast<size_t>(g) * ws.chunk + r];
                __syncthreads();
                if (r < cnt) ws.ties[offt[g] + r] = j;
                __syncthreads();
            }
        }
        uint32_t need = need0;
        int lo = 96;
        while (need > 0 && lo > 0) {
            const int w = lo >= 11 ? 11 : lo;
            lo -= w;
            for (int b = threadIdx.x; b < kBins; b += kThreads) hist[b] = 0u;
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < ntie; t += kThreads) {
                const int32_t j = ws.ties[t];
                atomicAdd(&hist[tie_digit(arrival_key(arrival[j]), static_cast<uint32_t>(j), lo, w)], 1u);
            }
            __syncthreads();
            constexpr int PER = kBins / kThreads;
            uint32_t h[PER], sum = 0;
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                h[q] = hist[threadIdx.x * PER + q];
                sum += h[q];
            }
            scan[threadIdx.x] = sum;
            __syncthreads();
            for (int off = 1; off < kThreads; off <<= 1) {
                const uint32_t v = threadIdx.x >= off ? scan[threadIdx.x - off] : 0u;
                __syncthreads();
                scan[threadIdx.x] += v;
                __syncthreads();
            }
            uint32_t below = scan[threadIdx.x] - sum;
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                if (below < need && need <= below + h[q]) {
                    sh_bucket = threadIdx.x * PER + q;
                    sh_below = below;
                    sh_cnt = h[q];
                }
                below += h[q];
            }
            __syncthreads();
            const uint32_t bucket = sh_bucket;
            const bool take_all = sh_cnt == need - sh_below;
            // digit < bucket (or == bucket when taken whole) -> picked; == bucket -> kept.
            uint32_t kept = 0, picked = npicked;
            for (uint32_t base = 0; base < ntie; base += kThreads) {
                const uint32_t t = base + threadIdx.x;
                int32_t j = 0;
                uint32_t dg = 0xffffffffu;
                if (t < ntie) {
                    j = ws.ties[t];
                    dg = tie_digit(arrival_key(arrival[j]), static_cast<uint32_t>(j), lo, w);
                }
                const bool ch = t < ntie && (dg < bucket || (dg == bucket && take_all));
                const bool kp = t < ntie && dg == bucket && !take_all;
                const uint32_t mine = (ch ? 1u : 0u) | (kp ? 0x10000u : 0u);
                scan[threadIdx.x] = mine;
                __syncthreads();
                for (int off = 1; off < kThreads; off <<= 1) {
                    const uint32_t v = threadIdx.x >= off ? scan[threadIdx.x - off] : 0u;
                    __syncthreads();
                    scan[threadIdx.x] += v;
                    __syncthreads();
                }
                const uint32_t ex = scan[threadIdx.x] - mine, tot = scan[kThreads - 1];
                if (ch) ws.picked[picked + (ex & 0xffffu)] = j;
                if (kp) ws.ties[kept + (ex >> 16)] = j;  // kept + rank <= t: in-place is safe
                picked += tot & 0xffffu;
                kept += tot >> 16;
                __syncthreads();
            }
            need = take_all ? 0u : need - (picked - npicked);
            npicked = picked;
            ntie = kept;
            __syncthreads();
        }
    }
    // The jobs chosen by the scatter behind the ties: one list of k, which the ranking kernel orders.
    for (int r = threadIdx.x; r < static_cast<int>(nchosen); r += kThreads) {
        const int g = find_group(offc, groups, static_cast<uint32_t>(r));
        ws.picked[npicked + r] = ws.chosen[static_cast<size_t>(g) * kSortMaxN + (r - static_cast<int>(offc[g]))];
    }
}

// Jobs named by a list of indices, for the ranking kernel.
struct ListedJobs {
    const float* pred;
    const int64_t* arrival;
    const int32_t* list;
    __device__ float key(int i) const { return pred[list[i]]; }
    __device__ int64_t arrived(int i) const { return arrival[list[i]]; }
    __device__ bool before(int i, int j) const { return list[i] < list[j]; }
    __device__ int32_t chosen(int i) const { return list[i]; }
    __device__ void check(int) const {}
};

// ------------------------------------------------------------------------------ group minima
// Selection in three launches where few jobs can come into question, from the smallest job (in the
// full order) of each of up to 4,096 groups: the k-th smallest of these minima bounds the k-th job
// from above, and only the k groups whose minimum it reaches hold candidates. At most k groups of
// jobs are candidates, whatever the data; on data without structure hardly more than k jobs are.
//   minima     every group's smallest job;
//   filter     every work-group finds the k-th smallest minimum by itself (block_kth, per 32-bit word
//              of the full key) and lists its own jobs up to it;
//   rank list  the candidates are ranked as in select_rank_kernel.
// The radix path takes nine launches and four reads of the keys: 45 us at 2^20 jobs, k = 64, this one
// 20 (4.5 + 9 + 6: launches, load latency and the barriers of the search; the keys are 4 MB).
// Equal keys cost the ranking a load of the index and one of the arrival per pair: up to 0.8 ms where all
// of the most candidates tie.
constexpr int kMinWgs = 256, kMinGroups = 16;  // work-groups, and groups of each
constexpr int kCandidates = 32768;             // most candidates: their keys are ranked out of LDS
constexpr int kMinMaxN = 1 << 21;

struct MinimaWs {
    uint32_t* key;    // [kMinWgs * kMinGroups] minima: ordered key and index (no job: the largest key, index -1)
    int32_t* idx;
    int32_t* count;   // [kMinWgs] candidates of each work-group
    uint32_t* ckey;   // [kMinWgs][cap] their keys and indices
    int32_t* cidx;
    int lanes;        // lanes (of 4 jobs a sweep) per group
    int sweeps;       // 1024-thread sweeps of a work-group's jobs
    int cap;          // jobs of a work-group, rounded up
};

// Quad u of work-group b: segments of 16 jobs are dealt out in turn, so that jobs in order of their
// keys spread over all work-groups and groups.
__device__ __forceinline__ int quad_first(int b, int u) { return ((u >> 2) * kMinWgs + b) * 16 + (u & 3) * 4; }

__device__ __forceinline__ bool job_less(uint32_t ka, int ia, uint32_t kb, int ib, const int64_t* arrival) {
    if (ia < 0 || ib < 0) return ib < 0 && ia >= 0;
    if (ka != kb) return ka < kb;
    const int64_t aa = arrival[ia], ab = arrival[ib];
    return aa != ab ? aa < ab : ia < ib;
}

__global__ __launch_bounds__(kThreads) void select_minima_kernel(const float* __restrict__ pred,
                                                                 const int64_t* __restrict__ arrival, int n,
                                                                 MinimaWs ws) {
    const bool vec = (reinterpret_cast<uintptr_t>(pred) & 15u) == 0;
    uint32_t bk = 0xffffffffu;
    int bi = -1;
    for (int s = 0; s < ws.sweeps; ++s) {
        const int i0 = quad_first(blockIdx.x, s * kThreads + threadIdx.x);
        if (i0 >= n) continue;
        float v[4];
        load4(pred, i0, n, vec, v);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t key = order_key(v[c]);
            if (i0 + c < n && job_less(key, i0 + c, bk, bi, arrival)) bk = key, bi = i0 + c;
        }
    }
    for (int o = 1; o < ws.lanes; o <<= 1) {
        const uint32_t ok = __shfl_xor(bk, o, kWave);
        const int oi = __shfl_xor(bi, o, kWave);
        if (job_less(ok, oi, bk, bi, arrival)) bk = ok, bi = oi;
    }
    const int g = static_cast<int>(threadIdx.x) / ws.lanes;
    if (threadIdx.x % ws.lanes == 0 && g < kMinGroups) {
        ws.key[blockIdx.x * kMinGroups + g] = bk;
        ws.idx[blockIdx.x * kMinGroups + g] = bi;
    }
}

// Scratch of block_kth.
static_assert(kKthBins == kThreads, "one bin per thread");
struct KthScratch {
    uint32_t range[2][kThreads / kWave];
    int wave[kThreads / kWave];
    int bin[kKthBins];
    int found, below;
};

// The smallest v such that at least need of the work-group's active values are <= v; need becomes its
// rank among the values equal to v, active their number, and only those stay active. The range of the
// active values (small arrival numbers and one round's predictions span far fewer than 32 bits) is cut to
// one of 1,024 equal parts at a time: two or three counting rounds in LDS (a binary search, two barriers
// for each of its 24 steps, took 13 us for 4,096 minima; this 3).
template <int PER>
__device__ __forceinline__ uint32_t block_kth(const uint32_t (&v)[PER], bool (&act)[PER], int& need, int& active,
                                              KthScratch& sh) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        lo = act[q] && v[q] < lo ? v[q] : lo;
        hi = act[q] && v[q] > hi ? v[q] : hi;
    }
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t a = __shfl_xor(lo, o, kWave), b = __shfl_xor(hi, o, kWave);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    __syncthreads();  // the scratch may still be read from the last call
    if (lane == 0) sh.range[0][wid] = lo, sh.range[1][wid] = hi;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) {
        lo = sh.range[0][w] < lo ? sh.range[0][w] : lo;
        hi = sh.range[1][w] > hi ? sh.range[1][w] : hi;
    }
    KthRange range{lo, hi};
    for (;;) {  // uniform: 32 bits are gone after four rounds
        const int shift = range.shift();
        sh.bin[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (act[q]) atomicAdd(&sh.bin[range.part(v[q], shift)], 1);
        __syncthreads();
        const int mine = sh.bin[tid];
        int incl = mine;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int u = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += u;
        }
        if (lane == kWave - 1) sh.wave[wid] = incl;
        __syncthreads();
        for (int w = 0; w < wid; ++w) incl += sh.wave[w];
        if (incl - mine < need && need <= incl) {  // one thread: the bin that holds the need-th value
            sh.found = tid;
            sh.below = incl - mine;
        }
        __syncthreads();
        const uint32_t bin = static_cast<uint32_t>(sh.found);
        need -= sh.below;
        active = sh.bin[bin];
#pragma unroll
        for (int q = 0; q < PER; ++q) act[q] = act[q] && range.part(v[q], shift) == bin;
        range.cut(bin, shift);
        if (shift == 0) return range.lo;
        __syncthreads();  // bins are cleared again
    }
}

__global__ __launch_bounds__(kThreads) void select_filter_kernel(const float* __restrict__ pred,
                                                                 const int64_t* __restrict__ arrival, int n, int k,
                                                                 MinimaWs ws) {
    __shared__ KthScratch sh;
    __shared__ int cnt[kThreads / kWave];
    __shared__ int listed;
    if (threadIdx.x == 0) listed = 0;
    constexpr int PER = kMinWgs * kMinGroups / kThreads, kSweeps = kMinMaxN / (4 * kThreads * kMinWgs);
    const bool vec = (reinterpret_cast<uintptr_t>(pred) & 15u) == 0;
    float v[kSweeps][4];  // this thread's jobs, requested before the search
#pragma unroll
    for (int s = 0; s < kSweeps; ++s) load4(pred, quad_first(blockIdx.x, s * kThreads + threadIdx.x), s < ws.sweeps ? n : 0, vec, v[s]);
    uint32_t mk[PER];
    int mi[PER];
    bool act[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        mk[q] = ws.key[q * kThreads + threadIdx.x];
        mi[q] = ws.idx[q * kThreads + threadIdx.x];
        act[q] = mi[q] >= 0;
    }
    int need = k, active = 0;
    // Bound: jobs below (key, arrival, index), the last two only when some of the minima with this key are above it.
    uint32_t bound_k = 0xffffffffu;
    uint64_t bound_a = ~0ull;
    int bound_i = INT_MAX;
    bool whole = true;  // every job with the bound's key is a candidate
    int jobs = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) jobs += __builtin_popcountll(__builtin_amdgcn_ballot_w64(act[q]));
    if ((threadIdx.x & (kWave - 1)) == 0) cnt[threadIdx.x / kWave] = jobs;
    __syncthreads();
    jobs = 0;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) jobs += cnt[w];
    if (jobs >= k) {  // else (fewer groups than k) every job is a candidate
        bound_k = block_kth(mk, act, need, active, sh);
        if (active > need) {
            whole = false;
            uint32_t w[PER];
            uint32_t word[2];
#pragma unroll
            for (int part = 0; part < 2; ++part) {
#pragma unroll
                for (int q = 0; q < PER; ++q)
                    w[q] = act[q] ? static_cast<uint32_t>(arrival_key(arrival[mi[q]]) >> (part ? 0 : 32)) : 0u;
                word[part] = block_kth(w, act, need, active, sh);
            }
            bound_a = (static_cast<uint64_t>(word[0]) << 32) | word[1];
#pragma unroll
            for (int q = 0; q < PER; ++q) w[q] = static_cast<uint32_t>(mi[q]);
            bound_i = static_cast<int>(block_kth(w, act, need, active, sh));
        }
    }
    uint32_t* ck = ws.ckey + static_cast<size_t>(blockIdx.x) * ws.cap;
    int32_t* ci = ws.cidx + static_cast<size_t>(blockIdx.x) * ws.cap;
#pragma unroll
    for (int s = 0; s < kSweeps; ++s) {
        const int i0 = quad_first(blockIdx.x, s * kThreads + threadIdx.x);
        if (s >= ws.sweeps || i0 >= n) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = i0 + c;
            const uint32_t key = order_key(v[s][c]);
            bool in = i < n && (key < bound_k || (key == bound_k && whole));
            if (i < n && key == bound_k && !whole) {
                const uint64_t a = arrival_key(arrival[i]);
                in = a < bound_a || (a == bound_a && i <= bound_i);
            }
            if (in) {
                const int at = atomicAdd(&listed, 1);
                ck[at] = key;
                ci[at] = i;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) ws.count[blockIdx.x] = listed;
}

__global__ __launch_bounds__(kThreads) void select_rank_list_kernel(const int64_t* __restrict__ arrival, int k,
                                                                    MinimaWs ws, int32_t* __restrict__ out_idx,
                                                                    int32_t* __restrict__ out_count,
                                                                    uint32_t* __restrict__ status) {
    constexpr int J = 16;
    __shared__ __attribute__((aligned(16))) uint32_t sk[kCandidates];
    __shared__ uint32_t off[kMinWgs];
    __shared__ uint32_t scan[kThreads];
    __shared__ int part[kThreads / kWave][J];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    if (blockIdx.x == 0 && tid == 0) {
        *out_count = k;
        *status = 0u;
    }
    const int mine = tid < kMinWgs ? ws.count[tid] : 0;
    int incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int v = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += v;
    }
    if (lane == kWave - 1) scan[wid] = static_cast<uint32_t>(incl);
    __syncthreads();
    int total = 0;
    for (int w = 0; w < kMinWgs / kWave; ++w) {
        if (w < wid) incl += static_cast<int>(scan[w]);
        total += static_cast<int>(scan[w]);
    }
    if (tid < kMinWgs) off[tid] = static_cast<uint32_t>(incl - mine);
    __syncthreads();
    if (static_cast<int>(blockIdx.x) * J >= total) return;  // uniform
    const int n4 = (total + 3) / 4;
    auto place = [&](int r) {
        const int g = find_group(off, kMinWgs, static_cast<uint32_t>(r));
        return static_cast<size_t>(g) * ws.cap + (r - static_cast<int>(off[g]));
    };
    for (int r = tid; r < 4 * n4; r += kThreads) sk[r] = r < total ? ws.ckey[place(r)] : 0xffffffffu;
    __syncthreads();
    const uint4* s4 = reinterpret_cast<const uint4*>(sk);
    for (int i0 = blockIdx.x * J; i0 < total; i0 += gridDim.x * J) {
        const int i = i0 + (tid & (J - 1));
        const uint32_t ki = sk[i < total ? i : 0];
        int below = 0;
#pragma unroll 4
        for (int q = tid / J; q < n4; q += kThreads / J) {
            const uint4 v = s4[q];
            below += static_cast<int>(v.x < ki) + static_cast<int>(v.y < ki) + static_cast<int>(v.z < ki) +
                     static_cast<int>(v.w < ki);
        }
#pragma unroll
        for (int o = J; o < kWave; o <<= 1) below += __shfl_xor(below, o, kWave);
        if (lane < J) part[wid][lane] = below;
        __syncthreads();
        const int r = i0 + wid;  // one wave per job
        int rank = k;
        if (r < total) {
            rank = 0;
#pragma unroll
            for (int w = 0; w < kThreads / kWave; ++w) rank += part[w][wid];
        }
        if (rank < k) {  // uniform over the wave
            const uint32_t kr = sk[r];
            const int32_t ir = ws.cidx[place(r)];
            int ties = 0;
#pragma unroll 4
            for (int q = lane; q < n4; q += kWave) {
                const uint4 v = s4[q];
                const uint32_t e[4] = {v.x, v.y, v.z, v.w};
                uint32_t same = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) same |= e[c] == kr && 4 * q + c != r && 4 * q + c < total ? 1u << c : 0u;
                if (!same) continue;
                const int64_t ar = arrival[ir];
                int g = find_group(off, kMinWgs, static_cast<uint32_t>(4 * q));  // of the first; the others follow it
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int j = 4 * q + c;
                    if (!((same >> c) & 1u)) continue;
                    while (g + 1 < kMinWgs && off[g + 1] <= static_cast<uint32_t>(j)) ++g;
                    const int32_t ij = ws.cidx[static_cast<size_t>(g) * ws.cap + (j - static_cast<int>(off[g]))];
                    const int64_t aj = arrival[ij];
                    ties += static_cast<int>((aj < ar) | ((aj == ar) & (ij < ir)));
                }
            }
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) ties += __shfl_xor(ties, o, kWave);
            rank += ties;
            if (lane == 0 && rank < k) out_idx[rank] = ir;
        }
        __syncthreads();  // part is written again
    }
}

}  // namespace

int select_max_n() { return kLargeMaxN; }
int select_max_k(int n) { return n <= kSortMaxN ? INT_MAX : kSortMaxN; }

namespace {

struct LargePlan {
    int groups, chunk;
};

LargePlan large_plan(int n) {
    // Chunks of at least two sweeps of a 1024-thread work-group reading 4 jobs per thread,
    // a multiple of 4096 jobs (16-byte aligned starts), at most kMaxGroups of them.
    constexpr int kSweep = 4 * kBlock;
    int groups = (n + 2 * kSweep - 1) / (2 * kSweep);
    groups = groups < kMaxGroups ? groups : kMaxGroups;
    const int chunk = ((n + groups - 1) / groups + kSweep - 1) / kSweep * kSweep;
    return LargePlan{(n + chunk - 1) / chunk, chunk};
}

size_t large_layout(int n, LargeWs* ws, char* base) {
    const LargePlan pl = large_plan(n);
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align_up(bytes);
        return base ? base + at : nullptr;
    };
    LargeWs w{};
    w.status = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t)));
    w.state = reinterpret_cast<SelState*>(take(sizeof(SelState)));
    w.totals = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * kBins));
    w.partial = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * kBins * static_cast<size_t>(pl.groups)));
    w.counts = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * 2 * static_cast<size_t>(pl.groups)));
    w.chosen = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * kSortMaxN * static_cast<size_t>(pl.groups)));
    w.ties = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * static_cast<size_t>(n)));
    w.picked = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * kSortMaxN));
    w.chunk = pl.chunk;
    w.groups = pl.groups;
    if (ws) *ws = w;
    return o;
}

// Group-minima layout for n jobs, in the workspace of the radix path; returns its bytes.
size_t minima_layout(int n, MinimaWs* ws, char* base) {
    const int segments = (n + 15) / 16, per_wg = (segments + kMinWgs - 1) / kMinWgs, quads = 4 * per_wg;
    MinimaWs w{};
    w.cap = 16 * per_wg;
    w.sweeps = (quads + kThreads - 1) / kThreads;
    w.lanes = 1;
    while (w.lanes * kMinGroups < (quads < kThreads ? quads : kThreads)) w.lanes <<= 1;
    size_t o = align_up(sizeof(uint32_t));  // the status word
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align_up(bytes);
        return base ? base + at : nullptr;
    };
    w.key = reinterpret_cast<uint32_t*>(take(4 * kMinWgs * kMinGroups));
    w.idx = reinterpret_cast<int32_t*>(take(4 * kMinWgs * kMinGroups));
    w.count = reinterpret_cast<int32_t*>(take(4 * kMinWgs));
    w.ckey = reinterpret_cast<uint32_t*>(take(4 * static_cast<size_t>(kMinWgs) * w.cap));
    w.cidx = reinterpret_cast<int32_t*>(take(4 * static_cast<size_t>(kMinWgs) * w.cap));
    if (ws) *ws = w;
    return o;
}

}  // namespace

size_t select_workspace_bytes(int n) {
    if (n < 1 || n > kLargeMaxN) return 0;
    if (n <= kSortMaxN) return align_up(sizeof(uint32_t));
    return large_layout(n, nullptr, nullptr);
}

hipError_t launch_select(const float* pred, const int64_t* arrival, int n, int k, int32_t* out_idx,
                         int32_t* out_count, void* workspace, hipStream_t st) {
    if (n < 1 || n > kLargeMaxN || k < 0) return hipErrorInvalidValue;
    uint32_t* status = static_cast<uint32_t*>(workspace);
    const PlainJobs all{pred, arrival, nullptr};
    if (n <= kSortMaxN) return launch_rank(all, n, k, out_idx, out_count, status, st);
    const int kk = k < n ? k : n;
    if (kk > kSortMaxN) return hipErrorInvalidValue;
    // Group minima while the candidates (k groups of at most lanes * 4 * sweeps jobs) fit the ranking kernel's LDS
    // and at most half of the groups hold any (beyond, nearly every job becomes one). Past that, up to 12,288 jobs are
    // ranked directly, more take the radix path. In us, distinct keys / one key for all jobs (FCFS):
    //                        minima       direct       radix
    //   8,193, k = 64       18 / 54        -          39 / 199
    //   8,193, k = 2,048    34 / 263    15 / 69       70 / 222
    //   12,288, k = 8,192   47 / 539    30 / 186     187 / 375
    //   65,536, k = 1,024   21 / 809       -          55 / 981
    //   2^20, k = 64        21 / 80        -          45 / 17,000
    MinimaWs mw;
    const bool fits = minima_layout(n, &mw, static_cast<char*>(workspace)) <= large_layout(n, nullptr, nullptr);
    const int most = kk * (mw.lanes * 4 * mw.sweeps);
    const bool few = 2 * most <= n;
    if (n <= kRankMaxN && !few) return launch_rank(all, n, kk, out_idx, out_count, status, st);
    if (kk > 0 && n <= kMinMaxN && fits && few && most <= kCandidates) {
        ELIS_TRY(launch_kernel(select_minima_kernel, dim3(kMinWgs), dim3(kThreads), 0, st, pred, arrival, n, mw));
        ELIS_TRY(launch_kernel(select_filter_kernel, dim3(kMinWgs), dim3(kThreads), 0, st, pred, arrival, n, kk, mw));
        ELIS_TRY(launch_kernel(select_rank_list_kernel, dim3(kMinWgs), dim3(kThreads), 0, st, arrival, kk, mw, out_idx, out_count,
                               status));
        return hipSuccess;
    }
    LargeWs ws;
    large_layout(n, &ws, static_cast<char*>(workspace));
    ELIS_TRY(launch_kernel(select_init_kernel, dim3(1), dim3(256), 0, st, ws, kk, out_count));
    if (kk == 0) return hipSuccess;
    const dim3 grid(ws.groups), red(kReduceBlocks);
    ELIS_TRY(launch_kernel((select_count_kernel<21, 11>), grid, dim3(kBlock), 0, st, pred, n, ws));
    ELIS_TRY(launch_kernel((select_reduce_kernel<11>), red, dim3(1024), 0, st, ws));
    ELIS_TRY(launch_kernel((select_count_kernel<10, 11>), grid, dim3(kBlock), 0, st, pred, n, ws));
    ELIS_TRY(launch_kernel((select_reduce_kernel<11>), red, dim3(1024), 0, st, ws));
    ELIS_TRY(launch_kernel((select_count_kernel<0, 10>), grid, dim3(kBlock), 0, st, pred, n, ws));
    ELIS_TRY(launch_kernel((select_reduce_kernel<10>), red, dim3(1024), 0, st, ws));
    ELIS_TRY(launch_kernel(select_scatter_kernel, grid, dim3(kBlock), 0, st, pred, n, ws));
    ELIS_TRY(launch_kernel(select_ties_kernel, dim3(1), dim3(kThreads), 0, st, arrival, ws));
    return launch_rank(ListedJobs{pred, arrival, ws.picked}, kk, kk, out_idx, out_count, nullptr, st);
}

hipError_t launch_jobs_select(JobTable t, const int32_t* slots, const float* wait, float aging, int a, int k,
                              int32_t* out_slots, int32_t* out_count, void* workspace, hipStream_t st) {
    // Up to 1,024 candidates (one per thread) the ranking kernel gathers them itself: one launch instead of the
    // gather, the select and the map back to slots.
    if (a <= kThreads) return launch_rank(TableJobs{t, slots, wait, aging}, a, k, out_slots, out_count, nullptr, st);
    const size_t n = static_cast<size_t>(a);
    char* p = static_cast<char*>(workspace);
    float* pred = reinterpret_cast<float*>(p);
    int64_t* arr = reinterpret_cast<int64_t*>(p + align_up(4 * n));
    int32_t* idx = reinterpret_cast<int32_t*>(p + align_up(4 * n) + align_up(8 * n));
    void* sel_ws = p + align_up(4 * n) + align_up(8 * n) + align_up(4 * n);
    // Bad slots are flagged in the table's status word: the select clears its own.
    ELIS_TRY(launch_jobs_gather(t, slots, wait, aging, a, pred, arr, st));
    if (a <= kSortMaxN)
        return launch_rank(PlainJobs{pred, arr, slots}, a, k, out_slots, out_count, static_cast<uint32_t*>(sel_ws), st);
    ELIS_TRY(launch_select(pred, arr, a, k, idx, out_count, sel_ws, st));
    const int kk = k < a ? k : a;
    return kk > 0 ? launch_jobs_map(slots, idx, out_count, kk, out_slots, st) : hipSuccess;
}

// ---------------------------------------------------------------------------------------------
// Allocation-free select: the same launches as launch_select on a fixed per-device scratch array
// instead of a caller workspace. `scratch` below is a device variable: in host code its name is
// only a stand-in, so the host takes the array's device address once per device with
// hipGetSymbolAddress and passes that address to the kernels. Each launch sequence initialises
// what it reads (select_init_kernel writes the selection state and status; every count, list and
// histogram is stored before it is read), so nothing needs clearing between calls.

namespace {

static_assert(kNoAllocScratchBytes % kAlign == 0, "scratch size");
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, once taken

hipError_t scratch_address(void** out) {
    int dev = 0;
    ELIS_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        ELIS_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

int select_noalloc_max_n() {
    static_assert(kNoAllocMaxN <= kLargeMaxN, "limit");
    return kNoAllocMaxN;
}

hipError_t launch_select_noalloc(const float* pred, const int64_t* arrival, int n, int k, int32_t* out_idx,
                                 int32_t* out_count, hipStream_t st) {
    if (n < 1 || n > kNoAllocMaxN || select_workspace_bytes(n) > kNoAllocScratchBytes) return hipErrorInvalidValue;
    void* ws = nullptr;
    ELIS_TRY(scratch_address(&ws));
    return launch_select(pred, arrival, n, k, out_idx, out_count, ws, st);
}

}  // namespace elis
