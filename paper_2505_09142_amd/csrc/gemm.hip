// Dense layers of the encoder on the CDNA4 matrix cores:
//   out[m, n] = epilogue( sum_k x[m, k] * w[n, k] + bias[n] )
// x is the activation, bf16 [M, K] row-major; w is the weight, bf16 [N, K]
// row-major ([out, in]); both operands are K-contiguous. fp32 accumulation.
// Epilogues: bf16 out; bf16 out after GELU; fp32 out plus a residual, which is
// either an fp32 matrix or a LayerNorm output rebuilt from its pre-norm rows and
// row statistics (Residual in kernels.h).
//
// Four kernels; launch_gemm plans each product (plan_gemm: one launch, or a
// launch of large tiles over whole rounds plus one of small tiles over the remaining rows):
//   gemm_kernel        register-staged k-slabs, 16 x 16 x 32 MFMA blocks; for N that
//                      is an odd multiple of 64;
//   gemm_sched_kernel  k-slabs go HBM -> LDS with global_load_lds_dwordx4 (no register
//                      staging), 32 x 32 x 16 MFMA blocks, a hand-scheduled k-loop
//                      (operand fragments double-buffered in registers, MFMAs of the
//                      last k-step of a slab issued after the slab barrier) and an
//                      epilogue staged through LDS for full-line stores; tiles of
//                      128 x 128, 64 x 128 and 64 x 64;
//   gemm_persist_kernel  256 x 256 tiles, one persistent work-group per CU whose two wave
//                      groups alternate between reading fragments and multiplying;
//   gemm_wave_kernel     32 x 32 tiles, one wave each, for products of few rows.
//
// LDS layout. A k-slab row of 64 bf16 is eight 16-byte chunks; the chunk index
// is XOR-swizzled with the row so the rows one MFMA operand read touches fall on
// different banks (see swz).
//
// Operand order. The MFMA is issued as (weight fragment, activation
// fragment), which computes the transposed tile: lane l then holds 4
// consecutive output columns of one output row, so the epilogue reads
// bias / residual and writes the output as 16-byte (fp32) or 8-byte (bf16)
// vectors.
//
// Work-group order. The hardware hands consecutive work-group ids round-robin
// to the 8 XCDs (each with its own L2). Ids are remapped so every XCD gets one
// contiguous range of tiles, grouped GROUP_M tile rows at a time: the tiles an
// XCD runs together share activation rows and weight columns in its L2.
#include <atomic>
#include <type_traits>

#include "gemm_common.h"
#include "kernels.h"

namespace elis {

// Compute units of the current device (the launch-time model below needs it). A device property,
// looked up once per device; the cache is safe to read and fill from several host threads.
int device_cus() {
    static std::atomic<int> cus[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int v = cus[dev].load(std::memory_order_relaxed);
    if (v == 0) {
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
        cus[dev].store(v, std::memory_order_relaxed);
    }
    return v;
}

namespace {

using namespace gemm;

constexpr int kBK = 64;

template <int EPI>
constexpr bool kF32Out = EPI == ELIS_EPI_BIAS_RES_F32 || EPI == kEpiResLn || EPI == kEpiResLnFfn2;
template <int EPI>
constexpr bool kResLn = EPI == kEpiResLn || EPI == kEpiResLnFfn2;
constexpr bool kResLnCode(int epi) { return epi == kEpiResLn || epi == kEpiResLnFfn2; }

// Residual of 4 consecutive columns n..n+3 of row m, given the 4 values h of res.x there.
template <int EPI>
__device__ __forceinline__ f32x4 residual4(const Residual& res, f32x4 h, int m, int n) {
    if constexpr (kResLn<EPI>) {
        const float2 st = res.stats[m];
        const f32x4 g = *reinterpret_cast<const f32x4*>(res.g + n);
        const f32x4 b = *reinterpret_cast<const f32x4*>(res.b + n);
#pragma unroll
        for (int c = 0; c < 4; ++c) h[c] = fmaf((h[c] - st.x) * st.y, g[c], b[c]);
    }
    return h;
}


// LDS chunk swizzle of the direct-to-LDS kernels: physical 16-byte chunk = logical chunk ^ swz(row).
// Measured free of bank conflicts on gfx950 for both 16-row and 32-row fragment reads (the
// plain row & 7 form conflicts 4-way on 32-row reads).
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

// GELU(x) = x * Phi(x) = max(x, 0) - a * Phi(-a) with a = |x| (as Phi(-a) = 1 - Phi(a)), so no
// branch or select on the sign. log2 Phi(-a) is smooth on [0, 5]: a degree-7 polynomial fitted
// there by weighted least squares (weight a * Phi(-a), the error it makes in GELU) gives Phi(-a)
// through one exp2. Past a = 5 the clamp leaves less than 5 * Phi(-5) < 1.5e-6 of error. Over
// all floats the result is within 1.5e-6 absolute and 3e-5 relative (where |GELU| > 1e-3) of
// x * Phi(x), far below the bf16 rounding of the output: one exp2, eight FMAs, a min and a max
// (a rational erf approximation needs a reciprocal as well, and measured 5% slower on FFN1).
__device__ __forceinline__ float gelu_erf(float x) {
    constexpr float c0 = -9.999995232e-01f, c1 = -1.151127219e+00f, c2 = -4.590456784e-01f,
                    c3 = -5.294791982e-02f, c4 = 7.674183231e-03f, c5 = -5.793952732e-04f,
                    c6 = -1.149886975e-05f, c7 = 4.121166967e-06f;
    const float a = fminf(fabsf(x), 5.0f);
    const float q = fmaf(fmaf(fmaf(fmaf(fmaf(fmaf(fmaf(c7, a, c6), a, c5), a, c4), a, c3), a, c2), a, c1), a, c0);
    return fmaf(-a, __builtin_amdgcn_exp2f(q), fmaxf(x, 0.f));
}


template <int BM, int BN, int WM, int WN, int MI, int EPI>
__global__ __launch_bounds__(WM* WN* kWave) void gemm_kernel(const uint16_t* __restrict__ A,
                                                             const uint16_t* __restrict__ B,
                                                             const float* __restrict__ bias,
                                                             Residual res, void* __restrict__ out,
                                                             int M, int N, int K) {
    typedef Mfma<MI> MF;
    typedef typename MF::acc_t acc_t;
    constexpr int NT = WM * WN * kWave;
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / MI, FN = TN / MI;
    constexpr int KSTEPS = kBK / MF::kDepth;
    constexpr int GROUPS = kWave / MI;  // lane groups along k (4 for MI 16, 2 for MI 32)
    constexpr int ACH = BM * 8 / NT, BCH = BN * 8 / NT;  // 16-byte chunks per thread per k-slab
    static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0, "tile must split evenly over the threads");
    static_assert(TM % MI == 0 && TN % MI == 0, "wave tile must be a multiple of the MFMA block");

    __shared__ __attribute__((aligned(16))) uint16_t sA[2][BM * kBK];
    __shared__ __attribute__((aligned(16))) uint16_t sB[2][BN * kBK];

    const int tiles_n = N / BN;
    const int tiles_m = (M + BM - 1) / BM;
    const int t = xcd_remap(blockIdx.x, tiles_m * tiles_n);
    const int m0 = (t / tiles_n) * BM, n0 = (t % tiles_n) * BN;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int wm = wid / WN, wn = wid % WN;

    // Per-thread global source pointers and LDS destinations of the k-slab chunks.
    const uint16_t* ga[ACH];
    const uint16_t* gb[BCH];
    int la[ACH], lb[BCH];
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
        const int id = tid + i * NT, row = id >> 3, c = id & 7;
        const int gr = (m0 + row < M) ? m0 + row : M - 1;  // ragged tail: re-read the last row
        ga[i] = A + static_cast<size_t>(gr) * K + c * 8;
        la[i] = row * kBK + ((c ^ (row & 7)) * 8);
    }
#pragma unroll
    for (int i = 0; i < BCH; ++i) {
        const int id = tid + i * NT, row = id >> 3, c = id & 7;
        gb[i] = B + static_cast<size_t>(n0 + row) * K + c * 8;
        lb[i] = row * kBK + ((c ^ (row & 7)) * 8);
    }

    u32x4 ra[ACH], rb[BCH];
    acc_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < MF::kRegs; ++r) acc[i][j][r] = 0.f;

    auto gload = [&](int k0) {
#pragma unroll
        for (int i = 0; i < ACH; ++i) ra[i] = *reinterpret_cast<const u32x4*>(ga[i] + k0);
#pragma unroll
        for (int i = 0; i < BCH; ++i) rb[i] = *reinterpret_cast<const u32x4*>(gb[i] + k0);
    };
    auto sstore = [&](int stg) {
#pragma unroll
        for (int i = 0; i < ACH; ++i) *reinterpret_cast<u32x4*>(&sA[stg][la[i]]) = ra[i];
#pragma unroll
        for (int i = 0; i < BCH; ++i) *reinterpret_cast<u32x4*>(&sB[stg][lb[i]]) = rb[i];
    };

    const int KT = K / kBK;
    gload(0);
    sstore(0);
    __syncthreads();

    const int rl = lane % MI, kg = lane / MI;
    for (int kt = 0; kt < KT; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < KT) gload((kt + 1) * kBK);
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            const int c = ks * GROUPS + kg;  // 16-byte chunk (8 k values) this lane feeds
            bf16x8 af[FM], bfr[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const int row = wm * TM + i * MI + rl;
                af[i] = *reinterpret_cast<const bf16x8*>(&sA[cur][row * kBK + ((c ^ (row & 7)) * 8)]);
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int row = wn * TN + j * MI + rl;
                bfr[j] = *reinterpret_cast<const bf16x8*>(&sB[cur][row * kBK + ((c ^ (row & 7)) * 8)]);
            }
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = MF::run(bfr[j], af[i], acc[i][j]);
        }
        if (kt + 1 < KT) sstore(cur ^ 1);
        __syncthreads();
    }

    // Epilogue. Lane holds, for output row m = rl of block i, groups of 4 consecutive
    // columns: MI 16: one group at 4*kg; MI 32: four groups at 8*q + 4*kg.
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int m = m0 + wm * TM + i * MI + rl;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
#pragma unroll
            for (int q = 0; q < MF::kRegs / 4; ++q) {
                const int n = n0 + wn * TN + j * MI + 8 * q + 4 * kg;
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * q + r];
                v += *reinterpret_cast<const f32x4*>(bias + n);
                const size_t o = static_cast<size_t>(m) * N + n;
                if constexpr (kF32Out<EPI>) {
                    v += residual4<EPI>(res, *reinterpret_cast<const f32x4*>(res.x + o), m, n);
                    *reinterpret_cast<f32x4*>(static_cast<float*>(out) + o) = v;
                } else {
                    if constexpr (EPI == ELIS_EPI_BIAS_GELU_BF16) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[c] = gelu_erf(v[c]);
                    }
                    u32x2 p;
                    p[0] = pack_bf16x2(v[0], v[1]);
                    p[1] = pack_bf16x2(v[2], v[3]);
                    *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(out) + o) = p;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Direct-to-LDS loading: k-slabs go from HBM straight into LDS (global_load_lds_dwordx4, no
// register staging), S stages deep, so S-1 slabs are in flight while one is multiplied.
// Each thread waits (vmcnt) only for its own loads of the slab about to be consumed; the
// barrier that follows makes every thread's part of that slab visible and also guarantees
// that every wave has finished reading the stage the next loads will overwrite.


// Tile index -> (tile row, tile col), grouping GM tile rows so that the tiles running
// together on one XCD share a small set of A rows and B columns (L2 reuse).
__device__ __forceinline__ void grouped_tile(int t, int tiles_m, int tiles_n, int gm, int& tm, int& tn) {
    const int per_group = gm * tiles_n;
    const int g = t / per_group, first = g * gm;
    const int rows = (tiles_m - first) < gm ? (tiles_m - first) : gm;
    const int r = t - g * per_group;
    tm = first + r % rows;
    tn = r / rows;
}

// ---------------------------------------------------------------------------------------------
// Scheduled variant: 4 waves (2 x 2), each owning a (BM/2) x (BN/2) block of MFMA tiles; two
// LDS stages filled by direct-to-LDS loads. A 64-deep k-slab is consumed in k-steps whose
// operand fragments are double-buffered in registers, so the LDS reads of the next k-step
// run under the MFMAs of the current one. The slab two steps ahead is requested right after
// the barrier that frees its stage (before the last k-step of the current slab), so a load
// has one full slab of MFMA work to arrive. sched_group_barrier spreads the LDS reads and the
// direct loads evenly between the MFMAs.
//
// LDS chunk swizzle: physical chunk = logical chunk ^ ((row >> 1) & 7). Measured free of bank
// conflicts on gfx950 for both the 16-row (16x16x32) and 32-row (32x32x16) fragment reads;
// the plain (row & 7) form conflicts 4-way on the 32-row reads.


// Bytes between the staged rows of a wave tile TN columns wide (16 bytes of padding).
template <int TN, int EPI>
constexpr int wave_tile_pitch() {
    return TN * (kF32Out<EPI> ? 4 : 2) + 16;
}

// Epilogue through LDS: each wave stages one 32-row block row of its output tile (bias,
// activation / residual applied), then writes it back as whole rows, 16 bytes per lane,
// so every store instruction covers full cache lines. bf16 outputs are stored
// non-temporally: they stream past the caches that hold the next tiles' operands (1% per
// predictor pass, up to 9% for a single GEMM). fp32 outputs (the pre-LayerNorm rows) are
// stored normally: the LayerNorm that reads them next then finds part of them in the
// memory-side cache (LayerNorm 21.4 -> 20.0 us at 24K tokens, 0.8% per pass).
// acc[i][j]: the 32 x 32 block at rows mw + 32 i, columns nw + 32 j, of a wave tile FM x FN blocks
// large; stg: 32 * wave_tile_pitch bytes of LDS of this wave's own.
template <int FM, int FN, int EPI>
__device__ __forceinline__ void store_wave_tile(const f32x16 (&acc)[FM][FN], char* stg, const float* __restrict__ bias,
                                                const Residual& res, void* __restrict__ out, int mw, int nw, int M,
                                                int N, int lane) {
    constexpr int TN = 32 * FN;
    const int rl = lane & 31, kg = lane >> 5;
    constexpr bool F32OUT = kF32Out<EPI>;
    constexpr int EB = F32OUT ? 4 : 2;          // output element bytes
    constexpr int ROWB = TN * EB;               // bytes of one wave-tile row
    constexpr int PITCH = wave_tile_pitch<TN, EPI>();
    constexpr int LPR = ROWB / 16;              // lanes per row on read-back
    constexpr int RPR = kWave / LPR;            // rows per read-back instruction
    // On read-back a lane always covers the same 16 output bytes of a row: columns nl ...
    const int ch = lane % LPR;
    const int nl = nw + ch * (16 / EB);
    f32x4 gl, bl;  // LayerNorm g, b of those columns (LayerNorm-form residual)
    if constexpr (kResLn<EPI>) {
        gl = *reinterpret_cast<const f32x4*>(res.g + nl);
        bl = *reinterpret_cast<const f32x4*>(res.b + nl);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int j = 0; j < FN; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = j * 32 + 8 * q + 4 * kg;
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * q + r];
                v += *reinterpret_cast<const f32x4*>(bias + nw + col);
                if constexpr (F32OUT) {
                    *reinterpret_cast<f32x4*>(stg + rl * PITCH + col * 4) = v;
                } else {
                    if constexpr (EPI == ELIS_EPI_BIAS_GELU_BF16) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[c] = gelu_erf(v[c]);
                    }
                    u32x2 pk;
                    pk[0] = pack_bf16x2(v[0], v[1]);
                    pk[1] = pack_bf16x2(v[2], v[3]);
                    *reinterpret_cast<u32x2*>(stg + rl * PITCH + col * 2) = pk;
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
        constexpr int NRR = 32 / RPR;  // read-back rows per lane per block row
        if constexpr (F32OUT) {
            // All residual vectors (and row statistics) of the block row are requested first.
            f32x4 hv[NRR];
            float2 sv[NRR];
#pragma unroll
            for (int rr = 0; rr < NRR; ++rr) {
                const int m = mw + i * 32 + rr * RPR + lane / LPR;
                const int mc = m < M ? m : M - 1;  // rows past the end load a valid row, store nothing
                hv[rr] = *reinterpret_cast<const f32x4*>(res.x + static_cast<size_t>(mc) * N + nl);
                if constexpr (kResLn<EPI>) sv[rr] = res.stats[mc];
            }
#pragma unroll
            for (int rr = 0; rr < NRR; ++rr) {
                const int row = rr * RPR + lane / LPR;
                const int m = mw + i * 32 + row;
                const u32x4 d = *reinterpret_cast<const u32x4*>(stg + row * PITCH + ch * 16);
                if (m < M) {
                    f32x4 h = hv[rr];
                    if constexpr (kResLn<EPI>) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) h[c] = fmaf((h[c] - sv[rr].x) * sv[rr].y, gl[c], bl[c]);
                    }
                    const f32x4 v = __builtin_bit_cast(f32x4, d) + h;
                    *reinterpret_cast<f32x4*>(static_cast<float*>(out) + static_cast<size_t>(m) * N + nl) = v;
                }
            }
        } else {
#pragma unroll
            for (int rr = 0; rr < NRR; ++rr) {
                const int row = rr * RPR + lane / LPR;
                const int m = mw + i * 32 + row;
                const u32x4 d = *reinterpret_cast<const u32x4*>(stg + row * PITCH + ch * 16);
                if (m < M) __builtin_nontemporal_store(d, reinterpret_cast<u32x4*>(static_cast<uint16_t*>(out) + static_cast<size_t>(m) * N + nl));
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
    }
}

template <int BM, int BN, int WM, int WN, int MI, int EPI, int OCC = 1, int S = 2>
__global__ __launch_bounds__(WM* WN* kWave) __attribute__((amdgpu_waves_per_eu(OCC * WM * WN / 4, OCC * WM * WN / 4))) void gemm_sched_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, const float* __restrict__ bias,
    Residual res, void* __restrict__ out, int M, int N, int K, int group_m) {
    typedef Mfma<MI> MF;
    typedef typename MF::acc_t acc_t;
    constexpr int BK = kBK;              // k-slab depth: 64 (eight 16-byte chunks per row)
    constexpr int NW = WM * WN;
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int FM = TM / MI, FN = TN / MI;
    constexpr int KS = BK / MF::kDepth;    // k-steps per slab
    constexpr int GROUPS = kWave / MI;     // lane groups along k
    constexpr int CPR = BK / 8;            // 16-byte chunks per slab row
    constexpr int RPI = kWave / CPR;       // slab rows covered by one wave-wide 16-byte load
    constexpr int LA = BM / RPI / NW, LB = BN / RPI / NW;  // direct loads per wave per stage
    static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "rows must split over the waves");
    constexpr int STAGE = (BM + BN) * BK;
    constexpr int NMF = FM * FN, NRD = FM + FN, NGL = LA + LB;
    static_assert(KS % 2 == 0, "fragment buffers alternate per k-step");
    static_assert(S >= 2 && S * NGL < 64, "pipeline depth");
    __shared__ __attribute__((aligned(1024))) uint16_t smem[S * STAGE];

    const int tiles_n = N / BN;
    const int tiles_m = (M + BM - 1) / BM;
    int tm, tn;
    grouped_tile(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, group_m, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WN, wn = wid % WN;
    auto sw = [](int row) { return (row >> 1) & (CPR - 1); };

    const uint16_t* ga[LA];
    const uint16_t* gb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int row = (wid * LA + i) * RPI + lane / CPR;
        const int c = (lane % CPR) ^ sw(row);
        const int gr = (m0 + row < M) ? m0 + row : M - 1;
        ga[i] = A + static_cast<size_t>(gr) * K + c * 8;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int row = (wid * LB + i) * RPI + lane / CPR;
        const int c = (lane % CPR) ^ sw(row);
        gb[i] = B + static_cast<size_t>(n0 + row) * K + c * 8;
    }
    auto issue = [&](int kt) {
        uint16_t* st = smem + (kt % S) * STAGE;
        const int k0 = kt * BK;
#pragma unroll
        for (int i = 0; i < LA; ++i) load_lds_16(ga[i] + k0, st + (wid * LA + i) * RPI * BK);
#pragma unroll
        for (int i = 0; i < LB; ++i) load_lds_16(gb[i] + k0, st + BM * BK + (wid * LB + i) * RPI * BK);
    };

    const int rl = lane % MI, kg = lane / MI;
    int offa[FM], offb[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) offa[i] = (wm * TM + i * MI + rl) * BK;
#pragma unroll
    for (int j = 0; j < FN; ++j) offb[j] = BM * BK + (wn * TN + j * MI + rl) * BK;
    const int rs = sw(rl);  // fragment rows start at multiples of 16, so sw(row) == sw(rl)

    bf16x8 fa[2][FM], fb[2][FN];
    auto load_frags = [&](int buf, int stage, int ks) {
        const uint16_t* st = smem + stage * STAGE;
        const int c = ((ks * GROUPS + kg) ^ rs) * 8;
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[buf][i] = *reinterpret_cast<const bf16x8*>(st + offa[i] + c);
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[buf][j] = *reinterpret_cast<const bf16x8*>(st + offb[j] + c);
    };

    acc_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < MF::kRegs; ++r) acc[i][j][r] = 0.f;

    auto mfma_all = [&](int buf) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = MF::run(fb[buf][j], fa[buf][i], acc[i][j]);
    };

    const int KT = K / BK;
    // Prologue: every stage gets a slab (slabs 0 .. S-1); wait for slab 0 only.
#pragma unroll
    for (int p = 0; p < S; ++p)
        if (p < KT) issue(p);
    if (KT >= S) wait_vmcnt<(S - 1) * NGL>();
    else wait_vmcnt<0>();
    block_sync_lds();
    load_frags(0, 0, 0);

    // One slab. WAIT: slabs still allowed in flight once slab kt+1 has landed; ISSUE: request
    // slab kt+S into the stage slab kt frees; NEXT: slab kt+1 exists (read its first
    // fragments). All compile-time, so the steady-state loop is straight-line code.
    auto slab = [&](int kt, auto wait_c, auto issue_c, auto next_c) {
        constexpr int WAIT = decltype(wait_c)::value;
        constexpr bool ISSUE = decltype(issue_c)::value, NEXT = decltype(next_c)::value;
        const int cur = kt % S;
#pragma unroll
        for (int ks = 0; ks < KS - 1; ++ks) {
            load_frags((ks + 1) & 1, cur, ks + 1);
            mfma_all(ks & 1);
            interleave_step<0, NMF, 0, NRD, 0>();
        }
        // Slab kt+1 has landed and every wave's reads of stage `cur` are complete.
        wait_vmcnt<WAIT * NGL>();
        wait_lgkm<0>();
        block_sync_lds();
        if constexpr (ISSUE) issue(kt + S);
        if constexpr (NEXT) load_frags(0, (kt + 1) % S, 0);
        mfma_all((KS - 1) & 1);
        interleave_step<0, NMF, ISSUE ? NGL : 0, NEXT ? NRD : 0, 1>();
    };
    typedef std::integral_constant<bool, true> T_;
    typedef std::integral_constant<bool, false> F_;
    typedef std::integral_constant<int, S - 2> WS_;
    typedef std::integral_constant<int, 0> W0_;
    int kt = 0;
    for (; kt + S < KT; ++kt) slab(kt, WS_(), T_(), T_());
    for (; kt + 1 < KT; ++kt) slab(kt, W0_(), F_(), T_());
    slab(kt, W0_(), F_(), F_());

    static_assert(NW * 32 * wave_tile_pitch<TN, EPI>() <= S * STAGE * 2, "staging must fit in the stage buffers");
    static_assert(MI == 32, "staged epilogue assumes 32-row MFMA blocks");
    block_sync_lds();  // every wave is done with the stage buffers
    store_wave_tile<FM, FN, EPI>(acc, reinterpret_cast<char*>(smem) + wid * 32 * wave_tile_pitch<TN, EPI>(), bias, res,
                                 out, m0 + wm * TM, n0 + wn * TN, M, N, lane);
}

// ---------------------------------------------------------------------------------------------
// Persistent 256 x 256 tiles, one work-group of 8 waves per CU; each wave owns a 128 x 64 block.
//
// k-loop. A 64-deep k-slab is four half-slabs in LDS (A rows / B rows that all waves read in the
// same phase) and four phases, one per (A half, B half) quadrant of the wave block: 8 MFMAs each.
// A phase is a memory part (LDS fragment reads, the direct loads of a half-slab two slabs ahead
// into the slot just read, the wait for the half-slab the next phase reads) and an MFMA part, with
// a barrier behind each. The two groups of four waves (one wave of each per SIMD) run one part
// apart, so on every SIMD one wave multiplies while the other reads.
//
// Tiles. A work-group walks its tiles as one stream of slabs: the loads of the next tile's first
// two slabs are in flight during a tile's last two slabs and land under its epilogue, whose
// stores in turn drain under the next tile's first slabs (their waits are left out: those slabs
// landed before the first store). Past the last tile the stream loads through empty buffer
// resources (no memory access), so every slab runs the same code and wait counts.
//
// The schedule (two wave groups a part apart, half-slab loads, raised priority around the products) is the published
// eight-wave ping-pong scheme for these matrix cores.
//
// What bounds it. On full rounds of a large square product the board's power limit: 8192 x 8192 x 8192 runs at
// 1,410 TFLOP/s with normal operands (clock 1.6 GHz) and 1,980 with zeros (2.27 GHz), 80% of the matrix cores'
// cycles both times. Where the last round is part-filled, that round: 92,000 x 1,024 x 4,096 is 5.63 rounds and
// hipBLASLt, which splits k over the last one, takes 0.86-0.89 times the time (two boxes). At k = 768 the
// epilogues take a quarter of the time (GELU's vector work and the stores; with both left out
// 93,014 x 3,072 x 768 takes 342 us). Against the one-tile-per-launch kernel with whole-slab waits that it
// replaces, in us (fp32 out with residual for n = 768):
//   93,014 x 3,072 x 768 + GELU 489 -> 446    93,014 x 2,304 x 768 315 -> 284
//   93,014 x 768 x 3,072        483 -> 453    21,760 x 3,072 x 768 + GELU 113 -> 104
//   102,548 x 1,024 x 4,096     863 -> 800    21,760 x 768 x 3,072 100 -> 97
// Two 256 x 128 work-groups per CU, which let one's epilogue run beside the other's k-loop, were
// 2-10% slower: half again the operand bytes costs power, and the overlap gains nothing under it.
template <int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_persist_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, const float* __restrict__ bias, Residual res,
    void* __restrict__ out, int M, int N, int K, int group_m) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass has no buffer-resource type
    constexpr int BM = 256, BN = 256, HALF = 128 * kBK, STAGE = 4 * HALF, STG = 2048;
    constexpr bool F32OUT = kF32Out<EPI>;
    constexpr int EB = F32OUT ? 4 : 2;
    __shared__ __attribute__((aligned(1024))) uint16_t smem[2 * STAGE + 8 * STG];
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wid >> 2, wn = wid & 3;
    const int tiles_n = N / BN, tiles_m = (M + BM - 1) / BM;
    // This work-group's tiles: every XCD owns one contiguous range, dealt out to its work-groups.
    const int tiles = tiles_m * tiles_n, xcd = blockIdx.x & 7, wgs = (static_cast<int>(gridDim.x) - xcd + 7) >> 3;
    const int per = tiles >> 3, rem = tiles & 7;
    const int t_end = xcd * per + (xcd < rem ? xcd : rem) + per + (xcd < rem ? 1 : 0);
    int tile = t_end - per - (xcd < rem ? 1 : 0) + static_cast<int>(blockIdx.x >> 3);
    auto origin = [&](int t, int& m0, int& n0) {
        int tm, tn;
        grouped_tile(t, tiles_m, tiles_n, group_m, tm, tn);
        m0 = __builtin_amdgcn_readfirstlane(tm * BM);
        n0 = __builtin_amdgcn_readfirstlane(tn * BN);
    };

    // Direct loads: wave w fills rows [16 w, 16 w + 16) of each half-slab with two wave-wide loads
    // of 8 rows. Row r of A half h is row 128 (r / 64) + 64 h + r % 64 of the tile, of B half h
    // column 64 (r / 32) + 32 h + r % 32, so a wave's quadrants make up a contiguous block. Rows
    // past the end of A are outside the resource and read as zeros.
    uint32_t oa[2][2], ob[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = wid * 16 + i * 8 + (lane >> 3), c = ((lane & 7) ^ swz(r)) * 8;
            oa[h][i] = static_cast<uint32_t>((((r >> 6) * 128 + h * 64 + (r & 63)) * K + c) * 2);
            ob[h][i] = static_cast<uint32_t>((((r >> 5) * 64 + h * 32 + (r & 31)) * K + c) * 2);
        }
    // The load stream: tile, k offset (bytes) and operands of the slab to request next.
    int lt = tile, lk = 0, lm = 0, ln = 0, la_bytes = 0, lb_bytes = 0;
    auto stream_tile = [&] {
        const bool more = lt < t_end;
        origin(more ? lt : t_end - 1, lm, ln);
        la_bytes = more ? (M - lm < BM ? M - lm : BM) * K * 2 : 0;
        lb_bytes = more ? BN * K * 2 : 0;
    };
    auto stream_next = [&] {
        lk += la_bytes ? kBK * 2 : 0;  // an empty resource is read at offset 0 only
        if (lk == K * 2) {
            lk = 0;
            lt += wgs;
            stream_tile();
        }
    };
    uint16_t* const my = smem + wid * 16 * kBK;
    auto load_a = [&](int st, int h) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(A) + static_cast<size_t>(lm) * K, 0, la_bytes, 0x00020000);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)(my + st + h * HALF + i * 8 * kBK), 16, oa[h][i], lk, 0, 0);
    };
    auto load_b = [&](int st, int h) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(B) + static_cast<size_t>(ln) * K, 0, lb_bytes, 0x00020000);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)(my + st + (2 + h) * HALF + i * 8 * kBK), 16, ob[h][i], lk, 0, 0);
    };

    const int rl = lane & 31, kg = lane >> 5;
    bf16x8 fa[2][4], fb[2][4];
    // This lane's 16 bytes of a 32-row block at each 16-deep k-step, in the stage of the current slab.
    int pa[4], pb[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const int l = rl * kBK + (((ks * 2 + kg) ^ swz(rl)) * 8);
        pa[ks] = wm * 64 * kBK + l;
        pb[ks] = 2 * HALF + wn * 32 * kBK + l;
    }
    auto read_a = [&](int h) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                fa[i][ks] = *reinterpret_cast<const bf16x8*>(smem + pa[ks] + h * HALF + i * 32 * kBK);
    };
    auto read_b = [&](int h) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) fb[h][ks] = *reinterpret_cast<const bf16x8*>(smem + pb[ks] + h * HALF);
    };
    f32x16 acc[4][2];
    auto multiply = [&](int ha, int hb) {
        __builtin_amdgcn_sched_barrier(0);
        wait_lgkm<0>();
        block_sync_lds();
        __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                acc[2 * ha + i][hb] = Mfma<32>::run(fb[hb][ks], fa[i][ks], acc[2 * ha + i][hb]);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        block_sync_lds();
        __builtin_amdgcn_sched_barrier(0);
    };

    // Bias (and LayerNorm g, b) of the wave's 64 columns, loaded into its staging area ahead of the epilogue.
    uint16_t* const stg = smem + 2 * STAGE + wid * STG;
    auto load_cols = [&](int n0) {
        auto one = [&](const float* p, int at) {
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p) + n0 + wn * 64, 0, 256, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)(stg + at * 128), 4, lane * 4, 0, 0, 0);
        };
        one(bias, 0);
        if constexpr (kResLn<EPI>) {
            one(res.g, 1);
            one(res.b, 2);
        }
    };

    int m0, n0, st = 0, landed = 0;  // landed: slabs from the current one on known to be in LDS
    origin(tile, m0, n0);
    load_cols(n0);
    stream_tile();
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        load_a(v * STAGE, 0);
        load_b(v * STAGE, 0);
        load_b(v * STAGE, 1);
        load_a(v * STAGE, 1);
        stream_next();
    }
    wait_vmcnt<12>();
    block_sync_lds();
    for (;;) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        if (wm == 1) block_sync_lds();
        for (int k = 0; k < K; k += kBK) {
            read_b(0);
            read_a(0);
            if (landed < 1) wait_vmcnt<10>();
            multiply(0, 0);
            read_b(1);
            load_a(st, 0);
            if (landed < 1) wait_vmcnt<10>();
            multiply(0, 1);
            read_a(1);
            load_b(st, 0);
            multiply(1, 1);
            load_b(st, 1);
            load_a(st, 1);
            if (landed < 2) wait_vmcnt<12>();
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) pa[ks] ^= STAGE, pb[ks] ^= STAGE;
            st ^= STAGE;
            landed = landed > 0 ? landed - 1 : 0;
            stream_next();
            multiply(1, 0);
        }
        if (wm == 0) block_sync_lds();

        // Epilogue: 32 rows x 128 bytes at a time through the wave's staging area, stored as whole lines.
        const int rows = M - m0 < BM ? M - m0 : BM;
        const uint32_t o_bytes = (static_cast<uint32_t>(rows) * N - n0) * EB;
        const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
            static_cast<char*>(out) + (static_cast<size_t>(m0) * N + n0) * EB, 0, o_bytes, 0x00020000);
        asm volatile("" ::: "memory");
        f32x4 bv[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) bv[j][q] = *reinterpret_cast<const f32x4*>(stg + (j * 32 + 8 * q + 4 * kg) * 2);
        const int ch = lane & 7, rr0 = lane >> 3;  // read-back: 16-byte chunk and row of 8
        // Output offset of the lane's first row (rows past the end of the matrix are outside the resource) and of 8
        // rows; formed anew for every tile, so that no row's offset is kept in a register through the k-loop.
        uint32_t ro0 = (static_cast<uint32_t>(wm * 128 + rr0) * N + wn * 64) * EB + ch * 16, row8 = 8u * N * EB;
        asm volatile("" : "+v"(ro0), "+s"(row8));
        if constexpr (F32OUT) {
            f32x4 gl[2], bl[2];
            if constexpr (kResLn<EPI>) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    gl[j] = *reinterpret_cast<const f32x4*>(stg + 128 + (j * 32 + ch * 4) * 2);
                    bl[j] = *reinterpret_cast<const f32x4*>(stg + 256 + (j * 32 + ch * 4) * 2);
                }
            }
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<float*>(res.x) + static_cast<size_t>(m0) * N + n0, 0, o_bytes, 0x00020000);
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<float2*>(res.stats) + (kResLn<EPI> ? m0 : 0), 0, kResLn<EPI> ? rows * 8 : 0, 0x00020000);
            f32x4 hv[2][4];
            f32x2 sv[2][4];
            // Residual rows (and statistics) of step b = 2 i + j, requested one step ahead.
            uint32_t fo = ro0, so = ro0;
            auto fetch = [&](int b) {
                const int i = b >> 1, j = b & 1;
                if (j == 1) fo -= 4 * row8;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr, fo += row8) {
                    hv[b & 1][rr] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, fo, j * 128, 0));
                    if constexpr (kResLn<EPI>)
                        if (j == 0)
                            sv[i & 1][rr] = __builtin_bit_cast(
                                f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, (wm * 128 + rr0 + i * 32 + rr * 8) * 8, 0, 0));
                }
            };
            fetch(0);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const int i = b >> 1, j = b & 1;
                if (b < 7) fetch(b + 1);
                asm volatile("" ::: "memory");
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * q + r];
                    *reinterpret_cast<f32x4*>(stg + rl * 64 + (((2 * q + kg) ^ swz(rl)) * 8)) = v + bv[j][q];
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int rr = 0; rr < 4; ++rr, so += row8) {
                    const int row = rr * 8 + rr0;
                    f32x4 h = hv[b & 1][rr];
                    if constexpr (kResLn<EPI>) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) h[c] = fmaf((h[c] - sv[i & 1][rr][0]) * sv[i & 1][rr][1], gl[j][c], bl[j][c]);
                    }
                    const f32x4 v = *reinterpret_cast<const f32x4*>(stg + row * 64 + ((ch ^ swz(row)) * 8)) + h;
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ro, so, j * 128, 0);
                }
                if (j == 0) so -= 4 * row8;
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                asm volatile("" ::: "memory");
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        f32x4 v;
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * q + r];
                        v += bv[j][q];
                        if constexpr (EPI == ELIS_EPI_BIAS_GELU_BF16) {
#pragma unroll
                            for (int c = 0; c < 4; ++c) v[c] = gelu_erf(v[c]);
                        }
                        u32x2 pk;
                        pk[0] = pack_bf16x2(v[0], v[1]);
                        pk[1] = pack_bf16x2(v[2], v[3]);
                        *reinterpret_cast<u32x2*>(stg + rl * 64 + (((4 * j + q) ^ swz(rl)) * 8 + 4 * kg)) = pk;
                    }
                if (i == 0) wait_vmcnt<0>();  // the next tile's first two slabs are in LDS before the first store
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int rr = 0; rr < 4; ++rr, ro0 += row8) {
                    const int row = rr * 8 + rr0;
                    const u32x4 d = *reinterpret_cast<const u32x4*>(stg + row * 64 + ((ch ^ swz(row)) * 8));
                    __builtin_amdgcn_raw_buffer_store_b128(d, ro, ro0, 0, 2);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        tile += wgs;
        if (tile >= t_end) break;
        origin(tile, m0, n0);
        load_cols(n0);
        landed = 2;
    }
    wait_vmcnt<0>();  // the empty loads of the stream's end write LDS: none may outlive the work-group
#endif
}

// ---------------------------------------------------------------------------------------------
// 32 x 32 tiles, one wave per work-group: products of few rows, where a wider tile would leave most
// CUs without one. The wave keeps six or seven 64-deep k-slabs (8 KB each) in flight into a ring of eight in
// LDS; nobody else reads them, so there is no barrier. Fragments of the next slab are read while the
// current one is multiplied, and the residual, bias and LayerNorm columns are requested up front.
// Bound by the CU's load path (8 KB per slab at about 37 bytes a cycle, 0.105 us; it takes 0.126):
// the 64 x 64 tile moves 16 KB per slab on a quarter of the CUs. That tile (four-stage, 0.22 us per
// slab) took 13.7 us at 200 x 768 x 3,072, this one 8.9; 64 rows 13.2 -> 8.6, 520 rows 14.4 -> 11.6;
// 200 x 768 x 768 5.4 -> 4.2. Past 512 tiles (two per CU) the wider tiles win: 193 x 3,072 x 768, 672
// tiles, 5.5 against 7.8.
template <int EPI>
__global__ __launch_bounds__(64) void gemm_wave_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                       const float* __restrict__ bias, Residual res,
                                                       void* __restrict__ out, int M, int N, int K) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass has no buffer-resource type
    constexpr int RING = 8, SLAB = 64 * kBK;
    constexpr bool F32OUT = kF32Out<EPI>;
    __shared__ __attribute__((aligned(1024))) uint16_t smem[RING * SLAB];
    // An XCD's work-groups share few rows of the larger operand and read the smaller one whole (1,978 x 256 x 4,096, where
    // that is the weights: 20.9 us with few weight rows shared instead, now 12.7; 64 x 64 tiles 17.1).
    const int tiles_m = (M + 31) / 32, tiles_n = N / 32, t = xcd_remap(blockIdx.x, tiles_m * tiles_n);
    const bool tall = M > N;
    const int inner = tall ? tiles_n : tiles_m, slow = t / inner, fast = t - slow * inner;
    const int m0 = (tall ? slow : fast) * 32, n0 = (tall ? fast : slow) * 32;
    const int lane = threadIdx.x, rl = lane & 31, kg = lane >> 5;
    const int rows = M - m0 < 32 ? M - m0 : 32, KT = K / kBK;

    const int m = m0 + (rl < rows ? rl : rows - 1);  // rows past the end compute on the last row, stored nowhere
    f32x4 bv[4], hv[4], gv[4], cv[4];
    float2 sv;
    // Buffer loads, which the compiler leaves ahead of the slabs' loads instead of moving them to their use.
    auto early = [&](const float* p, size_t base, uint32_t off) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p) + base, 0, 0xffffffffu, 0x00020000);
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off * 4u, 0, 0));
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t n = 8 * q + 4 * kg;
        bv[q] = early(bias, n0, n);
        if constexpr (F32OUT) hv[q] = early(res.x, static_cast<size_t>(m0) * N + n0, (m - m0) * N + n);
        if constexpr (kResLn<EPI>) {
            gv[q] = early(res.g, n0, n);
            cv[q] = early(res.b, n0, n);
        }
    }
    if constexpr (kResLn<EPI>) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(res.stats) + m0, 0, rows * 8, 0x00020000);
        sv = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, (m - m0) * 8, 0, 0));
    }

    uint32_t oa[4], ob[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = i * 8 + (lane >> 3), c = ((lane & 7) ^ swz(r)) * 8;
        oa[i] = static_cast<uint32_t>(((r < rows ? r : rows - 1) * K + c) * 2);
        ob[i] = static_cast<uint32_t>((r * K + c) * 2);
    }
    // Past the last slab the resource is empty (no memory access), so that every step runs the same code.
    auto load = [&](int kt) {
        const bool more = kt < KT;
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(A) + static_cast<size_t>(m0) * K, 0, more ? rows * K * 2 : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(B) + static_cast<size_t>(n0) * K, 0, more ? 32 * K * 2 : 0, 0x00020000);
        const int at = more ? kt * kBK * 2 : 0;
        uint16_t* d = smem + (kt % RING) * SLAB;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)(d + i * 8 * kBK), 16, oa[i], at, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void_t*)(d + (4 + i) * 8 * kBK), 16, ob[i], at, 0, 0);
    };
    int lo[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) lo[ks] = rl * kBK + (((ks * 2 + kg) ^ swz(rl)) * 8);
    bf16x8 fa[2][4], fb[2][4];
    auto read = [&](int buf, int kt) {
        const uint16_t* p = smem + (kt % RING) * SLAB;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            fa[buf][ks] = *reinterpret_cast<const bf16x8*>(p + lo[ks]);
            fb[buf][ks] = *reinterpret_cast<const bf16x8*>(p + 32 * kBK + lo[ks]);
        }
    };
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int p = 0; p < RING - 1; ++p) load(p);
    wait_vmcnt<(RING - 2) * 8>();
    read(0, 0);
    // Slab kt: wait for slab kt + 1 and read its fragments, request slab kt + 7 (into the slot of slab kt - 1, whose
    // fragments have been multiplied, hence read), multiply. The barriers keep the compiler to this order: left alone
    // it read every second slab's fragments only in front of their products, and nothing but its own schedule kept
    // a read ahead of the load over its slot. (Requesting before reading exposes the reads: 8.9 -> 9.9 us at
    // 193 x 768 x 3,072.)
    auto step = [&](int buf, int kt) {
        wait_vmcnt<(RING - 3) * 8>();
        read(buf ^ 1, kt + 1);
        __builtin_amdgcn_sched_barrier(0);
        load(kt + RING - 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc = Mfma<32>::run(fb[buf][ks], fa[buf][ks], acc);
        __builtin_amdgcn_sched_barrier(0);
    };
    int kt = 0;
    for (; kt + 1 < KT; kt += 2) {
        step(0, kt);
        step(1, kt + 1);
    }
    if (kt < KT) step(0, kt);
    wait_vmcnt<0>();  // the empty loads write LDS: none may outlive the work-group

    if (rl >= rows) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const size_t o = static_cast<size_t>(m) * N + n0 + 8 * q + 4 * kg;
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = acc[4 * q + r];
        v += bv[q];
        if constexpr (F32OUT) {
            f32x4 h = hv[q];
            if constexpr (kResLn<EPI>) {
#pragma unroll
                for (int c = 0; c < 4; ++c) h[c] = fmaf((h[c] - sv.x) * sv.y, gv[q][c], cv[q][c]);
            }
            *reinterpret_cast<f32x4*>(static_cast<float*>(out) + o) = v + h;
        } else {
            if constexpr (EPI == ELIS_EPI_BIAS_GELU_BF16) {
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = gelu_erf(v[c]);
            }
            u32x2 pk;
            pk[0] = pack_bf16x2(v[0], v[1]);
            pk[1] = pack_bf16x2(v[2], v[3]);
            *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(out) + o) = pk;
        }
    }
#endif
}

hipError_t launch_persist(const uint16_t* x, const uint16_t* w, const float* bias, Residual res, int m, int n, int k,
                           int epi, void* out, hipStream_t st, int group_m) {
    const int tiles = ((m + 255) / 256) * (n / 256), cus = device_cus();
    const dim3 grid(tiles < cus ? tiles : cus), block(512);
    auto go = [&](auto kernel) { return launch_kernel(kernel, grid, block, 0, st, x, w, bias, res, out, m, n, k, group_m); };
    switch (epi) {
        case ELIS_EPI_BIAS_BF16: return go(gemm_persist_kernel<ELIS_EPI_BIAS_BF16>);
        case ELIS_EPI_BIAS_GELU_BF16: return go(gemm_persist_kernel<ELIS_EPI_BIAS_GELU_BF16>);
        case ELIS_EPI_BIAS_RES_F32: return go(gemm_persist_kernel<ELIS_EPI_BIAS_RES_F32>);
        case kEpiResLn: return go(gemm_persist_kernel<kEpiResLn>);
        case kEpiResLnFfn2: return go(gemm_persist_kernel<kEpiResLnFfn2>);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_wave(const uint16_t* x, const uint16_t* w, const float* bias, Residual res, int m, int n, int k,
                       int epi, void* out, hipStream_t st) {
    const dim3 grid(((m + 31) / 32) * (n / 32)), block(kWave);
    auto go = [&](auto kernel) { return launch_kernel(kernel, grid, block, 0, st, x, w, bias, res, out, m, n, k); };
    switch (epi) {
        case ELIS_EPI_BIAS_BF16: return go(gemm_wave_kernel<ELIS_EPI_BIAS_BF16>);
        case ELIS_EPI_BIAS_GELU_BF16: return go(gemm_wave_kernel<ELIS_EPI_BIAS_GELU_BF16>);
        case ELIS_EPI_BIAS_RES_F32: return go(gemm_wave_kernel<ELIS_EPI_BIAS_RES_F32>);
        case kEpiResLn: return go(gemm_wave_kernel<kEpiResLn>);
        case kEpiResLnFfn2: return go(gemm_wave_kernel<kEpiResLnFfn2>);
        default: return hipErrorInvalidValue;
    }
}

template <int BM, int BN, int WM, int WN, int MI, int OCC = 1, int S = 2>
hipError_t launch_sched(const uint16_t* x, const uint16_t* w, const float* bias, Residual res, int m, int n,
                        int k, int epi, void* out, hipStream_t st, int group_m) {
    const dim3 grid(((m + BM - 1) / BM) * (n / BN)), block(WM * WN * kWave);
    auto go = [&](auto kernel) { return launch_kernel(kernel, grid, block, 0, st, x, w, bias, res, out, m, n, k, group_m); };
    switch (epi) {
        case ELIS_EPI_BIAS_BF16: return go(gemm_sched_kernel<BM, BN, WM, WN, MI, ELIS_EPI_BIAS_BF16, OCC, S>);
        case ELIS_EPI_BIAS_GELU_BF16: return go(gemm_sched_kernel<BM, BN, WM, WN, MI, ELIS_EPI_BIAS_GELU_BF16, OCC, S>);
        case ELIS_EPI_BIAS_RES_F32: return go(gemm_sched_kernel<BM, BN, WM, WN, MI, ELIS_EPI_BIAS_RES_F32, OCC, S>);
        case kEpiResLn: return go(gemm_sched_kernel<BM, BN, WM, WN, MI, kEpiResLn, OCC, S>);
        case kEpiResLnFfn2: return go(gemm_sched_kernel<BM, BN, WM, WN, MI, kEpiResLnFfn2, OCC, S>);
        default: return hipErrorInvalidValue;
    }
}

template <int BM, int BN, int WM, int WN, int MI>
hipError_t launch_tile(const uint16_t* x, const uint16_t* w, const float* bias, Residual res, int m, int n,
                       int k, int epi, void* out, hipStream_t st) {
    const dim3 grid(((m + BM - 1) / BM) * (n / BN)), block(WM * WN * kWave);
    switch (epi) {
        case ELIS_EPI_BIAS_BF16:
            ELIS_TRY(launch_kernel((gemm_kernel<BM, BN, WM, WN, MI, ELIS_EPI_BIAS_BF16>), grid, block, 0, st, x, w,
                               bias, res, out, m, n, k));
            break;
        case ELIS_EPI_BIAS_GELU_BF16:
            ELIS_TRY(launch_kernel((gemm_kernel<BM, BN, WM, WN, MI, ELIS_EPI_BIAS_GELU_BF16>), grid, block, 0, st, x,
                               w, bias, res, out, m, n, k));
            break;
        case ELIS_EPI_BIAS_RES_F32:
            ELIS_TRY(launch_kernel((gemm_kernel<BM, BN, WM, WN, MI, ELIS_EPI_BIAS_RES_F32>), grid, block, 0, st, x, w,
                               bias, res, out, m, n, k));
            break;
        case kEpiResLn:
            ELIS_TRY(launch_kernel((gemm_kernel<BM, BN, WM, WN, MI, kEpiResLn>), grid, block, 0, st, x, w, bias,
                               res, out, m, n, k));
            break;
        case kEpiResLnFfn2:
            ELIS_TRY(launch_kernel((gemm_kernel<BM, BN, WM, WN, MI, kEpiResLnFfn2>), grid, block, 0, st, x, w, bias,
                               res, out, m, n, k));
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipSuccess;
}

}  // namespace

// The persistent kernel needs two k-slabs, and both it and the 32 x 32 tiles 32-bit offsets inside a tile's operands
// and output. The 32 x 32 tiles leave an n that is an odd multiple of 64 to the kernel that accumulates it in
// 16 x 16 x 32 blocks.
bool gemm_persist_fits(int n, int k) { return n % 256 == 0 && k >= 2 * kBK && k <= (1 << 21) && n <= (1 << 20); }
bool gemm_wave_fits(int n, int k) { return n % 128 == 0 && k <= (1 << 21) && n <= (1 << 20); }

// Tile configurations (ids are internal; benchmarks sweep them).
hipError_t launch_gemm_config(int cfg, int group_m, const uint16_t* x, const uint16_t* w, const float* bias,
                              Residual res, int m, int n, int k, int epi, void* out, hipStream_t st) {
    switch (cfg) {
        case 1: return launch_tile<128, 64, 2, 2, 16>(x, w, bias, res, m, n, k, epi, out, st);
        case kPersistCfg:  // other depths: the same bits in 128 x 128 tiles
            if (gemm_persist_fits(n, k)) return launch_persist(x, w, bias, res, m, n, k, epi, out, st, group_m);
            return launch_sched<128, 128, 2, 2, 32, 2>(x, w, bias, res, m, n, k, epi, out, st, group_m);
        case 32: return launch_sched<128, 128, 2, 2, 32, 2>(x, w, bias, res, m, n, k, epi, out, st, group_m);
        case 33: return launch_sched<64, 128, 2, 2, 32, 2>(x, w, bias, res, m, n, k, epi, out, st, group_m);
        case 34: return launch_sched<64, 128, 2, 2, 32, 1, 4>(x, w, bias, res, m, n, k, epi, out, st, group_m);
        case 35: return launch_sched<64, 64, 2, 2, 32, 4, 2>(x, w, bias, res, m, n, k, epi, out, st, group_m);
        case 36: return launch_sched<64, 64, 2, 2, 32, 2, 4>(x, w, bias, res, m, n, k, epi, out, st, group_m);
        case kWaveCfg: return gemm_wave_fits(n, k) ? launch_wave(x, w, bias, res, m, n, k, epi, out, st) : hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

namespace {
struct TileShape {
    int cfg, bm, bn, wgs_per_cu;
};
constexpr TileShape kTileShapes[] = {{1, 128, 64, 2},  {21, 256, 256, 1}, {32, 128, 128, 2}, {33, 64, 128, 2},
                                     {34, 64, 128, 1}, {35, 64, 64, 4},   {36, 64, 64, 2},   {40, 32, 32, 2}};
}  // namespace

void gemm_config_tile(int cfg, int* bm, int* bn, int* wgs_per_cu) {
    *bm = *bn = *wgs_per_cu = 0;
    for (const TileShape& t : kTileShapes)
        if (t.cfg == cfg) *bm = t.bm, *bn = t.bn, *wgs_per_cu = t.wgs_per_cu;
}

int gemm_config_of_tile(int bm, int bn, int wgs_per_cu) {
    for (const TileShape& t : kTileShapes)
        if (t.bm == bm && t.bn == bn && t.wgs_per_cu == wgs_per_cu) return t.cfg;
    return -1;
}

namespace {

// Launch-time model of the tile configurations, in microseconds on MI355X (256 CUs), fitted to
// medians of repeated timings over K = 768, 1024, 3072, 4096, the three epilogue kinds and ten
// fills from a lone tile to four rounds, two sets of operands in turn (so that a product does not
// find its weights and activations in the L2, as inside the encoder; a fit with everything L2-hot
// had priced a lone two-stage 64 x 64 tile at half of what it takes there), then moved to where the choice among
// plans loses least, over 11,500 random products (k = 512 .. 4,096, up to 100,000 rows) with every plan timed.
// Depths below 512 have a fit of their own (kShallowModel): few slabs hide little of the prologue, and large
// outputs are bound by memory. Over 12,000 other random products the chosen plan takes 0.3-0.5% more than the best
// one in the mean (with one fit for all depths 0.9%, up to 1.4 times the best at k = 128), and 1.1% of them
// are more than 3% slower than the plan the L2-hot fit chooses (4.8%); most of those are GELU
// products in 64 x 64 tiles, among them n = 3,072, k = 768 at 330 to 470 rows (6.6 us, 7.1 as chosen).
// A launch whose tiles fill R rounds of work-group slots (work-groups per CU x CUs), the last
// one a fraction f full, takes part(f) for R = 1, else t1 + (R - 2) * beta + part(f)
// - (t1 - beta) * f; part is piecewise linear through lat (a lone tile, f -> 0), th (f = 1/2)
// and t1 (f = 1), beta is the cost of one more full round. Each quantity is a + s * K / 64: the
// slope per 64-deep k-slab is shared by the epilogue kinds, the intercept is per kind (bf16,
// bf16 + GELU, fp32 + residual). Full rounds of 256 x 256 tiles cost more per slab than a lone
// tile (1.4-1.8 against 1.0 us): with every matrix core busy the clock falls to about 1.7 GHz.
// The 64-row tiles are priced only up to the four rounds they were timed on and are not offered
// past that.
struct TileModel {
    int cfg, bm, bn, occ, max_rounds;  // max_rounds: 0 = any; else the fitted range
    float s[4];     // lat, th, t1, beta: slope per k-slab
    float a[3][4];  // intercept per epilogue kind
};
struct LaunchModel {
    TileModel tiles[6];
    TileModel wave;  // the one-wave 32 x 32 tile: up to one round, and never beside another launch (beta unused)
};
constexpr LaunchModel kDeepModel = {{
    {21, 256, 256, 1, 0, {1.009f, 1.150f, 1.420f, 1.765f},
     {{5.05f, 6.28f, 8.18f, 1.99f}, {9.49f, 9.77f, 9.86f, 5.44f}, {8.25f, 14.11f, 26.44f, 15.63f}}},
    {32, 128, 128, 2, 0, {0.618f, 0.648f, 1.070f, 1.180f},
     {{2.60f, 3.33f, 3.75f, 0.91f}, {4.27f, 4.83f, 4.73f, 2.55f}, {4.22f, 7.72f, 11.39f, 9.80f}}},
    {33, 64, 128, 2, 4, {0.354f, 0.576f, 0.605f, 0.770f},
     {{2.62f, 2.92f, 3.73f, -0.52f}, {4.32f, 3.46f, 4.22f, 0.59f}, {4.06f, 4.11f, 6.29f, 3.84f}}},
    {34, 64, 128, 1, 4, {0.321f, 0.304f, 0.367f, 0.372f},
     {{2.86f, 3.16f, 3.34f, 1.58f}, {3.87f, 3.49f, 3.78f, 2.14f}, {3.56f, 4.00f, 5.50f, 3.58f}}},
    {35, 64, 64, 4, 4, {0.342f, 0.456f, 0.771f, 0.869f},
     {{1.25f, 2.60f, 3.26f, -1.34f}, {2.71f, 3.17f, 3.50f, -0.58f}, {2.95f, 4.62f, 4.95f, 3.62f}}},
    {36, 64, 64, 2, 4, {0.182f, 0.237f, 0.377f, 0.380f},
     {{2.83f, 3.28f, 3.78f, 1.29f}, {3.46f, 3.07f, 3.61f, 1.50f}, {3.35f, 3.86f, 4.78f, 2.16f}}},
}, {kWaveCfg, 32, 32, 2, 1, {0.125f, 0.126f, 0.176f, 0.000f},
    {{2.62f, 2.83f, 2.66f, 0.00f}, {2.88f, 3.09f, 2.94f, 0.00f}, {2.68f, 2.82f, 3.04f, 0.00f}}}};
constexpr LaunchModel kShallowModel = {{
    {21, 256, 256, 1, 0, {0.867f, 1.035f, 1.632f, 1.530f},
     {{4.31f, 5.11f, 7.79f, 4.23f}, {8.83f, 10.05f, 8.07f, 6.63f}, {7.11f, 15.64f, 23.83f, 24.90f}}},
    {32, 128, 128, 2, 0, {0.418f, 0.487f, 1.173f, 0.892f},
     {{2.66f, 4.06f, 3.10f, 2.24f}, {2.99f, 5.10f, 4.91f, 3.89f}, {2.17f, 9.56f, 12.35f, 8.45f}}},
    {33, 64, 128, 2, 4, {0.336f, 0.438f, 0.597f, 0.678f},
     {{2.37f, 3.17f, 2.87f, 1.00f}, {2.99f, 4.23f, 4.19f, 1.86f}, {2.87f, 5.24f, 8.65f, 4.41f}}},
    {34, 64, 128, 1, 4, {0.341f, 0.395f, 0.479f, 0.359f},
     {{2.42f, 3.35f, 2.84f, 1.29f}, {3.07f, 3.66f, 3.49f, 1.91f}, {2.89f, 3.86f, 4.36f, 4.09f}}},
    {35, 64, 64, 4, 4, {0.197f, 0.364f, 0.698f, 0.667f},
     {{2.27f, 2.98f, 2.84f, 0.75f}, {2.54f, 3.11f, 3.63f, 1.27f}, {2.37f, 4.33f, 6.37f, 4.67f}}},
    {36, 64, 64, 2, 4, {0.238f, 0.244f, 0.519f, 0.304f},
     {{2.23f, 3.14f, 2.88f, 0.72f}, {2.63f, 3.01f, 3.17f, 1.11f}, {2.36f, 3.45f, 4.21f, 2.96f}}},
}, {kWaveCfg, 32, 32, 2, 1, {0.134f, 0.131f, 0.117f, 0.000f},
    {{1.73f, 2.65f, 3.18f, 0.00f}, {2.71f, 2.87f, 3.29f, 0.00f}, {2.38f, 2.70f, 3.32f, 0.00f}}}};
constexpr float kSecondLaunchUs = 1.0f;  // dispatch cost of the remainder launch

int epilogue_kind(int epi) {
    if (epi == ELIS_EPI_BIAS_RES_F32 || kResLnCode(epi)) return 2;
    return epi == ELIS_EPI_BIAS_GELU_BF16 ? 1 : 0;
}

double model_us(const TileModel& t, int kind, long long m, int n, int k, long long cus) {
    if (m <= 0) return 0.0;
    const long long tiles = (m + t.bm - 1) / t.bm * (n / t.bn), slots = t.occ * cus;
    const long long rounds = (tiles + slots - 1) / slots;
    // The small tiles were timed over one to four rounds only; past that their cost is not
    // extrapolated (their many-round behaviour differs) and they are not offered.
    if (t.max_rounds && rounds > t.max_rounds) return 1e30;
    const double f = static_cast<double>(tiles - (rounds - 1) * slots) / static_cast<double>(slots);
    double v[4];
    for (int q = 0; q < 4; ++q) v[q] = t.a[kind][q] + t.s[q] * (k / 64.0);
    const double part = f <= 0.5 ? v[0] + (v[1] - v[0]) * (f / 0.5) : v[1] + (v[2] - v[1]) * ((f - 0.5) / 0.5);
    if (rounds == 1) return part;
    // First round t1, full rounds after it beta each (they overlap the one before), and a last
    // round f full that overlaps the one before it by (t1 - beta) * f.
    return v[2] + static_cast<double>(rounds - 2) * v[3] + part - (v[2] - v[3]) * f;
}

}  // namespace

// The plan of one product: a single launch of one configuration, or (main, m1, rest): rows
// [0, m1) with `main` in whole rounds of tiles and rows [m1, m) with the smaller-tile `rest`,
// whichever the launch-time model above prices lowest. A 256 x 256 round costs about as much
// as two rounds of the 128 x 128 pairs, but a round that is only partly filled costs nearly a
// full one, so the rows past the last full round of large tiles go to a configuration whose
// tiles are small enough to finish them in one short round.
GemmPlan plan_gemm(int m, int n, int k, int epi) {
    if (n % 128 != 0) return {1, m, 0};
    const int kind = epilogue_kind(epi);
    const long long cus = device_cus();
    const LaunchModel& model = k < 512 ? kShallowModel : kDeepModel;
    GemmPlan best{0, m, 0};
    double best_us = -1.0;
    auto fits = [&](const TileModel& t) { return n % t.bn == 0 && (t.cfg != kPersistCfg || gemm_persist_fits(n, k)); };
    for (const TileModel& main : model.tiles) {
        if (!fits(main)) continue;
        const double t = model_us(main, kind, m, n, k, cus);
        if (best_us < 0.0 || t < best_us) {
            best_us = t;
            best = {main.cfg, m, 0};
        }
        // Whole rows of tiles that fill whole rounds.
        const long long per_row = n / main.bn, slots = main.occ * cus;
        const long long tiles = (static_cast<long long>(m) + main.bm - 1) / main.bm * per_row;
        const long long m1 = (tiles / slots) * slots / per_row * main.bm;
        if (m1 <= 0 || m1 >= m) continue;
        const double head = model_us(main, kind, m1, n, k, cus) + kSecondLaunchUs;
        for (const TileModel& rest : model.tiles) {
            if (rest.cfg == main.cfg || !fits(rest)) continue;
            const double tr = head + model_us(rest, kind, m - m1, n, k, cus);
            if (tr < best_us) {
                best_us = tr;
                best = {main.cfg, static_cast<int>(m1), rest.cfg};
            }
        }
    }
    // 32 x 32 tiles where they fill at most one round (512 tiles) and the model prices them lower: up to about 540 rows
    // at n = 768 or 1,024, 200 at n = 2,304 and 150 at n = 3,072 or 4,096.
    if (gemm_wave_fits(n, k) && model_us(model.wave, kind, m, n, k, cus) < best_us) best = {kWaveCfg, m, 0};
    return best;
}

hipError_t launch_gemm_plan(const GemmPlan& p, const uint16_t* x, const uint16_t* w, const float* bias,
                            Residual res, int m, int n, int k, int epi, void* out, hipStream_t st) {
    constexpr int kGroupM = 8;
    ELIS_TRY(launch_gemm_config(p.main, p.main == 1 ? 1 : kGroupM, x, w, bias, res, p.m1, n, k, epi, out, st));
    if (p.m1 >= m) return hipSuccess;
    const size_t r0 = static_cast<size_t>(p.m1);
    const bool f32out = epi == ELIS_EPI_BIAS_RES_F32 || kResLnCode(epi);
    Residual rr = res;
    if (rr.x) rr.x += r0 * n;
    if (rr.stats) rr.stats += r0;
    void* o2 = f32out ? static_cast<void*>(static_cast<float*>(out) + r0 * n)
                      : static_cast<void*>(static_cast<uint16_t*>(out) + r0 * n);
    return launch_gemm_config(p.rest, kGroupM, x + r0 * k, w, bias, rr, m - p.m1, n, k, epi, o2, st);
}

// Every 32 x 32 x 16 configuration accumulates each output element in the same order with the
// same MFMA instruction and applies the same epilogue arithmetic, so neither the plan nor the
// split ever changes a result.
hipError_t launch_gemm(const uint16_t* x, const uint16_t* w, const float* bias, Residual res, int m, int n,
                       int k, int epi, void* out, hipStream_t st) {
    if (m < 1 || n % 64 != 0 || k % kBK != 0 || n < 64 || k < kBK) return hipErrorInvalidValue;
    return launch_gemm_plan(plan_gemm(m, n, k, epi), x, w, bias, res, m, n, k, epi, out, st);
}

}  // namespace elis
