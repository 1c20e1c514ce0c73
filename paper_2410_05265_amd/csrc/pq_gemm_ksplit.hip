// Products whose output has too few large tiles for 256 CUs (up to a few hundred tokens): K is split
// over the wavefronts of a workgroup.
//
// The persistent and the tiled kernels give every CU one large tile and one wavefront per SIMD; with few tokens
// most CUs have no tile, and those that do walk K alone, waiting for one load after the other.  Here a workgroup
// of 4 or 8 wavefronts owns one small tile of the output (32 to 128 tokens x 32 to 128 channels, chosen so that
// the tiles go round the CUs once), every wavefront multiplies its own run of K for the whole tile, and the
// partial tiles are added through LDS at the end: no planes in memory, no second launch, no barrier in the main
// loop.  What bounds the prepacked form is the rate at which a CU takes its operands in, (tokens + channels) x K codes per tile
// at 85 KB/us; in the packed form the transfers through LDS, the expansion of the nibbles and the matrix instructions of a
// SIMD follow one another (200 x 6144 x 4096: 328 KB of operands per CU in about 9 us).  The rule that picks the tile
// minimises the estimated sum over the rounds.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "pq_internal.h"

namespace pq {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) uint8_t* lds_u8;

constexpr int kMaxLds = 160 * 1024;

// What the epilogue multiplies by and adds: one static step or the tokens' own (srow), and the zero-point's
// per-channel integers (zcorr), as in the tiled kernel.
struct Epilogue {
    const float* sw;
    float sx;
    const float* srow;
    const int32_t* zcorr;
    __half* out;
    int32_t* acc_out;
};

// A second weight matrix on the same tokens, in the same launch: its tiles follow the `first` tiles of the first one.
struct Second {
    const uint8_t* w;
    const float* sw;
    __half* out;
    int N, first;
};

// This workgroup's tile within its matrix (row tiles fastest: the tiles that share weights meet in one L2); w, ep and N become those of the second matrix where the tile is in that one.
template <bool TWO>
__device__ __forceinline__ int own_tile(const Second& two, const uint8_t* __restrict__& w, Epilogue& ep, int& N)
{
    int b = (int)blockIdx.x, total = (int)gridDim.x;
    if constexpr (TWO) {
        if (b >= two.first) {
            b -= two.first;
            total -= two.first;
            w = two.w;
            ep.sw = two.sw;
            ep.out = two.out;
            N = two.N;
        } else {
            total = two.first;
        }
    }
    return xcd_run(b, total);
}

// LDS bytes of the partial tiles, one copy per wavefront.
template <int TI, int CJ, int W>
struct Partial {
    static constexpr int kPitch = 128 * CJ + 16;              // a token's 32 CJ sums, padded (bank spread)
    static constexpr int kCopy = 32 * TI * kPitch;
    static constexpr int kSteps = 32 * CJ * 8 + 32 * TI * 4;  // channel steps, zero-point integers, token steps
    static constexpr int kBytes = W * kCopy;
    static_assert(kBytes + kSteps <= kMaxLds, "partial tiles do not fit LDS");
};

// Adds the W partial tiles (sums of 2^SHIFT acc, register v of lane l: token l % 32, channel 8 (v / 4) + 4 (l / 32)
// + v % 4) and writes the tile.  steps_at: LDS offset of the steps, filled by the caller before the first barrier here.
template <typename ACC, int TI, int CJ, int W, int SHIFT>
__device__ __forceinline__ void reduce_and_store(ACC (&acc)[CJ][TI], uint8_t* smem, int steps_at, const Epilogue& ep, int m0, int n0,
                                                 int M, int N)
{
    using P = Partial<TI, CJ, W>;
    using V4 = typename std::conditional<std::is_same<ACC, v16f>::value, v4f, v4i>::type;
    typedef __attribute__((address_space(3))) V4* lds4;
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(lds4)(lds_u8)(smem + wave * P::kCopy + (32 * i + r) * P::kPitch + (32 * j + 8 * q + 4 * g) * 4) =
                    (V4){acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
    __syncthreads();
    const float* steps = reinterpret_cast<const float*>(smem + steps_at);
    constexpr int UPR = 8 * CJ, ITEMS = 32 * TI * UPR;        // four channels of a token per item
#pragma unroll
    for (int it0 = 0; it0 < ITEMS; it0 += 64 * W) {
        const int it = it0 + tid;
        if (ITEMS % (64 * W) != 0 && it >= ITEMS) break;
        const int row = it / UPR, u = it % UPR, m = m0 + row, n = n0 + 4 * u;
        V4 s = *(lds4)(lds_u8)(smem + row * P::kPitch + u * 16);
#pragma unroll
        for (int c = 1; c < W; ++c) s += *(lds4)(lds_u8)(smem + c * P::kCopy + row * P::kPitch + u * 16);
        if (m >= M || n >= N) continue;
        const int64_t o = (int64_t)m * N + n;
        if (ep.acc_out) {
            const v4i a = {(int)s.x >> SHIFT, (int)s.y >> SHIFT, (int)s.z >> SHIFT, (int)s.w >> SHIFT};
            *reinterpret_cast<v4i*>(ep.acc_out + o) = a;
        }
        if (ep.out) {
            // the tiled kernel's two roundings: fp32(256 acc) * (sw * (step / 256)); the fp32 sums of the 6-bit instruction carry
            // no factor, theirs goes to the step
            const float f = (ep.srow ? steps[64 * CJ + row] : ep.sx) * (1.0f / 256.0f);
            const v4f c = *reinterpret_cast<const v4f*>(steps + 4 * u);
            float c0 = mul_rn(c.x, f), c1 = mul_rn(c.y, f), c2 = mul_rn(c.z, f), c3 = mul_rn(c.w, f);
            if constexpr (SHIFT == 0) { c0 *= 256.0f; c1 *= 256.0f; c2 *= 256.0f; c3 *= 256.0f; }
            if constexpr (SHIFT != 0) {
                if (ep.zcorr) {
                    const v4i z = *reinterpret_cast<const v4i*>(steps + 32 * CJ + 4 * u);
                    s.x += z.x << SHIFT; s.y += z.y << SHIFT; s.z += z.z << SHIFT; s.w += z.w << SHIFT;
                }
            }
            const __half2 lo = __floats2half2_rn(mul_rn((float)s.x, c0), mul_rn((float)s.y, c1));
            const __half2 hi = __floats2half2_rn(mul_rn((float)s.z, c2), mul_rn((float)s.w, c3));
            v2i val;
            val.x = *reinterpret_cast<const int*>(&lo);
            val.y = *reinterpret_cast<const int*>(&hi);
            *reinterpret_cast<v2i*>(ep.out + o) = val;
        }
    }
}

// The tile's steps: requested at the start of the kernel, one value per thread, and written to LDS in front of the
// reduction's barrier, so that no memory latency is left for the end.
template <int TI, int CJ>
struct Steps {
    float s, t;
    int z;
    __device__ __forceinline__ void request(const Epilogue& ep, int m0, int n0, int M, int N)
    {
        const int tid = threadIdx.x;
        s = t = 0.0f;
        z = 0;
        if (tid < 32 * CJ) {
            const int n = n0 + tid < N ? n0 + tid : N - 1;
            s = ep.sw[n];
            if (ep.zcorr) z = ep.zcorr[n];
        }
        if (ep.srow && tid < 32 * TI) t = ep.srow[m0 + tid < M ? m0 + tid : M - 1];
    }
    __device__ __forceinline__ void deposit(uint8_t* at) const
    {
        const int tid = threadIdx.x;
        float* p = reinterpret_cast<float*>(at);
        if (tid < 32 * CJ) {
            p[tid] = s;
            reinterpret_cast<int*>(p)[32 * CJ + tid] = z;
        }
        if (tid < 32 * TI) p[64 * CJ + tid] = t;
    }
};

// ---- prepacked operands (f6 tiles).  Every plane of a block is one contiguous load of a wavefront, so the operands
// go straight from memory to the registers the matrix instruction reads: a ring of U stages of 128 channels, each
// slot refilled as soon as its matrix instructions have been issued.  Four wavefronts: with eight the loads come in
// 15 % faster, but twice the partial tiles have to pass through LDS (333 x 4096 x 4096: 9.8 against 9.5 us, 128 x
// 14336 x 4096: 12.5 against 11.6), and two or three of the smaller workgroups share a CU (64 x 64 tiles in two
// rounds: 13.0 against 11.7).  A second stage in the ring of the larger tiles: 3 % slower.
template <int TI, int CJ, int W, int U, bool TWO>
__global__ __launch_bounds__(64 * W) void k_gemm_f6_ksplit(const uint8_t* __restrict__ x6, const uint8_t* __restrict__ w6, Epilogue ep,
                                                          int M, int N, int K, int GM, Second two)
{
    extern __shared__ __align__(16) uint8_t smem[];
    using P = Partial<TI, CJ, W>;
    constexpr int kBlock = 3072, kP1 = 1024, kP2 = 1536, kP3 = 2048;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t l16 = (uint32_t)lane * 16u, l8 = (uint32_t)lane * 8u;
    const int tile = own_tile<TWO>(two, w6, ep, N);
    const int mt = tile % GM, nt = tile / GM, m0 = mt * (32 * TI), n0 = nt * (32 * CJ);
    const int nk = K >> 7, RBX = (M + 31) >> 5, RBW = (N + 31) >> 5;
    const int k0 = (int)((int64_t)nk * wave / W), k1 = (int)((int64_t)nk * (wave + 1) / W), n = k1 - k0;

    Steps<TI, CJ> steps;
    steps.request(ep, m0, n0, M, N);

    const uint8_t *xp[TI], *wp[CJ];
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        const int rb = mt * TI + i < RBX ? mt * TI + i : RBX - 1;
        xp[i] = x6 + ((size_t)k0 * RBX + rb) * kBlock;
    }
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
        const int rb = nt * CJ + j < RBW ? nt * CJ + j : RBW - 1;
        wp[j] = w6 + ((size_t)k0 * RBW + rb) * kBlock;
    }
    v8i a[U][2][TI], b[U][2][CJ];
    v16f acc[CJ][TI];
#pragma unroll
    for (int j = 0; j < CJ; ++j)
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;

    auto image = [&](const uint8_t* blk, int st, v8i& d) {
        if (st == 0) {
            const v4i t = *reinterpret_cast<const v4i*>(blk + l16);
            const v2i u = *reinterpret_cast<const v2i*>(blk + kP1 + l8);
            d[0] = t.x; d[1] = t.y; d[2] = t.z; d[3] = t.w; d[4] = u.x; d[5] = u.y;
        } else {
            const v2i u = *reinterpret_cast<const v2i*>(blk + kP2 + l8);
            const v4i t = *reinterpret_cast<const v4i*>(blk + kP3 + l16);
            d[0] = u.x; d[1] = u.y; d[2] = t.x; d[3] = t.y; d[4] = t.z; d[5] = t.w;
        }
    };
    auto load_step = [&](auto slotc, auto stc, int s) {
        constexpr int slot = decltype(slotc)::value, st = decltype(stc)::value;
#pragma unroll
        for (int j = 0; j < CJ; ++j) image(wp[j] + (size_t)s * RBW * kBlock, st, b[slot][st][j]);
#pragma unroll
        for (int i = 0; i < TI; ++i) image(xp[i] + (size_t)s * RBX * kBlock, st, a[slot][st][i]);
    };
    auto multiply = [&](auto slotc, auto stc) {
        constexpr int slot = decltype(slotc)::value, st = decltype(stc)::value;
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int i = 0; i < TI; ++i)      // formats 3, 3: E3M2 both; no scales
                acc[j][i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b[slot][st][j], a[slot][st][i], acc[j][i], 3, 3, 0, 0, 0, 0);
    };
    auto S0 = std::integral_constant<int, 0>{};
    auto S1 = std::integral_constant<int, 1>{};
    auto stage = [&](auto slotc) { multiply(slotc, S0); multiply(slotc, S1); };
    auto stage_refill = [&](auto slotc, int s) {
        multiply(slotc, S0);
        load_step(slotc, S0, s);
        __builtin_amdgcn_sched_barrier(0);
        multiply(slotc, S1);
        load_step(slotc, S1, s);
        __builtin_amdgcn_sched_barrier(0);
    };
    if (n > 0) {
        load_step(S0, S0, 0);
        load_step(S0, S1, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (U == 1) {
            int s = 0;
            for (; s + 1 < n; ++s) stage_refill(S0, s + 1);
            stage(S0);
        } else {
            if (n > 1) {
                load_step(S1, S0, 1);
                load_step(S1, S1, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            int s = 0;
            for (; s + 3 < n; s += 2) {
                stage_refill(S0, s + 2);
                stage_refill(S1, s + 3);
            }
            const int left = n - s;                       // 1, 2 or 3
            if (left == 3) stage_refill(S0, s + 2); else stage(S0);
            if (left >= 2) stage(S1);
            if (left == 3) stage(S0);
        }
    }
    steps.deposit(smem + P::kBytes);
    reduce_and_store<v16f, TI, CJ, W, 0>(acc, smem, P::kBytes, ep, m0, n0, M, N);
}

// ---- packed nibbles (canonical operands) on the INT8 matrix instruction.  Rows lie K/2 bytes apart, and a load whose
// neighbouring lanes sit in different rows runs at one lane per clock, so the bytes go to LDS first, 128 contiguous ones
// per row and stage (a whole cache line, eight lanes each), in a ring of NS stages that belongs to the wavefront alone (no
// barrier); read back in the instruction's layout and expanded as in the tiled kernel.  Stages of 64 bytes a row, half
// lines, measured 8-22 % slower at every size (64 x 4096 x 14336: 11.9 against 9.3 us, 333 x 4096 x 4096: 11.7 against 10.7).
template <int TI, int CJ, int W, int NS, bool TWO>
__global__ __launch_bounds__(64 * W) void k_gemm_i8_ksplit(const uint8_t* __restrict__ xq, const uint8_t* __restrict__ wq, Epilogue ep,
                                                          int M, int N, int K, int GM, Second two)
{
    extern __shared__ __align__(16) uint8_t smem[];
    using P = Partial<TI, CJ, W>;
    constexpr int kStage = (TI + CJ) * 4096, PIECES = (TI + CJ) * 4;          // 32 rows x 128 bytes (256 channels) per block
    const int lane = threadIdx.x & 63, r = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = own_tile<TWO>(two, wq, ep, N);
    const int mt = tile % GM, nt = tile / GM, m0 = mt * (32 * TI), n0 = nt * (32 * CJ);
    const int nk = (K + 255) >> 8, Kb = K >> 1;
    const int k0 = (int)((int64_t)nk * wave / W), k1 = (int)((int64_t)nk * (wave + 1) / W), n = k1 - k0;
    // K an odd multiple of 128: the last stage of the row has only 128 channels; this wavefront's stages that are whole
    const int whole = (K & 128) && k1 == nk && n > 0 ? n - 1 : n;

    Steps<TI, CJ> steps;
    steps.request(ep, m0, n0, M, N);

    // piece p: 8 rows; lane l fetches row l / 8, the 16-byte chunk that belongs at position l % 8: chunk c of row t sits
    // at position c ^ ((t / 2) % 8), which spreads the reads of 32 rows over all banks
    uint32_t off[PIECES];
    const int chunk[2] = {(lane & 7) ^ (lane >> 4), (lane & 7) ^ (4 | (lane >> 4))};       // even and odd pieces
#pragma unroll
    for (int p = 0; p < PIECES; ++p) {
        const bool is_w = p < 4 * CJ;
        int row = (is_w ? n0 + p * 8 : m0 + (p - 4 * CJ) * 8) + (lane >> 3);
        const int last = (is_w ? N : M) - 1;
        row = row < last ? row : last;
        off[p] = (uint32_t)row * (uint32_t)Kb + (uint32_t)(chunk[p & 1] * 16);
    }
    // in a half stage the lanes of the upper four chunks re-read the lower ones (in bounds; never multiplied)
    const uint32_t back[2] = {chunk[0] >= 4 ? 64u : 0u, chunk[1] >= 4 ? 64u : 0u};
    const uint32_t ring = (uint32_t)(uintptr_t)(lds_u8)(smem + wave * (NS * kStage));
    const uint8_t *xk = xq + (size_t)k0 * 128, *wk = wq + (size_t)k0 * 128;
    auto request = [&](int s, int slot) {
        if (s < whole) {
#pragma unroll
            for (int p = 0; p < PIECES; ++p)
                lds_dma16((p < 4 * CJ ? wk : xk) + (size_t)s * 128, off[p], ring + slot * kStage + p * 1024);
        } else {
#pragma unroll
            for (int p = 0; p < PIECES; ++p)
                lds_dma16((p < 4 * CJ ? wk : xk) + (size_t)s * 128, off[p] - back[p & 1], ring + slot * kStage + p * 1024);
        }
    };
    const int swr = (r >> 1) & 7;
    int rd[4];                                                                // 16-byte chunk 2 kk + g of the lane's row
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) rd[kk] = r * 128 + (((2 * kk + g) ^ swr) << 4);

    v16i acc[CJ][TI];
#pragma unroll
    for (int j = 0; j < CJ; ++j)
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0;

    typedef __attribute__((address_space(3))) const uint8_t* lds_cu8;
    v4i p[2][2][TI + CJ];                 // packed operands of a stage: [128 channels][64 channels][block]
    auto fetch = [&](lds_cu8 st, int h) {
#pragma unroll
        for (int b = 0; b < TI + CJ; ++b) {
            p[h][0][b] = *(__attribute__((address_space(3))) const v4i*)(st + b * 4096 + rd[2 * h]);
            p[h][1][b] = *(__attribute__((address_space(3))) const v4i*)(st + b * 4096 + rd[2 * h + 1]);
        }
    };
    auto multiply = [&](int h) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            v4i e[TI + CJ], o[TI + CJ];
#pragma unroll
            for (int b = 0; b < TI + CJ; ++b) unpack16(p[h][kk][b], e[b], o[b]);
#pragma unroll
            for (int j = 0; j < CJ; ++j)
#pragma unroll
                for (int i = 0; i < TI; ++i) acc[j][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(e[j], e[CJ + i], acc[j][i], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < CJ; ++j)
#pragma unroll
                for (int i = 0; i < TI; ++i) acc[j][i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(o[j], o[CJ + i], acc[j][i], 0, 0, 0);
        }
    };
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < n) request(s, s);
    int slot = 0;
    for (int s = 0; s < whole; ++s) {
        // stage s has landed when at most the NS - 1 stages behind it are outstanding; near the end there are fewer
        if (s + NS - 1 < n) wait_vm<(NS - 1) * PIECES>();
        else wait_vm<0>();
        lds_cu8 st = (lds_cu8)(lds_u8)(smem + wave * (NS * kStage) + slot * kStage);
        fetch(st, 0);
        fetch(st, 1);                                            // (in flight while the first half is multiplied)
        multiply(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // (the slot has been read: it can be refilled)
        if (s + NS < n) request(s + NS, slot);
        slot = slot + 1 == NS ? 0 : slot + 1;
        multiply(1);
    }
    if (whole < n) {
        wait_vm<0>();
        fetch((lds_cu8)(lds_u8)(smem + wave * (NS * kStage) + slot * kStage), 0);
        multiply(0);
    }
    __syncthreads();                     // every wavefront is done with its ring: partial tiles and steps take its place
    steps.deposit(smem + P::kBytes);
    reduce_and_store<v16i, TI, CJ, W, 8>(acc, smem, P::kBytes, ep, m0, n0, M, N);
}

template <typename KERN>
int launch_tiles(KERN kern, std::atomic<uint64_t>& lds_ok, size_t lds, int tm, int tn, int threads, const void* x, const void* w,
                 const Epilogue& ep, int64_t M, int64_t N, int64_t K, Second two, hipStream_t st)
{
    const int GM = (int)((M + tm - 1) / tm), GN = (int)((N + tn - 1) / tn), GN2 = two.w ? (two.N + tn - 1) / tn : 0;
    if (lds > 48 * 1024 && allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds, lds_ok) != PQ_OK) return PQ_ERR_HIP;
    two.first = GM * GN;
    hipLaunchKernelGGL(kern, dim3((unsigned)(GM * (GN + GN2))), dim3((unsigned)threads), lds, st, static_cast<const uint8_t*>(x),
                       static_cast<const uint8_t*>(w), ep, (int)M, (int)N, (int)K, GM, two);
    return hip_status(hipGetLastError());
}

template <int TI, int CJ, int W, int U>
int launch_f6_tile(const void* x6, const void* w6, const Epilogue& ep, int64_t M, int64_t N, int64_t K, const Second& two, hipStream_t st)
{
    using P = Partial<TI, CJ, W>;
    constexpr size_t lds = P::kBytes + P::kSteps;
    static std::atomic<uint64_t> lds_ok[2] = {{0}, {0}};
    if (two.w) return launch_tiles(k_gemm_f6_ksplit<TI, CJ, W, U, true>, lds_ok[1], lds, 32 * TI, 32 * CJ, 64 * W, x6, w6, ep, M, N, K, two, st);
    return launch_tiles(k_gemm_f6_ksplit<TI, CJ, W, U, false>, lds_ok[0], lds, 32 * TI, 32 * CJ, 64 * W, x6, w6, ep, M, N, K, two, st);
}

template <int TI, int CJ, int W, int NS>
int launch_i8_tile(const void* xq, const void* wq, const Epilogue& ep, int64_t M, int64_t N, int64_t K, const Second& two, hipStream_t st)
{
    using P = Partial<TI, CJ, W>;
    constexpr size_t ring = (size_t)W * NS * (TI + CJ) * 4096;
    constexpr size_t lds = ring > (size_t)(P::kBytes + P::kSteps) ? ring : (size_t)(P::kBytes + P::kSteps);
    static_assert(lds <= (size_t)kMaxLds, "ring too large");
    static std::atomic<uint64_t> lds_ok[2] = {{0}, {0}};
    if (two.w) return launch_tiles(k_gemm_i8_ksplit<TI, CJ, W, NS, true>, lds_ok[1], lds, 32 * TI, 32 * CJ, 64 * W, xq, wq, ep, M, N, K, two, st);
    return launch_tiles(k_gemm_i8_ksplit<TI, CJ, W, NS, false>, lds_ok[0], lds, 32 * TI, 32 * CJ, 64 * W, xq, wq, ep, M, N, K, two, st);
}

// Tile of a launch and its estimated time in microseconds: a fixed part, per 128-channel stage of K the operands' way into
// the CU (and their expansion), and per tile the reduction and the epilogue (in proportion to the tile), which overlap another
// tile's stages where several workgroups fit a CU; tiles go round 256 CUs.
struct Plan {
    int ti, cj;
    double us;
};

struct TileShape {
    int ti, cj, resident;      // 32-row blocks of tokens and of channels; workgroups a CU holds at a time
};

struct PlanCosts {
    double launch, tile, per_area;      // microseconds: once, per tile, per tile and 32 x 32 block
};

// (two matrices: each ends in a tile of its own, so ragged heights can make one more column of tiles than their sum)
template <int COUNT, typename COST>
Plan best_plan(const TileShape (&tiles)[COUNT], int64_t M, int64_t N, int64_t Nb, int64_t K, PlanCosts c, COST stage_us)
{
    Plan best{0, 0, 1e300};
    for (const TileShape& t : tiles) {
        const int64_t tn = 32 * t.cj, count = ((M + 32 * t.ti - 1) / (32 * t.ti)) * ((N + tn - 1) / tn + (Nb + tn - 1) / tn);
        if (count > (1 << 20)) continue;
        const int64_t rounds = (count + 255) / 256;
        const double fill = count < 256 ? (double)count / 256 : 1.0;
        const double us = c.launch + (double)rounds * (double)(K / 128) * stage_us(t, fill) +
                          (double)((rounds + t.resident - 1) / t.resident) * (c.tile + c.per_area * t.ti * t.cj) + (double)M * (N + Nb) * 2 / 4.2e6;
        if (us < best.us) best = Plan{t.ti, t.cj, us};
    }
    return best;
}

constexpr TileShape kTilesF6[] = {{1, 1, 4}, {1, 2, 3}, {2, 2, 2}, {3, 2, 1}, {2, 3, 1}, {4, 2, 1}, {2, 4, 1}};
constexpr TileShape kTilesI8[] = {{1, 1, 1}, {1, 2, 1}, {2, 2, 1}, {3, 2, 1}, {2, 3, 1}};

// Prepacked: 0.035 us per stage and 32-row block of the tile (3 KiB at 85 KB/us).  Fitted to sweeps over 12 shapes (17 to 1111
// tokens, K 4096 and 14336), within about 10 % of what was measured; on 1500 random shapes (17-2500 tokens, K 128-30000) no
// product chosen by it was slower than the persistent launch.
Plan plan_f6(int64_t M, int64_t N, int64_t Nb, int64_t K)
{
    return best_plan(kTilesF6, M, N, Nb, K, PlanCosts{1.5, 0.5, 0.3}, [](const TileShape& t, double) { return 0.035 * (t.ti + t.cj); });
}

// Packed nibbles.  Fitted to 3300 random shapes (9-2500 tokens, K 128-28672, N 16-28672, weights from the memory-side cache and
// from HBM), every tile measured on each, so that the choice against the other kernels' estimates errs least: of 4796 choices
// (with and without planes) 45 are slower than the other kernel by more than 3 %, by 25 % at most.  A fit to warm weights and long
// rows alone (1.5 + 0.5 + 0.25 per block) missed the launch's cost on short rows, 892 x 256 -> 1216 3.9 -> 5.4 us, and on
// cold weights, 26 x 18816 -> 2352 13.0 -> 16.7 us: 111 of the same choices, by 38 % at most.  A stage takes 0.063 / 0.099 / 0.132 / 0.196 us
// for tiles of 1 x 1, 1 x 2, 2 x 2 and 2 x 3 blocks with every CU busy, less with few; 11 % more where rows are an odd multiple of 64
// bytes, so that a stage's 128 bytes of a row straddle two cache lines (40 % on long rows where one row of tiles leaves CUs idle:
// every workgroup then streams weights of its own, 1.5 instead of 1.05 us per 2048 channels); and no less than the weights' way
// from memory (2.8 us + bytes at 6.3 TB/s).
Plan plan_i8(int64_t M, int64_t N, int64_t Nb, int64_t K)
{
    Plan p = best_plan(kTilesI8, M, N, Nb, K, PlanCosts{1.4, 1.05, 0.35}, [M, K](const TileShape& t, double fill) {
        const int area = t.ti * t.cj;
        const double straddle = (K & 128) == 0 ? 1.0 : (M <= 32 && K >= 12800 && fill < 0.6 ? 1.4 : 1.11);
        const double idle = area <= 2 ? 0.4 : 0.1;                      // share of a stage that goes with the CUs' crowding
        return (area == 1 ? 0.063 : (area == 2 ? 0.099 : (area == 4 ? 0.132 : 0.196))) * (1.0 - idle + idle * fill) * straddle;
    });
    const double stream_us = 2.8 + (double)((N + Nb) * (K / 2)) / 6.3e6;
    if (p.us < stream_us) p.us = stream_us;
    return p;
}

}  // namespace

// Estimated microseconds; a large number where the kernel does not take the shape.
double gemm_ksplit_f6_cost_us(int64_t M, int64_t N, int64_t Nb, int64_t K) { return plan_f6(M, N, Nb, K).us; }

double gemm_ksplit_i8_cost_us(int64_t M, int64_t N, int64_t Nb, int64_t K)
{
    // (sums of 256 acc in int32, 32-bit byte offsets of the rows)
    if (K % 128 != 0 || K >= 131072 || M * (K / 2) >= ((int64_t)1 << 32) || (N + Nb) * (K / 2) >= ((int64_t)1 << 32)) return 1e300;
    return plan_i8(M, N, Nb, K).us;
}

int gemm_ksplit_f6_tile(int64_t M, int64_t N, int64_t Nb, int64_t K)
{
    const Plan p = plan_f6(M, N, Nb, K);
    return p.ti * 10 + p.cj;
}

int gemm_ksplit_i8_tile(int64_t M, int64_t N, int64_t Nb, int64_t K)
{
    const Plan p = plan_i8(M, N, Nb, K);
    return p.ti * 10 + p.cj;
}

int launch_gemm_ksplit_f6(const void* x6, const void* w6, const float* sw, float sx, int64_t M, int64_t N, int64_t K, void* out,
                          int32_t* acc, hipStream_t st, const void* w6b, const float* swb, int64_t Nb, void* outb)
{
    const Epilogue ep{sw, sx, nullptr, nullptr, static_cast<__half*>(out), acc};
    const Second two{static_cast<const uint8_t*>(w6b), swb, static_cast<__half*>(outb), (int)Nb, 0};
    const Plan p = plan_f6(M, N, Nb, K);
    switch (p.ti * 10 + p.cj) {
        case 11: return launch_f6_tile<1, 1, 4, 2>(x6, w6, ep, M, N, K, two, st);
        case 12: return launch_f6_tile<1, 2, 4, 2>(x6, w6, ep, M, N, K, two, st);
        case 22: return launch_f6_tile<2, 2, 4, 1>(x6, w6, ep, M, N, K, two, st);
        case 32: return launch_f6_tile<3, 2, 4, 1>(x6, w6, ep, M, N, K, two, st);
        case 23: return launch_f6_tile<2, 3, 4, 1>(x6, w6, ep, M, N, K, two, st);
        case 42: return launch_f6_tile<4, 2, 4, 1>(x6, w6, ep, M, N, K, two, st);
        case 24: return launch_f6_tile<2, 4, 4, 1>(x6, w6, ep, M, N, K, two, st);
        default: return PQ_ERR_UNSUPPORTED;
    }
}

int launch_gemm_ksplit_i8(const void* xq, const void* wq, const float* sw, float sx, const float* srow, const int32_t* zcorr, int64_t M,
                          int64_t N, int64_t K, void* out, int32_t* acc, hipStream_t st, const void* wqb, const float* swb, int64_t Nb,
                          void* outb)
{
    const Epilogue ep{sw, sx, srow, zcorr, static_cast<__half*>(out), acc};
    const Second two{static_cast<const uint8_t*>(wqb), swb, static_cast<__half*>(outb), (int)Nb, 0};
    const Plan p = plan_i8(M, N, Nb, K);
    switch (p.ti * 10 + p.cj) {
        case 11: return launch_i8_tile<1, 1, 8, 2>(xq, wq, ep, M, N, K, two, st);
        case 12: return launch_i8_tile<1, 2, 4, 2>(xq, wq, ep, M, N, K, two, st);
        case 22: return launch_i8_tile<2, 2, 4, 2>(xq, wq, ep, M, N, K, two, st);
        case 32: return launch_i8_tile<3, 2, 4, 2>(xq, wq, ep, M, N, K, two, st);
        case 23: return launch_i8_tile<2, 3, 4, 2>(xq, wq, ep, M, N, K, two, st);
        default: return PQ_ERR_UNSUPPORTED;
    }
}

}  // namespace pq
