// The product of int8 activations (grouped byte order) and packed 4-bit weights on tiles of 64 to 192 tokens x 128 channels.
//
// What bounds it: with random bytes the INT8 matrix instructions alone bring the chip to its power limit, and the form with
// 16 x 16 results needs less energy than the 32 x 32 one (all CUs, operands in registers: 3.71 against 2.72 POP/s, codes times
// 16 4.21 against 3.33; on another machine 3.94 against 3.38 and 4.58 against 4.07), so this kernel uses v_mfma_i32_16x16x64_i8.  Beside it only two other instructions fit
// without cost, so eight wavefronts (two to a SIMD) share the tile; and the tile's height comes in steps of 32, so that a
// shape finds one that fills the CUs (1500 x 4096: 8 x 32 = 256 tiles of 192 x 128, where 256 x 128 has 192).  Measured against
// the tiles of 32 x 32 results (pq_gemm_mfma.hip, which stays the faster on outputs that fill the chip with 256-wide ones):
// 1500 x 11008 -> 4096 85.5 -> 70.8 us, 877 x 15872 -> 2512 62.2 -> 49.4, 3774 x 5760 -> 1296 42.7 -> 35.0 on bytes uniform over the
// whole range; on activations as a quantizer leaves them the first is 71.6 -> 61.2, with all operands from HBM 77.4 -> 63.8.
//
// A stage is 128 channels: BM rows of 128 activation bytes and 128 rows of 64 packed bytes, fetched into an LDS ring of four
// by direct loads.  Wavefront (wm, wn) of 2 x 4 computes BM / 2 tokens x 32 channels: TM = BM / 32 token operands x 2 channel
// operands.  Lane l of an operand holds row l % 16 and the channels of chunk l / 16 (32 of them): the even ones feed one
// instruction, the odd ones another.  Activation bytes come from LDS as they stand; a packed operand is expanded once a stage
// into two of 16 * code (sums carry 16, taken out exactly).  A stage multiplies what the stage before it has read: token
// operand i is replaced by the next stage's as soon as its last instruction is issued, the weights are read early and
// expanded into a second set in the second half.
//
// LDS: a 16-byte read serves eight lanes a clock, four rows of chunk c and the other four of chunk c + 1 among them (not eight rows of one
// chunk), and the places are chosen so that those lie in different banks: of an activation row t, the even unit of chunk c at
// c ^ ((t >> 1) & 7) and the odd one at (c + 4) ^ ((t >> 1) & 7); chunk c of a weight row t at {0, 3, 1, 2}[c] ^ ((t >> 2) & 3).  1500 x 11008 ->
// 4096: conflicts 39735 -> 758 clocks a CU, LDS busy for 79 -> 40 thousand of 118 thousand clocks; the product 1 % faster, so LDS does not bound it.
#include "pq_internal.h"

#include <hip/hip_fp16.h>
#include <atomic>
#include <type_traits>

namespace pq {
namespace {

typedef int v2i __attribute__((ext_vector_type(2)));

#define PQB_LDS(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int kBN = 128, kWR = 2, kWC = 4, kNW = kWR * kWC, kRing = 4, kShift = 4;

// The accumulator is tied to the result: the builtin may write other registers and copy.  The compiler places no wait states
// around it: two are needed between a vector instruction that writes an operand and this one, eighteen between it and a read of
// its result.
__device__ __forceinline__ void mfma_i8(v4i& c, const v4i& a, const v4i& b)
{
    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

constexpr int stage_bytes(int bm) { return bm * 128 + kBN * 64; }

template <int BM, bool SPLIT>
__global__ __launch_bounds__(kNW * 64) void k_gemm_bytes(const uint8_t* __restrict__ xq, const uint8_t* __restrict__ wq,
                                                        const float* __restrict__ sw, float sx, int M, int N, int K, int GM,
                                                        int tiles, int S, __half* __restrict__ out,
                                                        int32_t* __restrict__ acc_out, const float* __restrict__ srow)
{
    extern __shared__ __align__(16) uint8_t smem[];
    constexpr int TM = BM / (16 * kWR), TN = kBN / (16 * kWC), STAGE = stage_bytes(BM);
    constexpr int BLK_A = BM / 8, BLK = BLK_A + kBN / 16;            // blocks of 1 KiB: 8 activation rows or 16 weight rows
    constexpr int LW = (BLK + kNW - 1) / kNW;                        // loads of a wavefront and stage
    const int item = xcd_run(blockIdx.x, gridDim.x);
    const int tile = SPLIT ? item % tiles : item, run = SPLIT ? item / tiles : 0;      // (an XCD's tiles share a run of K)
    const int m0 = (tile % GM) * BM, n0 = (tile / GM) * kBN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / kWC, wn = wave % kWC;
    const int r = lane & 15, g = lane >> 4;
    const int k0 = SPLIT ? (int)((int64_t)(K >> 7) * run / S) : 0;
    const int nk = (SPLIT ? (int)((int64_t)(K >> 7) * (run + 1) / S) : K >> 7) - k0;
    xq += (size_t)k0 * 128;
    wq += (size_t)k0 * 64;

    // ---- loader: block b = wave + 8 i; past the last one a wavefront fetches its previous block once more (the same bytes to
    // the same place), so that all of them count the same loads
    constexpr bool AGAIN = BLK % kNW != 0;
    const bool again = AGAIN && wave + kNW * (LW - 1) >= BLK;
    uint32_t goff[LW];
    static_for<0, LW>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const int blk = i == LW - 1 && again ? wave + kNW * (i - 1) : wave + kNW * i;
        const int lrow8 = lane >> 3, lrow16 = lane >> 2;
        int ra = m0 + blk * 8 + lrow8, rw = n0 + (blk - BLK_A) * 16 + lrow16;
        ra = ra < M ? ra : M - 1;
        rw = rw < N ? rw : N - 1;
        const int ua = (lane & 7) ^ (((blk * 8 + lrow8) >> 1) & 7), uw = (lane & 3) ^ ((lrow16 >> 2) & 3);      // as below, read backwards
        const uint32_t a = (uint32_t)ra * (uint32_t)K + (((ua & 3) << 1 | ua >> 2) << 4);
        const uint32_t w = (uint32_t)rw * (uint32_t)(K >> 1) + ((0x1320 >> 4 * uw & 3) << 4);
        goff[i] = blk < BLK_A ? a : w;
    });
    const uint32_t lds0 = (uint32_t)(uintptr_t)PQB_LDS(smem) + wave * 1024;
    auto dma = [&](auto ic, int kt, uint32_t fill) {
        constexpr int i = decltype(ic)::value;
        const uint8_t *xk = xq + (size_t)kt * 128, *wk = wq + (size_t)kt * 64;
        if constexpr (kNW * i + kNW <= BLK_A) lds_dma16_at<kNW * 1024 * i>(xk, goff[i], fill);
        else if constexpr (kNW * i >= BLK_A && (i < LW - 1 || !AGAIN)) lds_dma16_at<kNW * 1024 * i>(wk, goff[i], fill);
        else {
            const bool rep = i == LW - 1 && again;
            const int blk = rep ? wave + kNW * (i - 1) : wave + kNW * i;
            lds_dma16_at<kNW * 1024 * i>(blk < BLK_A ? xk : wk, goff[i], fill - (rep ? kNW * 1024 : 0));
        }
    };
    // ---- reader
    const uint32_t row_a = (wm * (TM * 16) + r) * 128, swz = (r >> 1) & 7;
    const uint32_t rd_a[2] = {row_a + ((g ^ swz) << 4), row_a + (((g + 4) ^ swz) << 4)};
    const uint32_t rd_b = BM * 128 + (wn * (TN * 16) + r) * 64 + (((0x2130 >> 4 * g & 3) ^ ((r >> 2) & 3)) << 4);
    auto from_lds = [&](uint32_t off) { return *(__attribute__((address_space(3))) const v4i*)(smem + off); };

    v4i acc[TM][TN], xa[2][TM], xb[2][2][TN], packed[TN];            // xa [even, odd]; xb [stage parity][even, odd]
    auto expand = [&](int par, int j) {
        constexpr int MASK = (int)0xF0F0F0F0u;
        const v4i p = packed[j];
        xb[par][0][j] = (v4i){(p.x << 4) & MASK, (p.y << 4) & MASK, (p.z << 4) & MASK, (p.w << 4) & MASK};
        xb[par][1][j] = (v4i){p.x & MASK, p.y & MASK, p.z & MASK, p.w & MASK};
        asm volatile("" : "+v"(xb[par][0][j]), "+v"(xb[par][1][j]));    // (here, not sunk to the first use)
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            acc[i][j] = (v4i){0, 0, 0, 0};
            asm volatile("" : "+v"(acc[i][j]));                      // (written here, not right in front of the first use)
        }

    auto stage = [&](auto parc, uint32_t next, int kt, uint32_t fill) {
        constexpr int par = decltype(parc)::value, NM = 2 * TM * TN, EXPAND = NM / 2;
        // the next stage has landed; everyone has read this one, whose slot is filled again
        wait_loads<(kRing - 2) * LW>();
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, NM>([&](auto nc) {
            constexpr int n = decltype(nc)::value, i = n / (2 * TN), ph = (n / TN) & 1, jj = n % TN, j = ph ? TN - 1 - jj : jj;
            mfma_i8(acc[i][j], xb[par][ph][j], xa[ph][i]);
            if constexpr (n < TN) packed[n] = from_lds(next + rd_b + n * 1024);
            if constexpr (n >= EXPAND) {
                constexpr int e0 = (n - EXPAND) * TN / (NM - EXPAND), e1 = (n + 1 - EXPAND) * TN / (NM - EXPAND);
                static_for<e0, e1>([&](auto ec) { expand(par ^ 1, decltype(ec)::value); });
            }
            if constexpr (jj == TN - 1) xa[ph][i] = from_lds(next + rd_a[ph] + i * 2048);
            if constexpr (n < LW) dma(std::integral_constant<int, n>{}, kt, fill);
            __builtin_amdgcn_sched_barrier(0);
        });
        wait_lds();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 1");
    };

    static_for<0, kRing>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        const uint32_t fill = __builtin_amdgcn_readfirstlane(lds0 + s * STAGE);
        static_for<0, LW>([&](auto ic) { dma(ic, s < nk ? s : nk - 1, fill); });
    });
    wait_loads<(kRing - 1) * LW>();
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, TN>([&](auto jc) { packed[decltype(jc)::value] = from_lds(rd_b + decltype(jc)::value * 1024); });
    static_for<0, TM>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        xa[0][i] = from_lds(rd_a[0] + i * 2048);
        xa[1][i] = from_lds(rd_a[1] + i * 2048);
    });
    static_for<0, TN>([&](auto jc) { expand(0, decltype(jc)::value); });
    wait_lds();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1");
    __builtin_amdgcn_sched_barrier(0);

    int slot = 0, kt = 0;
    auto after = [&](int s) { return s + 1 == kRing ? 0 : s + 1; };
    auto ahead = [&](int k) { return k + kRing < nk ? k + kRing : nk - 1; };       // past the end: harmless re-reads
    for (; kt + 2 <= nk; kt += 2) {
        const int s1 = after(slot), s2 = after(s1);
        stage(std::integral_constant<int, 0>{}, s1 * STAGE, ahead(kt), __builtin_amdgcn_readfirstlane(lds0 + slot * STAGE));
        stage(std::integral_constant<int, 1>{}, s2 * STAGE, ahead(kt + 1), __builtin_amdgcn_readfirstlane(lds0 + s1 * STAGE));
        slot = s2;
    }
    if (kt < nk) stage(std::integral_constant<int, 0>{}, after(slot) * STAGE, nk - 1, __builtin_amdgcn_readfirstlane(lds0 + slot * STAGE));
    wait_loads<0>();      // none may still be writing LDS
    asm volatile("s_nop 15\n\ts_nop 3\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(acc[i][j]));             // (read behind the wait states above)

    // ---- epilogue: the arithmetic of pq_gemm_mfma.hip.  A lane has four channels of token r; 16 tokens at a time are turned
    // through a padded region of the wavefront's own and stored as rows of 64 bytes.
    constexpr int PITCH = TN * 32 + 16, UPR = TN * 2;
    static_assert(16 * UPR == 64, "one store per 16 tokens");
    static_assert(kNW * 16 * PITCH <= kRing * STAGE, "staging fits the ring");
    uint8_t* stg = smem + wave * (16 * PITCH);
    constexpr float kUnshift = 1.0f / (float)(1 << kShift);
    const int nb = n0 + wn * (TN * 16);
    auto store = [&](auto dync) {
        constexpr bool DYN = decltype(dync)::value;
        float4 sc[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int n = nb + j * 16 + 4 * g;
            n = n + 4 <= N ? n : N - 4;
            sc[j] = *reinterpret_cast<const float4*>(sw + n);
            if constexpr (!DYN) {
                const float f = sx * kUnshift;
                sc[j].x *= f; sc[j].y *= f; sc[j].z *= f; sc[j].w *= f;
            }
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mb = m0 + wm * (TM * 16) + i * 16;
            const float fm = DYN ? srow[mb + r < M ? mb + r : M - 1] * kUnshift : 0.0f;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const v4i a = acc[i][j];
                const float4 s = sc[j];
                const __half2 lo = __floats2half2_rn(mul_rn((float)a.x, DYN ? s.x * fm : s.x), mul_rn((float)a.y, DYN ? s.y * fm : s.y));
                const __half2 hi = __floats2half2_rn(mul_rn((float)a.z, DYN ? s.z * fm : s.z), mul_rn((float)a.w, DYN ? s.w * fm : s.w));
                v2i val;
                val.x = *reinterpret_cast<const int*>(&lo);
                val.y = *reinterpret_cast<const int*>(&hi);
                *(__attribute__((address_space(3))) v2i*)(stg + r * PITCH + (j * 16 + 4 * g) * 2) = val;
            }
            // (LDS operations of a wavefront execute in order)
            const int row = lane / UPR, u = lane % UPR;
            const v4i val = *(__attribute__((address_space(3))) const v4i*)(stg + row * PITCH + u * 16);
            const int m = mb + row, n = nb + u * 8;
            if (m < M && n < N) __builtin_nontemporal_store(val, reinterpret_cast<v4i*>(out + (int64_t)m * N + n));
        }
    };
    if (SPLIT || acc_out) {
        int32_t* dst = SPLIT ? acc_out + (int64_t)run * M * N : acc_out;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int m = m0 + wm * (TM * 16) + i * 16 + r, n = nb + j * 16 + 4 * g;
                if (m < M && n + 4 <= N) *reinterpret_cast<v4i*>(dst + (int64_t)m * N + n) = acc[i][j] >> kShift;
            }
    }
    if (!SPLIT && out) {
        if (srow) store(std::true_type{});
        else store(std::false_type{});
    }
}

template <int BM, bool SPLIT>
int launch(const void* xq8, const void* wq, const float* sw, float sx, const float* srow, int64_t M, int64_t N, int64_t K, int S,
           void* out, int32_t* acc, hipStream_t st)
{
    const int GM = (int)((M + BM - 1) / BM), GN = (int)((N + kBN - 1) / kBN);
    constexpr size_t lds = (size_t)kRing * stage_bytes(BM);
    static_assert(lds <= 160 * 1024, "LDS ring too large");
    auto kern = k_gemm_bytes<BM, SPLIT>;
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds, lds_ok) != PQ_OK) return PQ_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)(GM * GN * S)), dim3(kNW * 64), lds, st, static_cast<const uint8_t*>(xq8),
                       static_cast<const uint8_t*>(wq), sw, sx, (int)M, (int)N, (int)K, GM, GM * GN, S, static_cast<__half*>(out), acc,
                       srow);
    return hip_status(hipGetLastError());
}

template <int BM>
int launch(const void* xq8, const void* wq, const float* sw, float sx, const float* srow, int64_t M, int64_t N, int64_t K, int S,
           void* out, int32_t* acc, hipStream_t st)
{
    return S > 1 ? launch<BM, true>(xq8, wq, sw, sx, srow, M, N, K, S, out, acc, st)
                 : launch<BM, false>(xq8, wq, sw, sx, srow, M, N, K, 1, out, acc, st);
}

}  // namespace

// Tiles of bm tokens.  S > 1: S runs of K, each a plane of sums at acc, and no output.
int launch_gemm_bytes(const void* xq8, const void* wq, const float* sw, float sx, const float* srow, int64_t M, int64_t N, int64_t K,
                      int bm, int S, void* out, int32_t* acc, hipStream_t st)
{
    switch (bm) {
        case 64: return launch<64>(xq8, wq, sw, sx, srow, M, N, K, S, out, acc, st);
        case 96: return launch<96>(xq8, wq, sw, sx, srow, M, N, K, S, out, acc, st);
        case 128: return launch<128>(xq8, wq, sw, sx, srow, M, N, K, S, out, acc, st);
        case 160: return launch<160>(xq8, wq, sw, sx, srow, M, N, K, S, out, acc, st);
        default: return launch<192>(xq8, wq, sw, sx, srow, M, N, K, S, out, acc, st);
    }
}

}  // namespace pq
