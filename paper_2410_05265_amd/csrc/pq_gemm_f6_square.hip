// The product of f6 tiles (layout and exactness: pq_gemm_f6.hip) on near-square tiles, 256 tokens x 256 channels and smaller ones, of one
// matrix or of two of one size for the same tokens.
//
// What bounds it: the operands' way into the CU and the chip's power limit.  A CU keeps about 32 KiB of lines in flight,
// whatever the depth of the ring in front of it, so it takes in 113 KiB/us of what the L2 holds, 80 of what the memory-side
// cache holds and 60-65 of a stream from HBM.  The 128 x 512 tiles of k_gemm_f6 ask for 60 KiB per 1024 clocks of matrix work
// and are bound by that (2048 x 28672 -> 8192, a copy of that kernel without its matrix instructions: 228 of 243 us); a square tile of the
// same area asks for 48 (a copy of this one: 173 us).  Both operands then pass through LDS (144 KiB of reads and writes per 1024 clocks of matrix work),
// which 128 bytes per clock still cover.  With that the kernel reaches the power limit: its clock falls from 2.0 to 1.75 GHz.
// So the matrix instruction is the 16 x 16 x 128 one: on the same operands, alone, it is 25 % above the 32 x 32 x 64 one at
// that limit (6.9 against 5.5 POP/s; on another machine 6.98 against 6.47), and neighbouring instructions share an operand.  2048 x 28672 -> 8192, three copies of
// the weights in turn: layer 272-277 -> 233-238 us (one copy 214 -> 201, product).
//
// A workgroup of four wavefronts, a wavefront 128 tokens x 128 channels: 64 accumulators of four registers.  One half stage =
// 128 channels of the product: step s of the two blocks 2 p and 2 p + 1 of 128 channels.  Lane l of an operand holds row l % 16
// and the image of half-wavefront (l / 16) % 2 of block 2 p + l / 32, which is 32 channels, the same ones for both operands; an
// image's two planes are two LDS reads.  A direct load fills 1 KiB: 512 bytes of a step of block 2 p, then the same 512 bytes
// of block 2 p + 1.  Operands are read a half stage ahead into a second register set, so a ring slot is free as soon as its
// half stage begins and three slots give the loads two half stages (1.3 us) of lead.
#include <hip/hip_fp16.h>

#include <atomic>
#include <type_traits>

#include "pq_internal.h"

namespace pq {
namespace {

typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

#define PQ_INLINE __attribute__((always_inline))      // lambdas: one left to the late inliner keeps its captures in scratch memory
#define PQS_LDS(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int kBlock = 3072, kStep = 1536;          // 32 rows x 128 channels of the tiles; one of its two steps
constexpr int kRing = 3;
constexpr int kWorkgroups = 256;                    // persistent, one per CU
// TM, TN: operands of 16 tokens and of 16 channels per wavefront
template <int TM_, int TN_> struct Tile {
    static constexpr int TM = TM_, TN = TN_, BM = 32 * TM, BN = 32 * TN;
    static constexpr int PIECES = 3 * (TM + TN);            // KiB of a half stage
    static constexpr int L = (PIECES + 3) / 4;              // direct loads per wavefront and half stage (past the last piece: that again, into the pad)
    static constexpr int STAGE = L * 4096, SCALES = kRing * STAGE, STEPS = (BN + 255) / 256 * 1024;
    // STREAM: per wavefront 16 tokens x 64 channels (an odd count: x all channels) between accumulators and memory, PITCH bytes a token
    static constexpr int TURN = SCALES + 2 * STEPS, PITCH = TN & 1 ? 32 * TN : 144;
    static constexpr size_t kLds = (size_t)TURN + 4 * 16 * PITCH;
    static_assert(kLds <= 160 * 1024, "LDS");
};

// The accumulator is tied to the result (the compiler's own form of the instruction may write another register and copy:
// 3.4 times the clocks), and operands are six registers, not the builtin's eight.  Formats 3, 3: E3M2.
// The compiler places no wait states around it: two are needed between a vector instruction that writes an operand and this
// one, eighteen between it and a read of its result (operands come from LDS alone).
__device__ __forceinline__ void mfma_e3m2(v4f& c, const v6i& a, const v6i& b)
{
    asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0 cbsz:3 blgp:3" : "+a"(c) : "v"(a), "v"(b));
}
template <bool RESULTS> __device__ __forceinline__ void settle()
{
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (RESULTS) asm volatile("s_nop 15\n\ts_nop 3");
    else asm volatile("s_nop 1");
    __builtin_amdgcn_sched_barrier(0);
}

// The lane number, taken afresh: what derives from threadIdx would be held, or spilled, across the main loop, and a reload
// behind direct loads waits for all of them.
__device__ __forceinline__ int fresh_lane()
{
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// (workgroup-uniform by construction: kept in scalar registers)
__device__ __forceinline__ const uint8_t* uniform(const uint8_t* p)
{
    const uint64_t a = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return reinterpret_cast<const uint8_t*>((uintptr_t)((uint64_t)hi << 32 | lo));
}

// Persistent workgroups walk a list of GM x GN tiles; in a round of 256 each XCD takes a contiguous run of 32.  The list goes
// through four panels at a time, and in those through strips of eight row tiles (fewer at the ends), row tiles fastest, so that a
// run is 8 row tiles x 4 panels and needs the least operand bytes.  With plain columns where GM is no multiple of 8 a run of 30000
// rows was 32 row tiles x one panel (30000 x 6144 -> 16384 1795 -> 1490 us, 20000 x 28672 -> 2048 755 -> 629, 7000 x 5120 -> 28000 583 ->
// 539; up to 16 row tiles level).
// A second matrix of the same size for the same tokens (w6 NULL: none); its tiles follow the first one's in the list.
struct Second {
    const uint8_t* w6;
    const float* sw;
    __half* out;
};

template <int TM, int TN, bool TWO, bool STREAM>
__global__ __launch_bounds__(256) void k_gemm_f6_square(const uint8_t* __restrict__ x6, const uint8_t* __restrict__ w6a,
                                                       const float* __restrict__ swa, float sx, int M, int N, int K, int GM,
                                                       int GN, __half* __restrict__ outa, int32_t* __restrict__ acc_out, Second two)
{
    using T = Tile<TM, TN>;
    constexpr int BM = T::BM, BN = T::BN, L = T::L, STAGE = T::STAGE, SCALES = T::SCALES;
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int H = K >> 7, np = H >> 1;                         // half stages (as many as blocks of 128 channels), pairs of blocks
    const int RBX = (M + 31) >> 5, RBW = (N + 31) >> 5;
    const uint32_t stride_x = (uint32_t)RBX * kBlock, stride_w = (uint32_t)RBW * kBlock;
    const uint32_t lds0 = (uint32_t)(uintptr_t)PQS_LDS(smem);
    const int G = gridDim.x, bid = blockIdx.x;
    const int total = (TWO ? 2 : 1) * GM * GN;
    // XCDs that read the same panels start an eighth of K apart (integer sums do not care about the order)
    const int p_first = (int)(((int64_t)(bid & 7) * np) >> 3);

    auto tile_of = [&](int seq) PQ_INLINE {                              // seq-th tile of this workgroup, -1 past the end
        const int base = seq * G;
        if (base >= total) return -1;
        const int cnt = total - base < G ? total - base : G;
        return bid < cnt ? base + xcd_run(bid, cnt) : -1;
    };
    int m0 = 0, n0 = 0;                                        // the tile whose loads are in flight or whose main loop runs
    const uint8_t* w6 = w6a;                                   // its matrix
    const float* sw = swa;
    __half* out = outa;
    auto move_to = [&](int t) PQ_INLINE {
        if constexpr (TWO) {
            const bool b = t >= GM * GN;
            w6 = b ? two.w6 : w6a;
            sw = b ? two.sw : swa;
            out = b ? two.out : outa;
            t = b ? t - GM * GN : t;
        }
        const int group = t / (4 * GM), in = t - group * 4 * GM, wide = GN - 4 * group < 4 ? GN - 4 * group : 4;
        const int strip = in / (8 * wide), at = in - strip * 8 * wide, high = GM - 8 * strip < 8 ? GM - 8 * strip : 8;
        const int mt = 8 * strip + at % high, nt = 4 * group + at / high;
        m0 = __builtin_amdgcn_readfirstlane(mt * BM);
        n0 = __builtin_amdgcn_readfirstlane(nt * BN);
    };
    auto pair_of = [&](int h) PQ_INLINE {                                // past the end: the last pair again (harmless re-reads)
        const int q = (h < H ? h >> 1 : np - 1) + p_first;
        return q >= np ? q - np : q;
    };

    uint32_t voff[L];                                          // lane offsets of the direct loads
    v6i tok[2][TM], wgt[2][TN];
    v4f acc[TN][TM];

    // piece q of a half stage: third q % 3 of row block q / 3 (tokens first); its upper lanes fetch from block 2 p + 1
    auto addresses = [&]() PQ_INLINE {
        const int lane = fresh_lane();
        // (copies: a choice between captured variables would put them in memory)
        const int rx = m0 >> 5, rw = n0 >> 5, last_x = RBX - 1, last_w = RBW - 1;
        const uint32_t next_x = lane < 32 ? 0u : stride_x, next_w = lane < 32 ? 0u : stride_w;
        const uint32_t at = (uint32_t)(lane & 31) * 16;
        static_for<0, L>([&](auto tc) PQ_INLINE {
            constexpr int t = decltype(tc)::value;
            const int q = wave + 4 * t < T::PIECES ? wave + 4 * t : T::PIECES - 1, b = q / 3, part = q % 3;
            int rb = rx + b;
            rb = rb < last_x ? rb : last_x;
            const uint32_t off_x = (uint32_t)rb * kBlock + next_x;
            rb = rw + b - TM;
            rb = rb < last_w ? rb : last_w;
            const uint32_t off_w = (uint32_t)rb * kBlock + next_w;
            voff[t] = (b < TM ? off_x : off_w) + part * 512 + at;
        });
    };
    auto dma = [&](auto tc, const uint8_t* xk, const uint8_t* wk, uint32_t fill) PQ_INLINE {
        constexpr int t = decltype(tc)::value;
        if constexpr (4 * t + 3 < 3 * TM) lds_dma16_at<t * 4096>(xk, voff[t], fill);
        else if constexpr (4 * t >= 3 * TM) lds_dma16_at<t * 4096>(wk, voff[t], fill);
        else lds_dma16_at<t * 4096>(wave + 4 * t < 3 * TM ? xk : wk, voff[t], fill);
    };
    // where this lane's images lie (an operand of odd number is the other half of the same block)
    const int g = (lane >> 4) & 1, b = lane >> 5, r = lane & 15;
    const uint32_t wide = (uint32_t)(g * 1024 + b * 512 + r * 16), narrow = (uint32_t)(b * 512 + g * 256 + r * 8);
    // With an odd count of operands the second wavefront starts inside a block: odd numbers then have a start of their own ([1]).
    auto start = [&](int o, uint32_t plane, uint32_t half) PQ_INLINE { return (uint32_t)(o >> 1) * kBlock + (uint32_t)(o & 1) * half + plane; };
    constexpr int XO = TM & 1, WO = TN & 1;
    const uint32_t xw[2] = {start(wm * TM, wide, 256), start(wm * TM + XO, wide, 256)}, xn[2] = {start(wm * TM, narrow, 128), start(wm * TM + XO, narrow, 128)};
    const uint32_t ww[2] = {start(2 * TM + wn * TN, wide, 256), start(2 * TM + wn * TN + WO, wide, 256)};
    const uint32_t wnr[2] = {start(2 * TM + wn * TN, narrow, 128), start(2 * TM + wn * TN + WO, narrow, 128)};
    // LDS read n of the 2 (TM + TN) of a half stage: even n the 16-byte plane of an operand's image, odd n the 8-byte one
    auto read = [&](auto stc, uint32_t slot, auto nc) PQ_INLINE {
        constexpr int st = decltype(stc)::value, n = decltype(nc)::value, f = n / 2, j = f < TM ? f : f - TM, own = (j & 1) & (f < TM ? XO : WO);
        v6i& d = f < TM ? tok[st][j] : wgt[st][j];
        if constexpr ((n & 1) == 0) {
            constexpr int off = (j >> 1) * kBlock + (own ? 0 : (j & 1) * 256) + (st == 0 ? 0 : 1024);
            uint32_t at;
            if constexpr (f < TM) at = xw[own]; else at = ww[own];
            const v4i t = *(__attribute__((address_space(3))) const v4i*)(smem + slot + at + off);
            if constexpr (st == 0) { d[0] = t.x; d[1] = t.y; d[2] = t.z; d[3] = t.w; }
            else { d[2] = t.x; d[3] = t.y; d[4] = t.z; d[5] = t.w; }
        } else {
            constexpr int off = (j >> 1) * kBlock + (own ? 0 : (j & 1) * 128) + (st == 0 ? 2048 : 0);
            uint32_t at;
            if constexpr (f < TM) at = xn[own]; else at = wnr[own];
            const v2i u = *(__attribute__((address_space(3))) const v2i*)(smem + slot + at + off);
            if constexpr (st == 0) { d[4] = u.x; d[5] = u.y; }
            else { d[0] = u.x; d[1] = u.y; }
        }
    };
    constexpr int READS = 2 * (TM + TN);
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;

    // The first loads of a tile: its channel steps (256 a load, one of the first wavefront; read back in the
    // epilogue, two regions in turn) and the whole ring.
    auto prefetch = [&](int parity) PQ_INLINE {
        addresses();
        if (out && wave < T::STEPS / 1024) {
            int n = n0 + 256 * wave + 4 * fresh_lane();
            n = n + 4 <= N ? n : N - 4;
            lds_dma16_at<0>(reinterpret_cast<const uint8_t*>(sw), (uint32_t)n * 4u, lds0 + SCALES + parity * T::STEPS + wave * 1024);
        }
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, kRing>([&](auto rc) PQ_INLINE {
            constexpr int s = decltype(rc)::value;
            const size_t at = (size_t)pair_of(s) * 2;
            const uint8_t *xk = uniform(x6 + at * stride_x + (s & 1) * kStep), *wk = uniform(w6 + at * stride_w + (s & 1) * kStep);
            const uint32_t fill = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024 + s * STAGE);
            static_for<0, L>([&](auto tc) PQ_INLINE { dma(tc, xk, wk, fill); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // stores of a full tile's output per wavefront, issued behind the next tile's first loads (STREAM: two per four operands, one per two or one)
    constexpr int STORES = TM * ((TN + 1) / 2);
    static_assert((kRing - 1) * L + STORES < 64, "vmcnt has six bits");

    // stores_behind: a full tile's stores were issued since this tile's first loads; they are not waited for
    auto compute = [&](bool stores_behind) PQ_INLINE {
        static_for<0, TN>([&](auto ic) PQ_INLINE { static_for<0, TM>([&](auto jc) PQ_INLINE { 
            v4f& a = acc[decltype(ic)::value][decltype(jc)::value];
            a = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
            asm volatile("" : "+a"(a));                        // (written here, not moved down to the first use)
        }); });
        // all matrix instructions of a half stage: channel operand i with every token operand, there and back
        auto multiply = [&](auto stc, auto&& between) PQ_INLINE {
            constexpr int st = decltype(stc)::value;
            static_for<0, TN * TM>([&](auto nc) PQ_INLINE {
                constexpr int n = decltype(nc)::value, i = n / TM, jj = n % TM, j = (i & 1) ? TM - 1 - jj : jj;
                mfma_e3m2(acc[i][j], wgt[st][i], tok[st][j]);
                between(nc);
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        auto half_stage = [&](auto stc, int h, int slot, int next) PQ_INLINE {
            constexpr int st = decltype(stc)::value;
            const size_t at = (size_t)pair_of(h + kRing) * 2;
            constexpr int fill_step = (st + kRing) & 1;
            const uint8_t *xk = uniform(x6 + at * stride_x + fill_step * kStep), *wk = uniform(w6 + at * stride_w + fill_step * kStep);
            const uint32_t fill = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024 + slot * STAGE);
            // half stage h + 1 has landed: behind its loads lie those of h + 2 (and, for h < 2, the stores)
            if (stores_behind && h < 2) wait_loads<L + STORES>();
            else wait_loads<L>();
            asm volatile("s_barrier" ::: "memory");            // for everyone, and everyone has read half stage h
            __builtin_amdgcn_sched_barrier(0);
            multiply(stc, [&](auto nc) PQ_INLINE {
                constexpr int n = decltype(nc)::value;
                if constexpr (n < READS) read(std::integral_constant<int, st ^ 1>{}, next * STAGE, nc);
                if constexpr ((n & 1) == 0 && n / 2 < L) dma(std::integral_constant<int, n / 2>{}, xk, wk, fill);
            });
            wait_lds();
            __builtin_amdgcn_sched_barrier(0);
        };
        static_assert(READS <= TM * TN && 2 * L <= TM * TN, "a read per instruction, a load per two");
        if (stores_behind) wait_loads<(kRing - 1) * L + STORES>();
        else wait_loads<(kRing - 1) * L>();
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        int slot = 0;
        asm volatile("" : "+s"(slot));                         // (addresses formed here, as for sx below)
        static_for<0, READS>([&](auto nc) PQ_INLINE { read(S0{}, slot * STAGE, nc); });
        wait_lds();
        settle<false>();                                       // (the zeroed accumulators)
        for (int h = 0; h < H; h += 2) {
            const int s1 = slot + 1 == kRing ? 0 : slot + 1, s2 = s1 + 1 == kRing ? 0 : s1 + 1;
            half_stage(S0{}, h, slot, s1);
            half_stage(S1{}, h + 1, s1, s2);
            slot = s2;
        }
        wait_loads<0>();                                       // none may still be writing LDS
        settle<true>();
        static_for<0, TN>([&](auto ic) PQ_INLINE { static_for<0, TM>([&](auto jc) PQ_INLINE {
            v4f& a = acc[decltype(ic)::value][decltype(jc)::value];
            asm volatile("" : "+a"(a));                        // (read behind the wait states above)
        }); });
        asm volatile("s_barrier" ::: "memory");                // nobody reads the ring any more
        __builtin_amdgcn_sched_barrier(0);
    };

    // out = fp16(fp32(acc * factor)), factor = 256 fl(sw * (sx / 256)): the same real product, hence the same rounding, as the
    // INT8 tiled kernel's (256 acc) * fl(sw * (sx / 256)).  A lane has four channels of one token per operand; neighbouring
    // rows of 16 lanes trade halves of two operands, so that a lane stores eight channels of its token: 16 bytes of 16 rows at a
    // time, in ordinary stores that wait in the L2 and the memory-side cache (non-temporal ones reach memory one by one: 2048 x 8192 ->
    // 28672 252 -> 276 us).  STREAM: 16 tokens x 64 channels turn through LDS instead, a wavefront's own part of it, and eight
    // neighbouring lanes store 128 bytes of a row non-temporally, past that cache; where it lies: streams_output.
    // (Rows of a turn lie 144 bytes apart, or 224 with the pieces of the upper eight rows swapped, which spreads them over the banks: 1.3 of 63
    // thousand clocks of a CU go to its conflicts, 1111 x 4096 -> 12288.)
    auto epilogue = [&](int m0, int n0, __half* out, int parity) PQ_INLINE {
        const int lane = fresh_lane();
        const int g4 = lane >> 4, r = lane & 15;
        const float* scl = reinterpret_cast<const float*>(smem + SCALES + parity * T::STEPS) + wn * (16 * TN);
        const int mb = m0 + wm * (16 * TM), nb = n0 + wn * (16 * TN);
        float step = sx;
        asm volatile("" : "+s"(step));                         // (the product is formed here, not held across the main loop)
        const float f = step * (1.0f / 256.0f);
        v4f sc[TN];
        if (out) {
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                v4f s = *(__attribute__((address_space(3))) const v4f*)(scl + i * 16 + 4 * g4);
                s.x = mul_rn(s.x, f) * 256.0f; s.y = mul_rn(s.y, f) * 256.0f; s.z = mul_rn(s.z, f) * 256.0f; s.w = mul_rn(s.w, f) * 256.0f;
                sc[i] = s;
            }
        }
        uint8_t* const turn = smem + T::TURN + wave * (16 * T::PITCH);
        static_for<0, TM>([&](auto jc) PQ_INLINE {
            constexpr int j = decltype(jc)::value;
            const int m16 = mb + j * 16;
            if (acc_out) {
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const int m = m16 + r, n = nb + i * 16 + 4 * g4;
                    const v4i iv = {(int)acc[i][j].x, (int)acc[i][j].y, (int)acc[i][j].z, (int)acc[i][j].w};
                    if (m < M && n + 4 <= N) *reinterpret_cast<v4i*>(acc_out + (int64_t)m * N + n) = iv;
                }
            }
            if (out) {
                auto pack = [&](const v4f& a, const v4f& s) PQ_INLINE {
                    const __half2 lo = __floats2half2_rn(mul_rn(a.x, s.x), mul_rn(a.y, s.y));
                    const __half2 hi = __floats2half2_rn(mul_rn(a.z, s.z), mul_rn(a.w, s.w));
                    v2i val;
                    val.x = *reinterpret_cast<const int*>(&lo);
                    val.y = *reinterpret_cast<const int*>(&hi);
                    return val;
                };
                if constexpr (STREAM) {
                    // CNT operands: from columns (of 8 channels) `at` on of the turned rows to the wavefront's columns `col` on
                    auto store = [&](auto cntc, int at, int col, auto nontemporal) PQ_INLINE {
                        constexpr int CNT = decltype(cntc)::value, LANES = 2 * CNT, ROWS = 64 / LANES < 16 ? 64 / LANES : 16;
                        const int c = lane % LANES, k = lane / LANES % ROWS;
                        static_for<0, 16 / ROWS>([&](auto pc) PQ_INLINE {
                            const int row = decltype(pc)::value * ROWS + k, m = m16 + row, n = nb + (col + c) * 8;
                            const int swapped = (at + c) ^ (TN & 1 ? row >> 3 : 0);
                            const v4i val = *(__attribute__((address_space(3))) const v4i*)(turn + row * T::PITCH + swapped * 16);
                            v4i* const to = reinterpret_cast<v4i*>(out + (int64_t)m * N + n);
                            if (lane < ROWS * LANES && m < M && n + 8 <= N) {
                                if constexpr (decltype(nontemporal)::value) __builtin_nontemporal_store(val, to);
                                else *to = val;
                            }
                        });
                    };
                    auto turned = [&](auto ic, int at) PQ_INLINE {
                        constexpr int i = decltype(ic)::value;
                        const int piece = g4 ^ (TN & 1 ? (r >> 3) << 1 : 0);
                        *(__attribute__((address_space(3))) v2i*)(turn + r * T::PITCH + at * 32 + piece * 8) = pack(acc[i][j], sc[i]);
                    };
                    if constexpr (TN & 1) {                    // the operand beside the other wavefront's shares its 64 bytes: ordinary
                        static_assert(TN == 7, "a chunk of four, of two and of one");
                        static_for<0, TN>([&](auto ic) PQ_INLINE { turned(ic, decltype(ic)::value); });
                        store(std::integral_constant<int, 4>{}, 2 * wn, 2 * wn, std::true_type{});
                        store(std::integral_constant<int, 2>{}, 2 * wn + 8, 2 * wn + 8, std::true_type{});
                        store(std::integral_constant<int, 1>{}, wn ? 0 : 12, wn ? 0 : 12, std::false_type{});
                    } else {
                        static_for<0, (TN + 2) / 4>([&](auto cc) PQ_INLINE {
                            constexpr int first = 4 * decltype(cc)::value, CNT = TN - first < 4 ? TN - first : 4;
                            static_for<0, CNT>([&](auto ic) PQ_INLINE { turned(std::integral_constant<int, first + decltype(ic)::value>{}, decltype(ic)::value); });
                            store(std::integral_constant<int, CNT>{}, 0, 2 * first, std::true_type{});
                        });
                    }
                } else {
                    const int m = m16 + r;
                    __half* const row = out + (int64_t)m * N;
                    if constexpr (TN & 1) {                        // the last operand alone: four channels a lane
                        const int n = nb + (TN - 1) * 16 + 4 * g4;
                        const v2i val = pack(acc[TN - 1][j], sc[TN - 1]);
                        if (m < M && n + 4 <= N) *reinterpret_cast<v2i*>(row + n) = val;
                    }
                    static_for<0, TN / 2>([&](auto pc) PQ_INLINE {
                        constexpr int i = 2 * decltype(pc)::value;
                        const v2i even = pack(acc[i][j], sc[i]);
                        // rows 0 .. 3 of 16 lanes hold channels 0-3, 4-7, 8-11, 12-15 of either operand; after the swap rows 0
                        // and 2 hold 0-7 and 8-15 of the even one, rows 1 and 3 of the odd one
                        const v2i odd = pack(acc[i + 1][j], sc[i + 1]);
                        const auto s0 = __builtin_amdgcn_permlane16_swap(even.x, odd.x, false, false);
                        const auto s1 = __builtin_amdgcn_permlane16_swap(even.y, odd.y, false, false);
                        const v4i val = {(int)s0[0], (int)s1[0], (int)s0[1], (int)s1[1]};
                        const int n = nb + i * 16 + (g4 & 1) * 16 + (g4 >> 1) * 8;
                        if (m < M && n + 8 <= N) *reinterpret_cast<v4i*>(row + n) = val;
                    });
                }
            }
        });
    };

    int t = tile_of(0);
    if (t < 0) return;
    move_to(t);
    prefetch(0);
    bool stores_behind = false;
    for (int seq = 1, parity = 0;; ++seq, parity ^= 1) {
        compute(stores_behind);
        const int m_done = m0, n_done = n0;
        __half* const out_done = out;
        t = tile_of(seq);
        if (t >= 0) {
            move_to(t);
            prefetch(parity ^ 1);
        }
        epilogue(m_done, n_done, out_done, parity);
        if (t < 0) break;
        stores_behind = out_done && m_done + BM <= M && n_done + BN <= N;
    }
}

// The tiles that are built, 10 * TM + TN.  (Of fifteen swept, those that were the fastest somewhere; the first one on equal estimates.)
constexpr int kTiles[] = {88, 78, 68, 58, 48, 87, 66, 46, 44, 64};

// Whether the output goes past the memory-side cache.  An output that stays there takes the place of operands that the next calls read again
// (471 x 8960 -> 12336, three copies in turn 47.3 -> 36.4 us, 1500 x 4096 -> 2 x 11008 100 -> 83.6, 2048 x 8192 -> 10240 102 -> 93, 4735 x
// 15360 -> 2288 96.2 -> 87); pieces that are no whole lines cost a non-temporal store more.  By the pieces of a wavefront's rows:
// - whole lines of 128 bytes (112 runs 0.964 x, geometric mean, 0.835 to 1.02), unless the operands alone fill the cache (2048 x 4096 -> 128256, one
//   copy 589 -> 615);
// - halves, up to half the cache (2048 x 8192 -> 28672 241 -> 259, 2867 x 7680 -> 14368, six copies, 166 -> 180; 259 x 3328 -> 2 x 24736, two
//   copies 51.0 -> 41.7);
// - 32 bytes, on long rows, whose outputs are few beside the operands (1724 x 1024 -> 15440 28.9 -> 37.5, 2195 x 4608 -> 3824 25.7 -> 28.2; 618 x
//   10496 -> 9904, three copies 52.0 -> 40.7).
bool streams_output(int TN, int64_t M, int64_t N, int64_t K, const void* out, const Second& two)
{
    const int64_t operands = (M + (two.w6 ? 2 : 1) * N) * K / 4 * 3, mib = 1 << 20;
    const uintptr_t start = (uintptr_t)out | (uintptr_t)two.out | (uintptr_t)(2 * N);
    if (start % 128 == 0 && TN % 4 == 0) return operands < 256 * mib;
    if (start % 64 == 0) return operands < 128 * mib;
    return TN % 2 == 0 && K >= 6144 && operands < 96 * mib;
}

template <int TM, int TN>
int launch_tile(const void* x6, const void* w6, const float* sw, float sx, int64_t M, int64_t N, int64_t K, void* out, int32_t* acc,
                hipStream_t st, const Second& two)
{
    using T = Tile<TM, TN>;
    const int GM = (int)((M + T::BM - 1) / T::BM), GN = (int)((N + T::BN - 1) / T::BN);
    const int64_t tiles = (two.w6 ? 2 : 1) * (int64_t)GM * GN;
    auto launch = [&](auto twoc, auto streamc) {
        auto kern = k_gemm_f6_square<TM, TN, decltype(twoc)::value, decltype(streamc)::value>;
        static std::atomic<uint64_t> lds_ok{0};      // (of this kernel: the lambda is instantiated per tile, count and kind of store)
        if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), T::kLds, lds_ok) != PQ_OK) return (int)PQ_ERR_HIP;
        hipLaunchKernelGGL(kern, dim3((unsigned)(tiles < kWorkgroups ? tiles : kWorkgroups)), dim3(256), T::kLds, st,
                           static_cast<const uint8_t*>(x6), static_cast<const uint8_t*>(w6), sw, sx, (int)M, (int)N, (int)K, GM, GN,
                           static_cast<__half*>(out), acc, two);
        return hip_status(hipGetLastError());
    };
    const std::true_type yes;
    const std::false_type no;
    if (out && streams_output(TN, M, N, K, out, two)) return two.w6 ? launch(yes, yes) : launch(no, yes);
    return two.w6 ? launch(yes, no) : launch(no, no);
}

}  // namespace

// The least estimate: the fits of the header, plus the output (0.08 us per MB beside the main loops), and a half stage takes up to a third
// less the fewer CUs share the memory side.  Rows under 1024 channels were not swept and stay with the other kernel (450 x 512 ->
// 400000 on 256 x 256 151 -> 169 us).
int gemm_f6_square_tile(int64_t M, int64_t N, int64_t K, bool two, double* us)
{
    *us = 1e30;
    if (K % 256 != 0 || K < 1024) return 0;
    const int64_t mats = two ? 2 : 1;
    const double H = (double)(K / 128), out_mb = (double)(mats * M) * N * 2e-6;
    int best = 0;
    for (const int tile : kTiles) {
        const int tm = tile / 10, tn = tile % 10;
        const int64_t gm = (M + 32 * tm - 1) / (32 * tm), gn = (N + 32 * tn - 1) / (32 * tn), tiles = mats * gm * gn;
        const int64_t rounds = (tiles + kWorkgroups - 1) / kWorkgroups;
        if (tiles >= (1 << 24)) continue;
        const double fill = (double)tiles / (double)(rounds * kWorkgroups);
        const double half_stage = (0.00798 * tm * tn + 0.02276 * (tm + tn)) * (1.0 - 0.33118 * (1.0 - fill));
        const double t = 1.74267 + 0.08083 * out_mb + (double)rounds * (1.05165 + 0.08898 * tm * tn + H * half_stage);
        if (t < *us) { *us = t; best = tile; }
    }
    return best;
}

int launch_gemm_f6_square(int tile, const void* x6, const void* w6, const float* sw, float sx, int64_t M, int64_t N, int64_t K, void* out,
                          int32_t* acc, hipStream_t st, const void* w6b, const float* swb, void* outb)
{
    const Second two{static_cast<const uint8_t*>(w6b), swb, static_cast<__half*>(outb)};
    switch (tile) {
    case 88: return launch_tile<8, 8>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 78: return launch_tile<7, 8>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 68: return launch_tile<6, 8>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 58: return launch_tile<5, 8>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 48: return launch_tile<4, 8>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 87: return launch_tile<8, 7>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 66: return launch_tile<6, 6>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 46: return launch_tile<4, 6>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 44: return launch_tile<4, 4>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    case 64: return launch_tile<6, 4>(x6, w6, sw, sx, M, N, K, out, acc, st, two);
    }
    return PQ_ERR_UNSUPPORTED;
}

}  // namespace pq
