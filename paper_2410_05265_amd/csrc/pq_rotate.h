// Device-side building blocks of the online rotation + quantizer, shared by the stand-alone
// kernels, the fused decode kernel and the calibration kernels (App. B "Online Rotation" and Eq. 1
// of the paper).  A workgroup of 256 threads transforms one chunk of a row; what the quantizer's
// step is (static, per head, per token, per group, with a zero-point) comes from a step provider,
// and an input transform can fuse an elementwise producer in front.
#pragma once

#include "pq_internal.h"

#include <hip/hip_fp16.h>
#include <type_traits>

namespace pq {
namespace rq {

constexpr int kThreads = 256;
constexpr int kChunk = 2048;  // channels per workgroup per group index

// ---- partner exchange between lanes: returns the value held by lane (id ^ (1 << B)).
// (Every lane of these moves has a source, so the old value is 0 with bound_ctrl set: only then does the compiler make move and addition
// one instruction, 16 instead of 24 for eight values.  Lanes 4 apart as two such moves, 7 - i within eight, then 3 - i within four: 24
// instead of 56 for two masked moves with their copies and wait states.)
template <int CTRL>
__device__ __forceinline__ int dpp_all(int iv)
{
    return __builtin_amdgcn_update_dpp(0, iv, CTRL, 0xF, 0xF, true);
}

template <int B>
__device__ __forceinline__ int lane_xor_i(int iv)
{
    int r;
    if constexpr (B == 0) {
        r = dpp_all<0xB1>(iv);                       // quad_perm [1,0,3,2]
    } else if constexpr (B == 1) {
        r = dpp_all<0x4E>(iv);                       // quad_perm [2,3,0,1]
    } else if constexpr (B == 2) {
        r = dpp_all<0x1B>(dpp_all<0x141>(iv));       // row_half_mirror, quad_perm [3,2,1,0]
    } else if constexpr (B == 3) {
        r = dpp_all<0x128>(iv);                      // row_ror:8
    } else if constexpr (B == 4) {
        r = __builtin_amdgcn_ds_swizzle(iv, 0x401F);  // bit-mask mode: and 0x1F, xor 0x10
    } else {
        r = __shfl_xor(iv, 32, 64);
    }
    return r;
}

template <int B>
__device__ __forceinline__ float lane_xor(float v)
{
    return __int_as_float(lane_xor_i<B>(__float_as_int(v)));
}

// One butterfly stage between lanes, up to sign: the lower lane of a pair ends with own + partner, the upper one with own - partner,
// the negative of its sum, which is one fused multiply-add with the exchange inside (a product with +-1 is exact: the roundings are the
// sum's).  Partners in the other stages carry the same sign, so after the stages of the low `bits` lane bits a lane's values are
// lane_sign(lane, bits) times the rotated ones; whoever takes them multiplies that into the step's reciprocal.
// The compiler makes a move and a multiply-add of it, and wait states where they share a register: written out for eight values, 9
// instructions a stage (17 for lanes 4 apart) against 24 (56) for move, select and addition.  Quantizers, us: silu x up 2048 x 14336 in blocks
// of 128 29.3 -> 24.3, per token 2048 x 11008 in blocks of 128 27.5 -> 21.1, 8 bits 1500 x 11008 13.2 -> 11.2, 2048 x 4096 in one block of 4096
// 8.5 -> 6.9.  The leading s_nop keeps two wait states between a vector instruction that writes a value and its exchange, and whole stages
// in one statement keep the compiler's own exchanges from following a write too closely.  (A value must not come straight from a matrix
// instruction, whose longer wait the compiler does not place in front of these.)
#define PQ_FMAC8(SRC, MOVE) \
    "v_fmac_f32_dpp %0, " SRC(0) ", %8 " MOVE "\n\tv_fmac_f32_dpp %1, " SRC(1) ", %8 " MOVE "\n\t" \
    "v_fmac_f32_dpp %2, " SRC(2) ", %8 " MOVE "\n\tv_fmac_f32_dpp %3, " SRC(3) ", %8 " MOVE "\n\t" \
    "v_fmac_f32_dpp %4, " SRC(4) ", %8 " MOVE "\n\tv_fmac_f32_dpp %5, " SRC(5) ", %8 " MOVE "\n\t" \
    "v_fmac_f32_dpp %6, " SRC(6) ", %8 " MOVE "\n\tv_fmac_f32_dpp %7, " SRC(7) ", %8 " MOVE
#define PQ_OWN(I) "%" #I
#define PQ_ALL " row_mask:0xf bank_mask:0xf bound_ctrl:1"
#define PQ_EIGHT(V) "+v"((V)[0]), "+v"((V)[1]), "+v"((V)[2]), "+v"((V)[3]), "+v"((V)[4]), "+v"((V)[5]), "+v"((V)[6]), "+v"((V)[7])
template <int B>
__device__ __forceinline__ void lane_stage8(float* v, float s)
{
    if constexpr (B == 0) {
        asm("s_nop 1\n\t" PQ_FMAC8(PQ_OWN, "quad_perm:[1,0,3,2]" PQ_ALL) : PQ_EIGHT(v) : "v"(s));
    } else if constexpr (B == 1) {
        asm("s_nop 1\n\t" PQ_FMAC8(PQ_OWN, "quad_perm:[2,3,0,1]" PQ_ALL) : PQ_EIGHT(v) : "v"(s));
    } else if constexpr (B == 3) {
        asm("s_nop 1\n\t" PQ_FMAC8(PQ_OWN, "row_ror:8" PQ_ALL) : PQ_EIGHT(v) : "v"(s));
    } else if constexpr (B == 2) {
        float t[8];
        asm("s_nop 1\n\t"
            "v_mov_b32_dpp %8, %0 row_half_mirror" PQ_ALL "\n\tv_mov_b32_dpp %9, %1 row_half_mirror" PQ_ALL "\n\t"
            "v_mov_b32_dpp %10, %2 row_half_mirror" PQ_ALL "\n\tv_mov_b32_dpp %11, %3 row_half_mirror" PQ_ALL "\n\t"
            "v_mov_b32_dpp %12, %4 row_half_mirror" PQ_ALL "\n\tv_mov_b32_dpp %13, %5 row_half_mirror" PQ_ALL "\n\t"
            "v_mov_b32_dpp %14, %6 row_half_mirror" PQ_ALL "\n\tv_mov_b32_dpp %15, %7 row_half_mirror" PQ_ALL "\n\t"
            "v_fmac_f32_dpp %0, %8, %16 quad_perm:[3,2,1,0]" PQ_ALL "\n\tv_fmac_f32_dpp %1, %9, %16 quad_perm:[3,2,1,0]" PQ_ALL "\n\t"
            "v_fmac_f32_dpp %2, %10, %16 quad_perm:[3,2,1,0]" PQ_ALL "\n\tv_fmac_f32_dpp %3, %11, %16 quad_perm:[3,2,1,0]" PQ_ALL "\n\t"
            "v_fmac_f32_dpp %4, %12, %16 quad_perm:[3,2,1,0]" PQ_ALL "\n\tv_fmac_f32_dpp %5, %13, %16 quad_perm:[3,2,1,0]" PQ_ALL "\n\t"
            "v_fmac_f32_dpp %6, %14, %16 quad_perm:[3,2,1,0]" PQ_ALL "\n\tv_fmac_f32_dpp %7, %15, %16 quad_perm:[3,2,1,0]" PQ_ALL
            : PQ_EIGHT(v), "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7])
            : "v"(s));
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = fmaf(lane_xor<B>(v[i]), s, v[i]);
    }
}
#undef PQ_FMAC8
#undef PQ_OWN
#undef PQ_ALL
#undef PQ_EIGHT

// SIGNED: the sums themselves (where a zero's sign is seen, or the caller takes the values).
template <int B, bool SIGNED = false, int NV>
__device__ __forceinline__ void lane_stage(float (&v)[NV], int lane)
{
    const bool upper = (lane >> B) & 1;
    if constexpr (SIGNED) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const float p = lane_xor<B>(v[i]);
            v[i] = upper ? (p - v[i]) : (p + v[i]);
        }
    } else {
        static_assert(NV % 8 == 0, "eight values at a time");
        const float s = upper ? -1.0f : 1.0f;
#pragma unroll
        for (int i = 0; i < NV; i += 8) lane_stage8<B>(v + i, s);
    }
}
__device__ __forceinline__ float lane_sign(int lane, int bits)
{
    return __builtin_popcount(lane & ((1 << bits) - 1)) & 1 ? -1.0f : 1.0f;
}

// d = 1, 2, 4 inside one group of 8
__device__ __forceinline__ void reg_stages8(float* v, int nstages)
{
    if (nstages >= 1) {
#pragma unroll
        for (int i = 0; i < 8; i += 2) { float a = v[i], b = v[i + 1]; v[i] = a + b; v[i + 1] = a - b; }
    }
    if (nstages >= 2) {
#pragma unroll
        for (int i = 0; i < 8; i += 4)
#pragma unroll
            for (int j = 0; j < 2; ++j) { float a = v[i + j], b = v[i + j + 2]; v[i + j] = a + b; v[i + j + 2] = a - b; }
    }
    if (nstages >= 3) {
#pragma unroll
        for (int j = 0; j < 4; ++j) { float a = v[j], b = v[j + 4]; v[j] = a + b; v[j + 4] = a - b; }
    }
}

// Round-to-nearest-even of eight scaled values, clamp to [-8,7], pack low nibble first.
// `magic` puts round(t) + 8 into the low mantissa bits of an fp32 in [2^23, 2^24).
constexpr float kMagic = 12582920.0f;            // 1.5 * 2^23 + 8, bit pattern 0x4B400008
constexpr uint32_t kMagicSum = 0x4B400000u * 0x11111111u;  // sum of (pattern - offset part) << 4i

// zo = zero-point - 8 (Eq. 1 with a zero-point z: stored code = clamp(round(t) + z, 0, 15) - 8); 0 for
// the symmetric quantizer, in which case the compiler drops every trace of it.
template <bool EXACT>
__device__ __forceinline__ uint32_t quant_pack8(const float* v, const float* raw, float mult, float step, int zo = 0)
{
    float t[8];
    uint32_t bits[8];
    bool suspect = false;
    const float lo = -8.0f - (float)zo, hi = 7.0f - (float)zo;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        t[i] = v[i] * mult;
        const float c = __builtin_amdgcn_fmed3f(t[i], lo, hi);
        const float r = c + kMagic;                 // fp32 add rounds to an integer, ties to even
        bits[i] = __float_as_uint(r) + (uint32_t)zo;   // the offset enters after the rounding (integer add)
        if constexpr (EXACT) {
            const float f = c - (r - kMagic);       // exact; |f| <= 0.5
            suspect |= (fabsf(f) > 0.5f - 0x1.0p-18f);
        }
    }
    if constexpr (EXACT) {
        // t carries two fp32 roundings (reciprocal and product), so a quotient within
        // ~1e-6 of k + 1/2 may have been rounded to the wrong side.  Decide those from
        // the sign of (k + 1/2) * step - x, which one fused multiply-add gives exactly.
        if (__builtin_amdgcn_ballot_w64(suspect) != 0) {   // wave-uniform: a real branch, taken rarely
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float c = __builtin_amdgcn_fmed3f(t[i], lo, hi);
                const float r = c + kMagic;
                const float f = c - (r - kMagic);
                if (fabsf(f) > 0.5f - 0x1.0p-18f) {
                    const float k = floorf(t[i]);
                    const float d = fmaf(k + 0.5f, step, -raw[i]);
                    const int ki = (int)k;
                    int q = (d > 0.0f ? ki : (d < 0.0f ? ki + 1 : ((ki & 1) ? ki + 1 : ki))) + zo;
                    q = q < -8 ? -8 : (q > 7 ? 7 : q);
                    bits[i] = 0x4B400008u + (uint32_t)q;
                }
            }
        }
    }
    uint32_t s = bits[7];
#pragma unroll
    for (int i = 6; i >= 0; --i) s = (s << 4) + bits[i];
    return (s - kMagicSum) ^ 0x88888888u;   // offset-binary nibbles -> two's complement
}

// The same codes for eight fp16 values as they were loaded, in half the instructions (34 against 65): the value times the
// reciprocal step is added to 200.5 + 2^-16 in one fused multiply-add, whose result has 16 fractional bits, clamped to the ends of the
// range, and its upper half is 0x4340 + 8 + floor(t + 1/2).  The sum is within 2^-17 + 2^-20 of the quotient's, so the floor is that of
// the exact quotient unless the lower half is 0, 1 or 2; then the group takes the path above.
__device__ __forceinline__ uint32_t quant_pack8_f16(const v4i raw, float mult, float step)
{
    constexpr float kMid = 200.5f + 0x1.0p-16f;
    typedef uint16_t v2u16 __attribute__((ext_vector_type(2)));
    float v[8];
    uint32_t bits[8];
    const __half2* h2 = reinterpret_cast<const __half2*>(&raw);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float2 f = __half22float2(h2[i]);
        v[2 * i] = f.x;
        v[2 * i + 1] = f.y;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) bits[i] = __float_as_uint(__builtin_amdgcn_fmed3f(fmaf(v[i], mult, kMid), kMid - 8.0f, kMid + 7.0f));
    uint32_t low[4], high[4];                              // values i and i + 4 in the halves
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        low[i] = __builtin_amdgcn_perm(bits[i + 4], bits[i], 0x05040100u);
        high[i] = __builtin_amdgcn_perm(bits[i + 4], bits[i], 0x07060302u);
    }
    v2u16 least = __builtin_bit_cast(v2u16, low[0]);
#pragma unroll
    for (int i = 1; i < 4; ++i) least = __builtin_elementwise_min(least, __builtin_bit_cast(v2u16, low[i]));
    least = __builtin_elementwise_min(least, (v2u16){3, 3});
    if (__builtin_amdgcn_ballot_w64(__builtin_bit_cast(uint32_t, least) != 0x00030003u) != 0) return quant_pack8<true>(v, v, mult, step);
    uint32_t s = high[3];
#pragma unroll
    for (int i = 2; i >= 0; --i) s = (s << 4) + high[i];
    return (s - 0x4340u * 0x1111u * 0x10001u) ^ 0x88888888u;
}

// 8-bit variant: codes in [-128, 127], one byte each.  The four even-channel bytes and the four
// odd-channel bytes of the thread's eight channels are returned as two dwords.
constexpr float kMagic8 = 12582912.0f;   // 1.5 * 2^23, bit pattern 0x4B400000: low byte = code

template <bool EXACT>
__device__ __forceinline__ void quant_bytes8(const float* v, const float* raw, float mult, float step, uint32_t& even4,
                                             uint32_t& odd4)
{
    float t[8];
    uint32_t bits[8];
    bool suspect = false;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        t[i] = v[i] * mult;
        const float c = __builtin_amdgcn_fmed3f(t[i], -128.0f, 127.0f);
        const float r = c + kMagic8;
        bits[i] = __float_as_uint(r);
        if constexpr (EXACT) {
            const float f = c - (r - kMagic8);
            suspect |= (fabsf(f) > 0.5f - 0x1.0p-14f);   // |t| <= 128: two roundings move t by < 2^-15
        }
    }
    if constexpr (EXACT) {
        if (__builtin_amdgcn_ballot_w64(suspect) != 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float c = __builtin_amdgcn_fmed3f(t[i], -128.0f, 127.0f);
                const float r = c + kMagic8;
                const float f = c - (r - kMagic8);
                if (fabsf(f) > 0.5f - 0x1.0p-14f) {
                    const float k = floorf(t[i]);
                    const float d = fmaf(k + 0.5f, step, -raw[i]);
                    const int ki = (int)k;
                    int q = d > 0.0f ? ki : (d < 0.0f ? ki + 1 : ((ki & 1) ? ki + 1 : ki));
                    q = q < -128 ? -128 : (q > 127 ? 127 : q);
                    bits[i] = 0x4B400000u + (uint32_t)q;
                }
            }
        }
    }
    // byte 0 of bits[i] is the code; gather bytes with v_perm_b32 (selector: 0-3 second operand, 4-7 first)
    even4 = __builtin_amdgcn_perm(bits[2], bits[0], 0x0c0c0400u) | __builtin_amdgcn_perm(bits[6], bits[4], 0x04000c0cu);
    odd4 = __builtin_amdgcn_perm(bits[3], bits[1], 0x0c0c0400u) | __builtin_amdgcn_perm(bits[7], bits[5], 0x04000c0cu);
}

// BITS = 0: no output.  BITS = 16: no quantizer, fp16 out (global memory only).
// BITS = 4: eight codes packed into dst_row[channel / 8].  BITS = 8: one byte per code; inside every
// group of 32 channels the 16 even channels come first, then the 16 odd ones (the order in which
// the matrix kernel consumes them), so a thread stores two dwords.
// A row of codes in global memory whose writer chooses how the dwords leave: STREAM = written through at once
// (non-temporal), else ordinary stores that wait in this XCD's L2.  The codes are read next by another launch,
// on every XCD, i.e. from the memory side in any case.  While all of a launch's codes fit the L2s, ordinary
// stores leave in one burst at the end of the kernel, and streaming them out during it is faster (canonical
// step of the five 2048-token linears with cold weights 415 -> 406 us); a larger output is evicted as the kernel
// goes anyway, and streaming costs 1 % (8192 tokens: 1419 -> 1434 us).  kStreamBelow is the sum of the eight L2s.
// (A compile-time choice: a run-time branch around every store cost the kernels 5 %.)
template <bool STREAM>
struct GlobalCodes {
    uint32_t* p;
};
constexpr int64_t kStreamBelow = 32ll << 20;

template <typename DST>
__device__ __forceinline__ void put_codes(DST dst_row, int64_t at, uint32_t w)
{
    if constexpr (std::is_same<DST, GlobalCodes<true>>::value) {
        __builtin_nontemporal_store(w, dst_row.p + at);
    } else if constexpr (std::is_same<DST, GlobalCodes<false>>::value) {
        dst_row.p[at] = w;
    } else {
        dst_row[at] = w;
    }
}

template <int BITS, bool EXACT, typename DST>
__device__ __forceinline__ void store_codes(const float* v, float mult, float step, DST dst_row, int64_t e0, int zo = 0)
{
    if constexpr (BITS == 0) {
        // nothing is stored: the caller took the values through its step provider
    } else if constexpr (BITS == 16) {
        // rotation only: the normalised values go out as fp16 (round to nearest even), 16 bytes
        v4i o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const __half2 h = __floats2half2_rn(v[2 * i] * mult, v[2 * i + 1] * mult);
            o[i] = *reinterpret_cast<const int*>(&h);
        }
        *reinterpret_cast<v4i*>(&dst_row[e0 >> 1]) = o;
    } else if constexpr (BITS == 4) {
        put_codes(dst_row, e0 >> 3, quant_pack8<EXACT>(v, v, mult, step, zo));
    } else {
        uint32_t ev, od;
        quant_bytes8<EXACT>(v, v, mult, step, ev, od);
        const int64_t d = (e0 >> 5) * 8 + ((e0 >> 3) & 3);
        put_codes(dst_row, d, ev);
        put_codes(dst_row, d + 4, od);
    }
}

// Rotate (block size 2^log2h, 0 = none), quantize and pack the channels [chunk0, chunk0 + 2048 G)
// of one row.  x_row points at the row's first channel; packed dwords go to dst_row[channel / 8]
// (global or LDS).  xch: LDS scratch of 2048 G floats, touched only when log2h > 9.  Must be
// called by all threads of the workgroup (it contains LDS barriers when log2h > 9): `tid` is
// the thread's index 0..255 inside the group of 256 that owns the chunk, and threads of other
// groups, or groups without a chunk, pass active = false and only take part in the barriers.
// LDS-only barrier: global loads that are still in flight stay in flight.
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

typedef __attribute__((address_space(3))) const v4i* lds_cv4_ptr;
typedef __attribute__((address_space(3))) uint32_t* lds_u32_ptr;
typedef __attribute__((address_space(3))) float* lds_f32_ptr;

// SRC: const __half* (global) or an LDS pointer to fp16; DST: uint32_t* (global) or
// lds_u32_ptr.  Explicit LDS pointers keep the accesses off the vector-memory counter.
//
// load_chunk only issues the loads (branch-free: threads without data read the row's first
// bytes), so a caller can have several chunks in flight before the arithmetic starts.
template <int G, typename SRC>
__device__ __forceinline__ void load_chunk(SRC x_row, int64_t K, int64_t chunk0, int tid, bool active, v4i (&raw)[G],
                                           bool (&live)[G])
{
    using src_v4 = std::conditional_t<std::is_same<SRC, const __half*>::value, const v4i*, lds_cv4_ptr>;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int64_t e0 = chunk0 + (int64_t)g * kChunk + tid * 8;
        live[g] = active && e0 < K;
        // (activations in global memory are read once: non-temporal, they leave the caches to what is read again)
        if constexpr (std::is_same<SRC, const __half*>::value)
            raw[g] = __builtin_nontemporal_load((src_v4)(x_row + (live[g] ? e0 : 0)));
        else
            raw[g] = *(src_v4)(x_row + (live[g] ? e0 : 0));
    }
}

// The step of a per-tensor static quantizer: known before the rotation, the same everywhere.
struct StaticStep {
    static constexpr bool kMagnitudes = true;
    float mult, step;
    template <int NV>
    __device__ __forceinline__ void prepare(const float (&)[NV]) {}
    __device__ __forceinline__ void get(int64_t, float& m, float& s) const { m = mult; s = step; }
    __device__ __forceinline__ int zero_offset() const { return 0; }
};

// Per-tensor static step with a zero-point (Eq. 1 in its general form): zo = zero-point - 8.
struct StaticStepZp {
    static constexpr bool kMagnitudes = true;
    float mult, step;
    int zo;
    template <int NV>
    __device__ __forceinline__ void prepare(const float (&)[NV]) {}
    __device__ __forceinline__ void get(int64_t, float& m, float& s) const { m = mult; s = step; }
    __device__ __forceinline__ int zero_offset() const { return zo; }
};

// Per-head static steps (one per block of 2^log2d consecutive channels), read from device memory;
// the reciprocal carries the 1/sqrt(h) of the rotation.
struct HeadStep {
    static constexpr bool kMagnitudes = true;
    const float* scales;
    int log2d;
    double inv_sqrt_h;
    template <int NV>
    __device__ __forceinline__ void prepare(const float (&)[NV]) {}
    __device__ __forceinline__ void get(int64_t e0, float& m, float& s) const
    {
        s = scales[e0 >> log2d];
        m = (float)(inv_sqrt_h / (double)s);
    }
    __device__ __forceinline__ int zero_offset() const { return 0; }
};

// A step provider has `prepare(values)`, called once after the rotation by every thread of the
// workgroup with its G * 8 rotated (unnormalised) values (a dynamic quantizer derives its step
// there and may synchronise the workgroup; kMagnitudes: it takes their magnitudes alone, so their signs need not be right yet), and `get(channel, mult, step)`, called per group of 8
// channels, which sets the quantizer's reciprocal step and step for that group.
//
// An input transform `xf.apply(g, values)` may rewrite the 8 fp32 values of group g right after
// they are converted from fp16 (before the rotation): the identity for a plain input, or the
// fusion of an elementwise producer (see SiluGate).
struct NoTransform {
    __device__ __forceinline__ void apply(int, float (&)[8]) const {}
};

// Producer fusion for down_proj: the layer input is silu(gate) * up, elementwise.  The values
// passed in are the gate's; the matching 16 bytes of `up` were loaded by the caller.
struct SiluGate {
    const v4i* up_raw;   // G loaded groups of the calling thread
    __device__ __forceinline__ void apply(int g, float (&v)[8]) const
    {
        const v4i u = up_raw[g];
        const __half2* h2 = reinterpret_cast<const __half2*>(&u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float2 f = __half22float2(h2[i]);
            // hardware exp2 and reciprocal (about 1 ulp each): far inside the quantizer's tie tolerance
            v[2 * i] = v[2 * i] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[2 * i])) * f.x;
            v[2 * i + 1] = v[2 * i + 1] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[2 * i + 1])) * f.y;
        }
    }
};

template <int G, bool EXACT, int BITS = 4, typename DST, typename STEPS, typename XF = NoTransform>
__device__ __forceinline__ void rotate_quant_regs_with(const v4i (&raw)[G], const bool (&live)[G], int64_t chunk0,
                                                       int log2h, STEPS steps, DST dst_row, lds_f32_ptr xch,
                                                       int tid, bool active, XF xf = XF{})
{
    float mult, step;
    const int lane = tid & 63;
    const int wave = tid >> 6;

    float v[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const v4i rg = live[g] ? raw[g] : (v4i){0, 0, 0, 0};
        const __half2* h2 = reinterpret_cast<const __half2*>(&rg);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float2 f = __half22float2(h2[i]);
            v[g][2 * i] = f.x;
            v[g][2 * i + 1] = f.y;
        }
        xf.apply(g, v[g]);
    }

    if constexpr (EXACT) {
        // no rotation: the unrotated value doubles as the exact tie-break operand
        steps.prepare(reinterpret_cast<float(&)[G * 8]>(v));
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (live[g]) {
                const int64_t e0 = chunk0 + (int64_t)g * kChunk + tid * 8;
                steps.get(e0, mult, step);
                store_codes<BITS, true>(v[g], mult, step, dst_row, e0, steps.zero_offset());
            }
        }
    } else {
        constexpr bool SIGNED = BITS == 16 || !STEPS::kMagnitudes;
#pragma unroll
        for (int g = 0; g < G; ++g) reg_stages8(v[g], log2h < 3 ? log2h : 3);
        float(&flat)[G * 8] = reinterpret_cast<float(&)[G * 8]>(v);
        if (log2h > 3) lane_stage<0, SIGNED>(flat, lane);
        if (log2h > 4) lane_stage<1, SIGNED>(flat, lane);
        if (log2h > 5) lane_stage<2, SIGNED>(flat, lane);
        if (log2h > 6) lane_stage<3, SIGNED>(flat, lane);
        if (log2h > 7) lane_stage<4, SIGNED>(flat, lane);
        if (log2h > 8) lane_stage<5, SIGNED>(flat, lane);
        if (log2h > 9) {
            // radix-4 (or radix-2 when h == 1024) exchange between the 4 wavefronts
            if (active) {
#pragma unroll
                for (int i = 0; i < G * 8; ++i) xch[(wave * G * 8 + i) * 64 + lane] = flat[i];
            }
            lds_sync();
            const bool two = log2h > 10;
            if (active) {
#pragma unroll
            for (int i = 0; i < G * 8; ++i) {
                const float a = xch[((wave ^ 1) * G * 8 + i) * 64 + lane];
                float r = (wave & 1) ? (a - flat[i]) : (a + flat[i]);
                if (two) {
                    const float b = xch[((wave ^ 2) * G * 8 + i) * 64 + lane];
                    const float c = xch[((wave ^ 3) * G * 8 + i) * 64 + lane];
                    const float rp = (wave & 1) ? (c - b) : (c + b);   // same stage-1 result in the partner pair
                    r = (wave & 2) ? (rp - r) : (rp + r);
                }
                flat[i] = r;
            }
            }
            lds_sync();   // the scratch may be reused by the next call
        }
        if constexpr (G > 1) {
            // d = 2048 * 2^j between groups
#pragma unroll
            for (int dg = 1; dg < G; dg <<= 1) {
                if (log2h > 11 + __builtin_ctz(dg)) {
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if ((g & dg) == 0) {
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const float a = v[g][i], b = v[g + dg][i];
                                v[g][i] = a + b;
                                v[g + dg][i] = a - b;
                            }
                        }
                    }
                }
            }
        }
        const float sign = SIGNED ? 1.0f : lane_sign(lane, log2h < 3 ? 0 : (log2h < 9 ? log2h - 3 : 6));
        steps.prepare(flat);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (live[g]) {
                const int64_t e0 = chunk0 + (int64_t)g * kChunk + tid * 8;
                steps.get(e0, mult, step);
                if constexpr (!SIGNED) mult *= sign;
                store_codes<BITS, false>(v[g], mult, step, dst_row, e0, steps.zero_offset());
            }
        }
    }
}

template <int G, bool EXACT, int BITS = 4, typename DST>
__device__ __forceinline__ void rotate_quant_regs(const v4i (&raw)[G], const bool (&live)[G], int64_t chunk0,
                                                  int log2h, float mult, float step, DST dst_row, lds_f32_ptr xch,
                                                  int tid, bool active)
{
    rotate_quant_regs_with<G, EXACT, BITS>(raw, live, chunk0, log2h, StaticStep{mult, step}, dst_row, xch, tid, active);
}

template <int G, bool EXACT, typename SRC, typename DST>
__device__ __forceinline__ void rotate_quant_chunk(SRC x_row, int64_t K, int64_t chunk0, int log2h, float mult,
                                                   float step, DST dst_row, lds_f32_ptr xch, int tid, bool active)
{
    v4i raw[G];
    bool live[G];
    load_chunk<G>(x_row, K, chunk0, tid, active, raw, live);
    rotate_quant_regs<G, EXACT>(raw, live, chunk0, log2h, mult, step, dst_row, xch, tid, active);
}

// ---- rotation blocks of 4096 channels on the matrix pipe: H_4096 = H_32 x H_128.  The 32 blocks of 128 channels are the
// columns of a product with H_128, the five outer stages are fp32 butterflies between the lanes that hold the columns.
// Every kernel that makes static 4-bit codes of such blocks calls this function, so a token has the same codes in
// whichever call, form and batch it arrives (with sums in another order a code can differ at a rounding tie).
constexpr int kXPitch = 272;      // LDS row of 128 fp16 + 16 bytes: the 16-byte operand reads of 32 rows spread over all banks
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// The output channels 32 n .. 32 n + 31 of all 32 blocks of 128, by one wavefront (n: uniform, 0..3).  stg: LDS, the fp16
// input, one row of kXPitch bytes per block.  Lane l returns the codes of block l % 32, channels 32 n + 16 (l / 32) + 0..15:
// two dwords of eight.
// (rotate4096_values leaves the sums times lane_sign(l, 5): lane l ends with block l % 32, channels 32 n + 8 (i / 4) + 4 (l / 32) + i % 4 in v[i])
__device__ __forceinline__ void rotate4096_values(const uint8_t* stg, int n, int lane, float (&v)[16])
{
    // The H operand needs no memory: the sign is the parity of popcount(i & j), j = 32 n + l % 32, i = 16 s + 8 (l / 32) + 0..7
    const int j = lane & 31, g = lane >> 5;
    uint32_t hreg[2][4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t lo = __builtin_popcount((2 * d) & j & 7) & 1, hi = __builtin_popcount((2 * d + 1) & j & 7) & 1;
        const uint32_t base = 0x3C003C00u ^ (lo << 15) ^ (hi << 31);
        const uint32_t f0 = (uint32_t)(g & (j >> 3)) & 1u, f1 = f0 ^ ((uint32_t)(j >> 4) & 1u);
        hreg[0][d] = base ^ (f0 * 0x80008000u);
        hreg[1][d] = base ^ (f1 * 0x80008000u);
    }
    // blocks x H_128: lane l ends with block l % 32, channels 32 n + 8 (v / 4) + 4 (l / 32) + v % 4
    v16f acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const v4i xi = *(lds_cv4_ptr)(stg + j * kXPitch + 32 * s + 16 * g);
        const uint32_t flip = (__builtin_popcount((s >> 1) & n) & 1) ? 0x80008000u : 0u;      // wavefront-uniform
        const v4i hi4 = {(int)(hreg[s & 1][0] ^ flip), (int)(hreg[s & 1][1] ^ flip), (int)(hreg[s & 1][2] ^ flip), (int)(hreg[s & 1][3] ^ flip)};
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, hi4), __builtin_bit_cast(v8h, xi), acc, 0, 0, 0);
    }
    // the outer stages: between blocks, i.e. between lanes
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = fmaf(lane_xor<0>(acc[i]), lane & 1 ? -1.0f : 1.0f, acc[i]);      // (lane_stage<0>, with the compiler's waits for acc)
    lane_stage<1>(v, lane);
    lane_stage<2>(v, lane);
    lane_stage<3>(v, lane);
    lane_stage<4>(v, lane);
}

// The codes of those sums; the half-wavefronts trade so that a lane has 16 consecutive channels.
__device__ __forceinline__ void rotate4096_codes(const float (&v)[16], int lane, float mult, float step, int zero_offset, uint32_t (&codes)[2])
{
    mult *= lane_sign(lane, 5);
    const uint32_t w01 = quant_pack8<false>(v, v, mult, step, zero_offset);
    const uint32_t w23 = quant_pack8<false>(v + 8, v + 8, mult, step, zero_offset);
    const auto sw = __builtin_amdgcn_permlane32_swap(w01, w23, false, false);
    const uint32_t mine = sw[0], theirs = sw[1];
    codes[0] = __builtin_amdgcn_perm(theirs, mine, 0x05040100u);
    codes[1] = __builtin_amdgcn_perm(theirs, mine, 0x07060302u);
}

template <typename STEPS>
__device__ __forceinline__ void rotate4096_quarter(const uint8_t* stg, int n, int lane, const STEPS& steps, uint32_t (&codes)[2])
{
    float v[16];
    rotate4096_values(stg, n, lane, v);
    rotate4096_codes(v, lane, steps.mult, steps.step, steps.zero_offset(), codes);
}

}  // namespace rq
}  // namespace pq
