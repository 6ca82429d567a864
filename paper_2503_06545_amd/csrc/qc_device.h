// Device helpers shared by the quantization and the GEMM translation units: groups of 128 columns of an
// activation row, the quantizer's exact quotient and cast, the epilogue's activations.
#pragma once

#include "qc_internal.h"

namespace qc {
namespace {

constexpr int kUnit = 16;  // elements handled as one unit: 16 codes = one 16 B store

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

template <bool NT>
__device__ inline uint4 load16(const void *p) {
    if constexpr (NT) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
        return make_uint4(v.x, v.y, v.z, v.w);
    } else {
        return *reinterpret_cast<const uint4 *>(p);
    }
}

template <bool NT>
__device__ inline void store16(void *p, const uint4 &v) {
    if constexpr (NT) __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(p));
    else *reinterpret_cast<uint4 *>(p) = v;
}

__device__ inline float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// Eight lanes' share of 128 consecutive columns of a row: 16 elements per lane.  Every load
// instruction covers whole 128 B lines (8 lanes x 16 B, consecutive), so a lane's elements are pieces
// of 16 B that lie 128 B apart: bf16 columns 64 j + 8 sub .. + 7 (j = 0, 1), binary32 columns
// 32 j + 4 sub .. + 3 (j = 0 .. 3), sub the lane's index among the eight.  (With 16 consecutive
// elements per lane instead, every load instruction touches each line in part, which costs 32 % of
// the time once the loads are non-temporal: binary32 16384 x 4608, 102 against 70 us.)
//   load()         columns col0 .. of a row of K (a multiple of 16); past its end the row's last piece
//                  is read again, which changes no maximum or minimum and is not stored
//   get(i)         element i of the lane, i = 0 .. 15 in that order, widened to float
//   gather_codes() turns dwords of four codes each, in that order, into the 16 codes of one unit of
//                  16 consecutive columns; lane sub gets unit unit_of(sub) of the eight.
//   absmax_into()  folds the elements' magnitudes into a running maximum, absmax_value() reads it; a NaN
//                  is passed over, like by fmaxf, so that it spoils no code but its own.
//                  For bf16 it stays two packed 16-bit patterns (Bf16Max): nothing is widened that the
//                  compiler would then keep in registers up to the cast.
//   load_ragged()  the same for a K that is no multiple of 16 (16 B or more): rows at any alignment (the hardware
//                  takes 16 B loads at any address).  The piece that holds the row's end is loaded so that it ends
//                  there, and settle_ragged(), after all loads, moves it down to its place, zeros following; pieces wholly past
//                  the end stay copies of the last one, as with load().
//                  (Its elements loaded one by one, each load waited for, in order: us 4099 x 1000 bf16 4.7 4.4, 30000 x 1156 bf16
//                  23.3 18.5, f32 39.7 30.4.)
template <typename XT>
struct Group;

// The largest magnitude of bf16 patterns, two at a time.  A pattern doubled is its magnitude without the
// sign, and magnitudes order like their patterns; 0xff more and infinity is the largest number of 16 bits,
// while every NaN wraps round to less than a zero's 0xff and loses to anything.  One v_pk_mad_u16 and one
// v_pk_max_u16 for two elements.
struct Bf16Max {
    u16x2 m = {0xff, 0xff};
    __device__ void fold(uint32_t two_patterns) {
        u16x2 twice = {2, 2};
        asm("" : "+s"(twice));   // a constant the compiler does not see: it would make two instructions of it, a shift and an add
        m = __builtin_elementwise_max(m, (u16x2)(__builtin_bit_cast(u16x2, two_patterns) * twice + u16x2{0xff, 0xff}));
    }
    __device__ float value() const { return __uint_as_float((uint32_t)(((m.x > m.y ? m.x : m.y) - 0xff) >> 1) << 16); }
};

typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));   // 16 B at any element

// a piece moved down by 1 .. 7 halfwords, zeros from above
__device__ inline uint4 move_down(uint4 v, int halfwords) {
    if (halfwords & 4) v = make_uint4(v.z, v.w, 0, 0);
    if (halfwords & 2) v = make_uint4(v.y, v.z, v.w, 0);
    if (halfwords & 1) v = make_uint4(v.x >> 16 | v.y << 16, v.y >> 16 | v.z << 16, v.z >> 16 | v.w << 16, v.w >> 16);
    return v;
}

template <int CTRL>
__device__ inline float dpp_max(float v) {
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false)));
}
template <int CTRL>
__device__ inline float dpp_min(float v) {
    return fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false)));
}
__device__ inline float min_of_eight(float v) { return dpp_min<0x141>(dpp_min<0x4E>(dpp_min<0xB1>(v))); }
// the maximum of eight consecutive lanes, in each of them (quad_perm [1, 0, 3, 2], [2, 3, 0, 1], row_half_mirror)
__device__ inline float max_of_eight(float v) { return dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(v))); }

// the dword of lane ^ 1 (quad_perm [1, 0, 3, 2])
__device__ inline uint32_t dpp_xor1(uint32_t v) { return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false); }
// the dword of lane ^ 2 (quad_perm [2, 3, 0, 1])
__device__ inline uint32_t dpp_xor2(uint32_t v) { return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false); }

template <>
struct Group<float> {
    uint4 v[4];
    template <bool NT>
    __device__ void load(const float *xrow, int col0, int K, int sub) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = col0 + 32 * j + 4 * sub;
            v[j] = load16<NT>(xrow + (col < K - 4 ? col : K - 4));
        }
    }
    __device__ void load_ragged(const float *xrow, int col0, int K, int sub) {
        const int most = K - 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = col0 + 32 * j + 4 * sub;
            const u32x4_any t = *reinterpret_cast<const u32x4_any *>(xrow + (col < most ? col : most));
            v[j] = make_uint4(t.x, t.y, t.z, t.w);
        }
    }
    __device__ void settle_ragged(int col0, int K, int sub) {
        const int most = K - 4;
        if (col0 + 128 > K) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int past = col0 + 32 * j + 4 * sub - most;   // elements of the piece past the row's end
                if (past > 0 && past < 4) v[j] = move_down(v[j], 2 * past);
            }
        }
    }
    __device__ float get(int i) const {
        const uint4 &f = v[i >> 2];
        switch (i & 3) {
            case 0: return __uint_as_float(f.x);
            case 1: return __uint_as_float(f.y);
            case 2: return __uint_as_float(f.z);
            default: return __uint_as_float(f.w);
        }
    }
    static __device__ int unit_of(int sub) { return 2 * (sub & 3) + (sub >> 2); }
    // dword j of the four lanes of a quad belongs to one unit: a 4 x 4 transpose inside the quad
    static __device__ uint4 gather_codes(const uint32_t (&w)[4], int sub) {
        const bool odd = sub & 1, high = sub & 2;
        // swap across lane ^ 1: afterwards a[2 p + o] holds dwords of columns j with j % 2 == own parity
        const uint32_t s0 = dpp_xor1(odd ? w[0] : w[1]), s1 = dpp_xor1(odd ? w[2] : w[3]);
        const uint32_t a0 = odd ? s0 : w[0], a1 = odd ? w[1] : s0;   // lanes (even, odd) of the pair, dword own parity
        const uint32_t b0 = odd ? s1 : w[2], b1 = odd ? w[3] : s1;   // the same for dword 2 + own parity
        const uint32_t t0 = dpp_xor2(high ? a0 : b0), t1 = dpp_xor2(high ? a1 : b1);
        return high ? make_uint4(t0, t1, b0, b1) : make_uint4(a0, a1, t0, t1);
    }
    typedef float Max;
    __device__ void absmax_into(Max &m) const {
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(get(i)));
    }
    static __device__ Max no_max() { return 0.0f; }
    static __device__ float absmax_value(Max m) { return m; }
};

template <>
struct Group<uint16_t> {  // bf16 bit patterns
    uint4 v[2];
    template <bool NT>
    __device__ void load(const uint16_t *xrow, int col0, int K, int sub) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = col0 + 64 * j + 8 * sub;
            v[j] = load16<NT>(xrow + (col < K - 8 ? col : K - 8));
        }
    }
    __device__ void load_ragged(const uint16_t *xrow, int col0, int K, int sub) {
        const int most = K - 8;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = col0 + 64 * j + 8 * sub;
            const u32x4_any t = *reinterpret_cast<const u32x4_any *>(xrow + (col < most ? col : most));
            v[j] = make_uint4(t.x, t.y, t.z, t.w);
        }
    }
    __device__ void settle_ragged(int col0, int K, int sub) {
        const int most = K - 8;
        if (col0 + 128 > K) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int past = col0 + 64 * j + 8 * sub - most;
                if (past > 0 && past < 8) v[j] = move_down(v[j], past);
            }
        }
    }
    __device__ float get(int i) const {
        const uint4 &u = v[i >> 3];
        uint32_t w;
        switch ((i >> 1) & 3) { case 0: w = u.x; break; case 1: w = u.y; break; case 2: w = u.z; break; default: w = u.w; }
        return (i & 1) ? bf16_hi(w) : bf16_lo(w);
    }
    static __device__ int unit_of(int sub) { return (sub >> 1) + 4 * (sub & 1); }
    static __device__ uint4 gather_codes(const uint32_t (&w)[4], int sub) {
        const bool odd = sub & 1;
        const uint32_t s0 = dpp_xor1(odd ? w[0] : w[2]), s1 = dpp_xor1(odd ? w[1] : w[3]);
        return odd ? make_uint4(s0, s1, w[2], w[3]) : make_uint4(w[0], w[1], s0, s1);
    }
    typedef Bf16Max Max;
    __device__ void absmax_into(Max &m) const {
        const uint32_t w[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
        for (int i = 0; i < 8; ++i) m.fold(w[i]);
    }
    static __device__ Max no_max() { return {}; }
    static __device__ float absmax_value(const Max &m) { return m.value(); }
};

// RN(x / s) from r = RN(1 / s): product, exact residual, one correction.
__device__ inline float quotient(float x, float s, float r) {
    const float q = x * r;
    return fmaf(fmaf(-s, q, x), r, q);
}

// Four quotients of the symmetric quantizer -> four int8 codes in one dword.  No clamp: with s =
// RN(a / qmax) and |x| <= a the quotient is at most qmax (1 + 2^-22), which rounds to qmax.  Adding
// 1.5 * 2^23 rounds to an integer (ties to even) and leaves its two's complement low byte in the
// low byte of the float.  A NaN gets some byte as its code.
__device__ inline uint32_t codes4(float q0, float q1, float q2, float q3) {
    const float magic = 12582912.0f;
    const uint32_t y0 = __float_as_uint(q0 + magic), y1 = __float_as_uint(q1 + magic);
    const uint32_t y2 = __float_as_uint(q2 + magic), y3 = __float_as_uint(q3 + magic);
    const uint32_t lo = __builtin_amdgcn_perm(y1, y0, 0x0c0c0400u);  // [y0.b0, y1.b0, 0, 0]
    const uint32_t hi = __builtin_amdgcn_perm(y3, y2, 0x04000c0cu);  // [0, 0, y2.b0, y3.b0]
    return lo | hi;
}

__device__ inline float scale_of(float absmax, float qmax) { return fmaxf(absmax, kAbsmaxFloor) / qmax; }

// Four quotients of the asymmetric quantizer -> four bytes in one dword: clamp(rne(q) + off, cmin, cmax).
__device__ inline uint32_t asym_codes4(float q0, float q1, float q2, float q3, float off, float cmin, float cmax) {
    const float magic = 12582912.0f;  // 1.5 * 2^23: the sum's low byte is the integer's low byte
    const float q[4] = {q0, q1, q2, q3};
    uint32_t y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = __float_as_uint(__builtin_amdgcn_fmed3f(rintf(q[e]) + off, cmin, cmax) + magic);
    return __builtin_amdgcn_perm(y[1], y[0], 0x0c0c0400u) | __builtin_amdgcn_perm(y[3], y[2], 0x04000c0cu);
}

// ---- rotation of a group of 128 columns (Section 3.2 AIGQ (1)) ------------------------------------
// Each block of `rot` consecutive columns (16, 32, 64 or 128) is multiplied by the Walsh-Hadamard
// matrix of that size before the absmax and the cast, as a butterfly network in binary32 with
// the strides in ascending order: one rounding per output and stage, so the bits do not depend
// on which lane does which butterfly.  The rows are loaded as in quant_rows_kernel, whole lines per
// instruction, so a group of 128 columns lies over eight lanes in pieces of E = 16 B: the strides below
// E and those of 8 E or more are butterflies between a lane's own values, the three between them pair
// lanes.
//
// A butterfly across lanes is one v_fmac_f32 with a DPP operand: own + sign * other.  It leaves the
// upper lane of a pair with minus its output, which every later stage carries along unchanged; the
// quotient takes the sign out again, because x / s and (-x) / (-s) are the same operations on the same
// magnitudes.  DPP reaches lanes sub ^ 1, ^ 2 and ^ 7 in one move, not ^ 4; so the lane takes the piece
// `label` of the eight, which differs in bit 2 alone between lanes sub and sub ^ 7.
// 65536 x 1152 bf16, blocks of 128, with a move and an fma (two moves for the third stage) and 16
// consecutive columns a lane: 52.7 us; this form 38.3 (binary32 72.1 and 60.0).
// (One asm block per stage: the compiler leaves the DPP move and the fma apart.  A DPP operand may be read two
// wait states after a VALU instruction has written it, hence the s_nop; inside the block no
// instruction reads what another has written.)
#define QC_BUTTERFLY(i, how) "v_fmac_f32_dpp %" #i ", %" #i ", %16 " how " row_mask:0xf bank_mask:0xf\n\t"
#define QC_BUTTERFLIES(f, sign, how)                                                                          \
    asm volatile("s_nop 1\n\t"                                                                               \
        QC_BUTTERFLY(0, how) QC_BUTTERFLY(1, how) QC_BUTTERFLY(2, how) QC_BUTTERFLY(3, how)                   \
        QC_BUTTERFLY(4, how) QC_BUTTERFLY(5, how) QC_BUTTERFLY(6, how) QC_BUTTERFLY(7, how)                   \
        QC_BUTTERFLY(8, how) QC_BUTTERFLY(9, how) QC_BUTTERFLY(10, how) QC_BUTTERFLY(11, how)                 \
        QC_BUTTERFLY(12, how) QC_BUTTERFLY(13, how) QC_BUTTERFLY(14, how) QC_BUTTERFLY(15, how)               \
        : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]), "+v"(f[6]), "+v"(f[7]),     \
          "+v"(f[8]), "+v"(f[9]), "+v"(f[10]), "+v"(f[11]), "+v"(f[12]), "+v"(f[13]), "+v"(f[14]), "+v"(f[15]) \
        : "v"(sign))
static_assert(kUnit == 16, "a stage's elements are written out");
__device__ inline void butterflies_xor1(float (&f)[kUnit], float sign) { QC_BUTTERFLIES(f, sign, "quad_perm:[1,0,3,2]"); }
__device__ inline void butterflies_xor2(float (&f)[kUnit], float sign) { QC_BUTTERFLIES(f, sign, "quad_perm:[2,3,0,1]"); }
__device__ inline void butterflies_xor7(float (&f)[kUnit], float sign) { QC_BUTTERFLIES(f, sign, "row_half_mirror"); }
#undef QC_BUTTERFLIES
#undef QC_BUTTERFLY

// Lane sub's piece of the eight, which the rotated forms use in the place of sub.
__device__ inline int rotation_label(int sub) { return sub < 4 ? sub : sub ^ 3; }

template <typename XT>
struct Rotation {
    static constexpr int E = 16 / (int)sizeof(XT);   // consecutive columns of a lane's pieces
    int rot, label;
    float sg1, sg2, sg4;
    __device__ Rotation(int rot_, int label_)
        : rot(rot_), label(label_), sg1(label_ & 1 ? -1.0f : 1.0f), sg2(label_ & 2 ? -1.0f : 1.0f), sg4(label_ & 4 ? -1.0f : 1.0f) {}
    static __device__ void own_lane(float (&f)[kUnit], int h) {   // butterflies between elements h apart
#pragma unroll
        for (int j = 0; j < kUnit; ++j)
            if ((j & h) == 0) {
                const float lo = f[j], hi = f[j + h];
                f[j] = lo + hi;
                f[j + h] = lo - hi;
            }
    }
    // f: the group's columns col0 .. of a row of K, widened.  Columns past the row's end, whole blocks of them, are
    // not the row's last piece again, as loaded, but zeros.
    __device__ void apply(float (&f)[kUnit], int col0, int K) const {
        if (col0 + 128 > K) {
#pragma unroll
            for (int e = 0; e < kUnit; ++e)
                if (col0 + e / E * (8 * E) + E * label >= K) f[e] = 0.0f;
        }
        own_lane(f, 1);
        own_lane(f, 2);
        if constexpr (E == 8) {   // strides 1 2 4 | 8 16 32 | 64
            own_lane(f, 4);
            butterflies_xor1(f, sg1);
            if (rot >= 32) butterflies_xor2(f, sg2);
            if (rot >= 64) butterflies_xor7(f, sg4);
            if (rot >= 128) own_lane(f, 8);
        } else {                  // strides 1 2 | 4 8 16 | 32 64
            butterflies_xor1(f, sg1);
            butterflies_xor2(f, sg2);
            if (rot >= 32) butterflies_xor7(f, sg4);
            if (rot >= 64) own_lane(f, 4);
            if (rot >= 128) own_lane(f, 8);
        }
    }
    // minus for the lanes that an odd number of the stages across lanes has negated
    __device__ float sign() const {
        float sign = sg1;
        if (rot >= 32 || E == 4) sign *= sg2;
        if (rot >= (E == 8 ? 64 : 32)) sign *= sg4;
        return sign;
    }
};

__device__ inline float gelu_tanh_f(float y) {
    // 0.5 y (1 + tanh(u)) = y / (1 + exp(-2u)),  u = sqrt(2/pi) (y + 0.044715 y^3)
    const float c1 = -2.0f * 0.7978845608028654f * 1.4426950408889634f;  // -2 sqrt(2/pi) log2(e)
    const float c2 = c1 * 0.044715f;
    const float t = y * fmaf(c2, y * y, c1);
    return y * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

// 0.5 y (1 + erf(y / sqrt 2)) with erfc(x) = t (a1 + t (a2 + .. a5 t)) exp(-x^2), t = 1 / (1 + p x)
// for x >= 0 (Abramowitz and Stegun 7.1.26, absolute error below 1.5e-7) and erf odd.  For
// negative y the product form keeps the small result's relative accuracy.  Far fewer registers
// than the math library's erff, which matters next to 128 live accumulators.
__device__ inline float gelu_erf_f(float y) {
    const float x = fabsf(y) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
    float p = fmaf(1.061405429f, t, -1.453152027f);
    p = fmaf(p, t, 1.421413741f);
    p = fmaf(p, t, -0.284496736f);
    p = fmaf(p, t, 0.254829592f);
    const float q = p * t * __builtin_amdgcn_exp2f(x * x * -1.4426950408889634f);  // erfc(x)
    const float gate = y >= 0.0f ? 2.0f - q : q;
    return 0.5f * y * gate;
}

// two floats -> two bf16 (round to nearest even), one v_cvt_pk_bf16_f32
__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
    typedef float f2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
    const f2v v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf2v));
}

}  // namespace
}  // namespace qc
