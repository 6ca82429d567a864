// Integer GEMM with fused dequantize / bias / GELU epilogue (Section 4.1 "Hardware
// Implementation": the DiT linears as low-bit GEMMs with quantization fused around them).
//
//   acc[m, n] = sum_k qx[m, k] * qw[n, k]          exact, int32, v_mfma_i32_16x16x64_i8
//   Y[m, n]   = act(acc * sx[m] * sw[n] + bias[n])
//
// Two kernels share the wavefront tile, the operand formats and the epilogue: gemm_kernel
// streams its weight tile through a ring in LDS and takes any K (gemm_mid_kernel and gemm_half_kernel the
// same with tiles of 192 and 128 tokens); gemm_resident_kernel (further down) keeps a whole weight tile in LDS and is taken for short reductions on large problems.
//
// gemm_kernel: block tile 256 tokens x 128 channels, 4 wavefronts stacked along the tokens, each
// 64 x 128 = 4 x 8 MFMA tiles (128 accumulator registers), two blocks per CU so that one
// block's epilogue overlaps the other's MFMA loop.  Operands arrive pre-arranged as 1 KiB
// MFMA fragments (see qc_internal.h).  The weight tile, which all four wavefronts use, goes
// HBM -> LDS by linear direct-to-LDS copies through a 3-deep ring of 64-k stages and is read
// back 16 B/lane, conflict free; the activation fragments are private to a wavefront and go
// HBM -> registers directly (LDS writes are the scarce resource: about 64 B/clk/CU against
// 256 B/clk/CU for reads).  Inside a stage the weight reads of the second half of the channels
// are in flight under the MFMAs of the first half.  Tokens are the MFMA "A" operand (rows of the
// result tile, four per lane) and channels the "B" operand (columns = lanes); the weight row
// permutation makes a lane's eight tiles eight consecutive channels, so 16 lanes store 128
// consecutive channels of one token at a time.  The 16x16x64 form of the MFMA is used because
// the chip holds a higher clock on it than on the 32x32x32 form under its power cap (measured:
// 4.1 against 3.4 POP/s on random operands, registers only).  Whole tiles of bf16 and int32 output
// are written with non-temporal stores: the output is not read again by this kernel and would
// otherwise push the operand panels out of the L2.  Float output that the last-level cache can hold,
// partly filled tiles and rows that are no multiple of 16 B go through the caches (keep_f32_output(),
// stream_bf16_edges()).
#pragma once

#include <type_traits>

#include "qc_device.h"
#include "qc_gemm.h"

namespace qc {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256, kSplitThreads = 2 * kThreads;
constexpr int kStages = 3;   // both rings: weight stages in LDS (4 and 6 were measured: 1.5 % and 3 % slower) and
                             // activation stages in registers.  The half-height tile gains nothing from 6
                             // either: alone on its CU a block waits for bandwidth, not for latency.

// LDS in front of the scales: the ring, or, split, two rings or what the groups exchange at a time
template <int BITS, bool SPLIT>
constexpr int kRingBytes = !SPLIT ? kStages * StageLayout<BITS>::kBytes
                           : 2 * kStages * StageLayout<BITS>::kBytes > kSplitThreads * 64 ? 2 * kStages * StageLayout<BITS>::kBytes : kSplitThreads * 64;

__device__ inline void lds_dma_16(const uint8_t *gsrc, uint8_t *lds_dst) {
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void *)gsrc,
        (__attribute__((address_space(3))) void *)lds_dst, 16, 0, 0);
}

// Map the launch's block index to a tile so that the blocks resident on one XCD at a time
// (block b runs on XCD b % 8) work on a compact 8 x 8 patch of tiles and share its operand
// panels through that XCD's L2.
__device__ inline void tile_of_block(int b, int nblocks, int m_tiles, int n_tiles, int group_m,
                                     int &mt, int &nt) {
    const int xcd = b % 8, slot = b / 8;
    const int per = nblocks / 8, extra = nblocks % 8;
    const int v = xcd * per + (xcd < extra ? xcd : extra) + slot;  // blocks of one XCD are consecutive
    const int kGroupM = group_m;
    const int per_group = kGroupM * n_tiles;
    const int g = v / per_group, r = v % per_group;
    const int m0 = g * kGroupM;
    const int gm = (m_tiles - m0) < kGroupM ? (m_tiles - m0) : kGroupM;
    mt = m0 + r % gm;
    nt = r / gm;
}

// vmcnt(n) with the other counters left unconstrained (gfx9 encoding: bits 3:0 and 15:14, n < 64)
#define QC_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// One piece of a row of Y.  ANY: at any alignment of its elements.  CACHED: not past the caches, where
// the pieces of a line that two tiles, two rows or two instructions share meet.
template <bool ANY, bool CACHED, typename T, typename V>
__device__ inline void store_piece(T *p, V v) {
    typedef V VAny __attribute__((aligned(2)));
    typedef std::conditional_t<ANY, VAny, V> P;
    if constexpr (CACHED) *reinterpret_cast<P *>(p) = v;
    else __builtin_nontemporal_store(v, reinterpret_cast<P *>(p));
}

// Epilogue of one wavefront's tile of 16 MI tokens x 128 channels: registers -> Y.  Lane (c = lane % 16, h = lane / 16)
// of MFMA tile (i, t) holds, in register r, token m_wave + 16 i + 4 h + r and channel
// 128 nt + 8 c + t.  sx64 / cx64: the tile's token scales / corrections, lds_sw / lds_bs /
// lds_rs: the channel tile's 128 scales, biases and code sums, all in LDS.  KEEP: interior tiles
// through the caches; a parameter of the kernel, because two copies of the straight-line path under a
// condition are merged by the compiler, which then drops the non-temporal hint of the one.
template <int BITS, int OUT, int EPI, bool ASYM, bool KEEP, int MI>
__device__ __forceinline__ void store_wave_tile(v4i (&acc)[MI][8], const GemmArgs &a, int64_t m_wave, int nt,
                                                int lane, const float *sx64, const float *cx64,
                                                const float *lds_sw, const float *lds_bs, const float *lds_rs) {
    const int c = lane & 15, h = lane >> 4;
    const int64_t n0 = (int64_t)nt * kTileN + 8 * c;
    const int64_t m0 = m_wave + 4 * h;
    constexpr int kOutBytes = OUT == QC_OUT_BF16 ? 2 : 4;
    constexpr int kVecChannels = 16 / kOutBytes;  // channels in one 16 B store
    const bool interior = m_wave + 16 * MI <= a.M && (int64_t)(nt + 1) * kTileN <= a.N &&
                          (a.N % kVecChannels) == 0;  // uniform over the wavefront
    char *const y_wave = reinterpret_cast<char *>(a.Y) + (m_wave * a.N + (int64_t)nt * kTileN) * kOutBytes;
    const uint32_t lane_off = (uint32_t)((4 * h * a.N + 8 * c) * kOutBytes);  // N <= 2^26

    auto write_tile = [&](auto checked_tag, auto cached_tag) {
        constexpr bool CHECKED = decltype(checked_tag)::value, CACHED = decltype(cached_tag)::value;
        if (CHECKED && n0 >= a.N) return;
        // Whole 16 B pieces are stored as such at any alignment, which the hardware takes; the 1 to 7 channels a lane
        // has left at the end of a row go out as four, two and one, each of them one store under a
        // mask made once.  Element by element under tests of their own, and so, us: 4291 x 208 x 1283 GELU (erf) 17.2 12.6,
        // 1113 x 1152 x 2819 W4 GELU 13.9 12.0, 3000 x 1152 x 1203 10.3 9.2, f32 65536 x 1152 x 1156 135 127.
        const int cols = CHECKED ? (int)(a.N - n0 < 8 ? a.N - n0 : 8) : 8;
        const int rows = CHECKED ? (int)(a.M - m0 < 16 * MI ? a.M - m0 : 16 * MI) : 16 * MI;
        const bool ragged = CHECKED && a.N % 8 && (int64_t)(nt + 1) * kTileN > a.N;   // uniform over the wavefront
        const bool four = cols & 4, two = cols & 2;

        float sw[8], bs[8], rs[8];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float4 s4 = *reinterpret_cast<const float4 *>(lds_sw + 8 * c + 4 * j);
            const float4 b4 = *reinterpret_cast<const float4 *>(lds_bs + 8 * c + 4 * j);
            sw[4 * j + 0] = s4.x; sw[4 * j + 1] = s4.y; sw[4 * j + 2] = s4.z; sw[4 * j + 3] = s4.w;
            bs[4 * j + 0] = b4.x; bs[4 * j + 1] = b4.y; bs[4 * j + 2] = b4.z; bs[4 * j + 3] = b4.w;
            if (ASYM) {
                const float4 r4 = *reinterpret_cast<const float4 *>(lds_rs + 8 * c + 4 * j);
                rs[4 * j + 0] = r4.x; rs[4 * j + 1] = r4.y; rs[4 * j + 2] = r4.z; rs[4 * j + 3] = r4.w;
            }
        }

#pragma unroll
        for (int i = 0; i < MI; ++i) {
            float sx[4] = {0.f, 0.f, 0.f, 0.f}, cx[4] = {0.f, 0.f, 0.f, 0.f};
            const float4 x4 = *reinterpret_cast<const float4 *>(sx64 + 16 * i + 4 * h);
            sx[0] = x4.x; sx[1] = x4.y; sx[2] = x4.z; sx[3] = x4.w;
            if (ASYM) {
                const float4 c4 = *reinterpret_cast<const float4 *>(cx64 + 16 * i + 4 * h);
                cx[0] = c4.x; cx[1] = c4.y; cx[2] = c4.z; cx[3] = c4.w;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (CHECKED && 16 * i + q >= rows) continue;
                char *const y_row = y_wave + (int64_t)(16 * i + q) * a.N * kOutBytes + lane_off;
                if (OUT == QC_OUT_BF16) {
                    uint32_t pk[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float v[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const int t = 2 * j + e;
                            float af = (float)acc[i][t][q];
                            if (ASYM) af = fmaf(cx[q], rs[t], af);
                            float y = fmaf(af * sx[q], sw[t], bs[t]);
                            if (EPI == QC_EPI_GELU_TANH) y = gelu_tanh_f(y);
                            else if (EPI == QC_EPI_GELU_ERF) y = gelu_erf_f(y);
                            v[e] = y;
                        }
                        pk[j] = pack_bf16x2(v[0], v[1]);
                    }
                    uint16_t *const y = reinterpret_cast<uint16_t *>(y_row);
                    if (cols == 8) store_piece<CHECKED, CACHED>(y, u4{pk[0], pk[1], pk[2], pk[3]});
                    if (ragged) {
                        if (cols < 8 && four) store_piece<true, CACHED>(y, u2{pk[0], pk[1]});
                        if (two) store_piece<true, CACHED>(y + (cols & 4), four ? pk[2] : pk[0]);
                        if (cols & 1) y[cols & 6] = (uint16_t)(four ? (two ? pk[3] : pk[2]) : (two ? pk[1] : pk[0]));
                    }
                } else {
                    float v[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        float af = (float)acc[i][t][q];
                        if (ASYM) af = fmaf(cx[q], rs[t], af);
                        float y = fmaf(af * sx[q], sw[t], bs[t]);
                        if (EPI == QC_EPI_GELU_TANH) y = gelu_tanh_f(y);
                        else if (EPI == QC_EPI_GELU_ERF) y = gelu_erf_f(y);
                        v[t] = y;
                    }
                    float *const y = reinterpret_cast<float *>(y_row);
                    if (cols >= 4) store_piece<CHECKED, CACHED>(y, f4{v[0], v[1], v[2], v[3]});
                    if (cols == 8) store_piece<CHECKED, CACHED>(y + 4, f4{v[4], v[5], v[6], v[7]});
                    if (ragged) {
                        if (two) store_piece<true, CACHED>(y + (cols & 4), four ? f2{v[4], v[5]} : f2{v[0], v[1]});
                        if (cols & 1) y[cols & 6] = four ? (two ? v[6] : v[4]) : (two ? v[2] : v[0]);
                    }
                }
            }
        }
    };
    // the raw accumulators (a test's output), in whole pieces or element by element
    auto write_raw = [&](auto checked_tag) {
        constexpr bool CHECKED = decltype(checked_tag)::value;
        if (CHECKED && n0 >= a.N) return;
        bool vec[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) vec[j] = !CHECKED || n0 + 4 * j + 4 <= a.N;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int64_t m4 = m0 + 16 * i;
            if (CHECKED && m4 >= a.M) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (CHECKED && m4 + q >= a.M) continue;
                int raw[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) raw[t] = BITS == 4 ? acc[i][t][q] >> 4 : acc[i][t][q];   // exact: multiples of 16
                int32_t *y = reinterpret_cast<int32_t *>(y_wave + (int64_t)(16 * i + q) * a.N * kOutBytes + lane_off);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if (vec[j]) {
                        store_piece<CHECKED, CHECKED>(y + 4 * j, v4i{raw[4 * j], raw[4 * j + 1], raw[4 * j + 2], raw[4 * j + 3]});
                    } else {
#pragma unroll
                        for (int t = 4 * j; t < 4 * j + 4; ++t) if (n0 + t < a.N) y[t] = raw[t];
                    }
                }
            }
        }
    };
    if constexpr (OUT == QC_OUT_I32_ACC) {
        if (interior) write_raw(std::false_type{});
        else write_raw(std::true_type{});
    } else {
        if (!interior && OUT == QC_OUT_BF16 && a.stream_edges) write_tile(std::true_type{}, std::bool_constant<OUT != QC_OUT_BF16>{});
        else if (!interior) write_tile(std::true_type{}, std::true_type{});
        else write_tile(std::false_type{}, std::bool_constant<KEEP>{});
    }
}

// ASYM: the activation codes are the unsigned codes of the asymmetric quantizer minus a shift h
// (128 for 8-bit codes, else 0; Section 3.1 Eq. (3)-(4) as printed).  With c[m] = h - z[m] the dequantized activation
// is sx (code + c), so the epilogue adds c[m] * sum_k qw[n, k] to the accumulator.
// SPLIT: eight wavefronts in two groups that each walk half of the reduction, with a ring of their own, and
// exchange sums at the end: see split_height().
template <int BITS, int OUT, int EPI, bool ASYM, bool KEEP, int MI, bool SPLIT = false>
__device__ __forceinline__ void ring_gemm(const GemmArgs &a) {
    using L = StageLayout<BITS>;
    constexpr int TM = 4 * 16 * MI;   // tokens of the block, 16 MI of them a wavefront's
    constexpr int FPW = L::kFragsPerWave;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

    const int lane = threadIdx.x & 63;
    const int wave_of_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = SPLIT ? wave_of_block & 3 : wave_of_block, group = SPLIT ? wave_of_block >> 2 : 0;
    int mt, nt;
    tile_of_block(blockIdx.x, gridDim.x, a.m_tiles, a.n_tiles, a.group_m, mt, nt);

    // this group's stages, in whole threes: the first group has three more if they do not come out even
    const int most = SPLIT ? 3 * ((a.KF / 3 + 1) / 2) : a.KF;
    const int stage0 = group ? most : 0, stages = group ? a.KF - most : most;
    uint8_t *const ring = lds + group * (kStages * L::kBytes);
    // The epilogue's scales and bias are fetched now (one value per thread) and handed round
    // through LDS after the main loop, so that the epilogue does not start with a chain of L2
    // round trips.
    float *lds_sx = reinterpret_cast<float *>(lds + kRingBytes<BITS, SPLIT>);  // TM token scales (room for 256)
    float *lds_sw = lds_sx + kTileM;                                       // 128 channel scales
    float *lds_bs = lds_sw + kTileN;                                       // 128 biases
    float *lds_cx = lds_bs + kTileN;                                       // ASYM: 256 corrections
    float *lds_rs = lds_cx + kTileM;                                       // ASYM: 128 code sums
    float my_sx = 0.0f, my_sw = 0.0f, my_bs = 0.0f, my_cx = 0.0f, my_rs = 0.0f;
    if (OUT != QC_OUT_I32_ACC) {
        int64_t m = (int64_t)mt * TM + threadIdx.x % TM;   // x_scale is padded to Mp
        if (MI == 3) m = min(m, (int64_t)a.x_frags * kFragRows - 1);
        my_sx = a.x_scale[m];
        if (ASYM) my_cx = a.x_corr[m];
        const int64_t n = (int64_t)nt * kTileN + threadIdx.x;
        if (threadIdx.x < kTileN && n < a.N) {
            my_sw = a.w_scale[n];
            if (BITS == 4) my_sw *= 0.0625f;  // operands carry codes times 16
            if (a.bias) my_bs = a.bias[n];
            if (ASYM) {
                my_rs = (float)a.w_rowsum[n];  // |sum| <= 127 K < 2^24: exact
                if (BITS == 4) my_rs *= 16.0f;
            }
        }
    }
    // The pieces of the weight stage tile this wavefront copies HBM -> LDS, at stage 0 (a
    // stage tile is contiguous in memory).
    const uint8_t *const wsrc = a.w_codes + ((int64_t)nt * a.KF + stage0) * L::kBytes + wave * FPW * kFragBytes + lane * 16;
    // copy the weight pieces of K stage `stage` into ring buffer `slot`
    auto issue_w = [&](int stage, int slot) {
        uint8_t *buf = ring + slot * L::kBytes;
#pragma unroll
        for (int j = 0; j < FPW; ++j)
            lds_dma_16(wsrc + (int64_t)stage * L::kBytes + j * kFragBytes, buf + (wave * FPW + j) * kFragBytes);
    };

    // Activation fragments are private to a wavefront (its 16 MI tokens), so they skip LDS:
    // HBM -> registers, 16 B per lane, two stages ahead.  xq[slot][i]: tokens 16 i .. of the
    // stage held in `slot`.  Loads and LDS reads are asm so that they stay
    // in flight across loop iterations under explicit s_waitcnt counts; each wait names the
    // registers it makes valid, which orders the MFMAs that consume them behind it.
    v4i xq[kStages][MI];
    // The stage's base is a scalar address and a lane's place in its fragment a 32-bit offset, so that a
    // stage costs no address arithmetic in vector registers.  A wavefront of 48 tokens may begin inside a
    // panel of 64 and end in the next: an offset per fragment.  Its tile may end past the padded
    // tokens, where it reads the last fragment again and stores nothing.
    const int frag0 = min((mt * 4 + wave) * MI, a.x_frags - 1);   // first of its blocks of 16 tokens, four to a panel
    const uint8_t *const xsrc = a.x_tiled + ((int64_t)(frag0 / 4) * a.KF + stage0) * (4 * kFragBytes);
    uint32_t xoff[MI == 3 ? 3 : 1];
    if constexpr (MI == 3) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int f = min(frag0 + i, a.x_frags - 1);
            xoff[i] = (uint32_t)((f / 4 - frag0 / 4) * a.KF) * (4 * kFragBytes) + f % 4 * kFragBytes + lane * 16;
        }
    } else {
        xoff[0] = frag0 % 4 * kFragBytes + lane * 16;
    }

// (s_nop: a vector instruction may have written the scalar base just before, and the compiler, which sees
// no memory instruction here, does not know that five wait states have to pass.)
#define QC_GLOBAL_LOAD_FIRST(dst, off, base) \
    asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(off), "s"(base) : "memory")
#define QC_GLOBAL_LOAD(dst, off, base, imm) \
    asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=v"(dst) : "v"(off), "s"(base), "n"(imm) : "memory")
#define QC_ISSUE_X(stage, SLOT)                                              \
    do {                                                                     \
        const uint8_t *p_ = xsrc + (int64_t)(stage) * (4 * kFragBytes);      \
        QC_GLOBAL_LOAD_FIRST(xq[SLOT][0], xoff[0], p_);                      \
        if constexpr (MI == 3) {                                             \
            QC_GLOBAL_LOAD(xq[SLOT][1], xoff[1], p_, 0);                     \
            QC_GLOBAL_LOAD(xq[SLOT][2], xoff[2], p_, 0);                     \
        } else {                                                             \
            QC_GLOBAL_LOAD(xq[SLOT][1], xoff[0], p_, kFragBytes);            \
        }                                                                    \
        if constexpr (MI == 4) {                                             \
            QC_GLOBAL_LOAD(xq[SLOT][2], xoff[0], p_, 2 * kFragBytes);        \
            QC_GLOBAL_LOAD(xq[SLOT][3], xoff[0], p_, 3 * kFragBytes);        \
        }                                                                    \
    } while (0)
#define QC_WAIT_X(n, SLOT)                                                                    \
    do {                                                                                      \
        if constexpr (MI == 4)                                                                \
            asm volatile("s_waitcnt vmcnt(%4)" : "+v"(xq[SLOT][0]), "+v"(xq[SLOT][1]),        \
                         "+v"(xq[SLOT][2]), "+v"(xq[SLOT][3]) : "n"(n));                      \
        else if constexpr (MI == 3)                                                           \
            asm volatile("s_waitcnt vmcnt(%3)" : "+v"(xq[SLOT][0]), "+v"(xq[SLOT][1]),        \
                         "+v"(xq[SLOT][2]) : "n"(n));                                         \
        else                                                                                  \
            asm volatile("s_waitcnt vmcnt(%2)" : "+v"(xq[SLOT][0]), "+v"(xq[SLOT][1]) : "n"(n)); \
    } while (0)

    // LDS -> registers for the weight fragments.
    //   wr[h][t]: 16-channel block 4 h + t (8 bit);  wr[0][u]: nibble unit of blocks 2 u, 2 u + 1 (4 bit)
    v4i wr[2][4];
    const uint32_t lds_lane = (uint32_t)(uintptr_t)ring + lane * 16;  // LDS byte address of this lane
#define QC_DS_READ(dst, addr, imm) \
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(imm))
#define QC_READ_W(SLOT, H)                                                           \
    do {                                                                             \
        const uint32_t base_ = lds_lane + (SLOT) * L::kBytes;                        \
        if (BITS == 8) {                                                             \
            QC_DS_READ(wr[H][0], base_, (4 * H + 0) * kFragBytes);                   \
            QC_DS_READ(wr[H][1], base_, (4 * H + 1) * kFragBytes);                   \
            QC_DS_READ(wr[H][2], base_, (4 * H + 2) * kFragBytes);                   \
            QC_DS_READ(wr[H][3], base_, (4 * H + 3) * kFragBytes);                   \
        } else if (H == 0) {                                                        \
            QC_DS_READ(wr[0][0], base_, 0 * kFragBytes);                             \
            QC_DS_READ(wr[0][1], base_, 1 * kFragBytes);                             \
            QC_DS_READ(wr[0][2], base_, 2 * kFragBytes);                             \
            QC_DS_READ(wr[0][3], base_, 3 * kFragBytes);                             \
        }                                                                            \
    } while (0)
#define QC_WAIT_W(n, H) \
    asm volatile("s_waitcnt lgkmcnt(" #n ")" : "+v"(wr[H][0]), "+v"(wr[H][1]), "+v"(wr[H][2]), "+v"(wr[H][3]))

    v4i acc[MI][8];   // [16-token block][16-channel block]
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[i][t] = v4i{0, 0, 0, 0};

    // 4 bit: nibbles -> int8 operand dwords holding 16 * code, channel blocks 4 h .. 4 h + 3
    auto unpack = [&](v4i (&w)[4], int h) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const v4i unit = wr[0][2 * h + t / 2];
            const uint32_t v0 = (uint32_t)unit[2 * (t % 2)], v1 = (uint32_t)unit[2 * (t % 2) + 1];
            w[t][0] = (int)((v0 << 4) & 0xF0F0F0F0u);
            w[t][1] = (int)(v0 & 0xF0F0F0F0u);
            w[t][2] = (int)((v1 << 4) & 0xF0F0F0F0u);
            w[t][3] = (int)(v1 & 0xF0F0F0F0u);
        }
    };

    // One 64-k stage.  SLOT = stage % 3 is a literal constant (the loop is unrolled by three) so that
    // the activation ring stays in fixed registers and the LDS ring needs no address arithmetic (with
    // the remainder taken at run time 16384 x 1152 x 3456 took 0 to 3 % longer).  VMEM operations complete
    // in issue order, which is W(0) X(0) W(1) X(1) W(2) before the loop, then X(s+2) and W(s+3) in stage s.
    // X(s+2) goes out after the wait for X(s), among the first MFMAs of the stage, so at that wait two
    // weight stages and one activation stage are behind X(s); at the wait for W(s+1) in the middle of
    // the stage, two activation stages and one weight stage are behind it.  (A deeper weight ring buys
    // nothing: the loop is not waiting for the weights.)  Past the end of K the stage index is clamped
    // to the last stage: those copies repeat data that is not used again (they hit in cache), which
    // keeps the instruction stream and the wait counts uniform.
    constexpr int kXBehind = 2 * FPW + MI, kWBehind = 2 * MI + FPW;
    static_assert(kStages == 3, "the loop is unrolled by the ring, and KF is a multiple of 3");
    const int last = stages - 1;
#define QC_CLAMP(st) ((st) < last ? (st) : last)
    // The 4 MI MFMAs of a half stage (MI token blocks x 4 channel blocks) are independent, so
    // their order is free.  8 bit: token block outer.  4 bit: channel block outer, so that the
    // MFMAs that share an unpacked weight fragment follow each other.
#define QC_MFMA_LOOPS                                                                           \
    _Pragma("unroll") for (int o_ = 0; o_ < 4 * MI; ++o_)                                       \
        for (int i = BITS == 8 ? o_ / 4 : o_ % MI, t = BITS == 8 ? o_ % 4 : o_ / MI, once_ = 1; once_; once_ = 0)
#define QC_STAGE(s, SLOT)                                                                      \
    do {                                                                                       \
        QC_WAIT_W(0, 0);                                  /* channel half 0 of W(s) is here */ \
        QC_WAIT_X(kXBehind, SLOT);                                         /* X(s) is here */  \
        v4i w4a[4], w4b[4];                                                                    \
        if (BITS == 4) unpack(w4a, 0);                                                         \
        /* issued here, not before the waits, so that the loads go out under the MFMAs */      \
        QC_ISSUE_X(QC_CLAMP((s) + 2), (SLOT + 2) % 3);                                                 \
        QC_READ_W(SLOT, 1);       /* channel half 1: lands under the MFMAs of channel half 0 */ \
        QC_MFMA_LOOPS                                                                          \
                acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(                             \
                    xq[SLOT][i], BITS == 8 ? wr[0][t] : w4a[t], acc[i][t], 0, 0, 0);           \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        QC_WAIT_VMCNT(kWBehind);                                        /* W(s+1) has landed */\
        /* this wavefront's reads of W(s) are done ... */                                      \
        if (BITS == 8) QC_WAIT_W(0, 1);                                                        \
        __builtin_amdgcn_s_barrier(); /* ... and everybody else's: ring buffer SLOT is free */\
        asm volatile("" ::: "memory");                                                         \
        if (BITS == 4) unpack(w4b, 1);   /* before the reads below overwrite the nibbles */     \
        issue_w(QC_CLAMP((s) + 3), SLOT);                                                      \
        /* after the last stage this reads data that is not used */                            \
        QC_READ_W((SLOT + 1) % 3, 0);                                                          \
        QC_MFMA_LOOPS                                                                          \
                acc[i][4 + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(                         \
                    xq[SLOT][i], BITS == 8 ? wr[1][t] : w4b[t], acc[i][4 + t], 0, 0, 0);       \
        __builtin_amdgcn_sched_barrier(0);                                                     \
    } while (0)

    // ---- main loop -------------------------------------------------------------------
    issue_w(0, 0);
    QC_ISSUE_X(0, 0);
    issue_w(QC_CLAMP(1), 1);
    QC_ISSUE_X(QC_CLAMP(1), 1);
    issue_w(QC_CLAMP(2), 2);
    QC_WAIT_VMCNT(2 * MI + 2 * FPW);   // W(0) has landed
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    QC_READ_W(0, 0);

    for (int s = 0; s < stages; s += 3) {
        QC_STAGE(s, 0);
        QC_STAGE(s + 1, 1);
        QC_STAGE(s + 2, 2);
    }
    // drain everything still in flight before the registers are reused
    QC_WAIT_W(0, 0);
    QC_WAIT_X(0, 0);
    QC_WAIT_X(0, 1);
    QC_WAIT_X(0, 2);
    // a barrier is for both groups, so the second meets the first at those of the stages it does not have
    for (int s = stages; s < most; ++s) __builtin_amdgcn_s_barrier();
#undef QC_MFMA_LOOPS
#undef QC_CLAMP
#undef QC_STAGE
#undef QC_WAIT_W
#undef QC_READ_W
#undef QC_DS_READ
#undef QC_WAIT_X
#undef QC_ISSUE_X
#undef QC_GLOBAL_LOAD_FIRST
#undef QC_GLOBAL_LOAD

    // park the scales (fetched at kernel start, long since arrived) where every lane can pick
    // the ones of its tokens and channels
    if (OUT != QC_OUT_I32_ACC) {
        if (threadIdx.x < TM) lds_sx[threadIdx.x] = my_sx;
        if (threadIdx.x < kTileN) { lds_sw[threadIdx.x] = my_sw; lds_bs[threadIdx.x] = my_bs; }
        if (ASYM) {
            if (threadIdx.x < TM) lds_cx[threadIdx.x] = my_cx;
            if (threadIdx.x < kTileN) lds_rs[threadIdx.x] = my_rs;
        }
        __syncthreads();
    }

    // ---- epilogue: registers -> Y --------------------------------------------------------
    if constexpr (SPLIT) {
        // Each group finishes half of the tokens: a wavefront hands its sums of the others to its counterpart in the other
        // group, 4 KiB at a time, where the rings were.
        constexpr int H = MI / 2;
        v4i half[H][8];
        v4i *const mine = reinterpret_cast<v4i *>(lds) + wave_of_block * 256 + lane;
        const v4i *const theirs = reinterpret_cast<const v4i *>(lds) + (wave_of_block ^ 4) * 256 + lane;
#pragma unroll
        for (int i = 0; i < H; ++i)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                __syncthreads();   // the rings, or the exchange before, have been read
#pragma unroll
                for (int t = 0; t < 4; ++t) mine[64 * t] = group ? acc[i][4 * r + t] : acc[H + i][4 * r + t];
                __syncthreads();
#pragma unroll
                for (int t = 0; t < 4; ++t) half[i][4 * r + t] = (group ? acc[H + i][4 * r + t] : acc[i][4 * r + t]) + theirs[64 * t];
            }
        const int at = wave * (16 * MI) + group * (16 * H);
        store_wave_tile<BITS, OUT, EPI, ASYM, KEEP>(half, a, (int64_t)mt * TM + at, nt, lane, lds_sx + at, lds_cx + at, lds_sw, lds_bs, lds_rs);
    } else {
        store_wave_tile<BITS, OUT, EPI, ASYM, KEEP>(acc, a, (int64_t)mt * TM + wave * (16 * MI), nt, lane,
                                                    lds_sx + wave * (16 * MI), lds_cx + wave * (16 * MI), lds_sw, lds_bs, lds_rs);
    }
}

template <int BITS, int OUT, int EPI, bool ASYM>
__global__ __launch_bounds__(kThreads, 2) void gemm_kernel(GemmArgs a) {
    ring_gemm<BITS, OUT, EPI, ASYM, false, 4>(a);
}

// tiles of 192 and of 128 tokens x 128 channels: see ring_height().  Three (with a zero point and 8-bit
// weights two) and four blocks fit a CU's registers; asked for three the compiler spills.
template <int BITS, int OUT, int EPI, bool ASYM>
__global__ __launch_bounds__(kThreads, 2) void gemm_mid_kernel(GemmArgs a) {
    ring_gemm<BITS, OUT, EPI, ASYM, false, 3>(a);
}
template <int BITS, int OUT, int EPI, bool ASYM>
__global__ __launch_bounds__(kThreads, 4) void gemm_half_kernel(GemmArgs a) {
    ring_gemm<BITS, OUT, EPI, ASYM, false, 2>(a);
}

// two groups of four wavefronts on tiles of 128 and, with 4-bit weights, 256 tokens: see split_height()
template <int BITS, int OUT, int EPI, bool ASYM>
__global__ __launch_bounds__(kSplitThreads, 2) void gemm_split_half_kernel(GemmArgs a) {
    ring_gemm<BITS, OUT, EPI, ASYM, false, 2, true>(a);
}
template <int OUT, int EPI, bool ASYM>
__global__ __launch_bounds__(kSplitThreads, 2) void gemm_split_kernel(GemmArgs a) {
    ring_gemm<4, OUT, EPI, ASYM, false, 4, true>(a);
}

// the first three with f32 output stored through the caches: see keep_f32_output()
template <int BITS, int EPI, bool ASYM>
__global__ __launch_bounds__(kThreads, 2) void gemm_cached_kernel(GemmArgs a) {
    ring_gemm<BITS, QC_OUT_F32, EPI, ASYM, true, 4>(a);
}
template <int BITS, int EPI, bool ASYM>
__global__ __launch_bounds__(kThreads, 2) void gemm_mid_cached_kernel(GemmArgs a) {
    ring_gemm<BITS, QC_OUT_F32, EPI, ASYM, true, 3>(a);
}
template <int BITS, int EPI, bool ASYM>
__global__ __launch_bounds__(kThreads, 4) void gemm_half_cached_kernel(GemmArgs a) {
    ring_gemm<BITS, QC_OUT_F32, EPI, ASYM, true, 2>(a);
}

// ---- the same GEMM with the weight tile resident in LDS (short reductions) ---------------------
// When a whole channel tile of the weights (128 channels x Kp) fits in LDS beside the scales, a
// block of eight wavefronts, one per CU, loads it once and then every wavefront walks token tiles
// of 64 on its own: no weight copies and no block barriers inside the reduction, which is what
// the ring version above spends 5-9 % of its time on when K is 1152.  Work is cut into rounds of
// (channel tile, 512 tokens = one 64-token tile per wavefront) and dealt to the blocks by the
// static schedule of resident_rounds() (qc_internal.h): a block changes its weight tile once or
// twice per launch, and the blocks of an XCD read the same few token chunks at the same time.

template <int BITS, int OUT, int EPI, bool ASYM>
__global__ __launch_bounds__(kResThreads, 1) void gemm_resident_kernel(GemmArgs a) {
    using L = StageLayout<BITS>;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kResLdsBytes];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int stages = a.KF;

    float *lds_sw = reinterpret_cast<float *>(lds + kResWeightBytes);      // 128 channel scales
    float *lds_bs = lds_sw + kTileN;                                       // 128 biases
    float *lds_rs = lds_bs + kTileN;                                       // ASYM: 128 code sums
    float *lds_sx = lds_rs + kTileN + wave * kWaveM;                       // this wavefront's 64 token scales
    float *lds_cx = lds_sx + kResWaves * kWaveM;                           // ASYM: its 64 corrections

    // this block's XCD (block b runs on XCD b % 8), its place there and the XCD's token chunks
    const ResidentXcd xs = resident_xcd((int)blockIdx.x, (int)gridDim.x, resident_chunks(a.m_tiles));
    const int slot = xs.slot, nbx = xs.blocks, c_lo = xs.c_lo, c_hi = xs.c_hi;
    const int wave_tiles = a.m_tiles * (kTileM / kWaveM);          // 64-token tiles inside Mp

    v4i xq[kStages][4];
    v4i wr[2][4];
    const uint32_t lds_lane = (uint32_t)(uintptr_t)lds + lane * 16;

#define QC_GLOBAL_LOAD(dst, ptr, imm) \
    asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=v"(dst) : "v"(ptr), "n"(imm) : "memory")
#define QC_ISSUE_X(ptr, SLOT)                                                \
    do {                                                                     \
        const uint8_t *p_ = (ptr);                                           \
        QC_GLOBAL_LOAD(xq[SLOT][0], p_, 0);                                  \
        QC_GLOBAL_LOAD(xq[SLOT][1], p_, kFragBytes);                         \
        QC_GLOBAL_LOAD(xq[SLOT][2], p_, 2 * kFragBytes);                     \
        QC_GLOBAL_LOAD(xq[SLOT][3], p_, 3 * kFragBytes);                     \
    } while (0)
#define QC_WAIT_X(n, SLOT)                                                                    \
    asm volatile("s_waitcnt vmcnt(" #n ")" : "+v"(xq[SLOT][0]), "+v"(xq[SLOT][1]),            \
                 "+v"(xq[SLOT][2]), "+v"(xq[SLOT][3]))
#define QC_DS_READ(dst, addr, imm) \
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(imm))
#define QC_READ_W(stage, H)                                                          \
    do {                                                                             \
        const uint32_t base_ = lds_lane + (uint32_t)(stage) * L::kBytes;             \
        if (BITS == 8) {                                                             \
            QC_DS_READ(wr[H][0], base_, (4 * H + 0) * kFragBytes);                   \
            QC_DS_READ(wr[H][1], base_, (4 * H + 1) * kFragBytes);                   \
            QC_DS_READ(wr[H][2], base_, (4 * H + 2) * kFragBytes);                   \
            QC_DS_READ(wr[H][3], base_, (4 * H + 3) * kFragBytes);                   \
        } else if (H == 0) {                                                        \
            QC_DS_READ(wr[0][0], base_, 0 * kFragBytes);                             \
            QC_DS_READ(wr[0][1], base_, 1 * kFragBytes);                             \
            QC_DS_READ(wr[0][2], base_, 2 * kFragBytes);                             \
            QC_DS_READ(wr[0][3], base_, 3 * kFragBytes);                             \
        }                                                                            \
    } while (0)
#define QC_WAIT_W(n, H) \
    asm volatile("s_waitcnt lgkmcnt(" #n ")" : "+v"(wr[H][0]), "+v"(wr[H][1]), "+v"(wr[H][2]), "+v"(wr[H][3]))
#define QC_MFMA_LOOPS                                                                           \
    _Pragma("unroll") for (int o_ = 0; o_ < 16; ++o_)                                           \
        for (int i = BITS == 8 ? o_ / 4 : o_ % 4, t = BITS == 8 ? o_ % 4 : o_ / 4, once_ = 1; once_; once_ = 0)
    const int last = stages - 1;
#define QC_CLAMP(st) ((st) < last ? (st) : last)
    // One 64-k stage.  The only vector memory operations of the loop are the activation loads,
    // which complete in issue order: at the wait for X(s), X(s+1) (four loads) is behind it.
    // Past the end of K the stage index is clamped (a repeat that hits in cache), which keeps
    // the instruction stream and the counts uniform.
#define QC_RES_STAGE(s, SLOT, NEXT2)                                                           \
    do {                                                                                       \
        QC_WAIT_W(0, 0);                                  /* channel half 0 of W(s) is here */ \
        QC_WAIT_X(4, SLOT);                                                /* X(s) is here */  \
        v4i w4a[4], w4b[4];                                                                    \
        if (BITS == 4) unpack(w4a, 0);                                                         \
        QC_ISSUE_X(xsrc + (int64_t)QC_CLAMP((s) + 2) * (4 * kFragBytes), NEXT2);               \
        QC_READ_W((s), 1);        /* channel half 1: lands under the MFMAs of channel half 0 */ \
        QC_MFMA_LOOPS                                                                          \
                acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(                             \
                    xq[SLOT][i], BITS == 8 ? wr[0][t] : w4a[t], acc[i][t], 0, 0, 0);           \
        __builtin_amdgcn_sched_barrier(0);                                                     \
        if (BITS == 8) QC_WAIT_W(0, 1);                                                        \
        if (BITS == 4) unpack(w4b, 1);   /* before the reads below overwrite the nibbles */     \
        QC_READ_W(QC_CLAMP((s) + 1), 0);                                                       \
        QC_MFMA_LOOPS                                                                          \
                acc[i][4 + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(                         \
                    xq[SLOT][i], BITS == 8 ? wr[1][t] : w4b[t], acc[i][4 + t], 0, 0, 0);       \
        __builtin_amdgcn_sched_barrier(0);                                                     \
    } while (0)

    // the rounds of this block, one after the other
    int pass = 0;
    RoundRange rr = resident_rounds(0, slot, nbx, a.n_tiles, c_hi - c_lo);
    int id = rr.id0 - 1;
    auto advance = [&]() -> bool {   // to the block's next round; false when there is none
        ++id;
        while (id >= rr.id1) {
            ++pass;
            if (pass * nbx >= a.n_tiles) return false;
            rr = resident_rounds(pass, slot, nbx, a.n_tiles, c_hi - c_lo);
            id = rr.id0;
        }
        return true;
    };
    auto x_of_tile = [&](int wt) { return a.x_tiled + ((int64_t)wt * stages) * (4 * kFragBytes) + lane * 16; };

    // Every wavefront runs every round of its block, so that no branch goes round the in-flight
    // loads: a wavefront whose tile lies past the end of the (padded) tokens, which only happens
    // in the last chunk, computes on the last tile instead and stores nothing.
    if (!advance()) return;   // the whole block: no round at all
    int nt = rr.nt_off + id / rr.w;
    int wt = (c_lo + rr.c_off + id % rr.w) * kResWaves + wave;
    int cur_nt = -1;
    bool have;
    do {
        const int wt_ld = wt < wave_tiles ? wt : wave_tiles - 1;   // where this tile's inputs are read
        const uint8_t *const xsrc = x_of_tile(wt_ld);
        if (nt != cur_nt) {   // uniform over the block
            cur_nt = nt;
            __syncthreads();  // every wavefront is done with the previous tile and its scales
            const uint8_t *wsrc = a.w_codes + (int64_t)nt * stages * L::kBytes + lane * 16;
            for (int st = wave; st < stages; st += kResWaves) {
#pragma unroll
                for (int j = 0; j < L::kWFrags; ++j)
                    lds_dma_16(wsrc + (int64_t)st * L::kBytes + j * kFragBytes, lds + st * L::kBytes + j * kFragBytes);
            }
            if (OUT != QC_OUT_I32_ACC && threadIdx.x < kTileN) {
                const int64_t n = (int64_t)nt * kTileN + threadIdx.x;
                float sw = 0.0f, bs = 0.0f, rs = 0.0f;
                if (n < a.N) {
                    sw = a.w_scale[n];
                    if (BITS == 4) sw *= 0.0625f;  // operands carry codes times 16
                    if (a.bias) bs = a.bias[n];
                    if (ASYM) {
                        rs = (float)a.w_rowsum[n];
                        if (BITS == 4) rs *= 16.0f;
                    }
                }
                lds_sw[threadIdx.x] = sw;
                lds_bs[threadIdx.x] = bs;
                if (ASYM) lds_rs[threadIdx.x] = rs;
            }
            QC_WAIT_VMCNT(0);
            __syncthreads();
        }
        const int nt_now = nt, wt_now = wt;
        have = advance();
        if (have) {
            nt = rr.nt_off + id / rr.w;
            wt = (c_lo + rr.c_off + id % rr.w) * kResWaves + wave;
        }

        float my_sx = 0.0f, my_cx = 0.0f;
        if (OUT != QC_OUT_I32_ACC) {
            my_sx = a.x_scale[(int64_t)wt_ld * kWaveM + lane];  // x_scale is padded to Mp
            if (ASYM) my_cx = a.x_corr[(int64_t)wt_ld * kWaveM + lane];
        }
        v4i acc[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[i][t] = v4i{0, 0, 0, 0};
        auto unpack = [&](v4i (&w)[4], int h) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const v4i unit = wr[0][2 * h + t / 2];
                const uint32_t v0 = (uint32_t)unit[2 * (t % 2)], v1 = (uint32_t)unit[2 * (t % 2) + 1];
                w[t][0] = (int)((v0 << 4) & 0xF0F0F0F0u);
                w[t][1] = (int)(v0 & 0xF0F0F0F0u);
                w[t][2] = (int)((v1 << 4) & 0xF0F0F0F0u);
                w[t][3] = (int)(v1 & 0xF0F0F0F0u);
            }
        };

        // Nothing of this wavefront is in flight here but the scale loads above and the stores of
        // its previous tile, all older than these loads.
        QC_ISSUE_X(xsrc, 0);
        QC_ISSUE_X(xsrc + (int64_t)QC_CLAMP(1) * (4 * kFragBytes), 1);
        QC_READ_W(0, 0);
        for (int s = 0; s < stages; s += 3) {
            QC_RES_STAGE(s, 0, 2);
            QC_RES_STAGE(s + 1, 1, 0);
            QC_RES_STAGE(s + 2, 2, 1);
        }
        // everything in flight has landed before the registers are used for anything else
        QC_WAIT_W(0, 0);
        QC_WAIT_X(0, 0);
        QC_WAIT_X(0, 1);
        QC_WAIT_X(0, 2);

        if (OUT != QC_OUT_I32_ACC) {   // hand the token scales round inside the wavefront
            lds_sx[lane] = my_sx;
            if (ASYM) lds_cx[lane] = my_cx;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        store_wave_tile<BITS, OUT, EPI, ASYM, false>(acc, a, (int64_t)wt_now * kWaveM, nt_now, lane, lds_sx, lds_cx,
                                               lds_sw, lds_bs, lds_rs);
    } while (have);
#undef QC_RES_STAGE
#undef QC_CLAMP
#undef QC_MFMA_LOOPS
#undef QC_WAIT_W
#undef QC_READ_W
#undef QC_DS_READ
#undef QC_WAIT_X
#undef QC_ISSUE_X
#undef QC_GLOBAL_LOAD
}

template <int BITS, int OUT, int EPI, bool ASYM>
hipError_t launch_variant(const GemmArgs &args, hipStream_t stream) {
    // the combinations gemm_resident_epilogue() lets through
    if constexpr (EPI == QC_EPI_NONE || (EPI == QC_EPI_GELU_TANH && BITS == 8 && OUT == QC_OUT_BF16)) {
        if (args.resident) {
            gemm_resident_kernel<BITS, OUT, EPI, ASYM><<<dim3(kResBlocks), dim3(kResThreads), 0, stream>>>(args);
            return hipGetLastError();
        }
    }
    constexpr int kLds = kRingBytes<BITS, false> +
                         (kTileM + 2 * kTileN + (ASYM ? kTileM + kTileN : 0)) * (int)sizeof(float);
    // far below the 64 KiB a kernel may use without an attribute, so the first launch of a
    // variant needs no set-up call and can be captured into a graph like any other
    static_assert(kLds <= 64 * 1024, "dynamic LDS beyond the default limit needs an attribute");
    const int blocks = args.m_tiles * args.n_tiles;
    const dim3 grid((unsigned)blocks), block(kThreads);
    if (args.split) {
        constexpr int kSplitLds = kLds - kRingBytes<BITS, false> + kRingBytes<BITS, true>;
        static_assert(kSplitLds <= 64 * 1024, "dynamic LDS beyond the default limit needs an attribute");
        if constexpr (BITS == 4) {
            if (args.height == 4) {
                gemm_split_kernel<OUT, EPI, ASYM><<<grid, dim3(kSplitThreads), kSplitLds, stream>>>(args);
                return hipGetLastError();
            }
        }
        gemm_split_half_kernel<BITS, OUT, EPI, ASYM><<<grid, dim3(kSplitThreads), kSplitLds, stream>>>(args);
        return hipGetLastError();
    }
    if constexpr (OUT == QC_OUT_F32) {
        if (args.keep_output) {
            if (args.height == 2) gemm_half_cached_kernel<BITS, EPI, ASYM><<<grid, block, kLds, stream>>>(args);
            else if (args.height == 3) gemm_mid_cached_kernel<BITS, EPI, ASYM><<<grid, block, kLds, stream>>>(args);
            else gemm_cached_kernel<BITS, EPI, ASYM><<<grid, block, kLds, stream>>>(args);
            return hipGetLastError();
        }
    }
    if (args.height == 2) gemm_half_kernel<BITS, OUT, EPI, ASYM><<<grid, block, kLds, stream>>>(args);
    else if (args.height == 3) gemm_mid_kernel<BITS, OUT, EPI, ASYM><<<grid, block, kLds, stream>>>(args);
    else gemm_kernel<BITS, OUT, EPI, ASYM><<<grid, block, kLds, stream>>>(args);
    return hipGetLastError();
}

template <int BITS, bool ASYM>
hipError_t launch_bits(const GemmArgs &args, qc_epilogue epi, qc_out ydt, hipStream_t stream) {
    // the raw accumulators are the same kernel with or without a zero point
    if (ydt == QC_OUT_I32_ACC) return launch_variant<BITS, QC_OUT_I32_ACC, QC_EPI_NONE, false>(args, stream);
#define QC_EPI_CASE(O)                                                                        \
    switch (epi) {                                                                            \
        case QC_EPI_NONE: return launch_variant<BITS, O, QC_EPI_NONE, ASYM>(args, stream);         \
        case QC_EPI_GELU_TANH: return launch_variant<BITS, O, QC_EPI_GELU_TANH, ASYM>(args, stream);\
        default: return launch_variant<BITS, O, QC_EPI_GELU_ERF, ASYM>(args, stream);             \
    }
    if (ydt == QC_OUT_F32) { QC_EPI_CASE(QC_OUT_F32) }
    QC_EPI_CASE(QC_OUT_BF16)
#undef QC_EPI_CASE
}

}  // namespace

template <int BITS>
hipError_t launch_gemm_kernel(const GemmArgs &args, qc_epilogue epi, qc_out ydt, hipStream_t stream) {
    return args.x_corr && args.w_rowsum ? launch_bits<BITS, true>(args, epi, ydt, stream) : launch_bits<BITS, false>(args, epi, ydt, stream);
}

}  // namespace qc
