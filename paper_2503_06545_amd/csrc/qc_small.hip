// The quantized linear on few tokens (Section 4.1 "Hardware Implementation"): too few output tiles of
// 256 x 128 to fill the chip, so what bounds the call is latency - the number of launches, each
// wavefront's chain of loads - and how many CUs pull the weights at once.
//
// small_kernel: a block of 8 wavefronts computes a tile of 16 or 32 or 64 tokens x 32 or 64 channels.  The
// wavefronts split the reduction (64-k stages dealt round-robin), load their operand fragments
// straight into registers, all of them ahead of the first use when K is short, and add their partial
// sums through LDS: exact, the sums are integers.  The smallest tile that gives at most one block per
// CU is taken: a second block on a CU only adds to what the CU has to load, and a single CU gets
// about 35 B/clk from beyond its L2 (every launch starts with that L2 invalid).
//
// fused_kernel: the whole linear is one launch: each block quantizes its token tile into
// LDS itself, redundantly over the channel tiles (that is cheap while there are few tokens in a tile), and the blocks
// of the first channel tile leave codes and scales in the workspace as the two-launch path does.
//
// Measured, K = 1152, W8, GPU time of quantization + GEMM on full tiles, and in one launch: 2 tokens x 6912 channels
// 4.7 + 8.2 -> 4.9 us, 64 x 1152 2.8 + 8.8 -> 5.2 us, 256 x 1152 2.8 + 8.8 -> 6.7 us; K = 4608: 2 x 1152 5.0 + 24.1 ->
// 5.7 us, 256 x 1152 4.2 + 25.0 -> 4.2 + 8.5 us in two (a 256-token tile there walks 72 stages alone).
#include <atomic>

#include "qc_device.h"

namespace qc {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int kGroup = 128;   // columns that eight lanes quantize per step
constexpr int kWaves = kThreads / 64;
constexpr int kLdsMost = 150 * 1024;

struct SmallArgs {
    const void *X;          // fused_kernel: the activations
    uint8_t *x_tiled;       // the workspace's codes: read (small_kernel) or written (fused_kernel)
    float *x_scale;
    float *x_corr;          // asymmetric activations only, with w_rowsum: read (small_kernel) or written
    const int32_t *w_rowsum;
    const uint8_t *w_codes;
    const float *w_scale;
    const float *bias;
    void *Y;
    int64_t M, N, K;
    int KF, m_tiles, n_tiles;
    int rows, groups;       // fused_kernel: rows of a tile that can be live, groups of 128 columns in a row
    uint32_t inv_groups;    // 2^20 / groups, rounded up
    float qmax, shift;      // fused_kernel: largest code; asymmetric: largest unsigned one and what is subtracted from it
    int rot, epi, out;
};

// partial sums of small_kernel in LDS: WK x TM x kLd int32
template <int MI, int NF, int WN>
struct Layout {
    static constexpr int kTM = 16 * MI;
    static constexpr int kWK = kWaves / WN;
    static constexpr int kLd = 16 * NF + 4;   // 4 rows apart = 16 banks apart: conflict-free
    static constexpr int kSums = kWK * kTM * kLd * 4;
};

// MI x 16 tokens by NF x 16 channels per block, codes from the workspace; WN wavefront columns, kWaves / WN
// ways over K; a register ring of D stages.
template <int BITS, int MI, int NF, int WN, int D>
__global__ __launch_bounds__(kThreads, 2) void small_kernel(SmallArgs a) {
    using L = Layout<MI, NF, WN>;
    constexpr int TM = L::kTM, WK = L::kWK, NFW = NF / WN;
    constexpr int NW = BITS == 8 ? NFW : NFW / 2;             // 1 KiB weight pieces per stage and wavefront
    constexpr int kStageBytes = BITS == 8 ? 8192 : 4096;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    int *const sums = reinterpret_cast<int *>(lds);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, h = lane >> 4;
    const int wk = wave % WK, wn = wave / WK;

    // block b runs on XCD b % 8: the blocks of one XCD take consecutive tiles, token tile fastest, so
    // that they share weight tiles in its L2
    const int nb = gridDim.x, b = blockIdx.x;
    const int v = (b % 8) * (nb / 8) + ((b % 8) < nb % 8 ? (b % 8) : nb % 8) + b / 8;
    const int mt = v % a.m_tiles, nt = v / a.m_tiles;
    const int64_t m0 = (int64_t)mt * TM;
    const int G = nt / (8 / NF), t0 = nt % (8 / NF) * NF;
    if ((int64_t)G * kTileN + t0 >= a.N) return;   // no live channel in this tile

    const int KF = a.KF;
    // what the epilogue needs, requested first: a thread keeps one column of channels, n0 .. n0 + NF - 1,
    // and the tokens tid / 16 + 32 j
    constexpr int kRows = TM < 32 ? 1 : TM / 32;
    const int ec = tid & 15, em = tid >> 4;
    const int64_t n0 = (int64_t)G * kTileN + 8 * ec + t0;
    float sw[NF], bs[NF], rs[NF], sx[kRows], cx[kRows];
#pragma unroll
    for (int t = 0; t < NF; ++t) {
        sw[t] = a.w_scale[n0 + t < a.N ? n0 + t : a.N - 1];
        bs[t] = rs[t] = 0.0f;
    }
    if (a.bias) {
#pragma unroll
        for (int t = 0; t < NF; ++t) bs[t] = a.bias[n0 + t < a.N ? n0 + t : a.N - 1];
    }
#pragma unroll
    for (int j = 0; j < kRows; ++j) {   // padded to a multiple of 256 tokens
        sx[j] = a.x_scale[m0 + (em + 32 * j) % TM];
        cx[j] = 0.0f;
    }
    if (a.x_corr) {
#pragma unroll
        for (int t = 0; t < NF; ++t)
            rs[t] = (float)a.w_rowsum[n0 + t < a.N ? n0 + t : a.N - 1] * (BITS == 4 ? 16.0f : 1.0f);
#pragma unroll
        for (int j = 0; j < kRows; ++j) cx[j] = a.x_corr[m0 + (em + 32 * j) % TM];
    }
    if (BITS == 4) {
#pragma unroll
        for (int t = 0; t < NF; ++t) sw[t] *= 0.0625f;   // operands carry codes times 16
    }

    // weights of this wavefront: stages wk, wk + WK, ..; a register ring of D of them
    v4i w[D][NW];
    v4i x[D][MI];
    const uint8_t *const wbase = a.w_codes + (int64_t)G * KF * kStageBytes +
                                 (BITS == 8 ? t0 + wn * NFW : (t0 + wn * NFW) / 2) * kFragBytes + lane * 16;
    const uint8_t *const xbase = a.x_tiled + (m0 / kWaveM) * (int64_t)KF * (4 * kFragBytes) +
                                 (m0 % kWaveM) / kFragRows * kFragBytes + lane * 16;
    auto request = [&](int s, int d) {
        const int sc = s < KF ? s : KF - 1;
        const uint8_t *p = wbase + (int64_t)sc * kStageBytes;
#pragma unroll
        for (int j = 0; j < NW; ++j) w[d][j] = *reinterpret_cast<const v4i *>(p + j * kFragBytes);
        const uint8_t *q = xbase + (int64_t)sc * (4 * kFragBytes);
#pragma unroll
        for (int i = 0; i < MI; ++i) x[d][i] = *reinterpret_cast<const v4i *>(q + i * kFragBytes);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(wk + d * WK, d);

    v4i acc[MI][NFW];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int t = 0; t < NFW; ++t) acc[i][t] = v4i{0, 0, 0, 0};

    auto multiply = [&](int d) {   // the stage in ring slot d
#pragma unroll
        for (int t = 0; t < NFW; ++t) {
            v4i wt;
            if constexpr (BITS == 8) {
                wt = w[d][t];
            } else {
                const v4i unit = w[d][t / 2];
                const uint32_t v0 = (uint32_t)unit[2 * (t % 2)], v1 = (uint32_t)unit[2 * (t % 2) + 1];
                wt[0] = (int)((v0 << 4) & 0xF0F0F0F0u);
                wt[1] = (int)(v0 & 0xF0F0F0F0u);
                wt[2] = (int)((v1 << 4) & 0xF0F0F0F0u);
                wt[3] = (int)(v1 & 0xF0F0F0F0u);
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
                acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x[d][i], wt, acc[i][t], 0, 0, 0);
        }
    };
    // Stages wk, wk + WK, ..: the loads are unconditional wherever there are any (past the end they
    // repeat the last stage), so that the compiler's waits count exactly.
    int s = wk;
    for (; s + (2 * D - 1) * WK < KF; s += D * WK) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(d);
            request(s + (d + D) * WK, d);
        }
    }
    if (s + D * WK < KF) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(d);
            request(s + (d + D) * WK, d);
        }
        s += D * WK;
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (s + d * WK < KF) multiply(d);

    // the wavefronts' partial sums meet in LDS (integers: exact in any order)
    int *const mine = sums + wk * TM * L::kLd + (4 * h) * L::kLd + wn * NFW * 16 + c;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int t = 0; t < NFW; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) mine[(16 * i + q) * L::kLd + t * 16] = acc[i][t][q];
    __syncthreads();

    const bool vec = n0 + NF <= a.N;   // stored in one piece, at any alignment of Y's elements
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int m = em + 32 * j;
        if (m >= TM || m0 + m >= a.M || n0 >= a.N) break;
        int raw[NF];
#pragma unroll
        for (int t = 0; t < NF; ++t) {
            raw[t] = 0;
#pragma unroll
            for (int k = 0; k < WK; ++k) raw[t] += sums[(k * TM + m) * L::kLd + t * 16 + ec];
        }
        const int64_t at = (m0 + m) * a.N + n0;
        if (a.out == QC_OUT_I32_ACC) {
            int32_t *y = reinterpret_cast<int32_t *>(a.Y) + at;
#pragma unroll
            for (int t = 0; t < NF; ++t)
                if (n0 + t < a.N) y[t] = BITS == 4 ? raw[t] >> 4 : raw[t];   // exact: multiples of 16
            continue;
        }
        float y[NF];
#pragma unroll
        for (int t = 0; t < NF; ++t) {
            float af = (float)raw[t];
            if (a.x_corr) af = fmaf(cx[j], rs[t], af);
            y[t] = fmaf(af * sx[j], sw[t], bs[t]);
        }
        if (a.epi == QC_EPI_GELU_TANH) {
#pragma unroll
            for (int t = 0; t < NF; ++t) y[t] = gelu_tanh_f(y[t]);
        } else if (a.epi == QC_EPI_GELU_ERF) {
#pragma unroll
            for (int t = 0; t < NF; ++t) y[t] = gelu_erf_f(y[t]);
        }
        if (a.out == QC_OUT_F32) {
            float *o = reinterpret_cast<float *>(a.Y) + at;
            if (vec) {
                __builtin_memcpy(o, y, sizeof(y));
            } else {
#pragma unroll
                for (int t = 0; t < NF; ++t)
                    if (n0 + t < a.N) o[t] = y[t];
            }
        } else {
            uint16_t *o = reinterpret_cast<uint16_t *>(a.Y) + at;
            uint32_t pk[NF / 2];
#pragma unroll
            for (int t = 0; t < NF / 2; ++t) pk[t] = pack_bf16x2(y[2 * t], y[2 * t + 1]);
            if (vec) {
                __builtin_memcpy(o, pk, sizeof(pk));
            } else {
#pragma unroll
                for (int t = 0; t < NF; ++t)
                    if (n0 + t < a.N) o[t] = (uint16_t)(t % 2 ? pk[t / 2] >> 16 : pk[t / 2] & 0xffffu);
            }
        }
    }
}

// ---- quantization and GEMM in one launch -------------------------------------------------------
// A block of 8 or 16 wavefronts quantizes its tokens into LDS, redundantly over the channel tiles, and multiplies:
// 16 MI tokens by 16 NF channels, the wavefronts NF / 2 across the channels (two fragments each) and WK ways over
// K.  What bounds it is a chain - the activations' way from memory, the maximum, the cast, the products,
// the sums' way through LDS - and on more than a few tokens the cast itself, six vector instructions an
// element on one CU for as many elements as the tile has tokens.  Hence
//   * tiles of few tokens and many channels, 16 x 128 rather than 32 x 64: half as much to cast for the same
//     number of blocks;
//   * rows dealt to the threads in pairs (row, group of 128 columns), eight lanes a pair, so that a row of 9
//     groups wastes nothing; what a wavefront has no pair for it skips;
//   * 16 wavefronts where there is much to cast: a SIMD with two issues an instruction every 5.4 clocks, with
//     four every 4; they take longer to start;
//   * all arguments in one load, all loads of activations and (up to K = 1152) weights ahead of the first use.
// us per call in a graph, with 512 threads, tiles of 16 x 32 to 32 x 64 and a power of two of threads per row, and so:
// 2 x 1152 x 6912 5.7 4.9, 1 x 1152 x 1152 4.8 4.0, 64 x 1152 x 1152 5.7 5.2, 256 x 1152 x 1152 bf16 8.7 6.7, f32 9.5
// 7.2, 100 x 1152 x 4608 GELU 10.8 6.8, 256 x 1154 x 1152 11.7 7.2, 8 x 4608 x 4608 11.4 9.1.
constexpr int kStepsMost = 3;   // of 8 pairs per wavefront and step

// bytes between the 16-k quarters of a stage in the code tile: 16 B per row and 16 B of padding, so that
// the quarters a row's units go to fall into different banks
__host__ __device__ inline int quarter_stride(int rows) { return 16 * rows + 16; }

// a float as a number that orders like it, and back
__device__ inline uint32_t ordered(float v) {
    const uint32_t b = __float_as_uint(v);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ inline float from_ordered(uint32_t u) { return __uint_as_float(u ^ (((u >> 31) - 1) | 0x80000000u)); }

// LDS: [ row maxima: TM ][ row minima: TM ][ token scales: TM ][ their reciprocals: TM ][ corrections: TM ]
// [ partial sums: WK x TM x kLd int32 ][ codes ]
template <int MI, int NF, int WAVES>
struct FusedLayout {
    static constexpr int kTM = 16 * MI;
    static constexpr int kWN = NF / 2, kWK = WAVES / kWN;
    static constexpr int kLt = 20;              // between the columns of two fragments
    static constexpr int kLd = NF * kLt + 4;    // four rows 16 banks apart
    static constexpr int kSumsAt = 5 * kTM * 4;
    static constexpr int kCodesAt = kSumsAt + kWK * kTM * kLd * 4;
};

template <int BITS, typename XT, int MI, int NF, int WAVES, int STEPS, int SCHEME>
__global__ __launch_bounds__(64 * WAVES) void fused_kernel(SmallArgs a) {
    using L = FusedLayout<MI, NF, WAVES>;
    constexpr int TM = L::kTM, WK = L::kWK, kPairs = 8 * WAVES;   // pairs cast per step
    constexpr int NW = BITS == 8 ? 2 : 1;       // 1 KiB weight pieces per stage and wavefront
    constexpr int D = WK == 16 ? 2 : WK == 8 ? 3 : SCHEME == kQuantToken ? 5 : 4;   // stages in flight: all of K = 1152, or what registers allow
    constexpr int kStageBytes = BITS == 8 ? 8192 : 4096;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    uint32_t *const row_max = reinterpret_cast<uint32_t *>(lds);
    uint32_t *const row_min = row_max + TM;
    float *const lds_s = reinterpret_cast<float *>(lds) + 2 * TM, *const lds_r = lds_s + TM, *const lds_c = lds_r + TM;
    int *const sums = reinterpret_cast<int *>(lds + L::kSumsAt);
    uint8_t *const codes = lds + L::kCodesAt;
    // all arguments in one go: fetched where they are first needed, they are three round trips
    asm volatile("" ::"s"(a.X), "s"(a.x_tiled), "s"(a.x_scale), "s"(a.w_codes), "s"(a.w_scale), "s"(a.bias), "s"(a.Y), "s"(a.M),
                 "s"(a.N), "s"(a.K), "s"(a.KF), "s"(a.m_tiles), "s"(a.n_tiles), "s"(a.rows), "s"(a.groups), "s"(a.inv_groups), "s"(a.qmax), "s"(a.epi), "s"(a.out), "s"(a.rot), "s"(a.shift), "s"(a.x_corr), "s"(a.w_rowsum));

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, h = lane >> 4;
    const int wk = wave % WK, wn = wave / WK;

    // block b runs on XCD b % 8: the blocks of one XCD take consecutive tiles, token tile fastest, so
    // that they share weight tiles in its L2
    const int nb = a.m_tiles * a.n_tiles, b = blockIdx.x;
    const int v = (b % 8) * (nb / 8) + ((b % 8) < nb % 8 ? (b % 8) : nb % 8) + b / 8;
    const int mt = v % a.m_tiles, nt = v / a.m_tiles;
    const int64_t m0 = (int64_t)mt * TM;
    const int G = nt / (8 / NF), t0 = nt % (8 / NF) * NF;
    if ((int64_t)G * kTileN + t0 >= a.N) return;   // no live channel in this tile
    if (tid < TM) {
        row_max[tid] = 0;
        if (SCHEME == kQuantAsym) row_min[tid] = 0xffffffffu;
    }

    const int K = (int)a.K, KF = a.KF, pairs = a.rows * a.groups;
    const int sub = lane & 7, p0 = tid >> 3, piece = SCHEME == kQuantRotated ? rotation_label(sub) : sub;
    Group<XT> u[STEPS];
    int row[STEPS], col0[STEPS];
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        if (i > 0 && wave * 8 + i * kPairs >= pairs) continue;   // uniform over the wavefront
        const int p = p0 + i * kPairs < pairs ? p0 + i * kPairs : pairs - 1;
        row[i] = (int)((uint32_t)p * a.inv_groups >> 20);
        col0[i] = (p - row[i] * a.groups) * kGroup;
        const int64_t m = m0 + row[i] < a.M ? m0 + row[i] : a.M - 1;
        const XT *xrow = reinterpret_cast<const XT *>(a.X) + m * a.K;
        u[i].load_ragged(xrow, col0[i], K, piece);
    }

    // weights of this wavefront: stages wk, wk + WK, ..; a register ring of D of them
    v4i w[D][NW];
    const uint8_t *const wbase = a.w_codes + (int64_t)G * KF * kStageBytes + (t0 + 2 * wn) * (BITS == 8 ? kFragBytes : kFragBytes / 2);
    auto request = [&](int s, int d) {
        const uint8_t *p = wbase + (int64_t)(s < KF ? s : KF - 1) * kStageBytes;
#pragma unroll
        for (int j = 0; j < NW; ++j) w[d][j] = *reinterpret_cast<const v4i *>(p + j * kFragBytes + lane * 16);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(wk + d * WK, d);

    // what the epilogue needs: a thread keeps two channels, n0 and n0 + 1, and one or two tokens
    constexpr int JT = NF / 2, kRowsPerPass = 64 * WAVES / (16 * JT);
    const int ej = tid % JT, ec = tid / JT % 16, em = tid / (16 * JT);
    const int64_t n0 = (int64_t)G * kTileN + 8 * ec + t0 + 2 * ej;
    const int64_t na = n0 < a.N ? n0 : a.N - 1, nb2 = n0 + 1 < a.N ? n0 + 1 : a.N - 1;
    float sw0 = a.w_scale[na], sw1 = a.w_scale[nb2], bs0 = 0.0f, bs1 = 0.0f;
    if (a.bias) { bs0 = a.bias[na]; bs1 = a.bias[nb2]; }
    int rs0 = 0, rs1 = 0;
    if (SCHEME == kQuantAsym) { rs0 = a.w_rowsum[na]; rs1 = a.w_rowsum[nb2]; }

    // the maximum of each row, over the lanes of its pairs
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the zeros above are there; the loads stay in flight
    const Rotation<XT> rotation(a.rot, piece);
    float f[SCHEME == kQuantRotated ? STEPS : 1][kUnit];
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        if (i > 0 && wave * 8 + i * kPairs >= pairs) continue;
        if (K % kUnit) u[i].settle_ragged(col0[i], K, piece);
        if constexpr (SCHEME == kQuantAsym) {
            float lo = __builtin_inff(), hi = -__builtin_inff();
#pragma unroll
            for (int e = 0; e < kUnit; ++e) {
                lo = fminf(lo, u[i].get(e));
                hi = fmaxf(hi, u[i].get(e));
            }
            lo = min_of_eight(lo);
            hi = max_of_eight(hi);
            if (sub == 0) {
                atomicMin(row_min + row[i], ordered(lo));
                atomicMax(row_max + row[i], ordered(hi));
            }
        } else {
            float m = 0.0f;
            if constexpr (SCHEME == kQuantRotated) {
#pragma unroll
                for (int e = 0; e < kUnit; ++e) f[i][e] = u[i].get(e);
                rotation.apply(f[i], col0[i], K);
#pragma unroll
                for (int e = 0; e < kUnit; ++e) m = fmaxf(m, fabsf(f[i][e]));
            } else {
                auto running = Group<XT>::no_max();
                u[i].absmax_into(running);
                m = Group<XT>::absmax_value(running);
            }
            m = max_of_eight(m);   // no NaN, not negative: ordered like its bits
            if (sub == 0) atomicMax(row_max + (SCHEME == kQuantTensor ? 0 : row[i]), __float_as_uint(m));
        }
    }
    if constexpr (SCHEME == kQuantTensor) {
        if (a.m_tiles > 1) {   // the rows of the other tiles: every block reads the whole tensor
            constexpr int kPer = 16 / (int)sizeof(XT);
            const XT *const X = reinterpret_cast<const XT *>(a.X);
            const int n = (int)(a.M * a.K), nv = n / kPer;
            Bf16Max packed;
            float m = 0.0f;
            for (int base = tid; base < nv; base += 64 * WAVES * 4) {
                uint4 piece4[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {   // past the end the last piece again: the same maximum
                    const int at = base + 64 * WAVES * k;
                    piece4[k] = reinterpret_cast<const uint4 *>(X)[at < nv ? at : nv - 1];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t word[4] = {piece4[k].x, piece4[k].y, piece4[k].z, piece4[k].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (sizeof(XT) == 2) packed.fold(word[e]);
                        else m = fmaxf(m, fabsf(__uint_as_float(word[e])));
                    }
                }
            }
            if (tid < n - nv * kPer) {
                if constexpr (sizeof(XT) == 2) m = fmaxf(m, fabsf(__uint_as_float((uint32_t)X[nv * kPer + tid] << 16)));
                else m = fmaxf(m, fabsf(X[nv * kPer + tid]));
            }
            if constexpr (sizeof(XT) == 2) m = fmaxf(m, packed.value());
            m = max_of_eight(m);
            if (sub == 0) atomicMax(row_max, __float_as_uint(m));
        }
    }
    __syncthreads();
    const bool first_tile = nt == 0;   // one block per token tile leaves codes and scales in the workspace
    float s1 = 0.0f, r1 = 0.0f;
    if constexpr (STEPS > 1 || SCHEME != kQuantToken) {
        if (tid < a.rows) {
            const bool keep = first_tile && m0 + tid < a.M;
            float s, r;
            if constexpr (SCHEME == kQuantAsym) {
                const float lo = from_ordered(row_min[tid]), hi = from_ordered(row_max[tid]);
                s = fmaxf(hi - lo, kAbsmaxFloor) / a.qmax;
                r = 1.0f / s;   // correctly rounded
                const float corr = a.shift - -rintf(quotient(lo, s, r));   // minus the zero point
                lds_c[tid] = corr;
                if (keep) a.x_corr[m0 + tid] = corr;
            } else {
                s = scale_of(__uint_as_float(row_max[SCHEME == kQuantTensor ? 0 : tid]), a.qmax);
                r = 1.0f / s;   // correctly rounded
            }
            lds_s[tid] = s;
            lds_r[tid] = r;
            if (keep) a.x_scale[m0 + tid] = s;
        }
        __syncthreads();
    } else {
        s1 = scale_of(__uint_as_float(row_max[row[0]]), a.qmax);
        r1 = 1.0f / s1;
        if (sub == 0 && col0[0] == 0 && p0 < pairs) {
            lds_s[row[0]] = s1;
            if (first_tile && m0 + row[0] < a.M) a.x_scale[m0 + row[0]] = s1;
        }
    }
    const int qs = quarter_stride(a.rows);
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        if (i > 0 && wave * 8 + i * kPairs >= pairs) continue;
        constexpr bool kTable = STEPS > 1 || SCHEME != kQuantToken;
        float s = kTable ? lds_s[row[i]] : s1, r = kTable ? lds_r[row[i]] : r1;
        uint32_t q[4];
        if constexpr (SCHEME == kQuantAsym) {
            const float off = -lds_c[row[i]], cmin = -a.shift, cmax = a.qmax - a.shift;
#pragma unroll
            for (int d = 0; d < 4; ++d)
                q[d] = asym_codes4(quotient(u[i].get(4 * d + 0), s, r), quotient(u[i].get(4 * d + 1), s, r),
                                   quotient(u[i].get(4 * d + 2), s, r), quotient(u[i].get(4 * d + 3), s, r), off, cmin, cmax);
        } else {
            if constexpr (SCHEME == kQuantRotated) {
                const float sign = rotation.sign();
                s *= sign;
                r *= sign;
            }
            auto get = [&](int e) { return SCHEME == kQuantRotated ? f[SCHEME == kQuantRotated ? i : 0][e] : u[i].get(e); };
#pragma unroll
            for (int d = 0; d < 4; ++d)
                q[d] = codes4(quotient(get(4 * d + 0), s, r), quotient(get(4 * d + 1), s, r),
                              quotient(get(4 * d + 2), s, r), quotient(get(4 * d + 3), s, r));
        }
        const uint4 o = Group<XT>::gather_codes(q, piece);
        const int ui = col0[i] / kUnit + Group<XT>::unit_of(piece);   // unit = quarter of a stage
        if (p0 + i * kPairs < pairs && ui * kUnit < K) {
            *reinterpret_cast<uint4 *>(codes + ui * qs + row[i] * 16) = o;
            if (first_tile && m0 + row[i] < a.M)
                store16<false>(a.x_tiled + act_frag_offset(m0 + row[i], 0, KF) + (int64_t)(ui >> 2) * (4 * kFragBytes) + (ui & 3) * 256, o);
        }
    }
    __syncthreads();

    v4i acc[MI][2];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[i][t] = v4i{0, 0, 0, 0};
    const uint8_t *xl[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) xl[i] = codes + h * qs + (16 * i + c < a.rows ? 16 * i + c : a.rows - 1) * 16;
    auto multiply = [&](int s, int d) {   // stage s, in ring slot d
        v4i wt[2];
        if constexpr (BITS == 8) {
            wt[0] = w[d][0];
            wt[1] = w[d][1];
        } else {
            const v4i unit = w[d][0];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint32_t v0 = (uint32_t)unit[2 * t], v1 = (uint32_t)unit[2 * t + 1];
                wt[t][0] = (int)((v0 << 4) & 0xF0F0F0F0u);
                wt[t][1] = (int)(v0 & 0xF0F0F0F0u);
                wt[t][2] = (int)((v1 << 4) & 0xF0F0F0F0u);
                wt[t][3] = (int)(v1 & 0xF0F0F0F0u);
            }
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const v4i xa = *reinterpret_cast<const v4i *>(xl[i] + s * 4 * qs);
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, wt[t], acc[i][t], 0, 0, 0);
        }
    };
    int s = wk;
    for (; s + (2 * D - 1) * WK < KF; s += D * WK) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(s + d * WK, d);
            request(s + (d + D) * WK, d);
        }
    }
    if (s + D * WK < KF) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(s + d * WK, d);
            request(s + (d + D) * WK, d);
        }
        s += D * WK;
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (s + d * WK < KF) multiply(s + d * WK, d);

    // the wavefronts' partial sums meet in LDS (integers: exact in any order)
    int *const mine = sums + (wk * TM + 4 * h) * L::kLd + 2 * wn * L::kLt + c;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) mine[(16 * i + q) * L::kLd + t * L::kLt] = acc[i][t][q];
    __syncthreads();

    if (BITS == 4) { sw0 *= 0.0625f; sw1 *= 0.0625f; }   // operands carry codes times 16
    for (int m = em; m < TM && m0 + m < a.M && n0 < a.N; m += kRowsPerPass) {
        int raw0 = 0, raw1 = 0;
#pragma unroll
        for (int k = 0; k < WK; ++k) {
            const int *p = sums + (k * TM + m) * L::kLd + 2 * ej * L::kLt + ec;
            raw0 += p[0];
            raw1 += p[L::kLt];
        }
        const bool both = n0 + 1 < a.N;   // stored in one piece, at any alignment of Y's elements
        const int64_t at = (m0 + m) * a.N + n0;
        if (a.out == QC_OUT_I32_ACC) {
            int32_t *y = reinterpret_cast<int32_t *>(a.Y) + at;
            y[0] = BITS == 4 ? raw0 >> 4 : raw0;   // exact: multiples of 16
            if (both) y[1] = BITS == 4 ? raw1 >> 4 : raw1;
            continue;
        }
        const float sx = lds_s[m];
        float f0 = (float)raw0, f1 = (float)raw1;
        if constexpr (SCHEME == kQuantAsym) {
            f0 = fmaf(lds_c[m], (float)rs0 * (BITS == 4 ? 16.0f : 1.0f), f0);
            f1 = fmaf(lds_c[m], (float)rs1 * (BITS == 4 ? 16.0f : 1.0f), f1);
        }
        float y[2] = {fmaf(f0 * sx, sw0, bs0), fmaf(f1 * sx, sw1, bs1)};
        if (a.epi == QC_EPI_GELU_TANH) {
            y[0] = gelu_tanh_f(y[0]);
            y[1] = gelu_tanh_f(y[1]);
        } else if (a.epi == QC_EPI_GELU_ERF) {
            y[0] = gelu_erf_f(y[0]);
            y[1] = gelu_erf_f(y[1]);
        }
        if (a.out == QC_OUT_F32) {
            float *o = reinterpret_cast<float *>(a.Y) + at;
            if (both) __builtin_memcpy(o, y, sizeof(y));
            else o[0] = y[0];
        } else {
            uint16_t *o = reinterpret_cast<uint16_t *>(a.Y) + at;
            const uint32_t pk = pack_bf16x2(y[0], y[1]);
            if (both) __builtin_memcpy(o, &pk, sizeof(pk));
            else o[0] = (uint16_t)(pk & 0xffffu);
        }
    }
}

// A kernel may use 64 KiB of LDS without asking; this asks for more, once per kernel and device.
hipError_t allow_lds(const void *kernel, std::atomic<uint64_t> &asked) {
    int device = 0;
    if (hipError_t e = hipGetDevice(&device); e != hipSuccess) return e;
    const uint64_t bit = 1ull << (device & 63);
    if (device < 64 && (asked.load(std::memory_order_acquire) & bit)) return hipSuccess;
    if (hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMost); e != hipSuccess)
        return e;
    if (device < 64) asked.fetch_or(bit, std::memory_order_release);   // racing threads ask for the same
    return hipSuccess;
}

template <int BITS, int MI, int NF, int WN, int D>
hipError_t launch_tile(SmallArgs a, hipStream_t stream) {
    using L = Layout<MI, NF, WN>;
    a.m_tiles = (int)((a.M + L::kTM - 1) / L::kTM);
    a.n_tiles = (int)(round_up(a.N, kTileN) / kTileN) * (8 / NF);
    if (L::kSums > 64 * 1024) {
        static std::atomic<uint64_t> asked{0};
        if (hipError_t e = allow_lds((const void *)small_kernel<BITS, MI, NF, WN, D>, asked); e != hipSuccess) return e;
    }
    small_kernel<BITS, MI, NF, WN, D><<<dim3((unsigned)(a.m_tiles * a.n_tiles)), dim3(kThreads), L::kSums, stream>>>(a);
    return hipGetLastError();
}

// The tiles of small_kernel, smallest first: tokens and channels.
struct TileShape { int tokens, channels; };
constexpr TileShape kTiles[] = {{16, 32}, {32, 32}, {32, 64}, {64, 64}};
constexpr int kTileCount = 4;
constexpr int kCus = 256;

template <int BITS>
hipError_t launch_bits(int tile, const SmallArgs &a, hipStream_t stream) {
    switch (tile) {
        case 0: return launch_tile<BITS, 1, 2, 1, 4>(a, stream);
        case 1: return launch_tile<BITS, 2, 2, 1, 4>(a, stream);
        case 2: return launch_tile<BITS, 2, 4, 2, 4>(a, stream);
        default: return launch_tile<BITS, 4, 4, 2, 3>(a, stream);
    }
}

// Tiles with a channel below N.  A group of 128 channels is cut into tiles of NF = channels / 16 of every
// eight (channel 8 c + t belongs to tile t / NF), so all tiles of a last group with 8 channels are live.
int64_t live_channel_tiles(int64_t N, int channels) {
    const int64_t nf = channels / 16, per_group = 8 / nf, last = (N % kTileN + nf - 1) / nf;
    return N / kTileN * per_group + (last < per_group ? last : per_group);
}

// The smallest tile that leaves at most one block per CU, -1 if none does.  Measured, K = 1152
// (blocks of a tile: us): 128 x 1152: 16 x 32 tiles 288: 5.4, 32 x 32 tiles 144: 4.1; 256 x 1152: 32 x 32
// 288: 6.0, 32 x 64 144: 5.5; 512 x 1152: 32 x 64 288: 8.7, 64 x 64 144: 6.7; 1000 x 1152: 64 x 64 288:
// 12.0, the ring kernel 9.1.  Narrow outputs, whose channel tiles are all live: 8192 x 32: 32 x 32 1024:
// 24.0, 64 x 64 256 (not fused): 17.4; 16384 x 64: 64 x 64 512: 23.6, the ring kernel 18.1.
bool one_block_per_cu(int64_t M, int64_t N, TileShape t) {
    const int64_t mt = (M + t.tokens - 1) / t.tokens, nt = live_channel_tiles(N, t.channels);
    return mt <= kCus && nt <= kCus && mt * nt <= kCus;
}
int pick_tile(int64_t M, int64_t N) {
    for (int t = 0; t < kTileCount; ++t)
        if (one_block_per_cu(M, N, kTiles[t])) return t;
    return -1;
}

// The same for fused_kernel, -1 if two launches are the better or the only way: the smallest tile again, with eight
// wavefronts while each lane has at most three pairs of a row and a group to cast.  us in a graph, 8 and 16
// wavefronts: 2 x 1152 x 6912 4.9 6.3, 64 x 1152 x 1152 5.2 6.1, 128 x 1152 x 1152 (16 x 64) 5.6 5.9, 200 x 640 x 1152
// 4.8 5.8, 256 x 1152 x 1152 (16 x 128) 6.9 6.7.  Tiles of 32 tokens, two launches and one: 512 x 1152 x 1152
// 10.9 9.8, 700 tokens 11.0 10.3, K = 1536, 600 tokens 11.2 12.1: up to nine groups a row.  The other quantizers, in two
// launches (one scale for the tensor: three) and one, rotated, asymmetric, tensor: 2 x 1152 x 6912 8.0 5.1, 7.7 5.0, 8.8
// 4.8; 64 x 1152 x 1152 7.6 6.1, 7.3 5.8, 8.9 7.5; 256 x 1152 x 1152 10.1 7.2, 10.4 7.1.
// The longest rows on 16 x 32 tiles, the same input again and again | four in turn: 32 x 2816 x 4096 8.2 8.3 | 9.4 8.7, K = 2944 8.2 8.8
// | 9.3 9.3, 4 bit 7.7 8.5 | 8.5 8.8: up to 22 groups on 16 rows (10 rows of 36 gain again, 0.91 of the time in two).  Where
// an XCD's L2 does not hold X beside the weights, what each of four channel tiles or more reads of it again comes from further away:
// binary32 687 x 2560 x 565 13.6 13.5 | 12.9 14.0, K = 2912 14.2 15.8 | 13.2 16.0, 991 x 2688 x 46 11.2 13.3 | 10.3 13.5; bf16 991 x 3072 x 46 11.4
// 11.2 | 9.7 12.4; but two or three channel tiles, 1091 x 2688 x 92, 11.5 8.9 | 10.5 10.1: up to 27 MB of it in all, asymmetric,
// where a launch of the quantizer costs more, 34 (420 x 3024 x 1152, 43 MB, 13.8 16.3 | 13.1 15.9).  Tiles
// of 32 tokens, whose rows are short, at any size (over 98 drawn calls one launch 0.88 | 1.05 of two).
struct FusedShape { TileShape tile; int waves, pairs; bool all_schemes; };   // pairs: most pairs of a row and a group that it is taken for
constexpr FusedShape kFusedShapes[] = {{{16, 32}, 8, 192, true},   {{16, 32}, 16, 384, false}, {{16, 64}, 8, 192, true},
                                       {{16, 64}, 16, 384, false}, {{16, 128}, 16, 384, true}, {{32, 128}, 16, 288, false}};
constexpr int kFusedShapeCount = 6;
constexpr int64_t kTensorMost = 320 << 10;   // bytes of X that every block may read for one scale for the tensor: 115 x 1152 x 3456 11.5 9.3 us
int pick_fused_shape(int64_t M, int64_t N, int64_t K, size_t x_elem_bytes, QuantScheme scheme) {
    if (K < 8 || K > QC_MAX_K) return -1;   // a row of less than 16 B has no whole piece to load
    if (scheme == kQuantAsym && !quant_vector_path(K)) return -1;
    int tile = 0;   // the smallest that gives at most one block per CU
    while (tile < kFusedShapeCount && !one_block_per_cu(M, N, kFusedShapes[tile].tile)) ++tile;
    for (int i = tile; i < kFusedShapeCount; ++i) {
        const FusedShape &f = kFusedShapes[i];
        if (f.tile.tokens != kFusedShapes[tile].tile.tokens || f.tile.channels != kFusedShapes[tile].tile.channels) break;
        if (scheme != kQuantToken && !f.all_schemes) continue;
        if (scheme == kQuantTensor && M > f.tile.tokens && M * K * (int64_t)x_elem_bytes > kTensorMost) continue;
        const int64_t rows = M < f.tile.tokens ? M : f.tile.tokens, groups = (K + kGroup - 1) / kGroup;
        if (rows * groups > f.pairs) continue;
        if (rows == 16 && f.tile.channels == 32 && groups > 22) continue;
        const int64_t x_bytes = M * K * (int64_t)x_elem_bytes, readers = live_channel_tiles(N, f.tile.channels);
        if (f.tile.tokens == 16 && readers >= 4 && x_bytes > 3 << 20 && readers * x_bytes > (scheme == kQuantAsym ? 34 : 27) << 20) continue;
        return i;
    }
    return -1;
}

template <int BITS, typename XT, int MI, int NF, int WAVES, int STEPS, int SCHEME>
hipError_t launch_fused_steps(const SmallArgs &a, size_t lds, hipStream_t stream) {
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> asked{0};
        if (hipError_t e = allow_lds((const void *)fused_kernel<BITS, XT, MI, NF, WAVES, STEPS, SCHEME>, asked); e != hipSuccess) return e;
    }
    fused_kernel<BITS, XT, MI, NF, WAVES, STEPS, SCHEME><<<dim3((unsigned)(a.m_tiles * a.n_tiles)), dim3(64 * WAVES), lds, stream>>>(a);
    return hipGetLastError();
}

template <int BITS, typename XT, int MI, int NF, int WAVES, int SCHEME>
hipError_t launch_fused(SmallArgs a, hipStream_t stream) {
    using L = FusedLayout<MI, NF, WAVES>;
    a.m_tiles = (int)((a.M + L::kTM - 1) / L::kTM);
    a.n_tiles = (int)(round_up(a.N, kTileN) / kTileN) * (8 / NF);
    a.rows = (int)(a.M < L::kTM ? a.M : L::kTM);
    a.groups = (int)((a.K + kGroup - 1) / kGroup);
    a.inv_groups = ((1u << 20) + a.groups - 1) / a.groups;   // exact for pairs below 384
    // 384 groups at most, so that the codes, 16 B per unit of 16 columns and row and 16 B of padding per unit, take
    // 96 KiB at most, with one row, and less than kLdsMost together with the sums (140 KiB on tiles of 16 x 32)
    static_assert(MI > 1 || L::kCodesAt + 96 * 1024 <= kLdsMost, "the longest rows fit");
    const size_t lds = L::kCodesAt + (size_t)a.KF * 4 * quarter_stride(a.rows);
    if (lds > (size_t)kLdsMost) return hipErrorInvalidValue;
    if constexpr (SCHEME == kQuantToken) {   // (the others: three steps whatever the rows)
        if (a.rows * a.groups <= 8 * WAVES) return launch_fused_steps<BITS, XT, MI, NF, WAVES, 1, SCHEME>(a, lds, stream);
    }
    return launch_fused_steps<BITS, XT, MI, NF, WAVES, kStepsMost, SCHEME>(a, lds, stream);
}

template <int BITS, typename XT, int SCHEME>
hipError_t launch_fused_scheme(int shape, const SmallArgs &a, hipStream_t stream) {
    switch (shape) {
        case 0: return launch_fused<BITS, XT, 1, 2, 8, SCHEME>(a, stream);
        case 2: return launch_fused<BITS, XT, 1, 4, 8, SCHEME>(a, stream);
        case 4: return launch_fused<BITS, XT, 1, 8, 16, SCHEME>(a, stream);
    }
    if constexpr (SCHEME == kQuantToken) {
        switch (shape) {
            case 1: return launch_fused<BITS, XT, 1, 2, 16, SCHEME>(a, stream);
            case 3: return launch_fused<BITS, XT, 1, 4, 16, SCHEME>(a, stream);
            default: return launch_fused<BITS, XT, 2, 8, 16, SCHEME>(a, stream);
        }
    }
    return hipErrorInvalidValue;
}

template <int BITS, typename XT>
hipError_t launch_fused_shape(int shape, QuantScheme scheme, const SmallArgs &a, hipStream_t stream) {
    switch (scheme) {
        case kQuantToken: return launch_fused_scheme<BITS, XT, kQuantToken>(shape, a, stream);
        case kQuantRotated: return launch_fused_scheme<BITS, XT, kQuantRotated>(shape, a, stream);
        case kQuantAsym: return launch_fused_scheme<BITS, XT, kQuantAsym>(shape, a, stream);
        default: return launch_fused_scheme<BITS, XT, kQuantTensor>(shape, a, stream);
    }
}

SmallArgs small_args(uint8_t *x_tiled, float *x_scale, const uint8_t *w_packed, const float *w_scale,
                     const float *bias, void *Y, int64_t M, int64_t N, int64_t K, qc_epilogue epi, qc_out ydt) {
    SmallArgs a{};
    a.x_tiled = x_tiled;
    a.x_scale = x_scale;
    a.w_codes = w_packed + kPackedHeaderBytes;
    a.w_scale = w_scale;
    a.bias = bias;
    a.Y = Y;
    a.M = M;
    a.N = N;
    a.K = K;
    a.KF = (int)(round_up(K, kKAlign) / kFragK);
    a.epi = epi;
    a.out = ydt;
    return a;
}

}  // namespace

bool gemm_small_chosen(int64_t M, int64_t N) { return pick_tile(M, N) >= 0; }

int gemm_small_tokens(int64_t M, int64_t N) { return kTiles[pick_tile(M, N)].tokens; }

hipError_t launch_gemm_small(const uint8_t *x_tiled, const float *x_scale, const uint8_t *w_packed,
                             const float *w_scale, const float *bias, void *Y, int64_t M, int64_t N,
                             int64_t K, int bits, qc_epilogue epi, qc_out ydt, const float *x_corr,
                             const int32_t *w_rowsum, hipStream_t stream) {
    const int tile = pick_tile(M, N);
    if (tile < 0) return hipErrorInvalidValue;
    SmallArgs a = small_args(const_cast<uint8_t *>(x_tiled), const_cast<float *>(x_scale), w_packed, w_scale,
                             bias, Y, M, N, K, epi, ydt);   // small_kernel only reads both
    if (x_corr && w_rowsum) {
        a.x_corr = const_cast<float *>(x_corr);
        a.w_rowsum = w_rowsum;
    }
    return bits == 8 ? launch_bits<8>(tile, a, stream) : launch_bits<4>(tile, a, stream);
}

bool qlinear_small_chosen(int64_t M, int64_t N, int64_t K, qc_dtype xdt, QuantScheme scheme) {
    return pick_fused_shape(M, N, K, xdt == QC_BF16 ? 2 : 4, scheme) >= 0;
}

int qlinear_small_tokens(int64_t M, int64_t N, int64_t K, qc_dtype xdt, QuantScheme scheme) {
    return kFusedShapes[pick_fused_shape(M, N, K, xdt == QC_BF16 ? 2 : 4, scheme)].tile.tokens;
}

hipError_t launch_qlinear_small(const void *X, qc_dtype xdt, uint8_t *x_tiled, float *x_scale, float *x_corr,
                                const uint8_t *w_packed, const float *w_scale, const int32_t *w_rowsum, const float *bias,
                                void *Y, int64_t M, int64_t N, int64_t K, QuantScheme scheme, int act_bits, int rot_block,
                                int bits, qc_epilogue epi, qc_out ydt, hipStream_t stream) {
    const int shape = pick_fused_shape(M, N, K, xdt == QC_BF16 ? 2 : 4, scheme);
    if (shape < 0) return hipErrorInvalidValue;
    SmallArgs a = small_args(x_tiled, x_scale, w_packed, w_scale, bias, Y, M, N, K, epi, ydt);
    a.X = X;
    a.x_corr = x_corr;
    a.w_rowsum = w_rowsum;
    a.qmax = (float)(scheme == kQuantAsym ? (1 << act_bits) - 1 : (1 << (act_bits - 1)) - 1);
    a.shift = (float)asym_code_shift(act_bits);
    a.rot = rot_block;
    if (xdt == QC_BF16)
        return bits == 8 ? launch_fused_shape<8, uint16_t>(shape, scheme, a, stream) : launch_fused_shape<4, uint16_t>(shape, scheme, a, stream);
    return bits == 8 ? launch_fused_shape<8, float>(shape, scheme, a, stream) : launch_fused_shape<4, float>(shape, scheme, a, stream);
}

}  // namespace qc
