// The quantized linear on few tokens (Section 4.1 "Hardware Implementation"): too few output tiles of
// 256 x 128 to fill the chip, so what bounds the call is latency - the number of launches, each
// wavefront's chain of loads - and how many CUs pull the weights at once.
//
// A block of 8 wavefronts computes a tile of 16 or 32 or 64 tokens x 32 or 64 channels.  The
// wavefronts split the reduction (64-k stages dealt round-robin), load their operand fragments
// straight into registers, all of them ahead of the first use when K is short, and add their partial
// sums through LDS: exact, the sums are integers.  The smallest tile that gives at most one block per
// CU is taken: a second block on a CU only adds to what the CU has to load, and a single CU gets
// about 35 B/clk from beyond its L2 (every launch starts with that L2 invalid).
//
// For per-token quantization the whole linear is one launch: each block quantizes its token tile into
// LDS itself, redundantly over the channel tiles (that is cheap while there are few), and the blocks
// of the first channel tile leave codes and scales in the workspace as the two-launch path does.
//
// Measured, K = 1152, W8, GPU time of quantization + GEMM: 2 tokens x 6912 channels 4.7 + 8.2 -> 5.1
// us, 64 x 1152 2.8 + 8.8 -> 5.5 us, 256 x 1152 2.8 + 8.8 -> 7.8 us; K = 4608: 2 x 1152 5.0 + 24.1 ->
// 6.1 us, 256 x 1152 4.2 + 25.0 -> 4.2 + 8.5 us (a 256-token tile there walks 72 stages alone).
#include <atomic>

#include "qc_device.h"

namespace qc {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int kGroup = 128;   // columns that eight lanes quantize per step
constexpr int kWaves = kThreads / 64;
constexpr int kLdsMost = 150 * 1024;

enum Source { kCodes = 0, kFusedBf16 = 1, kFusedF32 = 2 };

struct SmallArgs {
    const void *X;          // fused quantizer: the activations
    uint8_t *x_tiled;       // the workspace's codes: read (kCodes) or written (fused)
    float *x_scale;
    const float *x_corr;    // asymmetric activations only, with w_rowsum
    const int32_t *w_rowsum;
    const uint8_t *w_codes;
    const float *w_scale;
    const float *bias;
    void *Y;
    int64_t M, N, K;
    int KF, m_tiles, n_tiles;
    int rp_log2;            // fused: rows of a tile that can be live, rounded up to a power of two
    float qmax;
    int epi, out;
};

// LDS: [ token scales: TM ][ wavefront maxima: 8 ][ codes, later partial sums: WK x TM x LD int32 ]
template <int MI, int NF, int WN>
struct Layout {
    static constexpr int kTM = 16 * MI;
    static constexpr int kWK = kWaves / WN;
    static constexpr int kLd = 16 * NF + 4;   // 4 rows apart = 16 banks apart: conflict-free
    static constexpr int kSums = kWK * kTM * kLd * 4;
    static constexpr int kSumsAt = (kTM * 4 + kWaves * 4 + 15) / 16 * 16;
};
// bytes between the 16-k quarters of a stage in the fused kernel's code tile: 16 B per row and 16 B
// of padding, so that the quarters a row's units go to fall into different banks
__host__ __device__ inline int quarter_stride(int rp_log2) { return (16 << rp_log2) + 16; }

// MI x 16 tokens by NF x 16 channels per block; WN wavefront columns, kWaves / WN ways over K; a
// register ring of D stages.  UPT: groups of 128 columns a thread quantizes (fused only).
template <int BITS, int MI, int NF, int WN, int D, int SRC, int UPT>
__global__ __launch_bounds__(kThreads, 2) void small_kernel(SmallArgs a) {
    using L = Layout<MI, NF, WN>;
    constexpr int TM = L::kTM, WK = L::kWK, NFW = NF / WN;
    constexpr int NW = BITS == 8 ? NFW : NFW / 2;             // 1 KiB weight pieces per stage and wavefront
    constexpr int kStageBytes = BITS == 8 ? 8192 : 4096;
    constexpr bool FUSED = SRC != kCodes;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    float *const lds_sx = reinterpret_cast<float *>(lds);
    float *const lds_max = lds_sx + TM;
    uint8_t *const codes = lds + L::kSumsAt;
    int *const sums = reinterpret_cast<int *>(codes);

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
    typedef typename std::conditional<SRC == kFusedF32, float, uint16_t>::type XT;
    Group<XT> u[FUSED ? UPT : 1];
    const int tpr_log2 = 9 - a.rp_log2, tpr = 1 << tpr_log2;   // threads per row, 8 or more
    const int row = tid >> tpr_log2, sub = lane & 7;
    const int group0 = (tid & (tpr - 1)) >> 3, groups_per_step = tpr >> 3;
    const bool live = m0 + row < a.M;
    if constexpr (FUSED) {
        const XT *xrow = reinterpret_cast<const XT *>(a.X) + (live ? m0 + row : m0) * a.K;
        if (a.K % kUnit == 0) {
#pragma unroll
            for (int i = 0; i < UPT; ++i)
                u[i].template load<false>(xrow, (group0 + i * groups_per_step) * kGroup, (int)a.K, sub);
        } else {
#pragma unroll
            for (int i = 0; i < UPT; ++i) u[i].load_ragged(xrow, (group0 + i * groups_per_step) * kGroup, (int)a.K, sub);
        }
    }

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
        sx[j] = FUSED ? 0.0f : a.x_scale[m0 + (em + 32 * j) % TM];
        cx[j] = 0.0f;
    }
    if (!FUSED && a.x_corr) {
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
    v4i x[FUSED ? 1 : D][MI];
    const uint8_t *const wbase = a.w_codes + (int64_t)G * KF * kStageBytes +
                                 (BITS == 8 ? t0 + wn * NFW : (t0 + wn * NFW) / 2) * kFragBytes + lane * 16;
    const uint8_t *const xbase = a.x_tiled + (m0 / kWaveM) * (int64_t)KF * (4 * kFragBytes) +
                                 (m0 % kWaveM) / kFragRows * kFragBytes + lane * 16;
    auto request = [&](int s, int d) {
        const int sc = s < KF ? s : KF - 1;
        const uint8_t *p = wbase + (int64_t)sc * kStageBytes;
#pragma unroll
        for (int j = 0; j < NW; ++j) w[d][j] = *reinterpret_cast<const v4i *>(p + j * kFragBytes);
        if constexpr (!FUSED) {
            const uint8_t *q = xbase + (int64_t)sc * (4 * kFragBytes);
#pragma unroll
            for (int i = 0; i < MI; ++i) x[d][i] = *reinterpret_cast<const v4i *>(q + i * kFragBytes);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(wk + d * WK, d);

    const int qs = quarter_stride(a.rp_log2);
    if constexpr (FUSED) {
        auto running = Group<XT>::no_max();
#pragma unroll
        for (int i = 0; i < UPT; ++i) u[i].absmax_into(running);
        float amax = Group<XT>::absmax_value(running);
        for (int d = 1; d < tpr && d < 64; d <<= 1) amax = fmaxf(amax, __shfl_xor(amax, d));
        if (tpr > 64) {   // a row spans several wavefronts
            if (lane == 0) lds_max[wave] = amax;
            __syncthreads();
            const int first = row << (tpr_log2 - 6);
            for (int j = 0; j < tpr / 64; ++j) amax = fmaxf(amax, lds_max[first + j]);
        }
        const float s = scale_of(amax, a.qmax);
        const float r = 1.0f / s;  // correctly rounded
        const bool keep = nt == 0 && live;   // one block per token tile leaves the codes in the workspace
        if ((tid & (tpr - 1)) == 0) {
            lds_sx[row] = s;
            if (keep) a.x_scale[m0 + row] = s;
        }
        uint8_t *out_tiled = a.x_tiled + act_frag_offset(m0 + row, 0, KF);
#pragma unroll
        for (int i = 0; i < UPT; ++i) {
            const int g = group0 + i * groups_per_step;
            if (g * kGroup >= (int)a.K) break;   // the same for the eight lanes of a group
            uint32_t q[4];
#pragma unroll
            for (int d = 0; d < 4; ++d)
                q[d] = codes4(quotient(u[i].get(4 * d + 0), s, r), quotient(u[i].get(4 * d + 1), s, r),
                              quotient(u[i].get(4 * d + 2), s, r), quotient(u[i].get(4 * d + 3), s, r));
            const uint4 o = Group<XT>::gather_codes(q, sub);
            const int ui = g * 8 + Group<XT>::unit_of(sub);
            if (ui * kUnit >= (int)a.K) continue;
            *reinterpret_cast<uint4 *>(codes + ui * qs + row * 16) = o;   // unit = quarter of a stage
            if (keep) store16<false>(out_tiled + (int64_t)(ui >> 2) * (4 * kFragBytes) + (ui & 3) * 256, o);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kRows; ++j) sx[j] = lds_sx[(em + 32 * j) % TM];
    }

    v4i acc[MI][NFW];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int t = 0; t < NFW; ++t) acc[i][t] = v4i{0, 0, 0, 0};

    const uint8_t *const xl = codes + h * qs;
    const int rmask = (1 << a.rp_log2) - 1;
    auto multiply = [&](int s, int d) {   // stage s, in ring slot d
        v4i xa[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
            xa[i] = FUSED ? *reinterpret_cast<const v4i *>(xl + s * 4 * qs + ((16 * i + c) & rmask) * 16) : x[FUSED ? 0 : d][i];
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
                acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i], wt, acc[i][t], 0, 0, 0);
        }
    };
    // Stages wk, wk + WK, ..: the loads are unconditional wherever there are any (past the end they
    // repeat the last stage), so that the compiler's waits count exactly.
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
    if constexpr (FUSED) __syncthreads();   // in the place of the codes
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
            if (!FUSED && a.x_corr) af = fmaf(cx[j], rs[t], af);
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

int live_rows_log2(int64_t M, int tile) {   // rows of a tile that can be live, as a power of two
    int r = 0;
    while ((1 << r) < tile && (1 << r) < M) ++r;
    return r;
}

template <int BITS, int MI, int NF, int WN, int D, int SRC, int UPT>
hipError_t launch_tile(SmallArgs a, hipStream_t stream) {
    using L = Layout<MI, NF, WN>;
    a.m_tiles = (int)((a.M + L::kTM - 1) / L::kTM);
    a.n_tiles = (int)(round_up(a.N, kTileN) / kTileN) * (8 / NF);
    a.rp_log2 = live_rows_log2(a.M, L::kTM);
    const size_t codes = SRC != kCodes ? (size_t)a.KF * 4 * quarter_stride(a.rp_log2) : 0;
    const size_t lds = L::kSumsAt + (codes > (size_t)L::kSums ? codes : (size_t)L::kSums);
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> asked{0};
        if (hipError_t e = allow_lds((const void *)small_kernel<BITS, MI, NF, WN, D, SRC, UPT>, asked); e != hipSuccess) return e;
    }
    small_kernel<BITS, MI, NF, WN, D, SRC, UPT>
        <<<dim3((unsigned)(a.m_tiles * a.n_tiles)), dim3(kThreads), lds, stream>>>(a);
    return hipGetLastError();
}

// The tiles, smallest first: tokens, channels, and for the fused form how many groups of 128 columns
// a thread may hold.  The 64-token tile is not fused: its blocks would spend longer on the
// redundant quantization than a launch of its own takes (512 x 1152: 11.2 against 2.9 + 6.7 us).
struct TileShape { int tokens, channels, upt; };
constexpr TileShape kTiles[] = {{16, 32, 3}, {32, 32, 5}, {32, 64, 5}, {64, 64, 0}};
constexpr int kTileCount = 4;
constexpr int kCus = 256;

template <int BITS>
hipError_t launch_bits(int tile, int src, const SmallArgs &a, hipStream_t stream) {
    if (src == kCodes) {
        switch (tile) {
            case 0: return launch_tile<BITS, 1, 2, 1, 4, kCodes, 1>(a, stream);
            case 1: return launch_tile<BITS, 2, 2, 1, 4, kCodes, 1>(a, stream);
            case 2: return launch_tile<BITS, 2, 4, 2, 4, kCodes, 1>(a, stream);
            default: return launch_tile<BITS, 4, 4, 2, 3, kCodes, 1>(a, stream);
        }
    }
    if (src == kFusedBf16) {
        switch (tile) {
            case 0: return launch_tile<BITS, 1, 2, 1, 4, kFusedBf16, kTiles[0].upt>(a, stream);
            case 1: return launch_tile<BITS, 2, 2, 1, 4, kFusedBf16, kTiles[1].upt>(a, stream);
            default: return launch_tile<BITS, 2, 4, 2, 4, kFusedBf16, kTiles[2].upt>(a, stream);
        }
    }
    switch (tile) {
        case 0: return launch_tile<BITS, 1, 2, 1, 4, kFusedF32, kTiles[0].upt>(a, stream);
        case 1: return launch_tile<BITS, 2, 2, 1, 4, kFusedF32, kTiles[1].upt>(a, stream);
        default: return launch_tile<BITS, 2, 4, 2, 4, kFusedF32, kTiles[2].upt>(a, stream);
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
int pick_tile(int64_t M, int64_t N) {
    for (int t = 0; t < kTileCount; ++t) {
        const int64_t mt = (M + kTiles[t].tokens - 1) / kTiles[t].tokens, nt = live_channel_tiles(N, kTiles[t].channels);
        if (mt <= kCus && nt <= kCus && mt * nt <= kCus) return t;
    }
    return -1;
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

hipError_t launch_gemm_small(const uint8_t *x_tiled, const float *x_scale, const uint8_t *w_packed,
                             const float *w_scale, const float *bias, void *Y, int64_t M, int64_t N,
                             int64_t K, int bits, qc_epilogue epi, qc_out ydt, const float *x_corr,
                             const int32_t *w_rowsum, hipStream_t stream) {
    const int tile = pick_tile(M, N);
    if (tile < 0) return hipErrorInvalidValue;
    SmallArgs a = small_args(const_cast<uint8_t *>(x_tiled), const_cast<float *>(x_scale), w_packed, w_scale,
                             bias, Y, M, N, K, epi, ydt);   // kCodes reads both
    if (x_corr && w_rowsum) {
        a.x_corr = x_corr;
        a.w_rowsum = w_rowsum;
    }
    return bits == 8 ? launch_bits<8>(tile, kCodes, a, stream) : launch_bits<4>(tile, kCodes, a, stream);
}

// What limits the fused form, beyond the tile: the columns a thread holds.  They bound its codes in LDS too,
// 16 B per unit of 16 columns and live row and 16 B of padding per unit: at most 81 KiB, with one row of
// 40960 columns, far below kLdsMost.
bool qlinear_small_chosen(int64_t M, int64_t N, int64_t K) {
    const int tile = pick_tile(M, N);
    if (tile < 0 || kTiles[tile].upt == 0) return false;
    const int rp_log2 = live_rows_log2(M, kTiles[tile].tokens);
    const int64_t columns = (int64_t)kTiles[tile].upt * kUnit * (kThreads >> rp_log2);
    return K <= columns;
}

hipError_t launch_qlinear_small(const void *X, qc_dtype xdt, uint8_t *x_tiled, float *x_scale,
                                const uint8_t *w_packed, const float *w_scale, const float *bias, void *Y,
                                int64_t M, int64_t N, int64_t K, int act_bits, int bits, qc_epilogue epi,
                                qc_out ydt, hipStream_t stream) {
    if (!qlinear_small_chosen(M, N, K)) return hipErrorInvalidValue;
    SmallArgs a = small_args(x_tiled, x_scale, w_packed, w_scale, bias, Y, M, N, K, epi, ydt);
    a.X = X;
    a.qmax = (float)((1 << (act_bits - 1)) - 1);
    const int src = xdt == QC_BF16 ? kFusedBf16 : kFusedF32, tile = pick_tile(M, N);
    return bits == 8 ? launch_bits<8>(tile, src, a, stream) : launch_bits<4>(tile, src, a, stream);
}

}  // namespace qc
