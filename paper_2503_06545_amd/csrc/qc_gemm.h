// What the rules of the GEMM (qc_gemm.hip) and its kernels (qc_gemm_kernels.h, compiled for 8-bit and for
// 4-bit weights by qc_gemm_w8.hip and qc_gemm_w4.hip) share.
#pragma once

#include "qc_internal.h"

namespace qc {

template <int BITS>
struct StageLayout {
    // Only the weight tile goes through LDS (all four wavefronts use all of it).  1 KiB pieces
    // per 64-k stage: 8 bit one fragment per block of 16 channels; 4 bit one nibble unit per
    // two such blocks.
    static constexpr int kWFrags = BITS == 8 ? kTileN / kFragRows : kTileN / kFragRows / 2;
    static constexpr int kBytes = kWFrags * kFragBytes;
    static constexpr int kFragsPerWave = kWFrags / 4;
    static_assert(kWFrags % 4 == 0, "fragments must split evenly over 4 wavefronts");
};

struct GemmArgs {
    const uint8_t *x_tiled;
    const float *x_scale;   // Mp entries (padded), 16 B aligned
    const float *x_corr;    // asymmetric activations only: per token code shift - zero point, Mp entries
    const int32_t *w_rowsum;  // asymmetric activations only: per channel sum of the weight codes
    const uint8_t *w_codes;
    const float *w_scale;
    const float *bias;
    void *Y;
    int64_t M, N;
    int KF;         // 64-k stages (Kp / 64)
    int m_tiles, n_tiles;   // m_tiles: of 64 * height tokens
    int x_frags;    // blocks of 16 tokens in the workspace (Mp / 16)
    int group_m;    // token tiles per patch of the block -> tile map (ring kernel)
    bool resident;  // run the kernel that keeps the weight tile in LDS
    int height;     // ring kernel: 4, 3 or 2 blocks of 16 tokens per wavefront
    bool split;     // ring kernel, height 4 or 2: two groups of wavefronts, half of the reduction each
    bool keep_output;  // ring kernel, f32 output: the kernel that stores through the caches
    bool stream_edges; // bf16 output: non-temporal stores also for rows and tiles that are not whole
};

constexpr int kResThreads = 512;
constexpr int kResWaves = kResThreads / 64;
static_assert(kRoundTokens == kResWaves * kWaveM, "a round is one 64-token tile per wavefront");

// LDS of the resident kernel, a fixed layout whatever K is (one block per CU has the CU's 160 KiB
// to itself, and a static size needs no launch attribute): the weight tile, 128 channel scales,
// biases and code sums, 64 token scales and corrections per wavefront.
constexpr int kResWeightBytes = 18 * 8192;   // 128 channels x 1152 k of 8-bit codes, x 2304 k of 4-bit ones
constexpr int kResLdsBytes = kResWeightBytes + 3 * kTileN * (int)sizeof(float) + 2 * kResWaves * kWaveM * (int)sizeof(float);
static_assert(kResLdsBytes <= 160 * 1024, "more than the LDS of a CU");

constexpr int kResBlocks = 256;   // one block per CU

template <int BITS>
hipError_t launch_gemm_kernel(const GemmArgs &args, qc_epilogue epi, qc_out ydt, hipStream_t stream);
extern template hipError_t launch_gemm_kernel<8>(const GemmArgs &, qc_epilogue, qc_out, hipStream_t);
extern template hipError_t launch_gemm_kernel<4>(const GemmArgs &, qc_epilogue, qc_out, hipStream_t);

}  // namespace qc
