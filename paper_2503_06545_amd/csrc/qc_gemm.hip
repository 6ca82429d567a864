// Which kernel the integer GEMM runs, with tiles of what height and with what kind of stores
// (Section 4.1 "Hardware Implementation"); the kernels themselves: qc_gemm_kernels.h.
#include "qc_gemm.h"

namespace qc {

bool gemm_resident_fits(int64_t K, int bits) {
    const int64_t KF = round_up(K, kKAlign) / kFragK;
    return KF * (bits == 8 ? StageLayout<8>::kBytes : StageLayout<4>::kBytes) <= kResWeightBytes;
}

// The resident kernel is taken when the weight tile fits, the blocks get 6 rounds or more on
// average and the static schedule is within 4 % of an even split.  Measured against the ring
// kernel at K = 1152 (rounds per block: gain): 3.4: -9 %, 4.5: -6 % (the weight tile a block loads
// first and its last, partly idle rounds weigh too much), 6.8: +3.5 %, 9: 0 to +2.5 %, 13.5: +4 %,
// 18: +2 to +9 %, 27 (QKV at M = 131072): 434 -> 420 us, 36 (fc1 + GELU): 650 -> 625 us; K = 384,
// 36 rounds: +10 %.
bool gemm_resident_chosen(int64_t M, int64_t N, int64_t K, int bits) {
    if (!gemm_resident_fits(K, bits)) return false;
    const int m_tiles = (int)(round_up(M, kTileM) / kTileM), n_tiles = (int)(round_up(N, kTileN) / kTileN);
    const int64_t total = (int64_t)n_tiles * resident_chunks(m_tiles);
    if (total < 6 * kResBlocks) return false;
    int most = 0, seen[2] = {-1, -1};   // the XCDs' chunk counts differ by one at most
    for (int xcd = 0; xcd < 8; ++xcd) {
        const ResidentXcd x = resident_xcd(xcd, kResBlocks, resident_chunks(m_tiles));
        const int cx = x.c_hi - x.c_lo;
        if (cx == seen[0] || cx == seen[1]) continue;
        seen[seen[0] < 0 ? 0 : 1] = cx;
        for (int slot = 0; slot < x.blocks; ++slot) {
            const int r = resident_block_rounds(xcd + 8 * slot, kResBlocks, n_tiles, m_tiles, nullptr, 0);
            most = r > most ? r : most;
        }
    }
    return (int64_t)most * kResBlocks * 100 <= total * 104;
}

// Its one block per CU hides less of a GELU, or of an output that is long for the reduction, than two of the ring kernel's,
// which take its place for GELU (erf) (us under sustained load, ring and resident: 65536 x 1152 x 4608 375 382, 131072 x 384 x
// 4608 483 514), for GELU (tanh) to bf16 with 4-bit weights (131072 x 1152 x 4608 658 668) or a short
// reduction (K = 384 374 379; K = 1152, 8-bit weights 661 629), for GELU (tanh) to f32 (59454 x 1152 x 4608 416 463, 131072 x 1152 x
// 1152 238 272, 40000 x 768 x 2304 125 137) and for f32 with a short reduction (60000 x 768 x 4608 343 390, 131072 x 768 x 2304 382
// 422; K = 1152, 65536 x 4608, 427 403; with a zero point and 8-bit weights only up to K = 576: 81720 x
// 768 x 3456 420 348, 90440 x 688 x 3984 547 487).  In bursts of a few calls the ring kernel gains 5 % more.
static bool gemm_resident_epilogue(int64_t K, int bits, qc_epilogue epi, qc_out ydt, bool asym) {
    if (ydt == QC_OUT_I32_ACC) return true;
    if (epi == QC_EPI_NONE) return ydt == QC_OUT_BF16 || K > (asym && bits == 8 ? 576 : 768);
    return epi == QC_EPI_GELU_TANH && ydt == QC_OUT_BF16 && bits == 8 && K > 768;
}

int gemm_resident_blocks() { return kResBlocks; }

constexpr int kCus = 256;

// 32-bit output: non-temporal stores write it to memory at once, ordinary ones into the last-level
// cache, where the next layer finds it.  Ordinary ones win from 24 MB on, 15 MB with lower
// tiles (below, writing back the L2s at the end of the launch weighs more; half the height, K = 1152,
// N = 384, 9.8 MB 10.0 10.5, 15.8 MB 14.9 14.0) while output and codes fit the cache together; past that they push
// out codes that the next tiles need, unless the codes are few.  us, non-temporal and ordinary, K = 1152,
// N = 1152: output of 18 MB 17.3 18.6, 21 MB 19.3 19.5, 26 MB 21.8 20.4, 127 MB 70 63, with codes 239 MB
// 91 85, 262 MB 99.6 99.2, 318 MB 119 120, 412 MB 140 156; N = 3456 (an eighth in codes): output of 223
// MB 112 102, 297 MB 150 136, 398 MB 186 167; K = 2304, N = 640: with codes 242 MB 96 90, 365 MB 123 138;
// K = 4608, N = 1152: 254 MB 142 140, 320 MB 176 178, 383 MB 202 217; K = 192, N = 1152: 400 MB 176 93.
// With K up to 576 the output is nearly all there is to move, and the caches take it at any size while it is
// 16 times the codes: 57258 x 192 x 4608 443 207, 100000 x 384 x 2304 367 234, 150000 x 576 x 2304 496 403, 200000 x 384 x 1536 441 347; but
// 60000 x 768 x 4608 342 351.
// GELU (erf) leaves non-temporal stores the time to drain, and ordinary ones win from 60 MB on only and up to 192 MB
// with the codes: 27 MB 23.3 25.1, 46 MB 30.2 32.6, 53 MB 34.2 35.2, 69 MB 53.8 46.5, with codes 193 MB 89.9 88.2;
// K = 1824, with codes 204 MB 116 127; half the height, N = 3456, 41 MB 26.0 27.7.  Of those outputs that are nearly all there is, with K
// from 385 to 576 it takes ordinary stores up to 512 MB only (to 724 MB the two are equal, beyond non-temporal ones take 5 to 7 % less,
// over 33 drawn calls).
// bf16 output is up to 9 % slower with ordinary stores.
static bool keep_f32_output(int64_t M, int64_t N, int64_t K, int height, qc_epilogue epi) {
    constexpr int64_t MB = 1 << 20;
    const int64_t out = 4 * M * N, codes = M * round_up(K, kKAlign);
    const int64_t from = epi == QC_EPI_GELU_ERF ? 60 : height == 4 ? 24 : 15, most = epi == QC_EPI_GELU_ERF ? 192 : 256;
    const bool any_size = K <= 576 && 16 * codes <= out && (epi != QC_EPI_GELU_ERF || K <= 384 || out <= 512 * MB);
    return out >= from * MB && (out + codes <= most * MB || (8 * codes <= out && out <= 400 * MB) || any_size);
}

// What a CU takes for `per_cu` of the ring kernel's tiles of 64 h tokens x 128 channels, in hundredths of what it
// takes for 64 tokens of a tile of 256 that it has to itself.  Read off some 8000 calls of bf16 output drawn
// over K = 128 .. 4608, 300 to 131072 tokens and 100 to 4608 channels, each at every height.  Up to three
// tiles of 256 the blocks' own chains of waits count: two tiles cost little more than one (510 against
// 400), one of 192 saves an eighth of its quarter.  Beyond, multiplications do, 57 for each 64 tokens, and what a
// lower tile fetches more for them (none while the reduction is short), less what the more blocks per CU hide
// of a GELU.  Those calls read the same codes and weights again and again.  Where these come from beyond the L2s, two tiles
// of 128 with a long reduction lose to one of 256 what they gain otherwise (the whole linear at 256 and 128, the same operands again
// and again | four sets in turn: 12000 x 3072 x 576 42.3 42.7 | 45.3 49.3, 6400 x 4608 x 1152 49.6 49.5 | 51.9 57.2, 6145 x 3360 x
// 1152 39.2 38.6 | 40.3 45.8; but 6400 x 1536 x 1152 23.1 22.3 | 21.9 21.4; over 87 drawn calls +1 % | -5 %).
// extra: hundredths of the cost for what ring_height() knows of the stores and the zero point.
static int ring_cost(int h, int64_t per_cu, int64_t K, qc_epilogue epi, int extra) {
    const bool gelu = epi != QC_EPI_NONE, brief = K <= 384, lengthy = K > 1500;
    constexpr int kFull[] = {400, 510, 680}, kMid[] = {350, 440, 540, 666}, kHalf[] = {310, 380, 450, 535, 630, 707};
    if (h == 4 && per_cu <= 3) return kFull[per_cu - 1];
    if (h == 3 && per_cu <= 4) return kMid[per_cu - 1] * extra / 100;
    if (h == 2 && per_cu <= 6)
        return kHalf[per_cu - 1] * (per_cu == 1 ? 100 : per_cu == 2 && K > 2000 ? 108 : lengthy ? 105 : gelu || brief ? 95 : 100) / 100 * extra / 100;
    int more = 100;
    if (h == 3) more = lengthy ? 102 : per_cu < 12 ? 98 : 101;
    if (h == 2) more = brief ? 100 : lengthy ? 116 : gelu ? 106 : 113;
    return (int)(h * (per_cu < 100000 ? per_cu : 100000) * 57 * more / 100 * extra / 100);
}

// Height of the ring kernel's tiles in 64 tokens: the one whose tiles spread best over the CUs.  Full
// height, full or half by the rule before, and this rule, us: K = 1152, tiles of 256 / 192 / 128 tokens:
// 144 / 198 / 288 9.7 9.8 8.5, 351 / 468 / 693 16.3 16.3 13.6, 216 / 297 / 432 10.6 10.7 9.6; K = 4608: 198 of 192
// tokens 27.0 27.0 23.1, 288 / 387 / 576 47.6 43.9 39.7, 351 / 468 / 693 50.7 51.3 43.5.  Over the drawn calls, the GEMM alone:
// 4 to 6 % less time, slower by more than 3 % in 2 %.
// f32 output past the caches: the more blocks a CU holds the worse their stores drain (the whole linear at 256 and 128, the same
// operands again and again | four sets in turn: 2850 x 1152 x 4608 GELU (erf) 34.1 38.3 | 28.8 34.0, 3649 x 352 x 3456 the same 23.4
// 27.5 | 22.4 27.1, 11670 x 1152 x 1152 38.6 43.4; over 1400 drawn calls -1 % | -3 %).
// A zero point and 8-bit weights: of 192 tokens two blocks fit a CU, without them three (at 256 and 192: 37714 x 256 x 3456,
// binary32 to bf16, 78.8 83.9 | 77.1 81.3, 11666 x 1152 x 4608 74.7 76.2 | 72.9 84.9, 67636 x 1152 x 4608 370 394 | 355 384; over 150
// drawn calls -2 % | -2 %; with two tiles to a CU or one there is nothing to fit, 2478 x 1152 x 3456 24.0 20.4 | 21.9 18.8).
static int ring_height(int64_t M, int64_t N, int n_tiles, int64_t K, qc_epilogue epi, qc_out ydt, bool asym8) {
    int best = 4, least = 0;
    for (int h = 4; h >= 2; --h) {
        const int64_t tiles = (M + kWaveM * h - 1) / (kWaveM * h) * n_tiles;
        const bool streamed = ydt == QC_OUT_F32 && !keep_f32_output(M, N, K, h, epi);
        const int64_t per_cu = (tiles + kCus - 1) / kCus;
        const int cost = ring_cost(h, per_cu, K, epi, h == 2 && streamed ? 106 : h == 3 && asym8 && per_cu > 2 ? 108 : 100);
        if (h == 4 || cost < least) { best = h; least = cost; }
    }
    return best;
}

// Tiles of which a CU gets one at most leave its SIMDs a wavefront each, which waits out every load, unpacking and
// barrier on its own.  Eight wavefronts in two groups, each with half of the reduction, cover each other's waits and
// add their sums up through LDS at the end, which the reduction has to be worth.  Ring kernel, and so, us:
// 4 bit, tiles of 128 tokens, K = 4608: 96 25.3 18.8, 256 26.0 20.0; K = 1152: 96 8.9 7.8, 256 9.9 9.1; K = 768 7.1 6.6; but
// K = 384 5.0 5.2.  4 bit, tiles of 256: K = 4608: 144 28.4 25.6, 256 39.0 31.8; K = 2304: 144 16.6 16.1; but K = 1536
// 12.5 12.7.  8 bit, tiles of 128 (nothing to unpack): K = 4608: 96 17.5 15.6, 144 18.8 17.1; K = 2304: 126 10.9 10.5;
// but K = 1536 8.7 8.8, and 256 tiles K = 2304 12.6 13.1, K = 6144 25.9 26.6.  With two tiles of 128 or 256 to a CU the two
// hide each other's waits and the exchange is lost: 8192 x 4608 x 1152, 288 tiles of 256, 41.9 52.6.
// The split kernels have no form that keeps f32 output in the caches: where tiles of 256 should, it takes K = 4608 (7168 x 4608 x
// 1152 41.5 38.2, but 4096 x 2304 x 2048 24.3 28.2).  Height of the tiles to split, 0: none.
static int split_height(int64_t M, int n_tiles, int KF, int bits) {
    const int64_t half = (M + 2 * kWaveM - 1) / (2 * kWaveM) * n_tiles, full = (M + kTileM - 1) / kTileM * n_tiles;
    if (bits == 8) return half <= 160 && KF >= 36 ? 2 : 0;
    if (half <= kCus) return KF >= 12 ? 2 : 0;
    return full <= kCus && KF >= 36 ? 4 : 0;
}

// Rows of bf16 that are no multiple of 16 B long, and partly filled tiles: through the caches while the
// output fits the last-level cache, past them beyond (N = 3460, K = 1152, ordinary and non-temporal: 113 MB
// 72.3 78.6 us, 454 MB 333 287; N = 1156: 303 MB 286 253).  With 32-bit output a piece covers half of the
// bytes that its neighbours on the line need at once, and non-temporal stores always lose (N = 3457:
// 227 MB 101 189, 906 MB 500 674).
static bool stream_bf16_edges(int64_t M, int64_t N) { return 2 * M * N > (int64_t)256 << 20; }

GemmChoice choose_gemm(int64_t M, int64_t N, int64_t K, int bits, qc_epilogue epi, qc_out ydt, bool asym) {
    GemmChoice c{};
    const int n_tiles = (int)(round_up(N, kTileN) / kTileN);
    if (gemm_resident_chosen(M, N, K, bits) && gemm_resident_epilogue(K, bits, epi, ydt, asym)) {
        c.resident = true;
        c.height = 4;
        return c;
    }
    c.height = ring_height(M, N, n_tiles, K, ydt == QC_OUT_I32_ACC ? QC_EPI_NONE : epi, ydt, asym && bits == 8);
    c.keep_output = ydt == QC_OUT_F32 && keep_f32_output(M, N, K, c.height, epi);
    // Whole rows of 32 bits past the caches: the more blocks a CU holds the worse their stores drain (us at 256
    // and 192 tokens: 39510 x 1152 x 4608 274 324, 105656 x 784 x 1152 210 229; of less than 192 MB the spread over the CUs
    // counts: 42 MB 9149 x 4608 x 1152 58.1 49.0, 43 MB 5597 x 592 x 1920, 4 bit, 128 tokens 20.0 17.6, 29000 x 4608 x 1152 147 147).
    // Of more than 400 MB through the caches too (250000 x 192 x 1152 287 247, 100000 x 384 x 2304, 4 bit, GELU 257 222).
    const int64_t out32 = ydt == QC_OUT_BF16 || N % 4 ? 0 : 4 * M * N;
    if (c.height != 4 && (out32 > (int64_t)400 << 20 || (out32 > (int64_t)192 << 20 && !c.keep_output))) {
        c.height = 4;
        c.keep_output = ydt == QC_OUT_F32 && keep_f32_output(M, N, K, 4, epi);
    }
    const int KF = (int)(round_up(K, kKAlign) / kFragK), split = split_height(M, n_tiles, KF, bits);
    c.split = split == 2 || (split == 4 && (KF >= 72 || ydt != QC_OUT_F32 || !keep_f32_output(M, N, K, 4, epi)));
    if (c.split) {
        c.height = split;
        c.keep_output = false;
    }
    return c;
}

hipError_t launch_gemm(const uint8_t *x_tiled, const float *x_scale, const uint8_t *w_packed,
                       const float *w_scale, const float *bias, void *Y, int64_t M, int64_t N,
                       int64_t K, int bits, qc_epilogue epi, qc_out ydt, const float *x_corr,
                       const int32_t *w_rowsum, hipStream_t stream) {
    if (gemm_small_chosen(M, N))
        return launch_gemm_small(x_tiled, x_scale, w_packed, w_scale, bias, Y, M, N, K, bits, epi, ydt, x_corr,
                                 w_rowsum, stream);
    const GemmChoice choice = choose_gemm(M, N, K, bits, epi, ydt, x_corr && w_rowsum);
    GemmArgs args;
    args.resident = choice.resident;
    args.height = choice.height;
    args.split = choice.split;
    args.keep_output = choice.keep_output;
    args.x_tiled = x_tiled;
    args.x_scale = x_scale;
    args.x_corr = x_corr;
    args.w_rowsum = w_rowsum;
    args.w_codes = w_packed + kPackedHeaderBytes;
    args.w_scale = w_scale;
    args.bias = bias;
    args.Y = Y;
    args.M = M;
    args.N = N;
    args.KF = (int)(round_up(K, kKAlign) / kFragK);
    args.m_tiles = (int)(round_up(M, kTileM) / kTileM);
    args.n_tiles = (int)(round_up(N, kTileN) / kTileN);
    // The blocks resident on one XCD at a time cover a patch of group_m token tiles by as many
    // channel tiles as fit.  With many channel tiles an 8 x 8 patch keeps both operand panels of
    // the patch in that XCD's L2; with few (all of them resident at once anyway) a narrow patch
    // launches the blocks that share a token panel next to each other, so that they read it at
    // the same time (fc2, 9 channel tiles, K = 4608: 870 MB instead of 1370 MB fetched by the L2s).
    // Measured at M = 131072: 8 is the best of 4 .. 32 for the wide layers; for the narrow ones
    // 2 is the best of 1 .. 8 at K = 1152 and 3 the best of 2 .. 6 at K = 4608 (545 against
    // 557 us with 8-bit weights, no difference at M = 65536 or with 4-bit weights).
    args.x_frags = args.m_tiles * (kTileM / kFragRows);
    if (args.height != 4) args.m_tiles = (int)((M + kWaveM * args.height - 1) / (kWaveM * args.height));
    args.stream_edges = stream_bf16_edges(M, N);
    args.group_m = args.n_tiles > 16 ? 8 : (args.KF >= 36 ? 3 : 2);
    return bits == 8 ? launch_gemm_kernel<8>(args, epi, ydt, stream) : launch_gemm_kernel<4>(args, epi, ydt, stream);
}

}  // namespace qc
