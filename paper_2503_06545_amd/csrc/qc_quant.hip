// Per-token dynamic activation quantization (Section 4.1 "Quantization Scheme": activation
// parameters computed online; Section 3.1 Eq. (3)-(4) in symmetric signed form).
//
// HBM-bound: every element of X is read once and one int8 code is written.  A row is held in
// registers between the absmax pass and the cast, so there is no second read.  Wavefronts are short
// (at most 384 columns of 8 rows up to K = 6144) and many per CU, so that the load, arithmetic and
// store phases of different rows overlap; on few rows, where nothing fills the chip, a wavefront's
// own chain of instructions is what the call waits for, and it is made shorter still.
//
// The quotient x / s is the correctly rounded IEEE one, computed without a division per
// element: with r = RN(1 / s) (one true division per row) and q0 = RN(x * r), the residual
// e = x - s * q0 is exact in one fma and q = RN(q0 + e * r) is RN(x / s) for every |x / s| that
// can round to a non-zero code (Markstein's correction step: one suffices when the reciprocal
// is correctly rounded; checked against true division on the CPU over all bf16 inputs, random
// binary32 ones, constructed near-ties and the scales whose significand is all ones).
#include <type_traits>

#include "qc_device.h"

namespace qc {
namespace {

constexpr int kGenericThreads = 256;

// How a kernel treats the caches on its one pass (picked per call by cache_policy()): the chip's
// last-level cache in front of HBM holds 256 MiB, and what the pass leaves in it decides whether
// the GEMM that follows finds the codes there.
enum CachePolicy {
    kCachePlain = 0,    // input and codes fit with room to spare: ordinary loads and stores
    kStreamLoads = 1,   // non-temporal loads of X
    kStreamStores = 2,  // non-temporal stores of the codes
    kStreamBoth = 3,
    kSkipPast = 4,      // with kStreamLoads: nothing is loaded for columns wholly past the row, see load_group()
};

// code = clamp(rne(x / s), -qmax, qmax): true IEEE division, then round half to even.
__device__ inline int quant_code(float x, float s, float qmax) {
    float r = rintf(x / s);
    r = fminf(fmaxf(r, -qmax), qmax);
    return (int)r;
}

// One scale for a whole activation tensor (Section 4.1 "Quantization Scheme": activation
// quantization per layer, parameters computed online): a first launch leaves the absmax of up to
// 256 slabs of the tensor in `partials`; every wavefront of the quantization kernel combines
// them itself (max is exact in any order), which needs neither atomics nor a third launch.
struct TensorMax {
    const float *partials;  // nullptr: one scale per row
    int count;
    bool single_scale;      // write x_scale[0] only, not one (equal) value per row
};

constexpr int kMaxSlabs = 256;

// A wavefront asks for the partial maxima in one load, before its rows, and combines them with DPP
// moves and four readlanes afterwards (a chain of shuffles through LDS cost 4 us of 24 at
// 32768 x 1152, every wavefront doing it).
struct TensorMaxLoad {
    float4 v;
    __device__ void load(const TensorMax &t, int lane) {   // the array holds kMaxSlabs values, count of them written
        v = reinterpret_cast<const float4 *>(t.partials)[lane];
        const int i = 4 * lane;
        v.x = i < t.count ? v.x : 0.0f;
        v.y = i + 1 < t.count ? v.y : 0.0f;
        v.z = i + 2 < t.count ? v.z : 0.0f;
        v.w = i + 3 < t.count ? v.w : 0.0f;
    }
    __device__ float combine() const {
        float a = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
        a = dpp_max<0xB1>(a);    // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror: 16 lanes
        a = dpp_max<0x4E>(a);
        a = dpp_max<0x141>(a);
        a = dpp_max<0x140>(a);
        float r = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) r = fmaxf(r, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), 16 * i)));
        return r;
    }
};

// The slabs' maxima: at most one block of 1024 threads per CU, four 16 B loads in flight per lane
// (64 KiB per CU; with 256 threads and one load the pass ran at 2.3 TB/s: 32768 x 1152 bf16 33 us).
// bf16 magnitudes are compared as packed bit patterns, see Bf16Max.
constexpr int kSlabThreads = 1024;
constexpr int kSlabUnroll = 4;

template <typename XT>
__global__ __launch_bounds__(kSlabThreads) void tensor_absmax_kernel(const XT *__restrict__ X, int64_t n,
                                                                    float *__restrict__ partials) {
    __shared__ float wave_max[kSlabThreads / 64];
    constexpr int kPer = 16 / (int)sizeof(XT);  // elements per 16 B load
    const int64_t nv = n / kPer;
    const int64_t stride = (int64_t)gridDim.x * kSlabThreads * kSlabUnroll;
    Bf16Max packed;
    float a = 0.0f;
    auto fold = [&](const uint4 &v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (sizeof(XT) == 2) packed.fold(w[j]);
            else a = fmaxf(a, fabsf(__uint_as_float(w[j])));
        }
    };
    for (int64_t base = (int64_t)blockIdx.x * kSlabThreads * kSlabUnroll + threadIdx.x; base < nv; base += stride) {
        uint4 v[kSlabUnroll];
#pragma unroll
        for (int u = 0; u < kSlabUnroll; ++u) {   // past the end the last piece again: the same maximum
            const int64_t i = base + u * kSlabThreads;
            v[u] = reinterpret_cast<const uint4 *>(X)[i < nv ? i : nv - 1];
        }
#pragma unroll
        for (int u = 0; u < kSlabUnroll; ++u) fold(v[u]);
    }
    if (blockIdx.x == 0 && threadIdx.x < (int)(n - nv * kPer)) {  // trailing elements
        const XT t = X[nv * kPer + threadIdx.x];
        if constexpr (sizeof(XT) == 2) a = fmaxf(a, fabsf(__uint_as_float((uint32_t)t << 16)));
        else a = fmaxf(a, fabsf(t));
    }
    if constexpr (sizeof(XT) == 2) a = fmaxf(a, packed.value());
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) a = fmaxf(a, __shfl_xor(a, d));
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kSlabThreads / 64; ++w) a = fmaxf(a, wave_max[w]);
        partials[blockIdx.x] = a;
    }
}

// 8 lanes share a row and a wavefront holds 8 rows x 8 UPT units of 16 columns in registers (UPT
// units per lane, picked by units_per_lane()), so that every 16 B store of the fragment
// layout completes a 128 B line (8 rows x 16 B) within one instruction.  A row is cut into column
// slices of that width, one wavefront of the block per slice; the slices agree on the row absmax
// through LDS.  Needs K % 16 == 0 and K <= 9216.
constexpr int kLanesPerRow = 8;
constexpr int kRowsPerBlock = 64 / kLanesPerRow;
constexpr int kGroup = kLanesPerRow * kUnit;      // 128 columns: what the lanes of a row hold per step
constexpr int kUnitsMost = 9 * kLanesPerRow * 8;  // units of the longest row: 8 slices at UPT = 9

// Most wavefronts of a block: with 9 units per lane a wavefront holds 1152 columns and uses most of
// its registers; with fewer units the block takes up to 16 wavefronts.
template <int UPT>
constexpr int kMaxSlices = UPT == 9 ? 8 : 16;

// Group i of the columns of a slice.  One wholly past the row loads the row's last piece once more, which does not
// change a maximum.  Ordinary loads find that piece in the L1; non-temporal ones fetch its line again.  Under kSkipPast
// such a group is the slice's first one over again instead, which begins inside the row (the quantizer alone, us for ordinary
// loads, non-temporal ones and these, the same input again and again | four in turn: binary32, 195 MB of input and codes,
// 304690 x 128 28 51 32 | 36 49 33, 81253 x 480 30 42 32 | 38 42 34; bf16, 245 MB, 182294 x 448 42 51 43 | 50 52 46.  Whole
// linears, four in turn: 102673 x 480 x 1152 142 128 123, 183344 x 448 x 1152 227 205 198).
template <typename XT, int POLICY, int UPT>
__device__ inline void load_group(Group<XT> (&u)[UPT], int i, const XT *xrow, int slice, int K, int sub) {
    const int col0 = (slice * UPT + i) * kGroup;
    if ((POLICY & kSkipPast) != 0 && i > 0 && __builtin_amdgcn_readfirstlane(col0) >= K) u[i] = u[0];
    else u[i].template load<(POLICY & kStreamLoads) != 0>(xrow, col0, K, sub);
}

// TENSOR: the absmax comes from `tmax` (one scale for the whole tensor).  A template parameter
// rather than a test of tmax.partials, so that the per-token kernel is compiled exactly as if
// the other did not exist.  RAGGED: a K that is no multiple of 16, for the fragment layout only; the
// codes of columns K .. up to the next multiple of 16 are written too, where the weights are zero.
template <typename XT, bool TENSOR, int POLICY, int UPT, bool RAGGED>
__global__ __launch_bounds__(64 * kMaxSlices<UPT>) void quant_rows_kernel(
    const XT *__restrict__ X, int64_t M, int64_t K, int8_t *__restrict__ qx,
    uint8_t *__restrict__ qx_tiled, int64_t KF, float *__restrict__ x_scale, float qmax,
    TensorMax tmax) {
    __shared__ float slice_max[kMaxSlices<UPT>][kRowsPerBlock];
    const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6, slices = blockDim.x >> 6;
    const int sub = lane % kLanesPerRow, row_in_block = lane / kLanesPerRow;
    // TENSOR: the last rows first, which the pass for the maximum left in the last-level cache
    const int64_t row_block = TENSOR ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
    const int64_t row = row_block * kRowsPerBlock + row_in_block;
    const int units = (int)((K + kUnit - 1) / kUnit);
    const bool live = row < M;
    const XT *xrow = X + (live ? row : 0) * K;

    TensorMaxLoad slabs;
    if (TENSOR) slabs.load(tmax, lane);   // uniform over the launch
    Group<XT> u[UPT];
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        if constexpr (RAGGED) u[i].load_ragged(xrow, (slice * UPT + i) * kGroup, (int)K, sub);
        else load_group<XT, POLICY, UPT>(u, i, xrow, slice, (int)K, sub);
    }
    if constexpr (RAGGED) {
#pragma unroll
        for (int i = 0; i < UPT; ++i) u[i].settle_ragged((slice * UPT + i) * kGroup, (int)K, sub);
    }

    float a = 0.0f;
    if (TENSOR) {  // one scale for the whole tensor: its absmax was reduced beforehand
        a = slabs.combine();
    } else {
        auto running = Group<XT>::no_max();
#pragma unroll
        for (int i = 0; i < UPT; ++i) u[i].absmax_into(running);
        a = Group<XT>::absmax_value(running);
        a = max_of_eight(a);
        if (slices > 1) {  // uniform over the block
            if (sub == 0) slice_max[slice][row_in_block] = a;
            __syncthreads();
            for (int sl = 0; sl < slices; ++sl) a = fmaxf(a, slice_max[sl][row_in_block]);
        }
    }

    const float s = scale_of(a, qmax);
    const float r = 1.0f / s;  // correctly rounded
    if (TENSOR && tmax.single_scale) {
        if (blockIdx.x == 0 && threadIdx.x == 0) x_scale[0] = s;
    } else if (live && sub == 0 && slice == 0) {
        x_scale[row] = s;
    }
    if (!live) return;

    int8_t *out_rows = qx ? qx + row * K : nullptr;
    uint8_t *out_tiled = qx_tiled ? qx_tiled + act_frag_offset(row, 0, KF) : nullptr;
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        const int ui0 = (slice * UPT + i) * kLanesPerRow;   // first unit of the group
        if (ui0 >= units) break;                            // the same for all lanes
        uint32_t w[4];
#pragma unroll
        for (int d = 0; d < 4; ++d)
            w[d] = codes4(quotient(u[i].get(4 * d + 0), s, r), quotient(u[i].get(4 * d + 1), s, r),
                          quotient(u[i].get(4 * d + 2), s, r), quotient(u[i].get(4 * d + 3), s, r));
        const uint4 out = Group<XT>::gather_codes(w, sub);
        const int ui = ui0 + Group<XT>::unit_of(sub);
        if (ui >= units) continue;
        if (out_rows) store16<(POLICY & kStreamStores) != 0>(out_rows + (int64_t)ui * kUnit, out);
        // unit ui covers k = 16 ui ..: 64-k stage ui / 4, k quarter ui % 4 (see act_frag_offset)
        if (out_tiled)
            store16<(POLICY & kStreamStores) != 0>(out_tiled + (int64_t)(ui >> 2) * (4 * kFragBytes) + (ui & 3) * 256, out);
    }
}

// ---- rotation fused into the quantization (Section 3.2 AIGQ (1); Section 4.1 "Hardware
// Implementation") -----------------------------------------------------------------------------
// see Rotation (qc_device.h)
template <typename XT, int POLICY, int UPT>
__global__ __launch_bounds__(64 * kMaxSlices<UPT>) void quant_rows_rot_kernel(
    const XT *__restrict__ X, int64_t M, int64_t K, int8_t *__restrict__ qx,
    uint8_t *__restrict__ qx_tiled, int64_t KF, float *__restrict__ x_scale, float qmax, int rot) {
    __shared__ float slice_max[kMaxSlices<UPT>][kRowsPerBlock];
    const int lane = threadIdx.x & 63, slice = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), slices = blockDim.x >> 6;
    const int sub = lane % kLanesPerRow, row_in_block = lane / kLanesPerRow;
    const int label = rotation_label(sub);
    const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + row_in_block;
    const int units = (int)(K / kUnit);
    const bool live = row < M;
    const XT *xrow = X + (live ? row : 0) * K;

    Group<XT> u[UPT];
#pragma unroll
    for (int i = 0; i < UPT; ++i)
        load_group<XT, POLICY, UPT>(u, i, xrow, slice, (int)K, label);

    const Rotation<XT> rotation(rot, label);
    float f[UPT][kUnit];
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        // A group wholly past the row, the same for all lanes, has nothing to add (rotated all the same, and its zeros put in
        // place, us: 125000 x 128 bf16, blocks of 16 14.4 10.7, of 128 18.3 11.5, binary32 15.9 13.6; 300000 x 64 26.5 17.8)
        if (UPT > 1 && (slice * UPT + i) * kGroup >= (int)K) break;
#pragma unroll
        for (int e = 0; e < kUnit; ++e) f[i][e] = u[i].get(e);
        rotation.apply(f[i], (slice * UPT + i) * kGroup, (int)K);
#pragma unroll
        for (int e = 0; e < kUnit; ++e) a = fmaxf(a, fabsf(f[i][e]));
    }
    a = max_of_eight(a);
    if (slices > 1) {  // uniform over the block
        if (sub == 0) slice_max[slice][row_in_block] = a;
        __syncthreads();
        for (int sl = 0; sl < slices; ++sl) a = fmaxf(a, slice_max[sl][row_in_block]);
    }

    const float s = scale_of(a, qmax);
    const float r = 1.0f / s;  // correctly rounded
    if (live && sub == 0 && slice == 0) x_scale[row] = s;
    if (!live) return;
    const float sign = rotation.sign();
    const float ss = sign * s, sr = sign * r;

    int8_t *out_rows = qx ? qx + row * K : nullptr;
    uint8_t *out_tiled = qx_tiled ? qx_tiled + act_frag_offset(row, 0, KF) : nullptr;
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        const int ui0 = (slice * UPT + i) * kLanesPerRow;   // first unit of the group
        if (ui0 >= units) break;                            // the same for all lanes
        uint32_t w[4];
#pragma unroll
        for (int d = 0; d < 4; ++d)
            w[d] = codes4(quotient(f[i][4 * d + 0], ss, sr), quotient(f[i][4 * d + 1], ss, sr),
                          quotient(f[i][4 * d + 2], ss, sr), quotient(f[i][4 * d + 3], ss, sr));
        const uint4 out = Group<XT>::gather_codes(w, label);
        const int ui = ui0 + Group<XT>::unit_of(label);
        if (ui >= units) continue;
        if (out_rows) store16<(POLICY & kStreamStores) != 0>(out_rows + (int64_t)ui * kUnit, out);
        if (out_tiled)
            store16<(POLICY & kStreamStores) != 0>(out_tiled + (int64_t)(ui >> 2) * (4 * kFragBytes) + (ui & 3) * 256, out);
    }
}

// ---- the quantizer as printed, asymmetric (Section 3.1 Eq. (3)-(4)) ----------------------------
//   s = max(hi - lo, 2^-64) / levels,  z = -rne(lo / s),  code = clamp(rne(x / s) + z, 0, levels)
// with levels = 2^b - 1.  Same layout and the same division-free quotient as above (it is
// exact for these larger quotients as well, checked on the host).  `shifted` selects what is
// stored: the canonical unsigned code and z, or, for the GEMM, code - shift as a signed byte
// and the correction shift - z (shift = asym_code_shift(act_bits)).
template <typename XT, int POLICY, int UPT>
__global__ __launch_bounds__(64 * kMaxSlices<UPT>) void quant_rows_asym_kernel(
    const XT *__restrict__ X, int64_t M, int64_t K, uint8_t *__restrict__ qx,
    uint8_t *__restrict__ qx_tiled, int64_t KF, float *__restrict__ x_scale,
    float *__restrict__ x_aux, float levels, float shift, bool shifted) {
    __shared__ float slice_lo[kMaxSlices<UPT>][kRowsPerBlock], slice_hi[kMaxSlices<UPT>][kRowsPerBlock];
    const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6, slices = blockDim.x >> 6;
    const int sub = lane % kLanesPerRow, row_in_block = lane / kLanesPerRow;
    const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + row_in_block;
    const int units = (int)(K / kUnit);
    const bool live = row < M;
    const XT *xrow = X + (live ? row : 0) * K;

    Group<XT> u[UPT];
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        load_group<XT, POLICY, UPT>(u, i, xrow, slice, (int)K, sub);
    }

    float lo = __builtin_inff(), hi = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
#pragma unroll
        for (int e = 0; e < kUnit; ++e) {
            lo = fminf(lo, u[i].get(e));
            hi = fmaxf(hi, u[i].get(e));
        }
    }
    lo = min_of_eight(lo);
    hi = max_of_eight(hi);
    if (slices > 1) {  // uniform over the block
        if (sub == 0) { slice_lo[slice][row_in_block] = lo; slice_hi[slice][row_in_block] = hi; }
        __syncthreads();
        for (int sl = 0; sl < slices; ++sl) {
            lo = fminf(lo, slice_lo[sl][row_in_block]);
            hi = fmaxf(hi, slice_hi[sl][row_in_block]);
        }
    }
    if (!live) return;

    const float s = fmaxf(hi - lo, kAbsmaxFloor) / levels;
    const float r = 1.0f / s;  // correctly rounded
    const float z = -rintf(quotient(lo, s, r));
    if (sub == 0 && slice == 0) {
        x_scale[row] = s;
        x_aux[row] = shifted ? shift - z : z;
    }
    // clamp(rne(q) + z, 0, levels) - shift = clamp(rne(q) + (z - shift), -shift, levels - shift)
    const float off = shifted ? z - shift : z;
    const float cmin = shifted ? -shift : 0.0f, cmax = shifted ? levels - shift : levels;

    uint8_t *out_rows = qx ? qx + row * K : nullptr;
    uint8_t *out_tiled = qx_tiled ? qx_tiled + act_frag_offset(row, 0, KF) : nullptr;
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
        const int ui0 = (slice * UPT + i) * kLanesPerRow;   // first unit of the group
        if (ui0 >= units) break;                            // the same for all lanes
        uint32_t w[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            w[d] = asym_codes4(quotient(u[i].get(4 * d + 0), s, r), quotient(u[i].get(4 * d + 1), s, r),
                               quotient(u[i].get(4 * d + 2), s, r), quotient(u[i].get(4 * d + 3), s, r), off, cmin, cmax);
        }
        const uint4 out = Group<XT>::gather_codes(w, sub);
        const int ui = ui0 + Group<XT>::unit_of(sub);
        if (ui >= units) continue;
        if (out_rows) store16<(POLICY & kStreamStores) != 0>(out_rows + (int64_t)ui * kUnit, out);
        if (out_tiled)
            store16<(POLICY & kStreamStores) != 0>(out_tiled + (int64_t)(ui >> 2) * (4 * kFragBytes) + (ui & 3) * 256, out);
    }
}

// Any K, any alignment: one wavefront per row, two passes over the row (the second one is
// served by the caches).  For what the row kernels do not take: row-major codes of rows that are no
// multiple of 16 long, and rows longer than 9216.
template <typename XT>
__global__ __launch_bounds__(kGenericThreads) void quant_rows_generic_kernel(
    const XT *__restrict__ X, int64_t M, int64_t K, int8_t *__restrict__ qx,
    uint8_t *__restrict__ qx_tiled, int64_t KF, float *__restrict__ x_scale, float qmax,
    TensorMax tmax) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (kGenericThreads / 64) + (threadIdx.x >> 6);
    if (row >= M) return;
    const XT *xrow = X + row * K;
    auto widen = [](XT v) -> float {
        if constexpr (sizeof(XT) == 2) return __uint_as_float((uint32_t)v << 16);
        else return v;
    };
    float a = 0.0f;
    if (tmax.partials) {
        TensorMaxLoad slabs;
        slabs.load(tmax, lane);
        a = slabs.combine();
    } else {
        for (int64_t k = lane; k < K; k += 64) a = fmaxf(a, fabsf(widen(xrow[k])));
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) a = fmaxf(a, __shfl_xor(a, d));
    }
    const float s = scale_of(a, qmax);
    if (tmax.single_scale) {
        if (row == 0 && lane == 0) x_scale[0] = s;
    } else if (lane == 0) {
        x_scale[row] = s;
    }
    for (int64_t k = lane; k < K; k += 64) {
        const int8_t c = (int8_t)quant_code(widen(xrow[k]), s, qmax);
        if (qx) qx[row * K + k] = c;
        if (qx_tiled) qx_tiled[act_frag_offset(row, k, KF)] = (uint8_t)c;
    }
}

// Measured with the GEMM that follows included.  While input and codes leave room in the cache, ordinary
// accesses are the fastest (M = 16384, QKV: 68 us against 72 with non-temporal loads).  From 160 MB of them on what
// else is on its way through the cache counts, the output of this call and of the one before and an input that
// another kernel has just written, and non-temporal loads leave the codes there for the GEMM (us per call, ordinary
// and non-temporal loads, the same input again and again | four inputs, workspaces and outputs in turn | inputs
// written just before by another kernel, its time included: 216 MB, K = 1152, N = 4608, GELU 343 350 | 390 351 |
// 393 389, N = 3456 236 245 | 264 248 | 290 286; 162 MB, N = 3456 191 196 | 193 190 | 238 225, K = 4608, N =
// 1152 79 82 | 81 81 | 124 114; 130 MB, K = 4608, asymmetric 72 74 | 73 75 | 103 102; 108 MB, N = 3456 129
// 128 | 128 132 | 155 153).  Rows that are no whole lines, of which non-temporal loads fetch the shared lines twice, gain
// from them only where input and codes do not fit the cache (MB of input and codes, K, N, ordinary and
// non-temporal: 165, 544, 56 47 52 | 52 52 | 86 91; 177, 1552, 1152 103 110 | 106 111 | 144 155; 200, 1200, 64 51 58 | 63 65 | 105
// 113; 195, 2576, 45 52 59 | 64 65 | 106 111; 200, 1552, 3456 250 257 | 251 260 | 292 307; 245, 544, 1152 155 151 | 202 175 |
// 216 221; 245, 1200, 1152 142 143 | 166 151 | 199 205; the quantizer alone, 245, 1168 44 54 | 55 55).  With few channels of output whole lines gain as well, except from the same input
// again and again (165, 1152, 64 44 45 | 52 48 | 86 83; 237, 1152, 64 59 61 | 75 64 | 121 113; binary32 165, 1152, 288 48 52 | 55 50 | 97
// 93).  Far beyond, M = 131072, K = 1152, they take the quantization from 80 to 69 us and
// QKV whole from 562 to 502 us, also while the codes alone are a little larger than
// the cache (bf16, 1152 channels, 270 MB of codes, K = 1152: 415 us, with non-temporal stores as well 471;
// 302 MB, K = 4608: 424 and 419).  With more codes little of them is left to find, and non-temporal
// stores win too (340 MB, K = 1152: 586 and 556; 500 MB, K = 4608: 697 and 698).  Past that size there is
// nothing to keep X out of the cache for either: rows that are no whole lines, of which non-temporal
// loads fetch the shared lines twice, are loaded ordinarily (340 MB, K = 1200: 641 and 627 us, K = 3952: 513
// and 493; while the codes are to be kept non-temporal loads are the better ones here too, 220 MB, K =
// 1200: 426 and 346).
int cache_policy(int64_t M, int64_t K, size_t x_elem_bytes) {
    constexpr int64_t kLastLevelCache = (int64_t)256 << 20;
    const int64_t codes = M * K, input = codes * (int64_t)x_elem_bytes;
    const bool whole_lines = K * (int64_t)x_elem_bytes % 128 == 0;
    if (codes > kLastLevelCache * 9 / 8) return whole_lines ? kStreamBoth : kStreamStores;
    return input + codes > kLastLevelCache * (whole_lines ? 5 : 8) / 8 ? kStreamLoads : kCachePlain;
}

// Units per lane of the row kernels.  One unit, a wavefront per 128 columns, where a block of 16
// wavefronts holds the row and the call is bound by latency: a wavefront alone on its SIMD issues an
// instruction every 8 clocks or so, and nine units are some 1600 of them (K = 1152, M = 1024: 9 units
// 5.5 us, 3 units 3.6, 1 unit 3.3; equal from M = 8192 on).  Three units otherwise: against nine the
// registers allow more wavefronts per SIMD and more of them are at different phases (M = 131072,
// K = 1152: 71.6 -> 68.6 us, K = 4608: 300 -> 292 us).  Nine for the rows 16 x 384 columns do not cover.
constexpr int kBlockWaves = 16;
int units_per_lane(int64_t M, int64_t K) {
    if (K <= kBlockWaves * kGroup && M * K <= (int64_t)8192 * 1152) return 1;
    return K <= 3 * kBlockWaves * kGroup ? 3 : 9;
}

dim3 row_grid(int64_t M) { return dim3((unsigned)((M + kRowsPerBlock - 1) / kRowsPerBlock)); }
dim3 row_block(int64_t K, int upt) {
    return dim3((unsigned)(64 * ((K + (int64_t)upt * kGroup - 1) / ((int64_t)upt * kGroup))));
}

// calls f(policy, units per lane), both std::integral_constant, for the pair picked at run time
template <typename F>
void with_row_variant(int64_t M, int64_t K, size_t x_elem_bytes, F &&f) {
    const int upt = units_per_lane(M, K), policy = cache_policy(M, K, x_elem_bytes);
    // Full rows have nothing to skip and lose up to 5 % by the test (202549 x 1152 bf16 114 to 118 us).  It is worth it where
    // a third or more of the wavefronts' columns are past the row: in binary32 K = 480 of 768 columns takes 0.82 to 0.84 of
    // the time without it, 512 of them 0.93 to 0.96, in bf16 512 as much or more.
    const int64_t columns = (K + 3 * kGroup - 1) / (3 * kGroup) * (3 * kGroup);
    const bool skip = upt == 3 && 2 * columns > 3 * K;
    auto with_policy = [&](auto u) {
        if (policy == kStreamBoth) f(std::integral_constant<int, kStreamBoth>{}, u);
        else if (policy == kStreamStores) f(std::integral_constant<int, kStreamStores>{}, u);
        else if (policy == kStreamLoads) {
            if constexpr (decltype(u)::value == 3) {
                if (skip) return f(std::integral_constant<int, kStreamLoads | kSkipPast>{}, u);
            }
            f(std::integral_constant<int, kStreamLoads>{}, u);
        }
        else f(std::integral_constant<int, kCachePlain>{}, u);
    };
    if (upt == 1) f(std::integral_constant<int, kCachePlain>{}, std::integral_constant<int, 1>{});  // small: plain
    else if (upt == 3) with_policy(std::integral_constant<int, 3>{});
    else with_policy(std::integral_constant<int, 9>{});
}

template <typename XT>
hipError_t launch_typed(const XT *X, int64_t M, int64_t K, int8_t *qx, uint8_t *qx_tiled,
                        int64_t KF, float *x_scale, float qmax, int rot, TensorMax tmax,
                        hipStream_t stream) {
    const bool vec = quant_vector_path(K);
    if (rot) {
        if (!vec || K % rot) return hipErrorInvalidValue;  // the entry points reject these first
        with_row_variant(M, K, sizeof(XT), [&](auto pol, auto upt) {
            constexpr int P = decltype(pol)::value;
            quant_rows_rot_kernel<XT, P, decltype(upt)::value>
                <<<row_grid(M), row_block(K, decltype(upt)::value), 0, stream>>>(
                    X, M, K, qx, qx_tiled, KF, x_scale, qmax, rot);
        });
        return hipGetLastError();
    }
    // Rows of any other length: the same kernels when only the fragment layout is wanted (4099 x 1000
    // bf16: 12.2 us with a wavefront per row and byte stores); row-major codes of ragged rows, rows of less than 16 B and
    // rows longer than 9216 take the generic one.
    const bool ragged = !vec && !qx && K <= (int64_t)kUnitsMost * kUnit && K * (int64_t)sizeof(XT) >= 16;
    if (!vec && !ragged) {
        const int64_t blocks = (M + 3) / 4;
        quant_rows_generic_kernel<XT><<<dim3((unsigned)blocks), dim3(kGenericThreads), 0, stream>>>(
            X, M, K, qx, qx_tiled, KF, x_scale, qmax, tmax);
        return hipGetLastError();
    }
    with_row_variant(M, K, sizeof(XT), [&](auto pol, auto upt) {
        constexpr int P = decltype(pol)::value, U = decltype(upt)::value;
        const dim3 grid = row_grid(M), block = row_block(K, U);
        // the tensor was read once already for its absmax: what the caches still hold of it helps
        if (tmax.partials && ragged)
            quant_rows_kernel<XT, true, kCachePlain, U, true><<<grid, block, 0, stream>>>(X, M, K, qx, qx_tiled, KF, x_scale, qmax, tmax);
        else if (tmax.partials)
            quant_rows_kernel<XT, true, kCachePlain, U, false><<<grid, block, 0, stream>>>(X, M, K, qx, qx_tiled, KF, x_scale, qmax, tmax);
        else if (ragged)
            quant_rows_kernel<XT, false, kCachePlain, U, true><<<grid, block, 0, stream>>>(X, M, K, qx, qx_tiled, KF, x_scale, qmax, tmax);
        else
            quant_rows_kernel<XT, false, P, U, false><<<grid, block, 0, stream>>>(X, M, K, qx, qx_tiled, KF, x_scale, qmax, tmax);
    });
    return hipGetLastError();
}

}  // namespace

bool quant_vector_path(int64_t K) {
    return K % kUnit == 0 && K / kUnit <= kUnitsMost;
}

hipError_t launch_quant_act_asym(const void *X, qc_dtype xdt, int64_t M, int64_t K, uint8_t *qx_rowmajor,
                                 uint8_t *qx_tiled, int64_t KF, float *x_scale, float *x_aux,
                                 int act_bits, bool shifted, hipStream_t stream) {
    if (!quant_vector_path(K)) return hipErrorInvalidValue;  // the entry points reject these first
    const float levels = (float)((1 << act_bits) - 1), shift = (float)asym_code_shift(act_bits);
    auto launch = [&](const auto *typed) {
        typedef std::remove_cv_t<std::remove_pointer_t<decltype(typed)>> XT;
        with_row_variant(M, K, sizeof(XT), [&](auto pol, auto upt) {
            quant_rows_asym_kernel<XT, decltype(pol)::value, decltype(upt)::value>
                <<<row_grid(M), row_block(K, decltype(upt)::value), 0, stream>>>(
                    typed, M, K, qx_rowmajor, qx_tiled, KF, x_scale, x_aux, levels, shift, shifted);
        });
        return hipGetLastError();
    };
    return xdt == QC_BF16 ? launch((const uint16_t *)X) : launch((const float *)X);
}

int quant_cache_policy(int64_t M, int64_t K, qc_dtype xdt, QuantScheme scheme) {
    if (scheme == kQuantTensor || !quant_vector_path(K) || units_per_lane(M, K) == 1) return kCachePlain;
    return cache_policy(M, K, xdt == QC_BF16 ? 2 : 4);
}

bool quant_rotation_supported(int64_t K, int rot_block) {
    if (rot_block != 16 && rot_block != 32 && rot_block != 64 && rot_block != 128) return false;
    return K % rot_block == 0 && quant_vector_path(K);
}

hipError_t launch_quant_act(const void *X, qc_dtype xdt, int64_t M, int64_t K, int8_t *qx_rowmajor,
                            uint8_t *qx_tiled, int64_t KF, float *x_scale, int act_bits,
                            int rot_block, hipStream_t stream) {
    const float qmax = (float)((1 << (act_bits - 1)) - 1);  // 127, 31 or 7 in an int8 container
    const TensorMax per_row = {nullptr, 0, false};
    if (xdt == QC_BF16)
        return launch_typed<uint16_t>((const uint16_t *)X, M, K, qx_rowmajor, qx_tiled, KF, x_scale,
                                      qmax, rot_block, per_row, stream);
    return launch_typed<float>((const float *)X, M, K, qx_rowmajor, qx_tiled, KF, x_scale, qmax,
                               rot_block, per_row, stream);
}

size_t tensor_partials_bytes() { return (size_t)kMaxSlabs * sizeof(float); }

hipError_t launch_quant_act_tensor(const void *X, qc_dtype xdt, int64_t M, int64_t K,
                                   int8_t *qx_rowmajor, uint8_t *qx_tiled, int64_t KF,
                                   float *x_scale, bool single_scale, float *partials, int act_bits,
                                   hipStream_t stream) {
    const float qmax = (float)((1 << (act_bits - 1)) - 1);
    const int64_t n = M * K;
    const int per = xdt == QC_BF16 ? 8 : 4;
    int64_t slabs = (n / per + (int64_t)kSlabThreads * kSlabUnroll - 1) / ((int64_t)kSlabThreads * kSlabUnroll);
    if (slabs < 1) slabs = 1;
    if (slabs > kMaxSlabs) slabs = kMaxSlabs;
    if (xdt == QC_BF16)
        tensor_absmax_kernel<uint16_t><<<dim3((unsigned)slabs), dim3(kSlabThreads), 0, stream>>>(
            (const uint16_t *)X, n, partials);
    else
        tensor_absmax_kernel<float><<<dim3((unsigned)slabs), dim3(kSlabThreads), 0, stream>>>(
            (const float *)X, n, partials);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    const TensorMax tmax = {partials, (int)slabs, single_scale};
    if (xdt == QC_BF16)
        return launch_typed<uint16_t>((const uint16_t *)X, M, K, qx_rowmajor, qx_tiled, KF, x_scale,
                                      qmax, 0, tmax, stream);
    return launch_typed<float>((const float *)X, M, K, qx_rowmajor, qx_tiled, KF, x_scale, qmax, 0,
                               tmax, stream);
}

}  // namespace qc
