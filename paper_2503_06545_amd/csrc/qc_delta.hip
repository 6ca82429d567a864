// The decision reductions: latent change (Section 3.2 HLC, Eq. (5)), cosine similarity of two feature
// tensors (Section 3.3 SRAP, Eq. (9)), inter-frame gradient norm (second factor of Eq. (5)) and
// cumulative variation over the previous steps (Eq. (11)).  Each is one pass over its tensors with a
// deterministic result: groups of four terms are summed in binary32 (the frame gradient's squares in
// binary64, which costs 0.4 us of 6.9 on 16 million bf16 elements in the caches and less elsewhere), everything after that in
// binary64 and in an order that does not depend on scheduling.
//
// HBM-bound where they are large, bound by launches and dependent round trips where they are small,
// hence two forms of one kernel:
//   * Two launches: at most one block per CU (256); a second, single-block launch adds the blocks'
//     partial sums.
//   * One launch, for small tensors: at most 64 blocks, of which the one that sees all partial
//     sums finishes the job (finish_here() says how, without a counter that somebody would have to
//     clear).  What it saves is a launch, 3 us of host time (a call takes 4.1 and 7.1 us there); what it costs on
//     the GPU are the device fence of each block, the blocks' reading of each other's records, and, with
//     the size, that fewer blocks read.  Two chunks a block (one from five earlier tensors on), 16 blocks at least while there are as many
//     chunks: with 32 blocks at most it took 5.6 instead of 5.3 us for a latent delta of 390000 elements, 7.5
//     instead of 6.6 for a similarity of 1.2 million; with more than 64, whose records a lane reads in two goes, 7.3 to 7.7 instead of
//     6.2 to 6.4 for 1.18 to 1.31 million bf16 elements read again and again.  Each operation's limit (kOneMost) lies where it costs
//     no more than two launches, over inputs read again and again too (one launch for a latent delta of
//     540000 to 715000 elements 6 to 7.4 us where two took 4.6).  Only the similarity's lies higher, for the calls from the
//     host, which two launches take 7.1 us for whatever the size: binary32, in a graph and from the host, two launches and one, 400000
//     4.5 5.5, 7.8 5.2, 524288 4.5 5.2, 7.3 6.2, 653550 5.1 6.0, 7.3 7.0; bf16, whose features a step asks for from the host, 1.31 million
//     5.0 6.3, 7.1 6.4.  us per call in a graph, four sets of inputs in turn, two launches and one:
//       latent delta     65536 4.5 3.7   300000 5.4 4.6   500000 5.7 5.6   700000 6.0 6.3   1 million 6.2 7.4
//       similarity bf16  100000 4.8 4.0   300000 4.7 4.7   600000 5.4 5.6   1.3 million 5.6 6.5   1.7 million 5.4 7.4
//       frame gradient   binary32 65536 4.1 3.4   250000 4.2 4.2   400000 4.0 5.1; bf16 500000 4.4 4.5   900000 4.2 5.5
//       variation over 1, 3, 8 tensors of 65536 elements 4.0 5.2 8.0, 3.6 4.4 6.9; of 97000 4.0 5.2 8.3, 3.9 5.0
//       7.5; of 150000 3.6 4.9 8.0, 4.4 5.3 8.9
#include <atomic>

#include "qc_device.h"

namespace qc {
namespace {

constexpr int kFinalThreads = 64;   // the second launch
constexpr int kMaxBlocks = 256;     // two launches: one block per CU
constexpr int kOneThreads = 512;    // one launch
constexpr int kOneFew = 16, kOneBlocks = 64;
static_assert(kMaxBlocks % kFinalThreads == 0 && kOneBlocks <= 64, "whole wavefronts of blocks, a lane per block in the combines");

// the workspaces: a double per sum and block of the two-launch form
constexpr size_t kDeltaBytes = kMaxBlocks * 2 * sizeof(double), kSimilarityBytes = kMaxBlocks * 3 * sizeof(double);
constexpr size_t kGradientBytes = kMaxBlocks * sizeof(double), kVariationBytes = kMaxBlocks * QC_MAX_PREV * sizeof(double);

// one DPP move of a binary64 value (two 32-bit halves); CTRL as in the ISA's dpp_ctrl field
template <int CTRL>
__device__ inline double dpp_move(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes, the same bits in every lane: butterflies inside a row of 16 lanes
// (quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror), then the four row sums in
// index order.
__device__ inline double wave_sum(double v) {
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    double r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        r[i] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 16 * i),
                                __builtin_amdgcn_readlane(__double2loint(v), 16 * i));
    return (r[0] + r[1]) + (r[2] + r[3]);
}

// Block-wide sums of COUNT values, in a fixed order; the result is valid in wavefront 0.  sh holds
// COUNT * (THREADS / 64) doubles and may be reused after the next barrier.  (The wavefronts' sums are
// added one after the other by every lane of wavefront 0: a second wave_sum over them took up to 1.4 us
// longer per reduction, variation over 8 tensors 7.8 us instead of 6.4.)
template <int THREADS, int COUNT>
__device__ inline void block_sum(double (&v)[COUNT], double *sh) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < COUNT; ++c) {
        v[c] = wave_sum(v[c]);
        if (lane == 0) sh[COUNT * wave + c] = v[c];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int c = 0; c < COUNT; ++c) {
            v[c] = sh[c];
#pragma unroll
            for (int w = 1; w < THREADS / 64; ++w) v[c] += sh[COUNT * w + c];
        }
    }
}

// The one-launch form's end, for the first wavefront alone: v holds this block's sums.  Every block publishes its
// sums and a check word, a 64-bit hash of the launch's nonce and the sums, with device-scope stores,
// passes a sequentially consistent fence, and then reads everybody's.  A block's sums count once they
// fit their check.  Words of a record half written or left by something else fit it with a probability
// of 2^-64; a whole record of an earlier launch with the same nonce, a replay of this one from a
// graph, is not there, because a launch clears its checks before it ends.  The block whose stores come
// last sees all records: at least one block finds everything present, forms the totals (every block
// that does forms the same ones) and clears the checks.  Nobody waits for anybody.  Returns whether
// this block has the totals in v.
// The check is a sum of one term per word, each a bijection of the word under a nonce of its own, so that
// the multiplications do not wait for each other.
__device__ inline uint64_t term_of(uint64_t nonce, int c, uint64_t bits) {
    const uint64_t t = ((nonce + (uint64_t)c * 0xD1B54A32D192ED03ull) ^ bits) * 0x9E3779B97F4A7C15ull;
    return t ^ (t >> 32);
}

template <int COUNT>
__device__ inline bool finish_here(double (&v)[COUNT], uint64_t *records, uint64_t nonce) {
    constexpr int kWords = COUNT + 1;
    const int lane = threadIdx.x, blocks = gridDim.x;
    if (lane == 0) {
        uint64_t *r = records + kWords * blockIdx.x, check = 0;
#pragma unroll
        for (int c = 0; c < COUNT; ++c) {
            const uint64_t bits = (uint64_t)__double_as_longlong(v[c]);
            __hip_atomic_store(r + c, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            check += term_of(nonce, c, bits);
        }
        // 0 is what a cleared check holds
        __hip_atomic_store(r + COUNT, check ? check : 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "agent");   // the stores before anybody's loads below
    uint64_t *const mine = records + kWords * (lane < blocks ? lane : 0);   // the record this lane reads
    uint64_t word[kWords], check = 0;
#pragma unroll
    for (int c = 0; c < kWords; ++c) word[c] = __hip_atomic_load(mine + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int c = 0; c < COUNT; ++c) {
        check += term_of(nonce, c, word[c]);
        v[c] = lane < blocks ? __longlong_as_double((long long)word[c]) : 0.0;
    }
    if (!__all((check ? check : 1) == word[COUNT])) return false;
    if (lane < blocks) __hip_atomic_store(mine + COUNT, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int c = 0; c < COUNT; ++c) v[c] = wave_sum(v[c]);
    return true;
}

// ---- the passes ------------------------------------------------------------------------------
// An Op describes one reduction over packs of consecutive elements (16 B per tensor and pack):
//   kCount, kElems       sums it keeps; elements per pack
//   kThreads, kUnroll    launch shape of the two-launch form: threads, packs in flight per lane
//   kOneUnroll, kBytes   packs in flight in the one-launch form (512 threads); the workspace
//   kOneChunks           chunks a block takes there beyond 16 blocks
//   kOneMost, kOuts      elements up to which that form is taken (see the top); floats of output
//   kSlabs               how the blocks share the packs (see reduce_kernel)
//   Regs, load, add      what a pack occupies, how it is read and summed
//   tail                 one element past the last whole pack
//   finish               totals -> outputs
// A reduction reads its tensors once, so it loads them non-temporally: measured against ordinary
// loads this is 6 % faster on the 33.5 MB latent pair and 10-13 % faster from 0.5 GB on, provided
// every load instruction of a wavefront covers whole lines (a lane stride of 16 B); the exception is
// the frame gradient, whose second read of every element is meant to hit in the caches.

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float4 stream4f(const float *p) {
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ inline float abs4(const float4 &a, const float4 &b) {
    return (fabsf(a.x - b.x) + fabsf(a.y - b.y)) + (fabsf(a.z - b.z) + fabsf(a.w - b.w));
}
__device__ inline float abs4(const float4 &b) {
    return (fabsf(b.x) + fabsf(b.y)) + (fabsf(b.z) + fabsf(b.w));
}

// One 16 B piece of a float or bf16 tensor (4 or 8 consecutive elements), widened by get().
template <typename T>
struct Pack;
template <>
struct Pack<float> {
    static constexpr int kElems = 4;
    float4 v;
    __device__ void stream(const float *p) { v = stream4f(p); }
    __device__ void load(const float *p) {   // any alignment of p
        f32x4 t;
        __builtin_memcpy(&t, p, 16);
        v = make_float4(t.x, t.y, t.z, t.w);
    }
    __device__ float get(int i) const {
        switch (i) { case 0: return v.x; case 1: return v.y; case 2: return v.z; default: return v.w; }
    }
};
template <>
struct Pack<uint16_t> {  // bf16 bit patterns
    static constexpr int kElems = 8;
    uint4 v;
    __device__ void stream(const uint16_t *p) { v = load16<true>(p); }
    __device__ void load(const uint16_t *p) {
        u32x4 t;
        __builtin_memcpy(&t, p, 16);
        v = make_uint4(t.x, t.y, t.z, t.w);
    }
    __device__ float get(int i) const {
        uint32_t w;
        switch (i >> 1) { case 0: w = v.x; break; case 1: w = v.y; break; case 2: w = v.z; break; default: w = v.w; }
        return (i & 1) ? bf16_hi(w) : bf16_lo(w);
    }
};

__device__ inline float widen(float v) { return v; }
__device__ inline float widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

// sum|cur - prev|, sum|prev| -> both and their ratio
struct DeltaOp {
    static constexpr int kCount = 2, kElems = 4, kThreads = 1024, kUnroll = 4, kOneUnroll = 2, kOneChunks = 2, kOuts = 3;
    static constexpr bool kSlabs = false;
    static constexpr size_t kBytes = kDeltaBytes;
    static constexpr int64_t kOneMost = 3 << 17;
    const float *cur, *prev;
    struct Regs { float4 a, b; };
    __device__ void load(Regs &r, int64_t i) const { r.a = stream4f(cur + 4 * i); r.b = stream4f(prev + 4 * i); }
    __device__ void add(const Regs &r, double (&s)[kCount]) const {
        s[0] += (double)abs4(r.a, r.b);
        s[1] += (double)abs4(r.b);
    }
    __device__ void tail(int64_t j, double (&s)[kCount]) const {
        s[0] += (double)fabsf(cur[j] - prev[j]);
        s[1] += (double)fabsf(prev[j]);
    }
    __device__ static void finish(const double (&s)[kCount], float *out) {
        out[0] = (float)s[0];
        out[1] = (float)s[1];
        out[2] = s[1] > 0.0 ? (float)(s[0] / s[1]) : s[0] > 0.0 ? __builtin_inff() : 0.0f;
    }
};

// <a, b>, <a, a>, <b, b> -> all three and the cosine
// THREADS: us for 1024 and 512 threads: binary32, 2 x 0.65 million elements 6.2 4.6, 2 x 2 million 6.5 5.9, 2 x 4.2
// million 7.0 7.7, 2 x 8 million 12.0 13.4, 2 x 24 million 29.5 31.1; bf16, 2 x 2 million 5.7 5.4, 2 x 8.4 million
// 8.5 7.9, 2 x 75 million, cold, 54 50.6.
template <typename T, int THREADS = 512>
struct SimilarityOp {
    static constexpr int kCount = 3, kElems = Pack<T>::kElems, kThreads = THREADS, kUnroll = 4, kOneUnroll = 2, kOneChunks = 2, kOuts = 4;
    static constexpr bool kSlabs = false;
    static constexpr size_t kBytes = kSimilarityBytes;
    static constexpr int64_t kOneMost = sizeof(T) == 4 ? 1 << 19 : 5 << 18;
    const T *a, *b;
    struct Regs { Pack<T> x, y; };
    __device__ void load(Regs &r, int64_t i) const { r.x.stream(a + kElems * i); r.y.stream(b + kElems * i); }
    __device__ void add(const Regs &r, double (&s)[kCount]) const {
#pragma unroll
        for (int g = 0; g < kElems / 4; ++g) {
            float pab = 0.f, paa = 0.f, pbb = 0.f;
#pragma unroll
            for (int e = 4 * g; e < 4 * g + 4; ++e) {
                const float xv = r.x.get(e), yv = r.y.get(e);
                pab = fmaf(xv, yv, pab);
                paa = fmaf(xv, xv, paa);
                pbb = fmaf(yv, yv, pbb);
            }
            s[0] += (double)pab;
            s[1] += (double)paa;
            s[2] += (double)pbb;
        }
    }
    __device__ void tail(int64_t j, double (&s)[kCount]) const {
        const float xv = widen(a[j]), yv = widen(b[j]);
        s[0] += (double)(xv * yv);
        s[1] += (double)(xv * xv);
        s[2] += (double)(yv * yv);
    }
    __device__ static void finish(const double (&s)[kCount], float *out) {
        const double denom = sqrt(s[1]) * sqrt(s[2]);
        out[0] = (float)s[0];
        out[1] = (float)s[1];
        out[2] = (float)s[2];
        out[3] = denom > 0.0 ? (float)(s[0] / denom) : 0.0f;
    }
};

// The feature map is [frames, inner]; the gradient is the forward difference along the frame axis
// and the norm is Euclidean: a pass over the pair (m, m + inner), of which the second is aligned to
// its elements only (the hardware takes 16 B loads at any address).
template <typename T>
struct GradientOp {
    // us with chunks of 2 packs a lane, slabs per block; of 16 elements a lane, every 256th chunk; of 8
    // elements a lane, every 256th chunk (the last two read much of the map twice: the CU that has read
    // the frame before is another one).  binary32, 16.8 and 31 million elements, frames of 1288 12.7
    // 20.6, 17.4 33, 14.0 23; of 4096 12.9 20.8, 14.8 25, 17.3 30; of 16384 17.2 28, 22 38, 22 38.  bf16, 16.8
    // and 31 million, frames of 1288 7.1 12.6, 7.6 13.2, 9.1 13.7; of 8192 7.6 13.1, 10.8 17.0, 12.7 20.4.
    static constexpr int kCount = 1, kElems = Pack<T>::kElems, kThreads = 1024, kUnroll = 2, kOneUnroll = 2, kOneChunks = 2, kOuts = 2;
    static constexpr bool kSlabs = true;
    static constexpr size_t kBytes = kGradientBytes;
    static constexpr int64_t kOneMost = (1 << 20) / sizeof(T);
    const T *m;
    int64_t inner;
    struct Regs { Pack<T> x, y; };
    __device__ void load(Regs &r, int64_t i) const { r.x.load(m + kElems * i); r.y.load(m + inner + kElems * i); }
    __device__ void add(const Regs &r, double (&s)[kCount]) const {
#pragma unroll
        for (int g = 0; g < kElems / 4; ++g) {
            double p = 0.0;
#pragma unroll
            for (int e = 4 * g; e < 4 * g + 4; ++e) {
                const double d = (double)(r.y.get(e) - r.x.get(e));
                p = fma(d, d, p);
            }
            s[0] += p;
        }
    }
    __device__ void tail(int64_t j, double (&s)[kCount]) const {
        const float d = widen(m[inner + j]) - widen(m[j]);
        s[0] += (double)d * (double)d;
    }
    __device__ static void finish(const double (&s)[kCount], float *out) {
        out[0] = (float)s[0];
        out[1] = (float)sqrt(s[0]);
    }
};

// L1 distance of the current tensor to each of COUNT earlier ones: the current tensor is read once,
// not once per distance.
struct PrevList { const float *p[QC_MAX_PREV]; };

template <int COUNT>
struct VariationOp {
    // two wavefronts per SIMD: room for 2 x 2 (COUNT + 1) float4 per lane
    static constexpr int kCount = COUNT, kElems = 4, kThreads = 512, kUnroll = 2, kOneUnroll = 1, kOneChunks = COUNT > 4 ? 1 : 2, kOuts = COUNT + 1;
    static constexpr bool kSlabs = false;
    static constexpr size_t kBytes = kVariationBytes;
    static constexpr int64_t kOneMost = 3 << 15;
    const float *cur;
    PrevList prevs;
    struct Regs { float4 a, b[COUNT]; };
    __device__ void load(Regs &r, int64_t i) const {
        r.a = stream4f(cur + 4 * i);
#pragma unroll
        for (int c = 0; c < COUNT; ++c) r.b[c] = stream4f(prevs.p[c] + 4 * i);
    }
    __device__ void add(const Regs &r, double (&s)[kCount]) const {
#pragma unroll
        for (int c = 0; c < COUNT; ++c) s[c] += (double)abs4(r.a, r.b[c]);
    }
    __device__ void tail(int64_t j, double (&s)[kCount]) const {
#pragma unroll
        for (int c = 0; c < COUNT; ++c) s[c] += (double)fabsf(cur[j] - prevs.p[c][j]);
    }
    __device__ static void finish(const double (&s)[kCount], float *out) {
        double total = 0.0;
#pragma unroll
        for (int c = 0; c < COUNT; ++c) {
            out[c] = (float)s[c];
            total += s[c];
        }
        out[COUNT] = (float)total;
    }
};

// A block reads chunks of THREADS * U packs, consecutive lanes consecutive packs, all of a chunk's loads
// ahead of the first use: those at first, first + step, .. below `end`, of which the last may be partial.
//   kSlabs false   every gridDim.x-th chunk of the tensors
//   kSlabs true    one stretch of `slab` packs, a slab per block: where what a chunk reads overlaps the
//                  chunk after it, both are read through the same caches
// (Loading a chunk while the one before is summed gains nothing, at 16 wavefronts per CU, and the longer
// code costs the small calls 0.2 us; so did a division to count the chunks.)
template <typename Op, int THREADS, int U, bool ONE_LAUNCH>
__global__ __launch_bounds__(THREADS) void reduce_kernel(Op op, int64_t n, int64_t slab, double *__restrict__ partials,
                                                         float *__restrict__ out, uint64_t nonce) {
    constexpr int C = Op::kCount;
    __shared__ double sh[C * (THREADS / 64)];
    const int64_t packs = n / Op::kElems;
    constexpr int64_t kChunk = (int64_t)THREADS * U;
    double s[C];
#pragma unroll
    for (int c = 0; c < C; ++c) s[c] = 0.0;
    int64_t first = (int64_t)blockIdx.x * kChunk, end = packs, step = (int64_t)gridDim.x * kChunk;
    if constexpr (Op::kSlabs) {
        first = (int64_t)blockIdx.x * slab;
        end = first + slab < packs ? first + slab : packs;
        step = kChunk;
    }
    int64_t base = first + threadIdx.x;
    typename Op::Regs r[U];
    for (; first + kChunk <= end; first += step, base += step) {
#pragma unroll
        for (int u = 0; u < U; ++u) op.load(r[u], base + u * THREADS);
#pragma unroll
        for (int u = 0; u < U; ++u) op.add(r[u], s);
    }
    if (first < end) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = base + u * THREADS;
            op.load(r[u], i < end ? i : end - 1);   // a valid pack either way
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (base + u * THREADS < end) op.add(r[u], s);
    }
    if (blockIdx.x == 0 && threadIdx.x < (int)(n - packs * Op::kElems)) op.tail(packs * Op::kElems + threadIdx.x, s);
    block_sum<THREADS, C>(s, sh);
    if constexpr (ONE_LAUNCH) {
        if (threadIdx.x >= 64) return;
        if (finish_here(s, reinterpret_cast<uint64_t *>(partials), nonce) && threadIdx.x == 0)
            Op::finish(s, out);
    } else if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < C; ++c) partials[C * blockIdx.x + c] = s[c];
    }
}

// one wavefront: fixed-order combine of the partial sums, four blocks' a lane (with a thread per block, and the four wavefronts'
// sums through LDS, against this, us in a graph: latent delta of 4 million 6.34 6.20, frame gradient 5.30 5.20, variation over 8 tensors of 1 million
// 8.71 8.29, similarity of 4 million 6.67 6.56; nowhere faster)
template <typename Op>
__global__ __launch_bounds__(kFinalThreads) void final_kernel(const double *__restrict__ partials, int count,
                                                              float *__restrict__ out) {
    constexpr int C = Op::kCount, kPer = kMaxBlocks / kFinalThreads;
    double p[kPer][C], s[C];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int b = (int)threadIdx.x + kFinalThreads * i;
#pragma unroll
        for (int c = 0; c < C; ++c) p[i][c] = partials[C * (b < count ? b : 0) + c];
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        s[c] = 0.0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) s[c] += (int)threadIdx.x + kFinalThreads * i < count ? p[i][c] : 0.0;
        s[c] = wave_sum(s[c]);
    }
    if (threadIdx.x == 0) Op::finish(s, out);
}

// a number no earlier launch of this process has used (splitmix64 of a counter)
uint64_t next_nonce() {
    static std::atomic<uint64_t> counter{0};
    uint64_t z = (counter.fetch_add(1, std::memory_order_relaxed) + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

template <typename Op>
qc_status launch_reduction(const Op &op, int64_t n, float *out, void *workspace, void *stream) {
    double *partials = (double *)workspace;
    hipStream_t st = (hipStream_t)stream;
    auto blocks_for = [&](int64_t chunk, int most) {
        const int64_t b = (n / Op::kElems + chunk - 1) / chunk;
        return (unsigned)(b < 1 ? 1 : b > most ? most : b);
    };
    auto slab_for = [&](unsigned blocks) {   // whole wavefronts
        return round_up((n / Op::kElems + blocks - 1) / blocks, 64);
    };
    // One launch needs the records to itself until every block that has the totals has spoiled the
    // checks: outputs that lie in the workspace are written by the second launch.
    if (n <= Op::kOneMost && !overlap(out, Op::kOuts * sizeof(float), workspace, Op::kBytes)) {
        constexpr int U = Op::kOneUnroll;
        static_assert(kOneBlocks * (Op::kCount + 1) * sizeof(double) <= Op::kBytes, "room for the blocks' sums and check words");
        const int64_t chunk = (int64_t)kOneThreads * U;
        const unsigned few = blocks_for(chunk, kOneFew), more = blocks_for(chunk * Op::kOneChunks, kOneBlocks), blocks = few > more ? few : more;
        reduce_kernel<Op, kOneThreads, U, true><<<dim3(blocks), dim3(kOneThreads), 0, st>>>(op, n, slab_for(blocks), partials, out, next_nonce());
        return hipGetLastError() == hipSuccess ? QC_OK : QC_ERR_DEVICE;
    }
    const unsigned blocks = blocks_for((int64_t)Op::kThreads * Op::kUnroll, kMaxBlocks);
    reduce_kernel<Op, Op::kThreads, Op::kUnroll, false><<<dim3(blocks), dim3(Op::kThreads), 0, st>>>(op, n, slab_for(blocks), partials, nullptr, 0);
    if (hipGetLastError() != hipSuccess) return QC_ERR_DEVICE;
    final_kernel<Op><<<dim3(1), dim3(kFinalThreads), 0, st>>>(partials, (int)blocks, out);
    return hipGetLastError() == hipSuccess ? QC_OK : QC_ERR_DEVICE;
}

template <int COUNT>
qc_status launch_variation(const float *cur, const PrevList &prevs, int64_t n, float *out, void *workspace, void *stream) {
    return launch_reduction(VariationOp<COUNT>{cur, prevs}, n, out, workspace, stream);
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

}  // namespace
}  // namespace qc

using namespace qc;

extern "C" size_t qc_latent_delta_workspace_bytes(int64_t n) {
    if (n < 1) return 0;
    return kDeltaBytes;
}

extern "C" qc_status qc_latent_delta(const float *cur, const float *prev, int64_t n, float *out3,
                                     void *workspace, size_t workspace_bytes, void *stream) {
    if (!cur || !prev || !out3 || !workspace || n < 1) return QC_ERR_INVALID_ARG;
    if (!aligned(cur, 16) || !aligned(prev, 16) || !aligned(out3, 4) || !aligned(workspace, 256))
        return QC_ERR_INVALID_ARG;
    if (workspace_bytes < qc_latent_delta_workspace_bytes(n)) return QC_ERR_WORKSPACE;
    return launch_reduction(DeltaOp{cur, prev}, n, out3, workspace, stream);
}

// ---- qc_latent_delta for callers that cannot allocate ---------------------------------------
// The per-block partial sums live in a file-scope device array instead of a caller's workspace.
// `scratch` below is the host-side handle of that array, not a device address: host code asks
// the runtime once per device for the address of that device's copy and uses only that.
namespace {
constexpr size_t kStaticScratchBytes = kDeltaBytes;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::atomic<void *> g_scratch_ptr[kMaxDevices];

// device address of the current device's copy of `scratch`, resolved on first use
qc_status static_scratch(void **out) {
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0) return QC_ERR_DEVICE;
    if (device >= kMaxDevices) return QC_ERR_UNSUPPORTED;
    void *p = g_scratch_ptr[device].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return QC_ERR_DEVICE;
        g_scratch_ptr[device].store(p, std::memory_order_release);  // racing threads store the same value
    }
    *out = p;
    return QC_OK;
}
}  // namespace

extern "C" qc_status qc_latent_delta_static(const float *cur, const float *prev, int64_t n,
                                            float *out3, void *stream) {
    if (!cur || !prev || !out3 || n < 1) return QC_ERR_INVALID_ARG;
    if (n > QC_LATENT_DELTA_STATIC_MAX_N) return QC_ERR_UNSUPPORTED;
    void *ws = nullptr;
    if (qc_status st = static_scratch(&ws); st != QC_OK) return st;
    // nothing to clear: one launch rejects by their check words what earlier calls left there, and of two the
    // second reads only what the first has written
    return qc_latent_delta(cur, prev, n, out3, ws, kStaticScratchBytes, stream);
}

extern "C" size_t qc_layer_similarity_workspace_bytes(int64_t n) {
    if (n < 1) return 0;
    return kSimilarityBytes;
}

extern "C" qc_status qc_layer_similarity(const void *a, const void *b, qc_dtype dt, int64_t n,
                                         float *out4, void *workspace, size_t workspace_bytes,
                                         void *stream) {
    if (!a || !b || !out4 || !workspace || n < 1) return QC_ERR_INVALID_ARG;
    if (dt != QC_F32 && dt != QC_BF16) return QC_ERR_INVALID_ARG;
    if (!aligned(a, 16) || !aligned(b, 16) || !aligned(out4, 4) || !aligned(workspace, 256))
        return QC_ERR_INVALID_ARG;
    if (workspace_bytes < qc_layer_similarity_workspace_bytes(n)) return QC_ERR_WORKSPACE;
    if (dt == QC_BF16)
        return launch_reduction(SimilarityOp<uint16_t>{(const uint16_t *)a, (const uint16_t *)b}, n, out4,
                                workspace, stream);
    if (n > 1 << 21)
        return launch_reduction(SimilarityOp<float, 1024>{(const float *)a, (const float *)b}, n, out4, workspace, stream);
    return launch_reduction(SimilarityOp<float>{(const float *)a, (const float *)b}, n, out4, workspace, stream);
}

extern "C" size_t qc_frame_gradient_norm_workspace_bytes(int64_t frames, int64_t inner) {
    if (frames < 1 || inner < 1) return 0;
    return kGradientBytes;
}

extern "C" qc_status qc_frame_gradient_norm(const void *m, qc_dtype dt, int64_t frames,
                                            int64_t inner, float *out2, void *workspace,
                                            size_t workspace_bytes, void *stream) {
    if (!m || !out2 || !workspace || frames < 1 || inner < 1) return QC_ERR_INVALID_ARG;
    if (dt != QC_F32 && dt != QC_BF16) return QC_ERR_INVALID_ARG;
    if (!aligned(m, 16) || !aligned(out2, 4) || !aligned(workspace, 256)) return QC_ERR_INVALID_ARG;
    if (frames > INT64_MAX / inner) return QC_ERR_INVALID_ARG;
    if (workspace_bytes < qc_frame_gradient_norm_workspace_bytes(frames, inner)) return QC_ERR_WORKSPACE;
    const int64_t n = (frames - 1) * inner;  // number of differences
    if (dt == QC_BF16)
        return launch_reduction(GradientOp<uint16_t>{(const uint16_t *)m, inner}, n, out2, workspace, stream);
    return launch_reduction(GradientOp<float>{(const float *)m, inner}, n, out2, workspace, stream);
}

extern "C" size_t qc_cumulative_variation_workspace_bytes(int64_t n, int count) {
    if (n < 1 || count < 1 || count > QC_MAX_PREV) return 0;
    return kVariationBytes;
}

extern "C" qc_status qc_cumulative_variation(const float *cur, const float *const *prevs, int count,
                                             int64_t n, float *out, void *workspace,
                                             size_t workspace_bytes, void *stream) {
    if (!cur || !prevs || !out || !workspace || n < 1 || count < 1) return QC_ERR_INVALID_ARG;
    if (count > QC_MAX_PREV) return QC_ERR_UNSUPPORTED;
    if (!aligned(cur, 16) || !aligned(out, 4) || !aligned(workspace, 256)) return QC_ERR_INVALID_ARG;
    PrevList list;
    for (int c = 0; c < QC_MAX_PREV; ++c) {
        list.p[c] = c < count ? prevs[c] : nullptr;
        if (c < count && (!prevs[c] || !aligned(prevs[c], 16))) return QC_ERR_INVALID_ARG;
    }
    if (workspace_bytes < qc_cumulative_variation_workspace_bytes(n, count)) return QC_ERR_WORKSPACE;
    switch (count) {
        case 1: return launch_variation<1>(cur, list, n, out, workspace, stream);
        case 2: return launch_variation<2>(cur, list, n, out, workspace, stream);
        case 3: return launch_variation<3>(cur, list, n, out, workspace, stream);
        case 4: return launch_variation<4>(cur, list, n, out, workspace, stream);
        case 5: return launch_variation<5>(cur, list, n, out, workspace, stream);
        case 6: return launch_variation<6>(cur, list, n, out, workspace, stream);
        case 7: return launch_variation<7>(cur, list, n, out, workspace, stream);
        default: return launch_variation<8>(cur, list, n, out, workspace, stream);
    }
}
