// mlp.hip -- the learned subtree proposal: a small MLP that predicts, per
// segment, which depth-8 subtree of the BVH holds its first hit, so the
// traversal can visit that subtree first and stop early on a sure hit.  The
// exact traversal still decides every result; the proposal only changes the
// order of work.
//
// Network: 6 endpoint coordinates normalised to [-1, 1] over the mesh box,
// plus sin / cos (pi f_k x) for 16 bands f_k = 2^(k/2) per coordinate
// (198 features, padded to 224), three hidden layers of 256 with ReLU, 256
// logits (one per frontier bucket; unused buckets masked).  bf16 weights and
// activations, fp32 accumulation on the matrix cores (v_mfma_f32_16x16x32_bf16);
// fp32 master weights and Adam for training.
//
// MFMA 16x16x32 bf16 operand layout on a wave of 64 lanes (lane l):
//   A (16 x 32): row l % 16, k = 8 (l / 16) + j, j = 0..7
//   B (32 x 16): col l % 16, k = 8 (l / 16) + j
//   D (16 x 16): row 4 (l / 16) + i, col l % 16, i = 0..3
#include "rsi_internal.h"

namespace rsi {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// -------------------------------------------------------------- features
// Feature j of one segment (j < kMlpIn; zero past kMlpFeat).  Coordinates are
// normalised as n = (p - lo) / (hi - lo) (0 on a flat axis), x = 2 n - 1; the
// band frequencies are the float32 values 2^(k/2).
__device__ __forceinline__ float band_freq(int k) {
    return ldexpf((k & 1) ? 1.41421354f : 1.0f, k >> 1);
}

__device__ __forceinline__ float norm_coord(float p, float lo, float hi) {
#pragma clang fp contract(off)
    const float ext = hi - lo;
    const float n = ext > 0.0f ? (p - lo) / ext : 0.0f;
    return n * 2.0f - 1.0f;
}

// sin(pi a) and cos(pi a): the hardware sine / cosine take their argument in
// turns, so a / 2 is reduced exactly to [-1/2, 1/2] first.  The features are
// rounded to bf16 (8 bits), far coarser than the instruction's error.
__device__ __forceinline__ void sincospi_fast(float a, float &sn, float &cs) {
    float t = 0.5f * a;
    t = t - rintf(t);
    sn = __builtin_amdgcn_sinf(t);
    cs = __builtin_amdgcn_cosf(t);
}

// Writes the 33 features that depend on coordinate c (its value, then
// sin / cos of the 16 bands) into row[].
__device__ __forceinline__ void coord_features(float x, int c, __bf16 *row) {
#pragma clang fp contract(off)
    row[c] = (__bf16)x;
    for (int k = 0; k < kMlpBands; ++k) {
        const float a = band_freq(k) * x;
        float sn, cs;
        sincospi_fast(a, sn, cs);
        row[6 + c * 2 * kMlpBands + 2 * k] = (__bf16)sn;
        row[6 + c * 2 * kMlpBands + 2 * k + 1] = (__bf16)cs;
    }
}

__device__ __forceinline__ float seg_coord(const float *__restrict__ from, const float *__restrict__ to, int64_t i,
                                           int c) {
    return c < 3 ? from[3 * i + c] : to[3 * i + c - 3];
}

// X[r][0..kMlpIn) for rows [0, rows): segment index = ids ? ids[r0 + r] : r0 + r.
__global__ __launch_bounds__(256) void k_features(const float *__restrict__ from, const float *__restrict__ to,
                                                  const int32_t *__restrict__ ids, int64_t r0, int64_t rows,
                                                  const float *__restrict__ bounds, __bf16 *__restrict__ X) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = t / 7;
    const int part = (int)(t % 7);
    if (r >= rows)
        return;
    __bf16 *row = X + r * kMlpIn;
    if (part == 6) {
        for (int j = kMlpFeat; j < kMlpIn; ++j)
            row[j] = (__bf16)0.0f;
        return;
    }
    const int64_t seg = ids ? ids[r0 + r] : r0 + r;
    const int c = part;
    const float x = norm_coord(seg_coord(from, to, seg, c), bounds[c % 3], bounds[3 + c % 3]);
    coord_features(x, c, row);
}

// Uniform(-a, a) initial weights from a counter-based hash (seed, index).
__device__ __forceinline__ uint32_t mix32(uint64_t x) {
    x ^= x >> 33;
    x *= 0xff51afd7ed558ccdull;
    x ^= x >> 33;
    x *= 0xc4ceb9fe1a85ec53ull;
    x ^= x >> 33;
    return (uint32_t)x;
}

// The bf16 weights are kept in MFMA fragment order: a layer with K inputs is
// a sequence of 16-column x 32-k blocks (column tile major, then k step),
// each 1 KB block laid out as the B operand's lanes take it (lane l: column
// l % 16, k = 8 (l / 16) .. + 7), so one wave-wide 16-byte load reads one
// whole block, eight full cache lines.
__host__ __device__ constexpr int64_t frag_index(int col, int k, int K) {
    return ((((int64_t)(col >> 4) * (K >> 5) + (k >> 5)) * 64 + (col & 15) + 16 * ((k & 31) >> 3)) << 3) + (k & 7);
}

// bf16 copies of weight i (layer l's W[out][in]): Wb in fragment order with
// columns = outputs (the forward product), and for layers 2..4 WbT in
// fragment order with columns = inputs (the backward product)
__device__ __forceinline__ void store_weight(__bf16 *__restrict__ Wb, __bf16 *__restrict__ WbT, int64_t i, float w) {
    const __bf16 h = (__bf16)w;
    const int64_t first = (int64_t)kMlpOut * kMlpIn, hh = (int64_t)kMlpHidden * kMlpHidden;
    if (i < first) {
        Wb[frag_index((int)(i / kMlpIn), (int)(i % kMlpIn), kMlpIn)] = h;
    } else {
        const int64_t l = (i - first) / hh, j = (i - first) % hh;
        const int o = (int)(j / kMlpHidden), in = (int)(j % kMlpHidden);
        Wb[first + l * hh + frag_index(o, in, kMlpHidden)] = h;
        WbT[l * hh + frag_index(in, o, kMlpHidden)] = h;
    }
}

__global__ __launch_bounds__(256) void k_init_params(float *__restrict__ P, __bf16 *__restrict__ Wb,
                                                     __bf16 *__restrict__ WbT, float *__restrict__ m1,
                                                     float *__restrict__ m2, uint64_t seed) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kMlpParams)
        return;
    float w = 0.0f;
    if (i < kMlpWeights) {
        const int fan_in = i < (int64_t)kMlpOut * kMlpIn ? kMlpFeat : kMlpHidden;
        const float a = sqrtf(6.0f / (float)fan_in);
        const float u = (mix32(seed * 0x9e3779b97f4a7c15ull + (uint64_t)i) >> 8) * 0x1p-24f;
        w = (2.0f * u - 1.0f) * a;
        if (i < (int64_t)kMlpOut * kMlpIn && (i % kMlpIn) >= kMlpFeat)
            w = 0.0f;  // padding features carry no weight
        store_weight(Wb, WbT, i, w);
    }
    P[i] = w;
    m1[i] = 0.0f;
    m2[i] = 0.0f;
}

// ------------------------------------------------ fused inference kernel
// kPRows segments per tile; four waves, wave w producing output columns
// [64 w, 64 w + 64) of every layer for all rows (24 MFMA per k step, so each
// weight fragment fetched from L2 feeds 6 row tiles).  Activations stay in LDS
// in one bf16 buffer that each layer overwrites once every wave has read it
// (two workgroups per CU, two waves per SIMD).  Weight fragments load two
// k steps ahead of the multiplies that use them, activations one.
// The weights are the MFMA's row operand and the segments its columns, so a
// lane ends with four neighbouring outputs of one segment: the epilogue packs
// them into one 8-byte LDS write, and the argmax needs two exchanges between
// lanes per row tile.  2e6 segments take 957 us (1,060 TFLOP/s;
// 1,279 with segments as rows, 24 row exchanges of four steps and 2-byte LDS
// writes).  Measured: 80 rows 1,004, 112 rows 979 (they spill), weights three
// steps ahead 970, activations read in their own step 1,001.
// The accumulation order over k is the training pass's, so the logits are
// bit-identical to its forward pass.
constexpr int kPRows = 96;
constexpr int kPPitch = kMlpHidden + 8;
constexpr int kPRowTiles = kPRows / 16;
constexpr int kPWaves = 4;                          // waves per workgroup, each owning a column slice
constexpr int kPThreads = 64 * kPWaves;
constexpr int kPColTiles = kMlpHidden / 16 / kPWaves;  // 16-column tiles per wave
constexpr int kPAhead = 2;  // k steps the weight loads run ahead
constexpr int kPRead = 1;   // and the activations' reads

// One layer of the inference tile: acc[a][b] = outputs 64 wave + 16 b .. + 15
// (rows) of segments 16 a .. + 15 (columns).  K (224 or 256) is known at compile
// time and the k loop fully unrolled, so every step's fragments are registers
// of their own and its loads stay in flight across the steps before it.
template <int K>
__device__ __forceinline__ void layer_tile(const __bf16 *__restrict__ Xin, const __bf16 *__restrict__ Wt, int wave,
                                           int lane, f32x4 (&acc)[kPRowTiles][kPColTiles]) {
    static_assert(K % 32 == 0, "K must be a multiple of 32");
    constexpr int kSteps = K / 32;
#pragma unroll
    for (int a = 0; a < kPRowTiles; ++a)
#pragma unroll
        for (int b = 0; b < kPColTiles; ++b)
            acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // the wave's first column tile, this lane's 16 bytes of each block
    const __bf16 *wfrag = Wt + (int64_t)kPColTiles * wave * kSteps * 512 + 8 * lane;
    const __bf16 *xrow = Xin + (lane & 15) * kPPitch + 8 * (lane >> 4);
    bf16x8 f[kSteps][kPColTiles], x[kSteps][kPRowTiles];
    auto weights = [&](int st) {
#pragma unroll
        for (int b = 0; b < kPColTiles; ++b)
            f[st][b] = *reinterpret_cast<const bf16x8 *>(wfrag + (int64_t)(b * kSteps + st) * 512);
    };
    auto rows = [&](int st) {
#pragma unroll
        for (int a = 0; a < kPRowTiles; ++a)
            x[st][a] = *reinterpret_cast<const bf16x8 *>(xrow + 16 * a * kPPitch + 32 * st);
    };
#pragma unroll
    for (int st = 0; st < kPAhead; ++st)
        weights(st);
#pragma unroll
    for (int st = 0; st < kPRead; ++st)
        rows(st);
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
        if (st + kPAhead < kSteps)
            weights(st + kPAhead);
        if (st + kPRead < kSteps)
            rows(st + kPRead);
#pragma unroll
        for (int a = 0; a < kPRowTiles; ++a)
#pragma unroll
            for (int b = 0; b < kPColTiles; ++b)
                acc[a][b] = mfma16(f[st][b], x[st][a], acc[a][b]);
        __builtin_amdgcn_sched_barrier(0);  // keep each step's loads in its step: no hoisting past the register budget
    }
}

template <int RT, int CT>
__device__ __forceinline__ void tile_step(const __bf16 *__restrict__ xrow, int k0, const bf16x8 (&fb)[CT],
                                          f32x4 (&acc)[RT][CT]) {
#pragma unroll
    for (int a = 0; a < RT; ++a) {
        const bf16x8 fa = *reinterpret_cast<const bf16x8 *>(xrow + 16 * a * kPPitch + k0);
#pragma unroll
        for (int b = 0; b < CT; ++b)
            acc[a][b] = mfma16(fa, fb[b], acc[a][b]);
    }
}

// A layer of the training tile (segments as rows), in a chain: the first AHEAD k steps' fragments come
// in pf, and the last AHEAD steps load the next layer's first AHEAD steps
// (from Wn, with KN inputs; none when Wn is NULL) into pf, so a layer starts
// without waiting on memory and the epilogue between two layers hides the
// loads' latency.
template <int KN, int CT, int AHEAD>
__device__ __forceinline__ void prefetch_layer(const __bf16 *__restrict__ Wn, int wave, int lane,
                                               bf16x8 (&pf)[AHEAD][CT]) {
    constexpr int kStepsN = KN / 32;
    const __bf16 *nfrag = Wn + (int64_t)CT * wave * kStepsN * 512 + 8 * lane;
#pragma unroll
    for (int st = 0; st < AHEAD; ++st)
#pragma unroll
        for (int b = 0; b < CT; ++b)
            pf[st][b] = *reinterpret_cast<const bf16x8 *>(nfrag + (int64_t)(b * kStepsN + st) * 512);
}

template <int K, int KN, int RT, int CT, int AHEAD>
__device__ __forceinline__ void layer_chain(const __bf16 *__restrict__ Xin, const __bf16 *__restrict__ Wt,
                                            const __bf16 *__restrict__ Wn, int wave, int lane,
                                            f32x4 (&acc)[RT][CT], bf16x8 (&pf)[AHEAD][CT]) {
    constexpr int kSteps = K / 32, kStepsN = KN / 32;
    static_assert(K % 32 == 0 && KN % 32 == 0 && AHEAD <= kSteps && AHEAD <= kStepsN, "whole k steps");
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int b = 0; b < CT; ++b)
            acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int kq = 8 * (lane >> 4);
    const __bf16 *wfrag = Wt + (int64_t)CT * wave * kSteps * 512 + 8 * lane;
    const __bf16 *nfrag = Wn ? Wn + (int64_t)CT * wave * kStepsN * 512 + 8 * lane : nullptr;
    const __bf16 *xrow = Xin + (lane & 15) * kPPitch + kq;
    bf16x8 f[kSteps][CT];
#pragma unroll
    for (int st = 0; st < AHEAD; ++st)
#pragma unroll
        for (int b = 0; b < CT; ++b)
            f[st][b] = pf[st][b];
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
        if (st + AHEAD < kSteps) {
#pragma unroll
            for (int b = 0; b < CT; ++b)
                f[st + AHEAD][b] = *reinterpret_cast<const bf16x8 *>(wfrag + (int64_t)(b * kSteps + st + AHEAD) * 512);
        } else if (nfrag) {
#pragma unroll
            for (int b = 0; b < CT; ++b)
                pf[st + AHEAD - kSteps][b] =
                    *reinterpret_cast<const bf16x8 *>(nfrag + (int64_t)(b * kStepsN + st + AHEAD - kSteps) * 512);
        }
        tile_step(xrow, 32 * st, f[st], acc);
        __builtin_amdgcn_sched_barrier(0);
    }
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Half of the features that depend on coordinate c of value x (bands 8 h ..
// 8 h + 7, and with h = 0 the value) into row[].
__device__ __forceinline__ void half_features(float x, int c, int h, __bf16 *row) {
#pragma clang fp contract(off)
    if (h == 0)
        row[c] = (__bf16)x;
    const float f0 = h ? 16.0f : 1.0f;  // 2^(8 h / 2)
    __bf16 *out = row + 6 + c * 2 * kMlpBands + h * kMlpBands;
#pragma unroll
    for (int k = 0; k < kMlpBands / 2; ++k) {
        float sn, cs;
        sincospi_fast(f0 * band_freq(k) * x, sn, cs);
        *reinterpret_cast<bf16x2 *>(out + 2 * k) = bf16x2{(__bf16)sn, (__bf16)cs};
    }
}

__global__ __launch_bounds__(kPThreads) __attribute__((amdgpu_waves_per_eu(kPWaves / 2))) void k_mlp_propose(
    const float *__restrict__ from, const float *__restrict__ to, int64_t n, const float *__restrict__ bounds,
    const __bf16 *__restrict__ Wb, const float *__restrict__ P, int nb, uint8_t *__restrict__ bucket) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __bf16 *X = reinterpret_cast<__bf16 *>(lds_raw);  // activations, overwritten layer by layer
    float *best_v = reinterpret_cast<float *>(X + kPRows * kPPitch);  // [kPWaves][kPRows]
    int *best_i = reinterpret_cast<int *>(best_v + kPWaves * kPRows);  // [kPWaves][kPRows]
    float *bias = reinterpret_cast<float *>(best_i + kPWaves * kPRows);  // [4][kMlpOut]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g4 = lane >> 4;
    for (int i = tid; i < 4 * kMlpOut; i += kPThreads)
        bias[i] = P[kMlpWeights + i];
    // this lane's outputs: columns col0 + 16 b + i of segment l16 of each row tile
    const int col0 = 16 * kPColTiles * wave + 4 * g4;
    const int64_t tiles = (n + kPRows - 1) / kPRows;
#pragma unroll 1
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t r0 = tile * kPRows;
        // features -> X: 12 halves of a coordinate per segment, then the padding
#pragma unroll 1
        for (int q = tid; q < kPRows * 13; q += kPThreads) {
            const int r = q / 13, part = q % 13;
            __bf16 *row = X + r * kPPitch;
            if (part == 12) {
#pragma unroll
                for (int j = kMlpFeat; j < kMlpIn; j += 2)
                    *reinterpret_cast<bf16x2 *>(row + j) = bf16x2{(__bf16)0.0f, (__bf16)0.0f};
                continue;
            }
            const int64_t seg = r0 + r < n ? r0 + r : n - 1;
            const int c = part >> 1;
            half_features(norm_coord(seg_coord(from, to, seg, c), bounds[c % 3], bounds[3 + c % 3]), c, part & 1, row);
        }
        __syncthreads();
        // the four layers through one call site, so the accumulators keep one
        // register set; a layer's outputs go over its inputs in X once every
        // wave has read them
        f32x4 acc[kPRowTiles][kPColTiles];
#pragma unroll 1
        for (int l = 0; l < 4; ++l) {
            const int64_t woff = l == 0 ? 0 : (int64_t)kMlpOut * kMlpIn + (int64_t)(l - 1) * kMlpHidden * kMlpHidden;
            if (l == 0)
                layer_tile<kMlpIn>(X, Wb + woff, wave, lane, acc);
            else
                layer_tile<kMlpHidden>(X, Wb + woff, wave, lane, acc);
            if (l == 3)
                break;
            __syncthreads();  // every wave has read X before it is overwritten
#pragma unroll
            for (int b = 0; b < kPColTiles; ++b) {
                const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias + l * kMlpHidden + col0 + 16 * b);
#pragma unroll
                for (int a = 0; a < kPRowTiles; ++a) {
                    bf16x4 h;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        h[i] = (__bf16)fmaxf(acc[a][b][i] + bv[i], 0.0f);
                    *reinterpret_cast<bf16x4 *>(X + (16 * a + l16) * kPPitch + col0 + 16 * b) = h;
                }
            }
            __syncthreads();
        }
        // argmax over valid buckets (smallest index on ties): the lane's
        // columns ascend, then the four lanes of a segment, then the waves
#pragma unroll
        for (int a = 0; a < kPRowTiles; ++a) {
            float bv = -INFINITY;
            int bi = INT32_MAX;
#pragma unroll
            for (int b = 0; b < kPColTiles; ++b) {
                const f32x4 b4 = *reinterpret_cast<const f32x4 *>(bias + 3 * kMlpHidden + col0 + 16 * b);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = acc[a][b][i] + b4[i];
                    if (col0 + 16 * b + i < nb && (v > bv || (v == bv && bi == INT32_MAX))) {
                        bv = v;
                        bi = col0 + 16 * b + i;
                    }
                }
            }
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) {
                const float ov = __shfl_xor(bv, off);
                const int oi = __shfl_xor(bi, off);
                if (ov > bv || (ov == bv && oi < bi)) {
                    bv = ov;
                    bi = oi;
                }
            }
            if (g4 == 0) {
                best_v[wave * kPRows + 16 * a + l16] = bv;
                best_i[wave * kPRows + 16 * a + l16] = bi;
            }
        }
        __syncthreads();
        if (tid < kPRows && r0 + tid < n) {
            float bv = best_v[tid];
            int bi = best_i[tid];
            for (int w = 1; w < kPWaves; ++w) {
                const float v = best_v[w * kPRows + tid];
                const int i2 = best_i[w * kPRows + tid];
                if (v > bv || (v == bv && i2 < bi)) {
                    bv = v;
                    bi = i2;
                }
            }
            bucket[r0 + tid] = (uint8_t)(bi >= 0 && bi < nb ? bi : 0);
        }
        // no barrier: the next write of best_v / best_i and of X by a faster
        // wave comes after barriers that this wave has yet to reach
    }
}

constexpr size_t kProposeLds = (size_t)kPRows * kPPitch * sizeof(__bf16) + 2 * kPWaves * (size_t)kPRows * 4 +
                               4 * (size_t)kMlpOut * sizeof(float);

// ------------------------------------------------ fused training pass
// One workgroup per kTRows rows of a batch: the features, the four layers
// forward, softmax cross-entropy and the chain of input gradients back to
// the first layer, with the activations and gradients of the tile in LDS and
// written out in bf16 for the weight gradients.  The layer
// products accumulate over k as k_mlp_propose's do, so the logits equal its
// logits bit for bit.  A workgroup also writes the column sums of each
// layer's gradient over its rows (the bias gradients, added over the tiles in
// order by k_wgrad) and the sum of its rows' losses.  The backward products
// read the transposed copy of the hidden weights, so both directions load 16
// contiguous bytes per lane.
// A batch has fewer tiles than the chip has CUs, so a tile's chain of seven
// dependent products is what counts; its floor is the stream of 0.9 MB of
// weights through one CU's L2 port (64 B a clock: 6 us).  Eight waves of 32
// columns each leave two waves per SIMD to hide each other's latencies, and
// their loads run kTAhead k steps (and over the epilogues) ahead; hidden
// activations and gradients go out from the registers that hold them instead
// of being gathered from LDS; the ReLU masks stay in the lanes that need them
// again; the layers are written out one after the other, because a branch on
// the layer inside the epilogue made each wait for every load in flight (27 us).
// At 3,168 rows (99 tiles) 23.6 us; with four waves of 64 columns, LDS gathers
// and masks in LDS it took 33.9.  Of its 46,000 clocks the features take 6,000
// (two dependent gathers), the seven products 1,300 to 2,000 each, their
// epilogues about 2,000 each and the softmax 5,000 (both VALU issue).
constexpr int kTRows = 32;
constexpr int kTRowTiles = kTRows / 16;
constexpr int kTWaves = 8;
constexpr int kTThreads = 64 * kTWaves;
constexpr int kTColTiles = kMlpHidden / 16 / kTWaves;
constexpr int kTAhead = 4;  // 6 or 7: the same
static_assert(kTRows == 32 && kTThreads == 2 * kMlpOut, "two lanes per column and one wave per four rows of the softmax");
static_assert(3 * kTRowTiles * kTColTiles * 4 <= 64, "the ReLU masks of a lane fit one word");

// The arrays that the weight gradients read have one 1 KB block per 16 columns
// and tile of 32 rows, laid out as MFMA operands take it (lane l: column
// l % 16, rows 8 (l / 16) .. + 7), so a wave loads a whole block with one
// contiguous 16 bytes per lane.  (Column-major arrays, a 64-byte piece of 16
// columns per load, made the gradient kernel 18.5 us at
// 3,168 rows; these make it 9.7.)
// Offset of rows 8 g .. 8 g + 7 of column col in tile `tile` of `tiles`:
__device__ __forceinline__ int64_t tile_block(int col, int g, int tile, int tiles) {
    return (((int64_t)(col >> 4) * tiles + tile) * 64 + (col & 15) + 16 * g) * 8;
}

struct TrainArgs {
    const float *from, *to;
    const int32_t *seg;  // segment of batch row r0 + r (NULL: the segment is r0 + r)
    const int32_t *lab;  // label of batch row r0 + r
    int64_t r0;
    int rows, nb;
    const float *bounds;
    const __bf16 *Wb;    // [out][in] per layer
    const __bf16 *WbT;   // layers 2..4 transposed, [in][out]
    const float *bias;   // [4][256]
    int tiles;           // ceil(rows / kTRows)
    __bf16 *X0;          // 224 columns of features, in the blocks of tile_block
    __bf16 *H;           // 3 x 256 columns: the hidden activations
    __bf16 *dZ;          // 4 x 256 columns: gradients of the pre-activations
    float *logits;       // [rows][256], or NULL
    float *bias_part;    // [tiles][4][256]
    float *loss_part;    // [tiles]
    float inv_rows, loss_scale;
};

// LDS: the activations (the logits later take their place and more), the
// gradients and the row losses of the softmax.
constexpr size_t kTActBytes = (size_t)kTRows * kPPitch * sizeof(__bf16);
constexpr int kLPitch = kMlpOut + 16;  // logits row pitch (floats): four rows on disjoint LDS banks
constexpr size_t kTLogitBytes = (size_t)kTRows * kLPitch * sizeof(float);
static_assert(kTLogitBytes >= kTActBytes, "the logits take the activations' place");
constexpr size_t kTrainLds = kTLogitBytes + kTActBytes + (size_t)kTRows * sizeof(float);

// Max / sum over the 16 lanes of a DPP row, every lane ending with the same
// value: rotations by 8, 4, 2 and 1 within the row, each step adding two
// operands that are equal up to order (so every lane rounds the same sums).
__device__ __forceinline__ float dpp_ror(float v, int n) {
    switch (n) {
    case 8: return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, false));
    case 4: return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xf, 0xf, false));
    case 2: return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x122, 0xf, 0xf, false));
    default: return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x121, 0xf, 0xf, false));
    }
}
__device__ __forceinline__ float row16_max(float v) {
    v = fmaxf(v, dpp_ror(v, 8));
    v = fmaxf(v, dpp_ror(v, 4));
    v = fmaxf(v, dpp_ror(v, 2));
    return fmaxf(v, dpp_ror(v, 1));
}
__device__ __forceinline__ float row16_sum(float v) {
    v += dpp_ror(v, 8);
    v += dpp_ror(v, 4);
    v += dpp_ror(v, 2);
    return v + dpp_ror(v, 1);
}

__global__ __launch_bounds__(kTThreads) void k_train_tile(TrainArgs a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __bf16 *X = reinterpret_cast<__bf16 *>(lds_raw);                  // activations [kTRows][kPPitch]
    float *L = reinterpret_cast<float *>(lds_raw);                     // logits [kTRows][256], over X
    __bf16 *D = reinterpret_cast<__bf16 *>(lds_raw + kTLogitBytes);    // gradients [kTRows][kPPitch]
    float *rl = reinterpret_cast<float *>(lds_raw + kTLogitBytes + kTActBytes);  // [kTRows] row losses
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g4 = lane >> 4, l16 = lane & 15;
    const int tile = blockIdx.x, t0 = tile * kTRows;
    const int nrows = min(kTRows, a.rows - t0);
    // features: lane q of the first 384 has row q % 32, coordinate and half of
    // the bands q / 32; the others write the padding.  Rows past the batch are
    // zero.  Loads return in order: the segment's come first.
    const int fr = tid & (kTRows - 1), fpart = tid / kTRows, fc = fpart >> 1;
    float fp = 0.0f, flo = 0.0f, fhi = 0.0f;
    if (fpart < 12 && fr < nrows) {
        const int64_t br = a.r0 + t0 + fr;
        const int64_t seg = a.seg ? a.seg[br] : br;
        fp = seg_coord(a.from, a.to, seg, fc);
        flo = a.bounds[fc % 3];
        fhi = a.bounds[3 + fc % 3];
    }
    bf16x8 pf[kTAhead][kTColTiles];  // the next layer's first k steps, loaded ahead
    prefetch_layer<kMlpIn, kTColTiles, kTAhead>(a.Wb, wave, lane, pf);
    {
        __bf16 *row = X + fr * kPPitch;
        if (fpart >= 12) {
            for (int j = kMlpFeat + fpart - 12; j < kMlpIn; j += kTThreads / kTRows - 12)
                row[j] = (__bf16)0.0f;
        } else {
            const int k0 = (fpart & 1) * (kMlpBands / 2);
            const float x = fr < nrows ? norm_coord(fp, flo, fhi) : 0.0f;
            if (k0 == 0)
                row[fc] = (__bf16)x;
            for (int k = k0; k < k0 + kMlpBands / 2; ++k) {
                float sn, cs;
                sincospi_fast(band_freq(k) * x, sn, cs);
                const bf16x2 v = {(__bf16)sn, (__bf16)(fr < nrows ? cs : 0.0f)};
                *reinterpret_cast<bf16x2 *>(row + 6 + fc * 2 * kMlpBands + 2 * k) = v;
            }
        }
    }
    __syncthreads();
    // the features out, 16 bytes per lane, four lanes per column
    for (int i = tid; i < kMlpIn * (kTRows / 8); i += kTThreads) {
        const int col = (i & 15) + 16 * (i >> 6), g = (i >> 4) & 3;
        bf16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = X[(8 * g + j) * kPPitch + col];
        *reinterpret_cast<bf16x8 *>(a.X0 + tile_block(col, g, tile, a.tiles)) = v;
    }
    // forward: each layer's output over its input in X once every wave has read it
    f32x4 acc[kTRowTiles][kTColTiles];
    uint64_t relu = 0;  // where H_l > 0 in this lane's outputs, layer l in bits [16 l, 16 l + 16)
    auto wlayer = [&](int l) -> const __bf16 * {  // forward l = 0..3, then backward l = 3..1 as 4..6
        if (l == 0)
            return a.Wb;
        if (l < 4)
            return a.Wb + (int64_t)kMlpOut * kMlpIn + (int64_t)(l - 1) * kMlpHidden * kMlpHidden;
        return a.WbT + (int64_t)(6 - l) * kMlpHidden * kMlpHidden;
    };
    float bvs[4][kTColTiles];
#pragma unroll
    for (int l = 0; l < 4; ++l)
#pragma unroll
        for (int b = 0; b < kTColTiles; ++b)
            bvs[l][b] = a.bias[l * kMlpHidden + 16 * kTColTiles * wave + 16 * b + l16];
    // a hidden layer's outputs into X and out
    auto hidden = [&](int l, const float(&bv)[kTColTiles]) {
        __syncthreads();
        __bf16 *out = a.H + tile_block(l * kMlpHidden + 16 * kTColTiles * wave + l16, g4 >> 1, tile, a.tiles) + 4 * (g4 & 1);
        uint32_t on = 0;
#pragma unroll
        for (int b = 0; b < kTColTiles; ++b)
#pragma unroll
            for (int t = 0; t < kTRowTiles; ++t) {
                bf16x4 hv;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    hv[i] = (__bf16)fmaxf(acc[t][b][i] + bv[b], 0.0f);
                    X[(16 * t + 4 * g4 + i) * kPPitch + 16 * kTColTiles * wave + 16 * b + l16] = hv[i];
                    on |= (uint32_t)((float)hv[i] > 0.0f) << (4 * (t * kTColTiles + b) + i);
                }
                *reinterpret_cast<bf16x4 *>(out + (int64_t)b * a.tiles * 512 + 256 * t) = hv;
            }
        relu |= (uint64_t)on << (16 * l);
        __syncthreads();
    };
    layer_chain<kMlpIn, kMlpHidden, kTRowTiles, kTColTiles, kTAhead>(X, wlayer(0), wlayer(1), wave, lane, acc, pf);
    hidden(0, bvs[0]);
    layer_chain<kMlpHidden, kMlpHidden, kTRowTiles, kTColTiles, kTAhead>(X, wlayer(1), wlayer(2), wave, lane, acc, pf);
    hidden(1, bvs[1]);
    layer_chain<kMlpHidden, kMlpHidden, kTRowTiles, kTColTiles, kTAhead>(X, wlayer(2), wlayer(3), wave, lane, acc, pf);
    hidden(2, bvs[2]);
    layer_chain<kMlpHidden, kMlpHidden, kTRowTiles, kTColTiles, kTAhead>(X, wlayer(3), wlayer(4), wave, lane, acc, pf);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < kTColTiles; ++b)
#pragma unroll
        for (int t = 0; t < kTRowTiles; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                L[(16 * t + 4 * g4 + i) * kLPitch + 16 * kTColTiles * wave + 16 * b + l16] = acc[t][b][i] + bvs[3][b];
    __syncthreads();
    if (a.logits)
        for (int i = tid; i < nrows * kMlpOut; i += kTThreads)
            a.logits[(int64_t)t0 * kMlpOut + i] = L[(i / kMlpOut) * kLPitch + i % kMlpOut];
    // softmax cross-entropy: a wave has four rows, 16 lanes (one DPP row)
    // each, lane l16 holding columns l16 + 16 j
    {
        const int row = 4 * wave + g4;
        const float *z = L + row * kLPitch;
        float v[16];
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int c = l16 + 16 * j;
            v[j] = c < a.nb ? z[c] : -INFINITY;
            mx = fmaxf(mx, v[j]);
        }
        mx = row16_max(mx);
        float sum = 0.0f;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            v[j] = (l16 + 16 * j) < a.nb ? expf(v[j] - mx) : 0.0f;
            sum += v[j];
        }
        sum = row16_sum(sum);
        const bool valid = row < nrows;
        const int label = valid ? a.lab[a.r0 + t0 + row] : -1;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int c = l16 + 16 * j;
            const float g = valid && c < a.nb ? (v[j] / sum - (c == label ? 1.0f : 0.0f)) * a.inv_rows : 0.0f;
            D[row * kPPitch + c] = (__bf16)g;
        }
        if (l16 == 0)
            rl[row] = valid && label >= 0 && label < a.nb ? (logf(sum) + mx - z[label]) * a.loss_scale : 0.0f;
    }
    __syncthreads();
    // the logits' gradient out, and its column sums in a fixed order:
    // two lanes per column, 16 rows each; of eight rows, r and r + 4 first,
    // then neighbours, then pairs; the four eights one after the other
    {
        const int col = tid >> 1, half = tid & 1;
        bf16x8 v[2];
        float e8[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[q][j] = D[(16 * half + 8 * q + j) * kPPitch + col];
            float c4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                c4[j] = (0.0f + (float)v[q][j]) + (float)v[q][j + 4];
            e8[q] = (c4[0] + c4[1]) + (c4[2] + c4[3]);
            *reinterpret_cast<bf16x8 *>(a.dZ + tile_block(3 * kMlpOut + col, 2 * half + q, tile, a.tiles)) = v[q];
        }
        const float e2 = __shfl_xor(e8[0], 1), e3 = __shfl_xor(e8[1], 1);
        if (half == 0)
            a.bias_part[((int64_t)tile * 4 + 3) * kMlpOut + col] = ((e8[0] + e8[1]) + e2) + e3;
    }
    if (wave == 0) {
        float v = lane < kTRows ? rl[lane] : 0.0f;
        for (int off = 32; off > 0; off >>= 1)
            v += __shfl_xor(v, off);
        if (lane == 0)
            a.loss_part[tile] = v;
    }
    // backward: dZ(l - 1) = (dZ(l) W_l) where H_l > 0, in place in D; the
    // column sums (bias gradients) from the registers, over the lanes that
    // share a column
    auto back = [&](int l) {  // dZ(l) from acc
        __syncthreads();
        __bf16 *out = a.dZ + tile_block(l * kMlpOut + 16 * kTColTiles * wave + l16, g4 >> 1, tile, a.tiles) + 4 * (g4 & 1);
        const uint32_t on = (uint32_t)(relu >> (16 * l));
#pragma unroll
        for (int b = 0; b < kTColTiles; ++b) {
            const int col = 16 * kTColTiles * wave + 16 * b + l16;
            float colsum = 0.0f;
#pragma unroll
            for (int t = 0; t < kTRowTiles; ++t) {
                bf16x4 gv;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    gv[i] = (__bf16)((on >> (4 * (t * kTColTiles + b) + i)) & 1u ? acc[t][b][i] : 0.0f);
                    if (l > 0)
                        D[(16 * t + 4 * g4 + i) * kPPitch + col] = gv[i];
                    colsum += (float)gv[i];
                }
                *reinterpret_cast<bf16x4 *>(out + (int64_t)b * a.tiles * 512 + 256 * t) = gv;
            }
            colsum += __shfl_xor(colsum, 16);
            colsum += __shfl_xor(colsum, 32);
            if (lane < 16)
                a.bias_part[((int64_t)tile * 4 + l) * kMlpOut + col] = colsum;
        }
    };
    layer_chain<kMlpHidden, kMlpHidden, kTRowTiles, kTColTiles, kTAhead>(D, wlayer(4), wlayer(5), wave, lane, acc, pf);
    back(2);
    __syncthreads();
    layer_chain<kMlpHidden, kMlpHidden, kTRowTiles, kTColTiles, kTAhead>(D, wlayer(5), wlayer(6), wave, lane, acc, pf);
    back(1);
    __syncthreads();
    layer_chain<kMlpHidden, kMlpHidden, kTRowTiles, kTColTiles, kTAhead>(D, wlayer(6), nullptr, wave, lane, acc, pf);
    back(0);
}

// ------------------------------- weight gradients and the parameter step
// dW_l[n][k] = sum_r dZ_l[r][n] H_l[r][k] for the four layers, the sums of the
// bias and loss parts, and with `adam` the Adam step on the fp32 masters and
// the bf16 copies, in one launch.  Both operands come in the blocks
// of tile_block, one per MFMA operand: no staging.  A workgroup makes a 32 x 32 tile of
// one layer (248 of them: about one per CU), wave c the sum over row chunk c of
// chunk_tiles tiles (in r order, one accumulator per 16 x 16); the chunks are
// then added in chunk order from LDS and the step follows in the same lanes,
// so no partial sum leaves the CU.  XCD x (workgroups are dealt round-robin)
// gets tiles [31 x, 31 x + 31), half of one layer: 1.2 MB of operands in its
// L2 at 3,168 rows instead of all 13 MB.
// What bounds it is latency: two round trips to memory, the tile sum and the
// Adam traffic (7 MB).  At 3,168 rows 9.7 us; 128 x 128 tiles over the same
// chunks, their partial sums (13.6 MB) through memory and a second launch to
// add them took 12.1 + 10.1 us.
constexpr int kSplitMax = 16;    // row chunks at most: a wave each
constexpr int kSplitRows = 256;  // rows per chunk, up to kSplitMax of them
constexpr int kChunkUnit = 128;  // chunks are whole multiples of this many rows
constexpr int kWT = 32;          // tile edge
constexpr int kWAhead = 4;       // row tiles in flight per wave (2: the same, 6: 40.8 us a batch of 4,096 instead of 36.0)
constexpr int kWTilesFirst = (kMlpOut / kWT) * (kMlpIn / kWT), kWTilesHidden = (kMlpOut / kWT) * (kMlpHidden / kWT);
constexpr int kWTiles = kWTilesFirst + 3 * kWTilesHidden;
static_assert(kMlpOut % kWT == 0 && kMlpIn % kWT == 0 && kMlpHidden % kWT == 0 && kWTiles % 8 == 0, "whole tiles, dealt to 8 XCDs");
static_assert(kMlpOut <= 256, "the bias workgroups");
constexpr int kStepThreads = kWT * kWT / 4;  // lanes that make the Adam step, four parameters each
constexpr int kWPitch = kWT + 8;
static_assert(kStepThreads == 256 && 2 * kWT * kWPitch * sizeof(__bf16) <= 2 * kWT * kWT * sizeof(float), "the step's lanes and LDS");
constexpr size_t kWgradLds = (size_t)kSplitMax * kWT * kWT * sizeof(float);

struct GradArgs {
    const __bf16 *X0, *H, *dZ;  // as in TrainArgs; padding rows have zero gradients
    int tiles;
    int chunk_tiles, chunks;    // tiles per row chunk
    const float *bias_part;
    const float *loss_part;
    float *loss;
    float *G;                   // without the step: the gradient
    int adam;
    float *P, *m1, *m2;
    __bf16 *Wb, *WbT;
    float lr, b1, b2, eps, c1, c2;
};

// one parameter's step from its gradient; m, v and w in and out
__device__ __forceinline__ void adam_step(const GradArgs &f, float g, float &m, float &v, float &w) {
#pragma clang fp contract(off)
    m = __builtin_fmaf(1.0f - f.b1, g, f.b1 * m);
    v = __builtin_fmaf((1.0f - f.b2) * g, g, f.b2 * v);
    w = w - f.lr * (m * f.c1) / (sqrtf(v * f.c2) + f.eps);
}

__global__ __launch_bounds__(64 * kSplitMax) void k_wgrad(GradArgs f) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    float *part = reinterpret_cast<float *>(lds_raw);  // [chunks][kWT][kWT]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nthr = blockDim.x;
    if (blockIdx.x >= kWTiles) {  // the biases of a layer, or the loss: the tiles' parts in tile order
        const int l = blockIdx.x - kWTiles;
        if (l < 4) {
            if (tid < kMlpOut) {
                const int i = l * kMlpOut + tid;
                float g = 0.0f, m = 0.0f, v = 0.0f, w = 0.0f;
                if (f.adam) {
                    m = f.m1[kMlpWeights + i];
                    v = f.m2[kMlpWeights + i];
                    w = f.P[kMlpWeights + i];
                }
                for (int t0 = 0; t0 < f.tiles; t0 += 32) {  // 32 loads in flight, also in the last round
                    float x[32];
#pragma unroll
                    for (int t = 0; t < 32; ++t)
                        x[t] = f.bias_part[(int64_t)min(t0 + t, f.tiles - 1) * 4 * kMlpOut + i];
#pragma unroll
                    for (int t = 0; t < 32; ++t)
                        g += t0 + t < f.tiles ? x[t] : 0.0f;
                }
                const int64_t q = kMlpWeights + i;
                if (f.adam) {
                    adam_step(f, g, m, v, w);
                    f.m1[q] = m;
                    f.m2[q] = v;
                    f.P[q] = w;
                } else {
                    f.G[q] = g;
                }
            }
        } else if (f.loss) {
            float sum = 0.0f;
            for (int b0 = 0; b0 < f.tiles; b0 += nthr) {
                const int m = min(nthr, f.tiles - b0);
                if (tid < m)
                    part[tid] = f.loss_part[b0 + tid];
                __syncthreads();
                if (tid == 0)
                    for (int t = 0; t < m; ++t)
                        sum += part[t];
                __syncthreads();
            }
            if (tid == 0)
                *f.loss += sum;
        }
        return;
    }
    const int t = (blockIdx.x & 7) * (kWTiles / 8) + (blockIdx.x >> 3);
    const int layer = t < kWTilesFirst ? 0 : 1 + (t - kWTilesFirst) / kWTilesHidden;
    const int K = layer == 0 ? kMlpIn : kMlpHidden;
    const int tl = layer == 0 ? t : (t - kWTilesFirst) % kWTilesHidden;
    const int n0 = tl / (K / kWT) * kWT, k0 = tl % (K / kWT) * kWT;
    const int64_t woff = layer == 0 ? 0 : (int64_t)kMlpOut * kMlpIn + (int64_t)(layer - 1) * kMlpHidden * kMlpHidden;
    // the first kStepThreads lanes make the step for four parameters each:
    // their state loads while the products run
    const int n = n0 + tid / (kWT / 4), k = k0 + 4 * (tid % (kWT / 4));
    const int64_t at = woff + (int64_t)n * K + k;
    f32x4 m = {0, 0, 0, 0}, v2 = m, w = m;
    if (tid < kStepThreads && f.adam) {
        m = *reinterpret_cast<const f32x4 *>(f.m1 + at);
        v2 = *reinterpret_cast<const f32x4 *>(f.m2 + at);
        w = *reinterpret_cast<const f32x4 *>(f.P + at);
    }
    if (wave < f.chunks) {
        const int64_t col_tile = (int64_t)f.tiles * 512;  // elements of a column tile
        const __bf16 *A = f.dZ + (layer * (kMlpOut / 16) + (n0 >> 4)) * col_tile + 8 * lane;
        const __bf16 *B = (layer == 0 ? f.X0 : f.H + (layer - 1) * (kMlpHidden / 16) * col_tile) +
                          (k0 >> 4) * col_tile + 8 * lane;
        const int tb = wave * f.chunk_tiles, te = min(f.tiles, tb + f.chunk_tiles);
        f32x4 acc[2][2] = {{{0, 0, 0, 0}, {0, 0, 0, 0}}, {{0, 0, 0, 0}, {0, 0, 0, 0}}};
        bf16x8 v[kWAhead][4];  // [tile ahead][A low, A high, B low, B high]
        auto load = [&](int t, bf16x8(&d)[4]) {
            const int64_t o = (int64_t)t * 512;
            d[0] = *reinterpret_cast<const bf16x8 *>(A + o);
            d[1] = *reinterpret_cast<const bf16x8 *>(A + col_tile + o);
            d[2] = *reinterpret_cast<const bf16x8 *>(B + o);
            d[3] = *reinterpret_cast<const bf16x8 *>(B + col_tile + o);
        };
#pragma unroll
        for (int q = 0; q < kWAhead; ++q)
            if (tb + q < te)
                load(tb + q, v[q]);
        for (int t = tb; t < te; t += kWAhead) {
#pragma unroll
            for (int q = 0; q < kWAhead; ++q) {
                if (t + q >= te)
                    break;
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = mfma16(v[q][a], v[q][2 + b], acc[a][b]);
                if (t + q + kWAhead < te)
                    load(t + q + kWAhead, v[q]);
            }
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    part[(wave * kWT + 16 * a + 4 * (lane >> 4) + i) * kWT + 16 * b + (lane & 15)] = acc[a][b][i];
    }
    __syncthreads();
    f32x4 g = {0, 0, 0, 0};
    if (tid < kStepThreads) {
        for (int c = 0; c < f.chunks; ++c)
            g += *reinterpret_cast<const f32x4 *>(part + c * kWT * kWT + 4 * tid);
        if (!f.adam)
            *reinterpret_cast<f32x4 *>(f.G + at) = g;
    }
    if (!f.adam)
        return;
    __syncthreads();  // the partial sums have been read
    // the new weights, n-major and k-major in bf16, for the two fragment orders
    __bf16 *tn = reinterpret_cast<__bf16 *>(lds_raw), *tk = tn + kWT * kWPitch;
    if (tid < kStepThreads) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float mq = m[q], vq = v2[q], wq = w[q];
            adam_step(f, g[q], mq, vq, wq);
            m[q] = mq;
            v2[q] = vq;
            w[q] = wq;
            const __bf16 h = (__bf16)wq;
            tn[(n - n0) * kWPitch + k - k0 + q] = h;
            tk[(k - k0 + q) * kWPitch + n - n0] = h;
        }
        *reinterpret_cast<f32x4 *>(f.m1 + at) = m;
        *reinterpret_cast<f32x4 *>(f.m2 + at) = v2;
        *reinterpret_cast<f32x4 *>(f.P + at) = w;
    }
    __syncthreads();
    if (tid < kStepThreads) {  // 16 bytes each: 128 lanes for Wb, 128 for WbT
        const int o = (tid & 127) >> 2, c = 8 * (tid & 3);
        if (tid < 128)
            *reinterpret_cast<bf16x8 *>(f.Wb + woff + frag_index(n0 + o, k0 + c, K)) =
                *reinterpret_cast<const bf16x8 *>(tn + o * kWPitch + c);
        else if (layer > 0)
            *reinterpret_cast<bf16x8 *>(f.WbT + (int64_t)(layer - 1) * kMlpHidden * kMlpHidden +
                                        frag_index(k0 + o, n0 + c, kMlpOut)) =
                *reinterpret_cast<const bf16x8 *>(tk + o * kWPitch + c);
    }
}

// ------------------------------------------------ frontier and labels
// Exclusive prefix sum of v over a 256-lane workgroup; total = the sum.
__device__ __forceinline__ int block_excl_scan(int v, int &total) {
    __shared__ int wsum[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int u = __shfl_up(incl, d, 64);
        incl += lane >= d ? u : 0;
    }
    if (lane == 63)
        wsum[w] = incl;
    __syncthreads();
    int off = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        off += k < w ? wsum[k] : 0;
        total += wsum[k];
    }
    __syncthreads();  // wsum is reused by the next call
    return off + incl - v;
}

// Left-to-right frontier of the tree at depth 8: internal nodes at depth 8
// and leaves shallower than that, in order.  One workgroup opens it level by
// level: lane j has node j of the level, a prefix sum of the children's numbers
// gives their places.  Then each bucket's first leaf is found by descending left.
__global__ __launch_bounds__(kMlpOut) void k_frontier(const Node *__restrict__ nodes, int root, int nt,
                                                      int32_t *__restrict__ bucket_ref,
                                                      int32_t *__restrict__ bucket_first,
                                                      int32_t *__restrict__ n_buckets) {
    __shared__ int cur[kMlpOut];
    const int b = threadIdx.x;
    int count = 1;
    if (b == 0)
        cur[0] = root;
    for (int d = 0; d < kFrontierDepth; ++d) {  // at most 2^d nodes at depth d: they fit
        __syncthreads();
        const int r = b < count ? cur[b] : -1;
        int2 kids = {r, r};
        if (r >= 0) {
            kids.x = nodes[r].refs.x;
            kids.y = nodes[r].refs.y;
        }
        int total;
        const int at = block_excl_scan(b < count ? (r >= 0 ? 2 : 1) : 0, total);  // its barriers: every lane has read cur
        if (b < count) {
            cur[at] = kids.x;
            if (r >= 0)
                cur[at + 1] = kids.y;
        }
        count = total;
    }
    __syncthreads();
    if (b == 0)
        *n_buckets = count;
    if (b < count) {
        int x = cur[b];
        bucket_ref[b] = x;
        for (int guard = 0; x >= 0 && guard < nt; ++guard)  // a path has fewer than nt internal nodes
            x = nodes[x].refs.x;
        bucket_first[b] = ~x;
    }
}

// leaf_bucket[k] = the bucket whose subtree holds leaf k: each leaf climbs to
// the first ancestor (or itself) among the frontier's references, looked up in
// a hash table in LDS (512 places for at most 256 references; an empty place
// ends a search).  Bound by the latency of the climb, one parent at a time,
// with every leaf of the mesh in flight: 36 us at 522,242 triangles
// and 25 at 32,258; one lane walking each bucket's subtree took 26.8 and 1.6 ms.
constexpr int kFrontHash = 512;
__device__ __forceinline__ uint32_t front_hash(int ref) { return ((uint32_t)ref * 2654435769u) >> 23; }

__global__ __launch_bounds__(256) void k_leaf_buckets(const int32_t *__restrict__ parent, int nt,
                                                      const int32_t *__restrict__ bucket_ref,
                                                      const int32_t *__restrict__ n_buckets,
                                                      uint8_t *__restrict__ leaf_bucket) {
    static_assert(kFrontHash >= 2 * kMlpOut && kFrontHash == 1 << 9, "at most half full; front_hash has 9 bits");
    constexpr int kEmpty = 0x7fffffff;  // no reference: nodes and leaves are below 2^30
    __shared__ int key[kFrontHash], val[kFrontHash];
    for (int i = threadIdx.x; i < kFrontHash; i += blockDim.x)
        key[i] = kEmpty;
    __syncthreads();
    if (threadIdx.x < (unsigned)*n_buckets) {
        const int ref = bucket_ref[threadIdx.x];
        for (uint32_t h = front_hash(ref);; h = (h + 1) & (kFrontHash - 1))  // ends: half of the places stay empty
            if (atomicCAS(&key[h], kEmpty, ref) == kEmpty) {
                val[h] = threadIdx.x;
                break;
            }
    }
    __syncthreads();
    const int leaf = blockIdx.x * blockDim.x + threadIdx.x;
    if (leaf >= nt)
        return;
    int x = ~leaf;
    for (int guard = 0; guard <= nt; ++guard) {  // a path has at most nt nodes
        for (uint32_t h = front_hash(x); key[h] != kEmpty; h = (h + 1) & (kFrontHash - 1))
            if (key[h] == x) {
                leaf_bucket[leaf] = (uint8_t)val[h];
                return;
            }
        x = x >= 0 ? parent[x] : parent[(nt - 1) + ~x];
        if (x < 0 || x >= nt - 1)
            return;  // above the root: not reached, every path meets the frontier
    }
}

// rank[ids[k]] = k: sorted position of each input triangle.
__global__ void k_rank(const int32_t *__restrict__ ids, int nt, int32_t *__restrict__ rank) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nt)
        rank[ids[k]] = k;
}

// The training list: for every segment with a first hit, in segment order,
// the segment and its bucket (the frontier subtree that holds the hit leaf).
// A stable compaction -- per-workgroup counts, one scan of them, then each
// workgroup writes at its offset in order -- so the list, and the training
// that walks it batch by batch, do not depend on scheduling.
constexpr int kLabSeg = 16;                   // segments per lane
constexpr int kLabPerBlock = 256 * kLabSeg;   // per workgroup of 256

__device__ __forceinline__ int lane_hits(const int32_t *__restrict__ tri_id, int64_t n, int64_t base) {
    int c = 0;
    for (int j = 0; j < kLabSeg; ++j)
        c += base + j < n && tri_id[base + j] >= 0;
    return c;
}

__global__ __launch_bounds__(256) void k_label_count(const int32_t *__restrict__ tri_id, int64_t n,
                                                     int32_t *__restrict__ blk) {
    const int64_t base = (int64_t)blockIdx.x * kLabPerBlock + (int64_t)threadIdx.x * kLabSeg;
    int total;
    block_excl_scan(lane_hits(tri_id, n, base), total);
    if (threadIdx.x == 0)
        blk[blockIdx.x] = total;
}

// blk[b] = the list position of workgroup b's first entry; *count = the total.
__global__ __launch_bounds__(256) void k_label_scan(int32_t *__restrict__ blk, int nblk, uint32_t *__restrict__ count) {
    uint32_t carry = 0;
    for (int b0 = 0; b0 < nblk; b0 += 256) {
        const int b = b0 + threadIdx.x;
        const int v = b < nblk ? blk[b] : 0;
        int total;
        const int ex = block_excl_scan(v, total);
        if (b < nblk)
            blk[b] = (int32_t)(carry + ex);
        carry += (uint32_t)total;
    }
    if (threadIdx.x == 0)
        *count = carry;
}

__global__ __launch_bounds__(256) void k_labels(const int32_t *__restrict__ tri_id, int64_t n,
                                                const int32_t *__restrict__ rank,
                                                const uint8_t *__restrict__ leaf_bucket,
                                                const int32_t *__restrict__ blk, int32_t *__restrict__ seg_out,
                                                int32_t *__restrict__ label_out) {
    const int64_t base = (int64_t)blockIdx.x * kLabPerBlock + (int64_t)threadIdx.x * kLabSeg;
    int total;
    int pos = blk[blockIdx.x] + block_excl_scan(lane_hits(tri_id, n, base), total);
    for (int j = 0; j < kLabSeg; ++j) {
        const int64_t i = base + j;
        const int t = i < n ? tri_id[i] : -1;
        if (t >= 0) {
            seg_out[pos] = (int32_t)i;
            label_out[pos] = leaf_bucket[rank[t]];
            ++pos;
        }
    }
}

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

}  // namespace

// ===================================================================== host
hipError_t proposal_frontier(const MeshDev &m, Proposal &pr, hipStream_t s) {
    if (m.nt < 1)
        return hipErrorInvalidValue;
    k_rank<<<cdiv(m.nt, 256), 256, 0, s>>>(m.ids, (int)m.nt, pr.rank);
    k_frontier<<<1, kMlpOut, 0, s>>>(m.nodes, m.root, (int)m.nt, pr.bucket_ref, pr.bucket_first, pr.dev_n_buckets);
    k_leaf_buckets<<<cdiv(m.nt, 256), 256, 0, s>>>(m.parent, (int)m.nt, pr.bucket_ref, pr.dev_n_buckets,
                                                   pr.leaf_bucket);
    return hipGetLastError();
}

hipError_t proposal_init(Proposal &pr, uint64_t seed, hipStream_t s) {
    k_init_params<<<cdiv(kMlpParams, 256), 256, 0, s>>>(pr.P, pr.Wb, pr.WbT, pr.m1, pr.m2, seed);
    return hipGetLastError();
}

size_t proposal_label_scratch(int64_t n) { return 4 * (size_t)(n / kLabPerBlock + 1); }

hipError_t proposal_labels(const MeshDev &m, Proposal &pr, const int32_t *tri_id, int64_t n, int32_t *seg,
                           int32_t *label, uint32_t *count, int32_t *blk, hipStream_t s) {
    const int nblk = (int)((n + kLabPerBlock - 1) / kLabPerBlock);
    if (nblk == 0)
        return hipSuccess;
    k_label_count<<<nblk, 256, 0, s>>>(tri_id, n, blk);
    k_label_scan<<<1, 256, 0, s>>>(blk, nblk, count);
    k_labels<<<nblk, 256, 0, s>>>(tri_id, n, pr.rank, pr.leaf_bucket, blk, seg, label);
    return hipGetLastError();
}

hipError_t proposal_predict(const MeshDev &m, const Proposal &pr, const float *from, const float *to, int64_t n,
                            int nb, uint8_t *bucket, hipStream_t s) {
    if (n == 0)
        return hipSuccess;
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int64_t tiles = (n + kPRows - 1) / kPRows;
    const int grid = (int)(tiles < 2 * cus ? tiles : 2 * cus);
    static_assert(kProposeLds <= 64 * 1024, "the fused inference kernel fits the default dynamic LDS");
    k_mlp_propose<<<grid, kPThreads, kProposeLds, s>>>(from, to, n, m.bounds, pr.Wb, pr.P, nb, bucket);
    return hipGetLastError();
}

// Forward + backward of one batch (rows segments listed in seg[r0..r0+rows),
// labels lab[r0..]) in two launches: k_train_tile (features, forward, softmax
// cross-entropy, input gradients and bias / loss parts per tile of kTRows
// rows) and k_wgrad (every layer's weight gradient and the sums in fixed
// order; into pr.G without `adam`, else the Adam step).  ws must hold
// proposal_batch_scratch(rows) bytes.
hipError_t proposal_batch_grad(const MeshDev &m, Proposal &pr, const float *from, const float *to,
                               const int32_t *seg, const int32_t *lab, int64_t r0, int rows, int nb, float *loss,
                               float loss_scale, char *ws, hipStream_t s, float *logits_out, const AdamStep *adam) {
    const int tiles = cdiv(rows, kTRows);
    const int64_t ld = (int64_t)tiles * kTRows;
    __bf16 *X0 = reinterpret_cast<__bf16 *>(ws);  // 224 columns of ld rows
    __bf16 *H = X0 + ld * kMlpIn;                 // 3 x 256 columns
    __bf16 *dZ0 = H + 3 * ld * kMlpHidden;        // 4 x 256 columns
    float *bias_part = reinterpret_cast<float *>(dZ0 + 4 * ld * kMlpOut);  // [tiles][4][256]
    float *loss_part = bias_part + (int64_t)tiles * 4 * kMlpOut;           // [tiles]
    TrainArgs a{};
    a.from = from;
    a.to = to;
    a.seg = seg;
    a.lab = lab;
    a.r0 = r0;
    a.rows = rows;
    a.nb = nb;
    a.bounds = m.bounds;
    a.Wb = pr.Wb;
    a.WbT = pr.WbT;
    a.bias = pr.P + kMlpWeights;
    a.tiles = tiles;
    a.X0 = X0;
    a.H = H;
    a.dZ = dZ0;
    a.logits = logits_out;
    a.bias_part = bias_part;
    a.loss_part = loss_part;
    a.inv_rows = 1.0f / rows;
    a.loss_scale = loss_scale > 0.0f ? loss_scale : 1.0f / rows;
    static_assert(kTrainLds <= 64 * 1024 && kWgradLds <= 64 * 1024, "both fit the default dynamic LDS");
    k_train_tile<<<tiles, kTThreads, kTrainLds, s>>>(a);
    GradArgs f{};
    f.X0 = X0;
    f.H = H;
    f.dZ = dZ0;
    const int chunks = ld > kSplitRows ? (cdiv(ld, kSplitRows) < kSplitMax ? cdiv(ld, kSplitRows) : kSplitMax) : 1;
    f.chunk_tiles = cdiv(cdiv(ld, chunks), kChunkUnit) * (kChunkUnit / kTRows);
    f.chunks = cdiv(tiles, f.chunk_tiles);
    f.bias_part = bias_part;
    f.tiles = tiles;
    f.loss_part = loss_part;
    f.loss = loss;
    if (adam) {
        f.adam = 1;
        f.P = pr.P;
        f.m1 = pr.m1;
        f.m2 = pr.m2;
        f.Wb = pr.Wb;
        f.WbT = pr.WbT;
        f.lr = adam->lr;
        f.b1 = 0.9f;
        f.b2 = 0.999f;
        f.eps = 1e-8f;
        f.c1 = 1.0f / (1.0f - powf(f.b1, (float)adam->step));
        f.c2 = 1.0f / (1.0f - powf(f.b2, (float)adam->step));
    } else {
        f.G = pr.G;
    }
    // at least four waves, to share the tile's sums and steps
    const int parts = f.chunks > 4 ? f.chunks : 4;
    k_wgrad<<<kWTiles + 5, 64 * parts, (size_t)parts * kWT * kWT * sizeof(float), s>>>(f);
    return hipGetLastError();
}

namespace {
__global__ void k_params_to_bf16(const float *__restrict__ P, __bf16 *__restrict__ Wb, __bf16 *__restrict__ WbT) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMlpWeights)
        store_weight(Wb, WbT, i, P[i]);
}
}  // namespace

hipError_t proposal_set_params(Proposal &pr, hipStream_t s) {
    k_params_to_bf16<<<cdiv(kMlpWeights, 256), 256, 0, s>>>(pr.P, pr.Wb, pr.WbT);
    return hipGetLastError();
}

size_t proposal_batch_scratch(int rows) {
    const size_t tiles = (size_t)cdiv(rows, kTRows);
    return tiles * kTRows * (kMlpIn + 3 * kMlpHidden + 4 * kMlpOut) * 2 + tiles * 4 * kMlpOut * 4 + tiles * 4 + 256;
}

hipError_t proposal_features(const MeshDev &m, const float *from, const float *to, int64_t n, __bf16 *X,
                             hipStream_t s) {
    if (n == 0)
        return hipSuccess;
    k_features<<<cdiv(n * 7, 256), 256, 0, s>>>(from, to, nullptr, 0, n, m.bounds, X);
    return hipGetLastError();
}

}  // namespace rsi
