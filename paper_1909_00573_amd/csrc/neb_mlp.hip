// Learned density: a small MLP that maps a surface point and its normal to
// log(density of NEE vertices), trained on the octree's robust densities
// (Sec. 5 provides the targets; the model itself is not in the paper).
//
// Model: 80 encoded inputs (normalised point q, normal n, and sin/cos of
// 2^f pi c for the six coordinates c and octaves f = 0..5, two zero pads)
// -> 64 -> 64 -> 64 (ReLU) -> 1, output log rho = mu + sigma * y.
//
// gfx950 mapping.  The three 64-wide layers run on the matrix cores, bf16
// operands and FP32 accumulation: inference on v_mfma_f32_16x16x32_bf16,
// training on v_mfma_f32_16x16x16_bf16.
// A wave evaluates 16 samples at a time with the transposed product
//     Z^T (64 x 16) = W^T (64 x K) . X^T (K x 16),
// so the weights are the A operand and the samples the B operand.  The
// accumulator of output block ob holds, in lane l, features 16 ob +
// 4 (l / 16) + i (i = 0..3) of sample l % 16 -- exactly the B-operand
// layout of the next layer's k-block ob, so layers chain in registers
// without any transpose.  The backward data pass uses A = W the same way.
// Weight gradients are K = batch GEMMs over tile-major bf16 stores of
// the activations and deltas.  Weights are kept as
// FP32 master copies (Adam) and re-packed after every step into bf16 operand
// fragments, which the kernels stage in LDS.
#include <algorithm>

#include "neb_device.h"
#include "neb_mlp.h"

namespace neb {

typedef short bf16x4 __attribute__((ext_vector_type(4)));  // bf16 bit patterns
typedef short bf16x8b __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// bfloat16 of four floats, rounded to nearest, ties to even (the conversion
// instruction rounds two at a time)
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
struct Bf16Pairs {
    bf16x2 lo, hi;
};
__device__ __forceinline__ bf16x4 pack4(float a, float b, float c, float d) {
    Bf16Pairs r;
    r.lo = __builtin_convertvector((f32x2){a, b}, bf16x2);
    r.hi = __builtin_convertvector((f32x2){c, d}, bf16x2);
    return __builtin_bit_cast(bf16x4, r);
}
__device__ __forceinline__ uint16_t to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

// 16 x 16 x 16 product (four k per lane)
__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// a product over two 16-wide k blocks whose A fragments lie side by side:
// one 16 x 16 x 32 product of gfx950 (kK32; eight k per lane, twice the k in
// the same issue time; it sums the same terms over a permuted k), or two
// 16 x 16 x 16 ones.  (The waits between dependent matrix products of different
// length are left to software; a 16 x 16 x 16 product that took the accumulator
// of a 16 x 16 x 32 one right behind it, which is how the compiler schedules
// such a pair, gave wrong sums.  Where the two meet, wait_products stands
// between them.)
template <bool kK32>
__device__ __forceinline__ f32x4 mfma_pair(bf16x8b a, bf16x4 b0, bf16x4 b1, f32x4 c) {
    if (kK32) {
        const bf16x8b b = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    }
    c = mfma(bf16x4{a[0], a[1], a[2], a[3]}, b0, c);
    return mfma(bf16x4{a[4], a[5], a[6], a[7]}, b1, c);
}

// The products that made these accumulators are over once this is: 32 wait
// states, more than the 19 that the longest product asks for.  The accumulators
// pass through it, so neither what made them nor what takes them can move
// across (tests/test_mlp_products_host.py reads the distance off the assembly).
__device__ __forceinline__ void wait_products(f32x4 (&acc)[4]) {
    asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]));
}

// The encoded input of one sample as the B operand of layer 1: lane group g
// holds features 16 ks + 4 g .. + 3 of k-block ks, two pairs of features.
// Pair p is a raw pair (p < 3), the sine and cosine of 2^octave pi c for
// coordinate c = (p - 3) / 6 and octave (p - 3) % 6, or the two zero pads.
// Within a k-block a lane's pair is one of two coordinates, by its group.
__device__ __forceinline__ void mlp_encode(const float q[3], const float n[3], const float scale[10],
                                           bf16x4 x[5]) {
    const float c[6] = {q[0], q[1], q[2], n[0], n[1], n[2]};
    // (k-block, pair): the coordinates of the groups below and from `from` on
    // (lane masks held in scalar registers: one select each)
    constexpr int lo[5][2] = {{0, 0}, {0, 1}, {2, 2}, {3, 3}, {4, 5}};
    constexpr int hi[5][2] = {{0, 0}, {1, 2}, {3, 3}, {4, 4}, {5, 5}};
    constexpr int from[5][2] = {{0, 0}, {1, 3}, {3, 2}, {2, 1}, {1, 0}};
    auto upper = [](int k) {  // groups k and above, k = 1..3
        return __builtin_amdgcn_inverse_ballot_w64(~0ull << (16 * k));
    };
#pragma unroll
    for (int ks = 0; ks < 5; ++ks) {
        float v[4];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const float y = from[ks][p] == 0 ? c[hi[ks][p]] : (upper(from[ks][p]) ? c[hi[ks][p]] : c[lo[ks][p]]);
            sincospif(scale[2 * ks + p] * y, &v[2 * p], &v[2 * p + 1]);  // exact power-of-two scale
        }
        if (ks == 0) {
            v[0] = upper(2) ? v[0] : (upper(1) ? n[1] : q[0]);
            v[1] = upper(2) ? v[1] : (upper(1) ? n[2] : q[1]);
            v[2] = upper(1) ? v[2] : q[2];
            v[3] = upper(1) ? v[3] : n[0];
        }
        if (ks == 4) {
            v[2] = upper(3) ? 0.f : v[2];
            v[3] = upper(3) ? 0.f : v[3];
        }
        x[ks] = pack4(v[0], v[1], v[2], v[3]);
    }
}

// 2^octave of the lane group's ten pairs (0 where there is none)
__device__ __forceinline__ void mlp_scales(int g, float scale[10]) {
#pragma unroll
    for (int k = 0; k < 10; ++k) {
        const int j = 8 * (k >> 1) + 2 * g + (k & 1) - 3;
        scale[k] = j >= 0 && j < 36 ? (float)(1 << (j % 6)) : 0.f;
    }
}

// Fragment blob (offsets in bf16 elements).  The fragments of two 16-wide k
// blocks lie side by side, eight values (16 bytes) per lane: the A operand of
// one 16 x 16 x 32 product, or of two 16 x 16 x 16 ones.  Layer 1's fifth k
// block is paired with zeros.
constexpr int kPair = 64 * 8;
constexpr int kFragF1 = 0;                              // W1^T: 4 ob x 3 pairs
constexpr int kFragF2 = kFragF1 + 4 * 3 * kPair;        // W2^T: 4 ob x 2 pairs
constexpr int kFragF3 = kFragF2 + 4 * 2 * kPair;        // W3^T
constexpr int kFragB2 = kFragF3 + 4 * 2 * kPair;        // W2 (backward): 4 kb x 2 pairs of nb
constexpr int kFragB3 = kFragB2 + 4 * 2 * kPair;        // W3 (backward)
constexpr int kFragFwd = kFragB2;                       // forward part
constexpr int kFragAll = kFragB3 + 4 * 2 * kPair;       // 22528

// fragment index of W_l[k][n] in the forward (W^T as A) and backward (W as A) blobs
__device__ __forceinline__ int frag_fwd(int k, int n, int pairs) {
    int ob = n >> 4, ks = k >> 4, lane = (n & 15) + 16 * ((k & 15) >> 2);
    return ((ob * pairs + (ks >> 1)) * 64 + lane) * 8 + 4 * (ks & 1) + (k & 3);
}
__device__ __forceinline__ int frag_bwd(int k, int n) {
    int kb = k >> 4, nb = n >> 4, lane = (k & 15) + 16 * ((n & 15) >> 2);
    return ((kb * 2 + (nb >> 1)) * 64 + lane) * 8 + 4 * (nb & 1) + (n & 3);
}

// one parameter's bf16 copies into the blob (weights of layers 1..3 only)
__device__ __forceinline__ void pack_param(uint16_t* blob, int p, float w) {
    if (p < kMlpB1) {
        int k = p / kMlpWidth, n = p % kMlpWidth;
        blob[kFragF1 + frag_fwd(k, n, 3)] = to_bf16(w);
    } else if (p >= kMlpW2 && p < kMlpB2) {
        int e = p - kMlpW2, k = e / kMlpWidth, n = e % kMlpWidth;
        blob[kFragF2 + frag_fwd(k, n, 2)] = to_bf16(w);
        blob[kFragB2 + frag_bwd(k, n)] = to_bf16(w);
    } else if (p >= kMlpW3 && p < kMlpB3) {
        int e = p - kMlpW3, k = e / kMlpWidth, n = e % kMlpWidth;
        blob[kFragF3 + frag_fwd(k, n, 2)] = to_bf16(w);
        blob[kFragB3 + frag_bwd(k, n)] = to_bf16(w);
    }
}

__global__ void k_mlp_pack(const float* __restrict__ theta, uint16_t* __restrict__ blob) {
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < kMlpParams; p += gridDim.x * blockDim.x)
        pack_param(blob, p, theta[p]);
}

__device__ __forceinline__ void stage_blob(const uint16_t* __restrict__ blob, uint16_t* lds, int n) {
    const uint4* src = reinterpret_cast<const uint4*>(blob);
    uint4* dst = reinterpret_cast<uint4*>(lds);
    for (int i = threadIdx.x; i < n / 8; i += blockDim.x) dst[i] = src[i];
    __syncthreads();
}

__device__ __forceinline__ bf16x8b frag(const uint16_t* lds, int base, int pair, int lane) {
    return *reinterpret_cast<const bf16x8b*>(lds + base + (pair * 64 + lane) * 8);
}

// Inputs of one sample.  Sources: float3 arrays of normalised points (or
// positions to normalise with an octree's box) and normals, with strides.
struct MlpInput {
    const float* pos;
    int pos_stride;
    const float* nrm;
    int nrm_stride;
    const int32_t* n_dev;  // item count in device memory (or null)
    int32_t n_host;        // capacity / count
    int normalize;         // 1: q = (pos - min_bound) * size_inv, clamped to [0, 1)
    float min_bound[3], size_inv[3];
};

__device__ __forceinline__ void load_input(const MlpInput& in, int i, float q[3], float n[3]) {
    const float* p = in.pos + (size_t)in.pos_stride * i;
    const float* m = in.nrm + (size_t)in.nrm_stride * i;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float v = p[c];
        if (in.normalize) {
            v = __fmul_rn(__fsub_rn(v, in.min_bound[c]), in.size_inv[c]);
            v = fminf(fmaxf(v, 0.f), 0.99999994f);
        }
        q[c] = v;
        n[c] = m[c];
    }
}

// Forward pass of one 16-sample tile.  Lane l works on sample l % 16 and
// holds features 16 ob + 4 g + i (g = l / 16) of every layer.  Outputs:
// z (pre-activations, FP32) of the three hidden layers and y.
struct TileFwd {
    f32x4 z1[4], z2[4], z3[4];
    bf16x4 x[5];  // encoded input, bf16
    bf16x4 h1[4], h2[4];
    float y;
};

// max(x, 0) in one instruction (fmaxf of a matrix result takes a second one to quiet NaNs); 0 for a NaN, as fmaxf gives
__device__ __forceinline__ float relu(float x) { return __builtin_amdgcn_fmed3f(x, 0.f, INFINITY); }
__device__ __forceinline__ bf16x4 relu_pack(f32x4 z) { return pack4(relu(z[0]), relu(z[1]), relu(z[2]), relu(z[3])); }

// a product over 64 inputs
template <bool kK32>
__device__ __forceinline__ f32x4 product64(const uint16_t* lds, int base, int pair, int lane, const bf16x4 in[4]) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = mfma_pair<kK32>(frag(lds, base, pair, lane), in[0], in[1], acc);
    return mfma_pair<kK32>(frag(lds, base, pair + 1, lane), in[2], in[3], acc);
}

// sb: b1, b2, b3 and w4, 64 floats each (16-byte aligned).  kK32: inference;
// training keeps the 16 x 16 x 16 products (its time is not theirs, and
// its activations keep their bits)
template <bool kK32>
__device__ __forceinline__ void tile_forward(const uint16_t* lds, const float* __restrict__ sb, float b4,
                                             const float q[3], const float n[3], const float scale[10], TileFwd& T) {
    const int lane = threadIdx.x & 63, g = lane >> 4;
    auto biased = [&](f32x4 acc, int l, int ob) { return acc + *reinterpret_cast<const f32x4*>(sb + l * kMlpWidth + 16 * ob + 4 * g); };
    mlp_encode(q, n, scale, T.x);
    f32x4 acc[4];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) acc[ob] = product64<kK32>(lds, kFragF1, ob * 3, lane, T.x);
    // the last 16 inputs: a 16 x 16 x 16 product (a 16 x 16 x 32 one with zeros
    // takes as long and rounds differently)
    if (kK32) wait_products(acc);
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        const bf16x8b w = frag(lds, kFragF1, ob * 3 + 2, lane);
        T.z1[ob] = biased(mfma(bf16x4{w[0], w[1], w[2], w[3]}, T.x[4], acc[ob]), 0, ob);
    }
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) T.h1[ob] = relu_pack(T.z1[ob]);
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) T.z2[ob] = biased(product64<kK32>(lds, kFragF2, ob * 2, lane, T.h1), 1, ob);
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) T.h2[ob] = relu_pack(T.z2[ob]);
    // layer 3 and the linear output (FP32 dot product over the lane's 16 features)
    float part = 0.f;
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        T.z3[ob] = biased(product64<kK32>(lds, kFragF3, ob * 2, lane, T.h2), 2, ob);
        const f32x4 w = *reinterpret_cast<const f32x4*>(sb + 3 * kMlpWidth + 16 * ob + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) part += w[i] * relu(T.z3[ob][i]);
    }
    part += __shfl_xor(part, 16, 64);
    part += __shfl_xor(part, 32, 64);
    T.y = part + b4;
}

// b1, b2, b3 and w4 into LDS (theta's offsets are not 16-byte aligned);
// the caller's barrier follows
__device__ __forceinline__ void stage_small(const float* __restrict__ theta, float* sb) {
    for (int i = threadIdx.x; i < 4 * kMlpWidth; i += blockDim.x) {
        const int l = i / kMlpWidth, f = i % kMlpWidth;
        sb[i] = theta[(l == 0 ? kMlpB1 : (l == 1 ? kMlpB2 : (l == 2 ? kMlpB3 : kMlpW4))) + f];
    }
}

// Inference: out[i] = log rho (mode 0) or rho = exp(log rho) (mode 1).
// Bound by instruction issue: 620 vector instructions per 16-sample tile (half
// of them the ten sincospif of a lane) and 28 matrix products, 2 870 cycles per
// tile and SIMD at 1.835 M samples, 163 -> 134 us (uniform random points and
// normals; points on a few planes and a ball, whose operands change less from
// sample to sample, 148 -> 110).  Before: 906 instructions
// (rounding to bf16 in integers, selecting a pair's coordinate through five
// compares, quieting NaNs before each ReLU).  Four waves per SIMD or two
// measure the same; 2 048 blocks beat the 1 280 that are resident at once (141
// us), 1 024 and 2 560 (146, 135).
__global__ void __launch_bounds__(256, 4) k_mlp_infer(const uint16_t* __restrict__ blob, const float* __restrict__ theta,
                                                   const MlpNorm* norm, MlpInput in, float* __restrict__ out,
                                                   int mode) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[kFragFwd];
    __shared__ __attribute__((aligned(16))) float sb[4 * kMlpWidth];
    stage_small(theta, sb);
    stage_blob(blob, lds, kFragFwd);
    const int lane = threadIdx.x & 63, s = lane & 15;
    float scale[10];
    mlp_scales(lane >> 4, scale);
    const float b4 = theta[kMlpB4];
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, n_waves = (gridDim.x * blockDim.x) >> 6;
    const int n = in.n_dev ? min(*in.n_dev, in.n_host) : in.n_host;
    const float mu = norm->mu, sigma = norm->sigma;
    for (int base = wave * 16; base < n; base += n_waves * 16) {
        int i = base + s;
        float q[3] = {0.f, 0.f, 0.f}, nn[3] = {0.f, 0.f, 1.f};
        if (i < n) load_input(in, i, q, nn);
        TileFwd T;
        // an offset the compiler cannot see through: the weights' fragments
        // are the same for every tile, and kept in registers over the loop they
        // would leave room for two waves per SIMD instead of four
        int at = 0;
        asm volatile("" : "+s"(at));
        tile_forward<true>(lds + at, sb + at, b4, q, nn, scale, T);
        if (lane < 16 && i < n) {
            float lr = mu + sigma * T.y;
            out[i] = mode ? __expf(lr) : lr;
        }
    }
}

// Training batch: items [0, n) of the given arrays, or n draws (with
// replacement, Philox) from a pool whose size is in device memory.
struct MlpBatch {
    MlpInput in;
    const float* target;       // log rho per item of in
    int32_t n;                 // batch size
    int32_t sample;            // 1: draw from the pool
    uint32_t k0, k1, step;     // Philox key and counter word for the draws
};

// per-wave partial sums of the small gradients: b1, b2, b3, w4 (64 each),
// b4, loss
constexpr int kPartStride = 4 * kMlpWidth + 2;
// Activations and deltas of a batch, tile-major: per 16-sample tile 400 rows
// of 16 bf16 (X rows 0..79, H1, H2, D1, D2, D3 64 rows each), so a wave
// writes whole cache lines and a 16 x 16 operand fragment is 8 contiguous
// bytes per lane.
constexpr int kRowsX = 0, kRowsH1 = kMlpIn, kRowsH2 = kRowsH1 + kMlpWidth, kRowsD1 = kRowsH2 + kMlpWidth,
              kRowsD2 = kRowsD1 + kMlpWidth, kRowsD3 = kRowsD2 + kMlpWidth, kRowsTile = kRowsD3 + kMlpWidth;
constexpr int kTrainWaves = 8;  // waves per block; the block's LDS fills a CU

// Forward, output gradient, backward data pass, the wave's partial sums of
// the bias and output-layer gradients and of the loss (plain stores, summed
// by k_mlp_wgrad), and the tile-major bf16 stores the weight-gradient GEMMs
// read.  A lane holds four rows of its sample, a fragment four samples of a row:
// the tile is turned in LDS, so that it leaves in 25 stores of 8 bytes per
// lane instead of 100 of 2.
// Bound by instruction issue (two waves per SIMD): the encoding, the roundings,
// the 2-byte stores into LDS.  65 536 samples: 40 -> 25 us.
__global__ void __launch_bounds__(64 * kTrainWaves) k_mlp_train_fb(const uint16_t* __restrict__ blob,
                                                                   const float* __restrict__ theta, const MlpNorm* norm,
                                                                   MlpBatch B, uint16_t* __restrict__ acts,
                                                                   int n_tiles, float* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[kFragAll];
    __shared__ __attribute__((aligned(16))) uint16_t turn[kTrainWaves][kRowsTile * 16];
    __shared__ __attribute__((aligned(16))) float sb[4 * kMlpWidth];
    stage_small(theta, sb);
    stage_blob(blob, lds, kFragAll);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, s = lane & 15, g = lane >> 4;
    const float mu = norm->mu, inv_sigma = 1.0f / norm->sigma, b4 = theta[kMlpB4];
    const float inv_n = 2.0f / (float)B.n;
    float scale[10];
    mlp_scales(g, scale);
    f32x4 gb1[4], gb2[4], gb3[4], gw4[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) gb1[k] = gb2[k] = gb3[k] = gw4[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    float gb4 = 0.f, lsum = 0.f;
    const int pool = B.sample ? (B.in.n_dev ? min(*B.in.n_dev, B.in.n_host) : B.in.n_host) : B.n;
    uint16_t* const mine = turn[wave];
    for (int tile = blockIdx.x * kTrainWaves + wave; tile < n_tiles; tile += gridDim.x * kTrainWaves) {
        const int j = 16 * tile + s;
        const bool live = j < B.n && pool > 0;
        float q[3] = {0.f, 0.f, 0.f}, nn[3] = {0.f, 0.f, 1.f}, t = 0.f;
        if (live) {
            int item = j;
            if (B.sample) {
                uint4 r = philox10(make_uint4((uint32_t)j, B.step, 0u, kTagMlp), B.k0, B.k1);
                item = (int)(((uint64_t)r.x * (uint64_t)pool) >> 32);
            }
            load_input(B.in, item, q, nn);
            t = (B.target[item] - mu) * inv_sigma;
        }
        TileFwd T;
        tile_forward<false>(lds, sb, b4, q, nn, scale, T);
        uint16_t* col = mine + s;
#pragma unroll
        for (int ks = 0; ks < 5; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i) col[(kRowsX + 16 * ks + 4 * g + i) * 16] = (uint16_t)T.x[ks][i];
        const float e = live ? T.y - t : 0.f;
        const float dy = e * inv_n;
        if (g == 0) {
            lsum += e * e;
            gb4 += dy;
        }
        // output layer and delta 3
        bf16x4 d3[4];
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            const f32x4 w = *reinterpret_cast<const f32x4*>(sb + 3 * kMlpWidth + 16 * ob + 4 * g);
            f32x4 d;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                gw4[ob][i] += dy * relu(T.z3[ob][i]);
                d[i] = T.z3[ob][i] > 0.f ? dy * w[i] : 0.f;
                gb3[ob][i] += d[i];
            }
            d3[ob] = pack4(d[0], d[1], d[2], d[3]);
        }
        // delta of the layer below: (W delta) . [z > 0]
        auto back = [&](int frags, const bf16x4 din[4], const f32x4 z[4], f32x4 gb[4], bf16x4 dout[4]) {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                f32x4 acc = product64<false>(lds, frags, kb * 2, lane, din);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[i] = z[kb][i] > 0.f ? acc[i] : 0.f;
                    gb[kb][i] += acc[i];
                }
                dout[kb] = pack4(acc[0], acc[1], acc[2], acc[3]);
            }
        };
        bf16x4 d2[4], d1[4];
        back(kFragB3, d3, T.z2, gb2, d2);
        back(kFragB2, d2, T.z1, gb1, d1);
#pragma unroll
        for (int ob = 0; ob < 4; ++ob)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int f = (16 * ob + 4 * g + i) * 16;
                col[kRowsH1 * 16 + f] = (uint16_t)T.h1[ob][i];
                col[kRowsH2 * 16 + f] = (uint16_t)T.h2[ob][i];
                col[kRowsD1 * 16 + f] = (uint16_t)d1[ob][i];
                col[kRowsD2 * 16 + f] = (uint16_t)d2[ob][i];
                col[kRowsD3 * 16 + f] = (uint16_t)d3[ob][i];
            }
        // the wave's own LDS, in order: no barrier needed
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint16_t* out = acts + (size_t)tile * (kRowsTile * 16) + 4 * lane;
#pragma unroll
        for (int rb = 0; rb < kRowsTile / 16; ++rb)
            *reinterpret_cast<bf16x4*>(out + 256 * rb) = *reinterpret_cast<const bf16x4*>(mine + 256 * rb + 4 * lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    // the wave's small gradients: over the 16 sample lanes of each group
    auto over_samples = [&](float v) {
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) v += __shfl_xor(v, off, 64);
        return v;
    };
    float* P = part + (size_t)(blockIdx.x * kTrainWaves + wave) * kPartStride;
#pragma unroll
    for (int ob = 0; ob < 4; ++ob)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int f = 16 * ob + 4 * g + i;
            const float v1 = over_samples(gb1[ob][i]), v2 = over_samples(gb2[ob][i]), v3 = over_samples(gb3[ob][i]),
                        v4 = over_samples(gw4[ob][i]);
            if (s == 0) {
                P[f] = v1;
                P[kMlpWidth + f] = v2;
                P[2 * kMlpWidth + f] = v3;
                P[3 * kMlpWidth + f] = v4;
            }
        }
    gb4 = over_samples(gb4);
    lsum = over_samples(lsum);
    if (lane == 0) {
        P[4 * kMlpWidth] = gb4;
        P[4 * kMlpWidth + 1] = lsum;
    }
}

// Weight gradients dW_l[k][n] = sum_s Hin[k][s] D[n][s] as K = batch GEMMs.
// One wave per slice of 512 samples and column of 16 x 16 tiles (16 input
// rows of a layer, 13 columns, against all 64 delta rows): it runs through its
// slice's samples in order and stores its part of dW^T (k_mlp_reduce sums the
// slices).  A wave per layer, four or five columns, read every row once but left
// the chip at 384 waves: 65 536 samples 26 -> 14 us.  Five more jobs per slice sum
// the training kernel's per-wave partials, each a share of the waves.  All
// jobs of a slice run on one XCD (blocks b, b + 8, ... do), whose L2 then
// reads the slice once.
constexpr int kWgSlice = 512;
constexpr int kWgCols = 13;
constexpr int kWgJobs = kWgCols + (kPartStride + 63) / 64;
// a slice's part: the gradient in theta's layout, then the loss sum
constexpr int kWPartLoss = kMlpParams;
constexpr int kWPart = (kMlpParams + 1 + 31) & ~31;

__global__ void __launch_bounds__(64) k_mlp_wgrad(const uint16_t* __restrict__ acts, int n_tiles, int n_slices,
                                                  const float* __restrict__ part, int n_waves,
                                                  float* __restrict__ wpart) {
    const int lane = threadIdx.x;
    const int slice = (blockIdx.x / (8 * kWgJobs)) * 8 + blockIdx.x % 8, job = (blockIdx.x / 8) % kWgJobs;
    if (slice >= n_slices) return;
    float* wp = wpart + (size_t)slice * kWPart;
    if (job >= kWgCols) {
        const int j = (job - kWgCols) * 64 + lane;
        if (j >= kPartStride) return;
        const int share = (n_waves + n_slices - 1) / n_slices;
        const int w0 = slice * share, w1 = min(n_waves, w0 + share);
        float sum = 0.f;
        for (int w = w0; w < w1; ++w) sum += part[(size_t)w * kPartStride + j];
        const int l = j / kMlpWidth, f = j % kMlpWidth;
        wp[l == 4 ? (f == 0 ? kMlpB4 : kWPartLoss)
                  : (l == 0 ? kMlpB1 : (l == 1 ? kMlpB2 : (l == 2 ? kMlpB3 : kMlpW4))) + f] = sum;
        return;
    }
    const int g = lane >> 4, r = lane & 15;
    const int in = job < 5 ? kRowsX + 16 * job : (job < 9 ? kRowsH1 + 16 * (job - 5) : kRowsH2 + 16 * (job - 9));
    const int de = job < 5 ? kRowsD1 : (job < 9 ? kRowsD2 : kRowsD3);
    constexpr size_t kTile = (size_t)kRowsTile * 16;
    const uint16_t* pa = acts + (de + r) * 16 + 4 * g;
    const uint16_t* pb = acts + (in + r) * 16 + 4 * g;
    f32x4 acc[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int t_end = min(n_tiles, (slice + 1) * (kWgSlice / 16));
    // U tiles' fragments are loaded before any of them is used
    constexpr int U = 8;
    int t = slice * (kWgSlice / 16);
    for (; t + U <= t_end; t += U) {
        bf16x4 a[U][4], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t off = (size_t)(t + u) * kTile;
            b[u] = *reinterpret_cast<const bf16x4*>(pb + off);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) a[u][nb] = *reinterpret_cast<const bf16x4*>(pa + off + 256 * nb);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) acc[nb] = mfma(a[u][nb], b[u], acc[nb]);
    }
    for (; t < t_end; ++t) {
        const size_t off = (size_t)t * kTile;
        const bf16x4 b = *reinterpret_cast<const bf16x4*>(pb + off);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[nb] = mfma(*reinterpret_cast<const bf16x4*>(pa + off + 256 * nb), b, acc[nb]);
    }
    // acc[nb][i] = dW[16 column + r][16 nb + 4 g + i]
    float* w = wp + (job < 5 ? kMlpW1 + 16 * job * kMlpWidth
                             : (job < 9 ? kMlpW2 + 16 * (job - 5) * kMlpWidth : kMlpW3 + 16 * (job - 9) * kMlpWidth)) +
               r * kMlpWidth + 4 * g;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) *reinterpret_cast<f32x4*>(w + 16 * nb) = acc[nb];
}

// Sums the slices' parts, 32 parameters per block of 256 threads (eight
// threads per parameter; whole 128-byte lines), eight slices at a time in order
// and then the groups in order (in FP64: the groups used to be added in any
// order, by atomics, and this stays in the middle of what that could give),
// and either takes one Adam step on the FP32
// master parameters and re-packs the bf16 operand fragments (kAdam), or writes
// the gradient.  The loss sum is added to *loss.  One launch for the sums
// (4.6 us, with atomics), Adam (4.7) and the fills (3.6): 6 us.
constexpr int kWrGroup = 8;
template <bool kAdam>
__global__ void __launch_bounds__(256) k_mlp_reduce(const float* __restrict__ wpart, int n_slices, float* loss,
                                                    float* __restrict__ grad, float* __restrict__ theta,
                                                    float* __restrict__ m, float* __restrict__ v,
                                                    uint16_t* __restrict__ blob, MlpAdam A) {
    __shared__ float sh[256 / 32][32];
    const int c = threadIdx.x & 31, q = threadIdx.x >> 5;
    const int p = blockIdx.x * 32 + c;
    double total = 0.0;
    for (int s0 = 0; s0 < n_slices; s0 += kWrGroup * (256 / 32)) {
        // this thread's group of the next eight
        const int s = s0 + kWrGroup * q;
        float x[kWrGroup];
#pragma unroll
        for (int u = 0; u < kWrGroup; ++u) x[u] = s + u < n_slices ? wpart[(size_t)(s + u) * kWPart + p] : 0.f;
        float sum = 0.f;
#pragma unroll
        for (int u = 0; u < kWrGroup; ++u) sum += x[u];
        sh[q][c] = sum;
        __syncthreads();
        if (q == 0)
#pragma unroll
            for (int u = 0; u < 256 / 32; ++u)
                if (s0 + kWrGroup * u < n_slices) total += (double)sh[u][c];
        __syncthreads();
    }
    if (q != 0 || p > kWPartLoss) return;
    const float gr = (float)total;
    if (p == kWPartLoss) {
        *loss += gr;
        return;
    }
    if (!kAdam) {
        grad[p] = gr;
        return;
    }
    float mm = A.beta1 * m[p] + (1.0f - A.beta1) * gr;
    float vv = A.beta2 * v[p] + (1.0f - A.beta2) * gr * gr;
    m[p] = mm;
    v[p] = vv;
    float mh = mm / A.bias1, vh = vv / A.bias2;
    float w = theta[p] - A.lr * mh / (sqrtf(vh) + A.eps);
    theta[p] = w;
    pack_param(blob, p, w);
}

__global__ void k_mlp_set_norm(MlpNorm* norm, float mu, float sigma) {
    norm->mu = mu;
    norm->sigma = sigma;
}

// mean and standard deviation of the pool's targets (FP64 sums)
__global__ void k_mlp_moments(const float* __restrict__ t, const int32_t* n_dev, int32_t n_host, double* sums) {
    int n = n_dev ? min(*n_dev, n_host) : n_host;
    double a = 0.0, b = 0.0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        double x = t[i];
        a += x;
        b += x * x;
    }
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(sums, a);
        atomicAdd(sums + 1, b);
    }
}

__global__ void k_mlp_norm_from_moments(const double* sums, const int32_t* n_dev, int32_t n_host, MlpNorm* norm) {
    int n = n_dev ? min(*n_dev, n_host) : n_host;
    if (n <= 0) {
        norm->mu = 0.f;
        norm->sigma = 1.f;
        return;
    }
    double mean = sums[0] / n;
    double var = fmax(sums[1] / n - mean * mean, 0.0);
    norm->mu = (float)mean;
    norm->sigma = (float)fmax(sqrt(var), 1e-3);
}

__global__ void k_mlp_zero_f64(double* p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0.0;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int blocks_for(int64_t n, int per_block, int cap) {
    int64_t b = (n + per_block - 1) / per_block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

// blocks of the training kernel: one per CU, at most
static int train_blocks(int tiles) { return blocks_for(tiles, kTrainWaves, 256); }

hipError_t mlp_alloc(Mlp& m, int32_t max_batch) {
    m.max_batch = max_batch;
    hipError_t e = hipMalloc(&m.theta, 4 * (size_t)kMlpParams);
    if (e == hipSuccess) e = hipMalloc(&m.m, 4 * (size_t)kMlpParams);
    if (e == hipSuccess) e = hipMalloc(&m.v, 4 * (size_t)kMlpParams);
    if (e == hipSuccess) e = hipMalloc(&m.blob, 2 * (size_t)kFragAll);
    if (e == hipSuccess) e = hipMalloc(&m.norm, sizeof(MlpNorm));
    if (e == hipSuccess) e = hipMalloc(&m.loss, sizeof(float));
    if (e == hipSuccess) e = hipMalloc(&m.moments, 2 * sizeof(double));
    const int tiles = (max_batch + 15) / 16;
    if (e == hipSuccess) e = hipMalloc(&m.acts, 2 * (size_t)kRowsTile * 16 * tiles);
    // one partial row per wave of the training kernel at its largest grid
    if (e == hipSuccess) e = hipMalloc(&m.part, 4 * (size_t)kPartStride * kTrainWaves * train_blocks(tiles));
    m.max_slices = (tiles * 16 + kWgSlice - 1) / kWgSlice;
    if (e == hipSuccess) e = hipMalloc(&m.wpart, 4 * (size_t)kWPart * m.max_slices);
    return e;
}

void mlp_free(Mlp& m) {
    void* ps[] = {m.theta, m.m, m.v, m.blob, m.norm, m.loss, m.moments, m.acts, m.part, m.wpart};
    for (void* p : ps)
        if (p) (void)hipFree(p);
    m = Mlp();
}

hipError_t mlp_set_weights(Mlp& m, const float* host_theta, hipStream_t s) {
    hipError_t e = hipMemcpyAsync(m.theta, host_theta, 4 * (size_t)kMlpParams, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    e = hipMemsetAsync(m.m, 0, 4 * (size_t)kMlpParams, s);
    if (e == hipSuccess) e = hipMemsetAsync(m.v, 0, 4 * (size_t)kMlpParams, s);
    if (e == hipSuccess) e = hipMemsetAsync(m.blob, 0, 2 * (size_t)kFragAll, s);
    if (e == hipSuccess) e = hipMemsetAsync(m.loss, 0, sizeof(float), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_pack, dim3(blocks_for(kMlpParams, 256, 64)), dim3(256), 0, s, (const float*)m.theta,
                       m.blob);
    m.step = 0;
    return hipGetLastError();
}

hipError_t mlp_set_norm(Mlp& m, float mu, float sigma, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_set_norm, dim3(1), dim3(1), 0, s, m.norm, mu, sigma);
    return hipGetLastError();
}

hipError_t mlp_norm_from_pool(Mlp& m, const float* target, const int32_t* n_dev, int32_t n_host, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_zero_f64, dim3(1), dim3(64), 0, s, m.moments, 2);
    hipLaunchKernelGGL(k_mlp_moments, dim3(blocks_for(n_host, 256, 1024)), dim3(256), 0, s, target, n_dev, n_host,
                       m.moments);
    hipLaunchKernelGGL(k_mlp_norm_from_moments, dim3(1), dim3(1), 0, s, (const double*)m.moments, n_dev, n_host,
                       m.norm);
    return hipGetLastError();
}

static MlpInput make_input(const float* pos, int pos_stride, const float* nrm, int nrm_stride, const int32_t* n_dev,
                           int32_t n_host, const OctParams* box) {
    MlpInput in;
    in.pos = pos;
    in.pos_stride = pos_stride;
    in.nrm = nrm;
    in.nrm_stride = nrm_stride;
    in.n_dev = n_dev;
    in.n_host = n_host;
    in.normalize = box ? 1 : 0;
    for (int c = 0; c < 3; ++c) {
        in.min_bound[c] = box ? box->min_bound[c] : 0.f;
        in.size_inv[c] = box ? box->size_inv[c] : 1.f;
    }
    return in;
}

hipError_t mlp_infer(const Mlp& m, const float* pos, int pos_stride, const float* nrm, int nrm_stride,
                     const int32_t* n_dev, int32_t n_host, const OctParams* box, float* out, int mode,
                     hipStream_t s) {
    if (n_host <= 0) return hipSuccess;
    MlpInput in = make_input(pos, pos_stride, nrm, nrm_stride, n_dev, n_host, box);
    hipLaunchKernelGGL(k_mlp_infer, dim3(blocks_for((n_host + 15) / 16, 4, 2048)), dim3(256), 0, s,
                       (const uint16_t*)m.blob, (const float*)m.theta, (const MlpNorm*)m.norm, in, out, mode);
    return hipGetLastError();
}

// gradient of the mean loss over one batch, left as parts for mlp_adam or
// mlp_write_gradient, which also add its loss sum to m.loss
hipError_t mlp_gradient(Mlp& m, const float* pos, int pos_stride, const float* nrm, int nrm_stride,
                        const float* target, const int32_t* pool_dev, int32_t pool_host, int32_t batch, int sample,
                        uint32_t k0, uint32_t k1, const OctParams* box, hipStream_t s) {
    if (batch <= 0 || batch > m.max_batch) return hipErrorInvalidValue;
    MlpBatch B;
    B.in = make_input(pos, pos_stride, nrm, nrm_stride, pool_dev, pool_host, box);
    B.target = target;
    B.n = batch;
    B.sample = sample;
    B.k0 = k0;
    B.k1 = k1;
    B.step = (uint32_t)m.step;
    const int tiles = (batch + 15) / 16, blocks = train_blocks(tiles);
    hipLaunchKernelGGL(k_mlp_train_fb, dim3(blocks), dim3(64 * kTrainWaves), 0, s, (const uint16_t*)m.blob,
                       (const float*)m.theta, (const MlpNorm*)m.norm, B, m.acts, tiles, m.part);
    m.slices = (16 * tiles + kWgSlice - 1) / kWgSlice;
    if (m.slices > m.max_slices) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mlp_wgrad, dim3((m.slices + 7) / 8 * 8 * kWgJobs), dim3(64), 0, s, (const uint16_t*)m.acts,
                       tiles, m.slices, (const float*)m.part, kTrainWaves * blocks, m.wpart);
    return hipGetLastError();
}

constexpr int kReduceGrid = kWPart / 32;

hipError_t mlp_adam(Mlp& m, float lr, float beta1, float beta2, float eps, hipStream_t s) {
    m.step += 1;
    MlpAdam A;
    A.lr = lr;
    A.beta1 = beta1;
    A.beta2 = beta2;
    A.eps = eps;
    A.bias1 = (float)(1.0 - std::pow((double)beta1, (double)m.step));
    A.bias2 = (float)(1.0 - std::pow((double)beta2, (double)m.step));
    hipLaunchKernelGGL(k_mlp_reduce<true>, dim3(kReduceGrid), dim3(256), 0, s, (const float*)m.wpart, m.slices, m.loss,
                       (float*)nullptr, m.theta, m.m, m.v, m.blob, A);
    return hipGetLastError();
}

hipError_t mlp_write_gradient(Mlp& m, float* grad, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_reduce<false>, dim3(kReduceGrid), dim3(256), 0, s, (const float*)m.wpart, m.slices, m.loss,
                       grad, (float*)nullptr, (float*)nullptr, (float*)nullptr, (uint16_t*)nullptr, MlpAdam{});
    return hipGetLastError();
}

}  // namespace neb
