// k_mlp.hip - the warm-start surrogate: an 8 -> 64 -> 64 -> 6 tanh MLP whose
// forward and backward passes run on the gfx950 matrix cores (bfloat16
// operands, FP32 accumulation), plus the gradient reduction and the Adam
// update (Kingma & Ba 2015).
//
// Work split: a work-group of four waves owns a tile of 16 samples; wave w
// computes the hidden units [16 w, 16 w + 16) of every layer (forward and
// back) and those units' weight gradients, and the activations are exchanged
// through LDS.  Products over the 64 hidden units (forward layers 2
// and 3, the error back-propagated into layer 1) are sums of 16 x 16 x 32
// tiles (v_mfma_f32_16x16x32_bf16); products over 16 (the padded inputs and
// outputs, and the weight gradients over the tile's 16 samples) take the
// 16 x 16 x 16 shape (v_mfma_f32_16x16x16_bf16).
// Rounding points (mirrored by the FP64 reference): inputs, weights, hidden
// activations and back-propagated errors are rounded to bfloat16 where they
// enter a product; biases, tanh, error terms and all sums stay FP32.  Each
// tile writes its own partial gradient, and one thread per parameter sums the
// tiles in a fixed order, so results do not depend on scheduling.
#include "lbell_dev.h"
#include "lbell_launch.h"

namespace lbd {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t to_bf16(float v) {  // round to nearest even (finite inputs)
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Operand layouts of the two products.  16 x 16 x 16: lane l (r = l % 16,
// g = l / 16) supplies A[r][4 g + j] and B[4 g + j][r], j = 0..3.
// 16 x 16 x 32: A[r][8 g + j] and B[8 g + j][r], j = 0..7 (A and B take the
// same K order, so the sum pairs A[m][k] with B[k][n] whatever K order the
// unit uses).  Both give D[4 g + j][r].  A result rounded to bfloat16 is
// therefore, as it stands, an operand of a product over its rows (the 16
// samples), which is what every weight gradient is.
__device__ __forceinline__ f32x4 mma16(bf16x4 a, bf16x4 b, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma32(bf16x8 a, bf16x8 b, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}

// Four consecutive floats of a caller's array (4-byte aligned only).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4u ld4(const float* p) { return *reinterpret_cast<const f32x4u*>(p); }

__device__ __forceinline__ bf16x4 pack4(float v0, float v1, float v2, float v3) {
    return bf16x4{(short)to_bf16(v0), (short)to_bf16(v1), (short)to_bf16(v2), (short)to_bf16(v3)};
}
__device__ __forceinline__ bf16x8 pack8(f32x4u lo, f32x4u hi) {
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = __builtin_bit_cast(__bf16, to_bf16(lo[j]));
        v[4 + j] = __builtin_bit_cast(__bf16, to_bf16(hi[j]));
    }
    return v;
}

constexpr int MLP_ROW = MLP_H + 8;  // padded row of 64 units: 16-byte aligned, 4 rows apart on other banks
struct alignas(16) MlpShm {
    uint16_t h1[16][MLP_ROW], h2[16][MLP_ROW], d2[16][MLP_ROW];  // [sample][unit]
    bf16x4 h1p[4][64];   // h1 as results lie: block of 16 units, lane -> 4 samples of one unit
    uint16_t d3[4][16][20];  // [wave][sample][output], each wave's own copy
};

// Sums e over the 16 samples in order (lane (r, g) holds samples 4 g + j of
// unit r); lanes with g = 3 return the total.  The terms are added as rounded
// (contraction off: e is a product in the caller).
__device__ __forceinline__ float sum_samples(const float (&e)[4], int r) {
#pragma clang fp contract(off)
    float s = 0.f, t = 0.f;
#pragma unroll
    for (int gg = 0; gg < 4; ++gg) {
        t = s;
#pragma unroll
        for (int j = 0; j < 4; ++j) t += e[j];
        if (gg < 3) s = __shfl(t, 16 * gg + r);
    }
    return t;
}

// mode 0: outputs for n samples -> out (n x 6).  mode 1: loss and gradient of
// the mean squared error against Y, scaled so that the tiles' partial
// gradients sum to the gradient of L = scale / 2 * sum (y - Y)^2; partial of
// tile t at G + t * MLP_NP, its sum of squared errors at Lpart[t].
//
// Bound by latency: a tile is 68 small matrix products, so what counts is
// the length of the chain and how many compute units share a mini-batch.  Each
// lane loads the weights of its wave's units straight into operand
// registers, all loads in flight at once (no LDS copy of the weights, whose
// staging loops were most of the kernel's time), and a tile has a
// work-group, so a mini-batch of 256 runs on 16 compute units instead of 4:
// 6.4 us (22.2 us with four tiles to a work-group and weights staged in LDS);
// 2048 samples forward and back 9.5 us, forward alone 6.6 us (22 and 15).
template <int MODE>
__global__ __launch_bounds__(256) void k_mlp(MlpArgs a) {
    __shared__ MlpShm sh;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int base = blockIdx.x * 16, unit = 16 * w + r;
    const float* P = a.P;
    // weights, inputs and targets
    f32x4u x4 = {0, 0, 0, 0}, w1 = {0, 0, 0, 0};
    if (g < 2) {
        w1 = ld4(P + MLP_OW1 + unit * MLP_IN + 4 * g);
        if (base + r < a.n) x4 = ld4(a.X + (long long)(base + r) * MLP_IN + 4 * g);
    }
    f32x4u w2[4], w3[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int col = 32 * (k >> 1) + 8 * g + 4 * (k & 1);
        w2[k] = ld4(P + MLP_OW2 + unit * MLP_H + col);
        w3[k] = f32x4u{0, 0, 0, 0};
        if (r < MLP_OUT) w3[k] = ld4(P + MLP_OW3 + r * MLP_H + col);
    }
    const float b1 = P[MLP_OB1 + unit], b2 = P[MLP_OB2 + unit], b3 = r < MLP_OUT ? P[MLP_OB3 + r] : 0.f;
    float xt[4], yt[4], w3t[4], w2t[2][8];  // mode 1: targets, and weights and inputs as the backward products take them
    if constexpr (MODE == 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = base + 4 * g + j;
            xt[j] = r < MLP_IN && m < a.n ? a.X[(long long)m * MLP_IN + r] : 0.f;
            yt[j] = r < MLP_OUT && m < a.n ? a.Y[(long long)m * MLP_OUT + r] : 0.f;
            w3t[j] = 4 * g + j < MLP_OUT ? P[MLP_OW3 + (4 * g + j) * MLP_H + unit] : 0.f;
        }
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
            for (int j = 0; j < 8; ++j) w2t[ot][j] = P[MLP_OW2 + (32 * ot + 8 * g + j) * MLP_H + unit];
    }
    const f32x4 zero = {0, 0, 0, 0};

    // forward
    f32x4 acc = mma16(pack4(x4[0], x4[1], x4[2], x4[3]), pack4(w1[0], w1[1], w1[2], w1[3]), zero);
    uint16_t h1[4], h2[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        h1[j] = to_bf16(tanhf(acc[j] + b1));
        sh.h1[4 * g + j][unit] = h1[j];
    }
    if constexpr (MODE == 1) sh.h1p[w][lane] = bf16x4{(short)h1[0], (short)h1[1], (short)h1[2], (short)h1[3]};
    __syncthreads();
    acc = zero;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
        acc = mma32(*reinterpret_cast<const bf16x8*>(&sh.h1[r][32 * kt + 8 * g]), pack8(w2[2 * kt], w2[2 * kt + 1]),
                    acc);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        h2[j] = to_bf16(tanhf(acc[j] + b2));
        sh.h2[4 * g + j][unit] = h2[j];
    }
    __syncthreads();
    f32x4 y = zero;  // every wave: the next product needs all of it
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
        y = mma32(*reinterpret_cast<const bf16x8*>(&sh.h2[r][32 * kt + 8 * g]), pack8(w3[2 * kt], w3[2 * kt + 1]), y);
    if constexpr (MODE == 0) {
        if (w == 0 && r < MLP_OUT)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m = base + 4 * g + j;
                if (m < a.n) a.out[(long long)m * MLP_OUT + r] = y[j] + b3;
            }
        return;
    }

    // backward: e3 = dL/dy
    float* G = a.G + (long long)blockIdx.x * MLP_NP;
    float sq = 0.f, e[4];
    bf16x4 d3;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int m = base + 4 * g + j;
        e[j] = 0.f;
        if (r < MLP_OUT && m < a.n) {
            const float d = y[j] + b3 - yt[j];
            sq += d * d;
            e[j] = a.scale * d;
        }
        d3[j] = (short)to_bf16(e[j]);
        sh.d3[w][4 * g + j][r] = (uint16_t)d3[j];
    }
    if (w == 0) {
        // squared error of the tile (lanes hold disjoint entries)
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
        if (lane == 0) a.Lpart[blockIdx.x] = sq;
        const float s = sum_samples(e, r);
        if (g == 3 && r < MLP_OUT) G[MLP_OB3 + r] = s;
    }
    // dW3[n][k] = sum_m e3[m][n] h2[m][k]
    const bf16x4 h2v = {(short)h2[0], (short)h2[1], (short)h2[2], (short)h2[3]};
    acc = mma16(d3, h2v, zero);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (4 * g + j < MLP_OUT) G[MLP_OW3 + (4 * g + j) * MLP_H + unit] = acc[j];
    // e2 = (e3 W3) * (1 - h2^2); d3 comes back in another layout through this
    // wave's own part of LDS, after its own writes
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    acc = mma16(*reinterpret_cast<const bf16x4*>(&sh.d3[w][r][4 * g]), pack4(w3t[0], w3t[1], w3t[2], w3t[3]), zero);
    bf16x4 d2;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float h = from_bf16(h2[j]);
        e[j] = acc[j] * (1.f - h * h);
        d2[j] = (short)to_bf16(e[j]);
        sh.d2[4 * g + j][unit] = (uint16_t)d2[j];
    }
    __syncthreads();
    // e1 = (e2 W2) * (1 - h1^2)
    acc = zero;
#pragma unroll
    for (int ot = 0; ot < 2; ++ot) {
        bf16x8 b;
#pragma unroll
        for (int j = 0; j < 8; ++j) b[j] = __builtin_bit_cast(__bf16, to_bf16(w2t[ot][j]));
        acc = mma32(*reinterpret_cast<const bf16x8*>(&sh.d2[r][32 * ot + 8 * g]), b, acc);
    }
    // dW2[o][k] = sum_m e2[m][o] h1[m][k]
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
        const f32x4 v = mma16(d2, sh.h1p[kt][lane], zero);
#pragma unroll
        for (int j = 0; j < 4; ++j) G[MLP_OW2 + (16 * w + 4 * g + j) * MLP_H + 16 * kt + r] = v[j];
    }
    float s = sum_samples(e, r);
    if (g == 3) G[MLP_OB2 + unit] = s;
    bf16x4 d1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float h = from_bf16(h1[j]);
        e[j] = acc[j] * (1.f - h * h);
        d1[j] = (short)to_bf16(e[j]);
    }
    s = sum_samples(e, r);
    if (g == 3) G[MLP_OB1 + unit] = s;
    // dW1[o][i] = sum_m e1[m][o] x[m][i]
    acc = mma16(d1, pack4(xt[0], xt[1], xt[2], xt[3]), zero);
    if (r < MLP_IN)
#pragma unroll
        for (int j = 0; j < 4; ++j) G[MLP_OW1 + (16 * w + 4 * g + j) * MLP_IN + r] = acc[j];
}

// One thread per parameter: sum of the tiles' partial gradients in tile
// order; mode 0 applies Adam (c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t)),
// mode 1 writes the sum to gsum.  The last work-group also sums the tiles'
// squared errors, adding to *loss_acc (or setting it, loss_first) or writing
// the sum over loss_div to *loss_out.
// Bound by latency: RED_LOADS loads of a thread are in flight together (the
// sums stay in tile order), and work-groups of one wave spread the 5126
// parameters over 81 compute units: 2.7 us for 16 tiles, 6.5 us for 128 (one
// load at a time on 21 work-groups of 256: 6.1 and 35.8 us).
constexpr int RED_BLOCK = 64, RED_LOADS = 32;
__global__ __launch_bounds__(RED_BLOCK) void k_mlp_reduce(MlpReduceArgs a) {
    const int lane = threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) {
        if (!a.loss_acc && !a.loss_out) return;
        double s = 0.0;
        for (int t0 = 0; t0 < a.ntiles; t0 += RED_BLOCK) {
            const float v = t0 + lane < a.ntiles ? a.Lpart[t0 + lane] : 0.f;
            const int cnt = min(RED_BLOCK, a.ntiles - t0);
            for (int k = 0; k < cnt; ++k) s += (double)__shfl(v, k);
        }
        if (lane == 0) {
            if (a.loss_acc) *a.loss_acc = a.loss_first ? s : *a.loss_acc + s;
            if (a.loss_out) *a.loss_out = (float)(s / a.loss_div);
        }
        return;
    }
    const int p = blockIdx.x * RED_BLOCK + lane;
    if (p >= MLP_NP) return;
    float m0 = 0.f, v0 = 0.f, p0 = 0.f;
    if (a.mode == 0) {
        m0 = a.M[p];
        v0 = a.V[p];
        p0 = a.P[p];
    }
    float gsum = 0.f;
    const float* G = a.G + p;
    int t0 = 0;
    for (; t0 + RED_LOADS <= a.ntiles; t0 += RED_LOADS) {
        float v[RED_LOADS];
#pragma unroll
        for (int k = 0; k < RED_LOADS; ++k) v[k] = G[(long long)(t0 + k) * MLP_NP];
#pragma unroll
        for (int k = 0; k < RED_LOADS; ++k) gsum += v[k];
    }
    for (; t0 < a.ntiles; t0 += 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = G[(long long)min(t0 + k, a.ntiles - 1) * MLP_NP];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (t0 + k < a.ntiles) gsum += v[k];
    }
    if (a.mode == 1) {
        a.gsum[p] = gsum;
        return;
    }
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float m = b1 * m0 + (1.f - b1) * gsum;
    const float v = b2 * v0 + (1.f - b2) * gsum * gsum;
    a.M[p] = m;
    a.V[p] = v;
    a.P[p] = p0 - a.lr * (m * a.c1) / (sqrtf(v * a.c2) + eps);
}

hipError_t launch_mlp(const MlpArgs& a, hipStream_t st) {
    if (a.n <= 0) return hipSuccess;
    const int tiles = (a.n + 15) / 16;
    if (a.mode == 0)
        hipLaunchKernelGGL(k_mlp<0>, dim3(tiles), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(k_mlp<1>, dim3(tiles), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_mlp_reduce(const MlpReduceArgs& a, hipStream_t st) {
    // the parameters, and one work-group for the loss
    hipLaunchKernelGGL(k_mlp_reduce, dim3((MLP_NP + RED_BLOCK - 1) / RED_BLOCK + 1), dim3(RED_BLOCK), 0, st, a);
    return hipGetLastError();
}

}  // namespace lbd
