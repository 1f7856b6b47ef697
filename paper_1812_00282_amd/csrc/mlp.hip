// Learned estimator for VATE on MI355X: a 64 -> 64 -> 64 -> 1 GELU network
// that maps a host's sketch features (distance histogram, live fraction, pool
// occupancy) to the log of its window cardinality, on top of the log of the
// closed-form estimate (a fixed residual branch).  Hand-written training and
// inference kernels on gfx950's BF16 matrix cores
// (v_mfma_f32_16x16x32_bf16: 16x32 by 32x16 tiles, FP32 accumulate).
//
// Numerics (mirrored by the CPU oracle): BF16 round-to-nearest-even of the
// features, W1, W2, a1 = GELU(z1), a2 = GELU(z2), and of the pre-activation
// gradients dz2, dz1 before the products that consume them; every sum, bias,
// GELU, the output layer and Adam in FP32.
//
// Tile organisation: inference gives a wavefront 16 samples, whose layers are
// (16 x 64) x (64 x 64) products; training gives a workgroup 64 samples and
// each of its 16 wavefronts one 16 x 16 tile of every product (k_train), the
// weight gradients accumulated across workgroups with FP32 atomics.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "vate.h"
#include "vate_mlp.h"
#include "mlp_core.h"

namespace vate {
namespace mlp {

// ---------------------------------------------------------------------------
// Pack FP32 parameters into the inference layout.
// ---------------------------------------------------------------------------
__global__ void k_pack(const float *__restrict__ theta, Packed *__restrict__ P)
{
    for (int i = threadIdx.x + blockIdx.x * blockDim.x; i < HD * F; i += blockDim.x * gridDim.x) {
        P->W1b[i] = bf16_bits(theta[OFF_W1 + i]);
        const int n = i / HD, k = i % HD;
        const uint16_t w2 = bf16_bits(theta[OFF_W2 + i]);
        P->W2b[i] = w2;
        P->W2bT[k * HD + n] = w2;
    }
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < HD; i += blockDim.x) {
            P->b1[i] = theta[OFF_B1 + i];
            P->b2[i] = theta[OFF_B2 + i];
            P->w3[i] = theta[OFF_W3 + i];
        }
        if (threadIdx.x == 0) {
            P->b3 = theta[OFF_B3];
            P->env.magic = 0;         // packing switches the envelope off
        }
        for (int i = threadIdx.x; i < kFallbackSlots; i += blockDim.x) P->fallbacks[i] = 0;
    }
}

// Load 16 feature rows of this wavefront into LDS (zero beyond n).
__device__ __forceinline__ void stage_rows(const uint16_t *__restrict__ X, uint64_t row0, uint64_t n, uint16_t *xs)
{
    const int l = threadIdx.x & 63;
    // 16 rows x 64 bf16 = 16 x 8 uint4; 64 lanes take two each
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int idx = l + 64 * t, m = idx >> 3, part = idx & 7;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row0 + m < n) v = reinterpret_cast<const uint4 *>(X + (row0 + m) * F)[part];
        *reinterpret_cast<uint4 *>(xs + m * LDS_STRIDE + part * 8) = v;
    }
}

// ---------------------------------------------------------------------------
// Inference over a feature matrix: o[i] = network(x_i) + r[i].
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_forward(const Packed *__restrict__ P, const uint16_t *__restrict__ X,
                                                 const float *__restrict__ R, uint64_t n, float *__restrict__ O)
{
    __shared__ __attribute__((aligned(16))) uint16_t xs_all[4][16 * LDS_STRIDE];
    __shared__ __attribute__((aligned(16))) uint16_t a1_all[4][16 * LDS_STRIDE];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, q = l >> 4, c = l & 15;
    const uint64_t row0 = (uint64_t)blockIdx.x * 64 + 16 * w;
    stage_rows(X, row0, n, xs_all[w]);
    __syncthreads();
    float r4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) r4[r] = row0 + 4 * q + r < n ? R[row0 + 4 * q + r] : 0.f;
    f32x4 z1[4], z2[4];
    float a2v[4][4], o4[4];
    forward16(P, xs_all[w], a1_all[w], r4, z1, z2, a2v, o4);
    if (c < 4 && row0 + 4 * q + c < n) O[row0 + 4 * q + c] = o4[c];
}

// ---------------------------------------------------------------------------
// One training pass over a minibatch: forward, loss gradient, backward; the
// parameter gradient (FP32, VATE_MLP_PARAMS entries, caller-zeroed) and the
// loss sum are accumulated with atomics.  Loss = mean |exp(o - y) - 1|.
//
// A workgroup of 4 S wavefronts takes 16 S samples at a time, each wavefront
// one 16 x 16 tile of every product (sample slab w / 4, unit tile w mod 4; of
// the weight gradients 4 / S tiles, column tile w mod 4), with the weights of
// its tiles loaded at the start together with the samples.  Its time is one
// workgroup's chain of steps (8 us with 32 samples, 10 with 64; the GELUs and
// their derivatives most of it) plus about 48 ns per workgroup for the 8385
// gradient atomics of each: so 32 samples a workgroup up to 2048, else 64 (at
// 4096 samples 13.7 us against 14.1 with 32, at 8192 16.7 against 20.8; four
// wavefronts with whole 16-sample slabs took 20 us at 4096 and 76 at 65,536,
// which now take 13.7 and 43).  Beyond 256 workgroups each goes on with the
// next samples and keeps its sums in registers.
// ---------------------------------------------------------------------------
constexpr unsigned kTrainBlocks = 256;       // the CUs of an MI355X

// One 16 x 16 tile, K = 64: rows of A from arow, rows of B already in registers.
__device__ __forceinline__ f32x4 tile64(const uint16_t *arow, const bf16x8 b0, const bf16x8 b1, int q)
{
    f32x4 d = {0.f, 0.f, 0.f, 0.f};
    d = mfma(frag(arow, 0, q), b0, d);
    return mfma(frag(arow, 1, q), b1, d);
}

// A tile of a weight gradient over K = 16 S samples, both operands from LDS.
template <int S>
__device__ __forceinline__ f32x4 grad_tile(const uint16_t *arow, const uint16_t *brow, int q)
{
    f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < S / 2; ++s) d = mfma(frag(arow, s, q), frag(brow, s, q), d);
    return d;
}

template <int S>
__global__ void __launch_bounds__(256 * S) k_train(const Packed *__restrict__ P, const uint16_t *__restrict__ X,
                                                   const float *__restrict__ R, const float *__restrict__ Y,
                                                   uint64_t n, float inv_batch, float *__restrict__ grad,
                                                   float *__restrict__ loss)
{
    static_assert(S == 2 || S == 4, "weight gradients in steps of 32 samples");
    constexpr int NT = 256 * S, ROWS = 16 * S, TILES = 4 / S;
    __shared__ __attribute__((aligned(16))) uint16_t xs[ROWS * LDS_STRIDE];    // [sample][feature]
    __shared__ __attribute__((aligned(16))) uint16_t xT[64 * LDS_STRIDE];      // [feature][sample]
    __shared__ __attribute__((aligned(16))) uint16_t a1s[ROWS * LDS_STRIDE];   // [sample][unit]
    __shared__ __attribute__((aligned(16))) uint16_t a1T[64 * LDS_STRIDE];     // [unit][sample]
    __shared__ __attribute__((aligned(16))) uint16_t dz2s[ROWS * LDS_STRIDE];  // [sample][unit]
    __shared__ __attribute__((aligned(16))) uint16_t dz2T[64 * LDS_STRIDE];    // [unit][sample]
    __shared__ __attribute__((aligned(16))) uint16_t dz1T[64 * LDS_STRIDE];    // [unit][sample]
    __shared__ float opart[4][ROWS];                                            // output layer, per unit tile
    __shared__ float gsmall[3 * HD + 1];                                        // db1, db2, dw3, db3
    __shared__ float lsum;
    const int t = threadIdx.x, w = t >> 6, l = t & 63, q = l >> 4, c = l & 15;
    const int sw = w >> 2, nt = w & 3, u = 16 * nt + c, m0 = 16 * sw + 4 * q;   // this lane's unit, first sample
    for (int i = t; i < 3 * HD + 1; i += NT) gsmall[i] = 0.f;
    if (t == 0) lsum = 0.f;
    const bf16x8 w1a = frag(P->W1b + u * F, 0, q), w1b = frag(P->W1b + u * F, 1, q);
    const bf16x8 w2a = frag(P->W2b + u * HD, 0, q), w2b = frag(P->W2b + u * HD, 1, q);
    const bf16x8 w2ta = frag(P->W2bT + u * HD, 0, q), w2tb = frag(P->W2bT + u * HD, 1, q);
    const float b1 = P->b1[u], b2 = P->b2[u], w3 = P->w3[u], b3 = P->b3;
    f32x4 gW1[TILES] = {}, gW2[TILES] = {};
    float gw3 = 0.f, gb2 = 0.f, gb1 = 0.f, gb3 = 0.f, ls = 0.f;

    for (uint64_t row0 = (uint64_t)blockIdx.x * ROWS; row0 < n; row0 += (uint64_t)gridDim.x * ROWS) {
        float r4[4], y4[4];
        bool v4[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint64_t row = row0 + m0 + r;
            v4[r] = row < n;
            r4[r] = v4[r] ? R[row] : 0.f;
            y4[r] = v4[r] ? Y[row] : 0.f;
        }
        if (t < 8 * ROWS) {      // rows of 8 16-byte parts (zero beyond n), and the transposed copy
            const int m = t >> 3, part = t & 7;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (row0 + m < n) v = reinterpret_cast<const uint4 *>(X + (row0 + m) * F)[part];
            *reinterpret_cast<uint4 *>(xs + m * LDS_STRIDE + part * 8) = v;
            const uint32_t w4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                xT[(8 * part + 2 * j) * LDS_STRIDE + m] = (uint16_t)w4[j];
                xT[(8 * part + 2 * j + 1) * LDS_STRIDE + m] = (uint16_t)(w4[j] >> 16);
            }
        }
        __syncthreads();
        // layer 1: this wavefront's 16 samples, 16 units
        f32x4 z1 = tile64(xs + (16 * sw + c) * LDS_STRIDE, w1a, w1b, q);
        uint32_t pk[2];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z1[r] += b1;
            const uint32_t b = bf16_bits(gelu(z1[r]));
            a1s[(m0 + r) * LDS_STRIDE + u] = (uint16_t)b;
            pk[r >> 1] = (r & 1) ? pk[r >> 1] | b << 16 : b;
        }
        *reinterpret_cast<uint2 *>(a1T + u * LDS_STRIDE + m0) = make_uint2(pk[0], pk[1]);
        __syncthreads();
        // layer 2 and the output layer's sum over this tile's units
        f32x4 z2 = tile64(a1s + (16 * sw + c) * LDS_STRIDE, w2a, w2b, q);
        float a2[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z2[r] += b2;
            a2[r] = bf16_float(bf16_bits(gelu(z2[r])));
            float part = a2[r] * w3;
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) part += __shfl_xor(part, off, 64);
            if (c == 0) opart[nt][m0 + r] = part;
        }
        __syncthreads();
        // loss gradient, output layer gradients, dz2
        uint32_t pd[2];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float o = opart[0][m0 + r] + opart[1][m0 + r] + opart[2][m0 + r] + opart[3][m0 + r] + b3 + r4[r];
            const float e = expf(o - y4[r]), d = e - 1.0f;
            const float dor = v4[r] ? (d > 0.f ? e : (d < 0.f ? -e : 0.f)) * inv_batch : 0.f;
            if (nt == 0 && c == 0) {       // once per sample
                gb3 += dor;
                if (v4[r]) ls += fabsf(d);
            }
            gw3 += dor * a2[r];
            const float dz = dor * w3 * gelu_grad(z2[r]);
            gb2 += dz;
            const uint32_t b = bf16_bits(dz);
            dz2s[(m0 + r) * LDS_STRIDE + u] = (uint16_t)b;
            pd[r >> 1] = (r & 1) ? pd[r >> 1] | b << 16 : b;
        }
        *reinterpret_cast<uint2 *>(dz2T + u * LDS_STRIDE + m0) = make_uint2(pd[0], pd[1]);
        __syncthreads();
        // dW2[i][k] += sum_m dz2[m][i] a1[m][k]: row tiles sw + S j, column tile nt
#pragma unroll
        for (int j = 0; j < TILES; ++j)
            gW2[j] += grad_tile<S>(dz2T + (16 * (sw + S * j) + c) * LDS_STRIDE, a1T + u * LDS_STRIDE, q);
        // da1 = dz2 W2, dz1 = da1 * gelu'(z1)
        {
            const f32x4 da = tile64(dz2s + (16 * sw + c) * LDS_STRIDE, w2ta, w2tb, q);
            uint32_t p1[2];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float dz = da[r] * gelu_grad(z1[r]);
                gb1 += dz;
                const uint32_t b = bf16_bits(dz);
                p1[r >> 1] = (r & 1) ? p1[r >> 1] | b << 16 : b;
            }
            *reinterpret_cast<uint2 *>(dz1T + u * LDS_STRIDE + m0) = make_uint2(p1[0], p1[1]);
        }
        __syncthreads();
        // dW1[j][f] += sum_m dz1[m][j] x[m][f]
#pragma unroll
        for (int j = 0; j < TILES; ++j)
            gW1[j] += grad_tile<S>(dz1T + (16 * (sw + S * j) + c) * LDS_STRIDE, xT + u * LDS_STRIDE, q);
        __syncthreads();       // xs and xT are free for the next samples
    }

#pragma unroll
    for (int j = 0; j < TILES; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * (sw + S * j) + 4 * q + r;
            atomicAdd(&grad[OFF_W2 + row * HD + u], gW2[j][r]);
            atomicAdd(&grad[OFF_W1 + row * F + u], gW1[j][r]);
        }
    // the four row groups of a unit's lanes, then the sample slabs
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
        gw3 += __shfl_xor(gw3, off, 64);
        gb2 += __shfl_xor(gb2, off, 64);
        gb1 += __shfl_xor(gb1, off, 64);
    }
    if (q == 0) {
        atomicAdd(&gsmall[u], gb1);
        atomicAdd(&gsmall[HD + u], gb2);
        atomicAdd(&gsmall[2 * HD + u], gw3);
    }
    if (nt == 0 && c == 0) {
        atomicAdd(&gsmall[3 * HD], gb3);
        atomicAdd(&lsum, ls);
    }
    __syncthreads();
    if (t < HD) {
        atomicAdd(&grad[OFF_B1 + t], gsmall[t]);
        atomicAdd(&grad[OFF_B2 + t], gsmall[HD + t]);
        atomicAdd(&grad[OFF_W3 + t], gsmall[2 * HD + t]);
    }
    if (t == 0) {
        atomicAdd(&grad[OFF_B3], gsmall[3 * HD]);
        atomicAdd(loss, lsum * inv_batch);
    }
}

// ---------------------------------------------------------------------------
// Adam (Kingma & Ba), bias-corrected, on FP32 parameters.
// ---------------------------------------------------------------------------
__global__ void k_adam(float *__restrict__ theta, const float *__restrict__ grad, float *__restrict__ m,
                       float *__restrict__ v, int count, float lr, float beta1, float beta2, float eps,
                       float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float g = grad[i];
    const float mi = beta1 * m[i] + (1.f - beta1) * g;
    const float vi = beta2 * v[i] + (1.f - beta2) * g * g;
    m[i] = mi;
    v[i] = vi;
    theta[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Features of hosts from vate_estimate's histogram output, a wavefront per
// host: lane f builds feature f, so a row is read and written in one piece.
// (A thread per host took 20 us for 331 hosts, row by row through scratch.)
__global__ void __launch_bounds__(256) k_features(const uint32_t *__restrict__ hist, const float *__restrict__ est,
                                                  uint64_t n, uint32_t k, uint32_t g, float occupancy,
                                                  uint16_t *__restrict__ X, float *__restrict__ R)
{
    const uint32_t f = threadIdx.x & 63u;
    const float fg = (float)g;
    for (uint64_t h = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6); h < n; h += (uint64_t)gridDim.x * 4) {
        const uint32_t bin = f < k ? hist[h * (k + 1) + f] : 0u;      // k < 64
        const float r = logf(fmaxf(est[h], 1.0f));
        uint32_t live = bin;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) live += __shfl_xor(live, off, 64);
        const float x = f <= k ? (float)(f < k ? bin : live) / fg : f == k + 1 ? occupancy : f == k + 2 ? r * 0.0625f : 0.f;
        X[h * F + f] = bf16_bits(x);
        if (f == 0) R[h] = r;
    }
}

__global__ void k_fill(float *__restrict__ p, int count, float value)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = value;
}

// Layout self-check of the matrix-core fragments: D = A * B for one 16x32 by
// 32x16 tile, with A and B row-major bf16 and D row-major FP32.
__global__ void k_mfma_selftest(const uint16_t *__restrict__ A, const uint16_t *__restrict__ B,
                                float *__restrict__ D)
{
    const int l = threadIdx.x & 63, q = l >> 4, c = l & 15;
    uint32_t bw[4];
    for (int j = 0; j < 4; ++j)
        bw[j] = (uint32_t)B[(8 * q + 2 * j) * 16 + c] | ((uint32_t)B[(8 * q + 2 * j + 1) * 16 + c] << 16);
    const bf16x8 a = as_bf16x8(*reinterpret_cast<const uint4 *>(A + c * 32 + 8 * q));
    const bf16x8 b = as_bf16x8(make_uint4(bw[0], bw[1], bw[2], bw[3]));
    f32x4 d = {0.f, 0.f, 0.f, 0.f};
    d = mfma(a, b, d);
    for (int r = 0; r < 4; ++r) D[(4 * q + r) * 16 + c] = d[r];
}

}  // namespace mlp
}  // namespace vate

using namespace vate::mlp;

static int mlp_check(const char *what)
{
    (void)what;
    return hipGetLastError() == hipSuccess ? VATE_OK : VATE_E_DEVICE;
}

extern "C" {

int vate_mlp_pack(const float *theta_dev, void *weights_dev, void *stream)
{
    if (!theta_dev || !weights_dev || (reinterpret_cast<uintptr_t>(weights_dev) & 255u)) return VATE_E_INVAL;
    k_pack<<<16, 256, 0, static_cast<hipStream_t>(stream)>>>(theta_dev, static_cast<Packed *>(weights_dev));
    return mlp_check("pack");
}

int vate_mlp_set_envelope(void *weights_dev, const vate_mlp_envelope *env, void *stream)
{
    if (!weights_dev || (reinterpret_cast<uintptr_t>(weights_dev) & 255u)) return VATE_E_INVAL;
    Envelope e{};
    if (env) {
        for (int f = 0; f < F; ++f)
            if (!(env->lo[f] <= env->hi[f])) return VATE_E_INVAL;
        e.magic = kEnvMagic;
        e.k = env->k;
        e.g = env->g;
        e.log2_pool = env->log2_pool;
        e.width = env->width;
        for (int f = 0; f < F; ++f) e.lo[f] = env->lo[f], e.hi[f] = env->hi[f];
    }
    Packed *P = static_cast<Packed *>(weights_dev);
    const unsigned long long zero[kFallbackSlots] = {};
    hipError_t err = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    if (err == hipSuccess) err = hipMemcpy(&P->env, &e, sizeof(Envelope), hipMemcpyHostToDevice);
    if (err == hipSuccess) err = hipMemcpy(P->fallbacks, zero, sizeof(zero), hipMemcpyHostToDevice);
    return err == hipSuccess ? VATE_OK : VATE_E_DEVICE;
}

int vate_mlp_fallbacks(const void *weights_dev, uint64_t *count, int reset, void *stream)
{
    if (!weights_dev || !count || (reinterpret_cast<uintptr_t>(weights_dev) & 255u)) return VATE_E_INVAL;
    const Packed *P = static_cast<const Packed *>(weights_dev);
    unsigned long long c[kFallbackSlots] = {};
    hipError_t err = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    if (err == hipSuccess) err = hipMemcpy(c, P->fallbacks, sizeof(c), hipMemcpyDeviceToHost);
    if (err == hipSuccess && reset) {
        const unsigned long long zero[kFallbackSlots] = {};
        err = hipMemcpy(const_cast<unsigned long long *>(P->fallbacks), zero, sizeof(zero), hipMemcpyHostToDevice);
    }
    if (err != hipSuccess) return VATE_E_DEVICE;
    uint64_t sum = 0;
    for (int i = 0; i < kFallbackSlots; ++i) sum += c[i];
    *count = sum;
    return VATE_OK;
}

int vate_mlp_forward(const void *weights_dev, const uint16_t *x_dev, const float *r_dev, size_t n, float *o_dev,
                     void *stream)
{
    if (n == 0) return VATE_OK;
    if (!weights_dev || !x_dev || !r_dev || !o_dev || (reinterpret_cast<uintptr_t>(x_dev) & 15u))
        return VATE_E_INVAL;
    const uint64_t blocks = (n + 63) / 64;
    if (blocks > 0x7FFFFFFFull) return VATE_E_INVAL;
    k_forward<<<(unsigned)blocks, 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<const Packed *>(weights_dev), x_dev, r_dev, n, o_dev);
    return mlp_check("forward");
}

int vate_mlp_train_step(const void *weights_dev, const uint16_t *x_dev, const float *r_dev, const float *y_dev,
                        size_t n, float *grad_dev, float *loss_dev, void *stream)
{
    if (n == 0) return VATE_OK;
    if (!weights_dev || !x_dev || !r_dev || !y_dev || !grad_dev || !loss_dev ||
        (reinterpret_cast<uintptr_t>(x_dev) & 15u))
        return VATE_E_INVAL;
    const uint64_t blocks = (n + 63) / 64;
    if (blocks > 0x7FFFFFFFull) return VATE_E_INVAL;
    const Packed *P = static_cast<const Packed *>(weights_dev);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const float inv = 1.0f / (float)n;
    if (n <= 2048)
        k_train<2><<<(unsigned)((n + 31) / 32), 512, 0, st>>>(P, x_dev, r_dev, y_dev, n, inv, grad_dev, loss_dev);
    else
        k_train<4><<<(unsigned)(blocks < kTrainBlocks ? blocks : kTrainBlocks), 1024, 0, st>>>(
            P, x_dev, r_dev, y_dev, n, inv, grad_dev, loss_dev);
    return mlp_check("train");
}

int vate_mlp_adam(float *theta_dev, const float *grad_dev, float *m_dev, float *v_dev, uint32_t step, float lr,
                  float beta1, float beta2, float eps, void *stream)
{
    if (!theta_dev || !grad_dev || !m_dev || !v_dev || step < 1) return VATE_E_INVAL;
    const float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
    k_adam<<<(VATE_MLP_PARAMS + 255) / 256, 256, 0, static_cast<hipStream_t>(stream)>>>(
        theta_dev, grad_dev, m_dev, v_dev, VATE_MLP_PARAMS, lr, beta1, beta2, eps, c1, c2);
    return mlp_check("adam");
}

int vate_mlp_fill(float *dst_dev, size_t count, float value, void *stream)
{
    if (!dst_dev || count > 0x7FFFFFFFull) return VATE_E_INVAL;
    if (count == 0) return VATE_OK;
    k_fill<<<(unsigned)((count + 255) / 256), 256, 0, static_cast<hipStream_t>(stream)>>>(dst_dev, (int)count,
                                                                                            value);
    return mlp_check("fill");
}

int vate_mlp_features(const uint32_t *hist_dev, const float *est_dev, size_t n, uint32_t k, uint32_t g,
                      float pool_active_fraction, uint16_t *x_dev, float *r_dev, void *stream)
{
    if (n == 0) return VATE_OK;
    if (k < 1 || k + 3 > (uint32_t)F) return VATE_E_UNSUPPORTED;
    if (!hist_dev || !est_dev || !x_dev || !r_dev || g < 1 || (reinterpret_cast<uintptr_t>(x_dev) & 15u))
        return VATE_E_INVAL;
    if ((n + 255) / 256 > 0x7FFFFFFFull) return VATE_E_INVAL;
    const uint64_t blocks = (n + 3) / 4;
    k_features<<<(unsigned)(blocks < 16384 ? blocks : 16384), 256, 0, static_cast<hipStream_t>(stream)>>>(
        hist_dev, est_dev, n, k, g, pool_active_fraction, x_dev, r_dev);
    return mlp_check("features");
}

int vate_mlp_mfma_selftest(const uint16_t *a_dev, const uint16_t *b_dev, float *d_dev, void *stream)
{
    if (!a_dev || !b_dev || !d_dev || (reinterpret_cast<uintptr_t>(a_dev) & 15u)) return VATE_E_INVAL;
    k_mfma_selftest<<<1, 64, 0, static_cast<hipStream_t>(stream)>>>(a_dev, b_dev, d_dev);
    return mlp_check("selftest");
}

}  // extern "C"
