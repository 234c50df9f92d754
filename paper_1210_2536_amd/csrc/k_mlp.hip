// K9 / K10: the learned format-and-kernel selector (the paper's offline data
// mining model of Section 5, Equation 1, here a 12-64-64-C perceptron) --
// inference on raw features, and the forward, backward and Adam kernels that
// train it.  float32 throughout; every reduction runs in a fixed order, so
// results are deterministic.
//
// Parameter order (flat float32): W1 [64 x 12], b1 [64], W2 [64 x 64],
// b2 [64], W3 [C x 64], b3 [C], row-major.
#include "internal.hpp"

namespace smat {
namespace {

constexpr int kIn = 12;
constexpr int kHid = 64;

struct Net {
    const float *W1, *b1, *W2, *b2, *W3, *b3;
};

__host__ __device__ inline Net unpack(const float *p, int n_out) {
    Net n;
    n.W1 = p;
    n.b1 = n.W1 + kHid * kIn;
    n.W2 = n.b1 + kHid;
    n.b2 = n.W2 + kHid * kHid;
    n.W3 = n.b2 + kHid;
    n.b3 = n.W3 + n_out * kHid;
    return n;
}

__device__ __forceinline__ bool is_log_feature(int j) { return j <= 5 || j == 9; }

// One workgroup of 64 threads per feature row.
__global__ __launch_bounds__(64) void k_mlp_infer(const float *__restrict__ params, int n_out,
                                                  const float *__restrict__ mean,
                                                  const float *__restrict__ stdv,
                                                  const float *__restrict__ raw,
                                                  float *__restrict__ scores) {
    __shared__ float z[kIn];
    __shared__ float h1[kHid];
    __shared__ float h2[kHid];
    const Net net = unpack(params, n_out);
    const int t = threadIdx.x;
    const int64_t row = blockIdx.x;
    if (t < kIn) {
        float g = raw[row * kIn + t];
        if (is_log_feature(t)) g = log1pf(fmaxf(g, 0.0f));
        z[t] = (g - mean[t]) / stdv[t];
    }
    __syncthreads();
    float a = net.b1[t];
    for (int k = 0; k < kIn; ++k) a = fmaf(net.W1[t * kIn + k], z[k], a);
    h1[t] = fmaxf(a, 0.0f);
    __syncthreads();
    a = net.b2[t];
    for (int k = 0; k < kHid; ++k) a = fmaf(net.W2[t * kHid + k], h1[k], a);
    h2[t] = fmaxf(a, 0.0f);
    __syncthreads();
    if (t < n_out) {
        a = net.b3[t];
        for (int k = 0; k < kHid; ++k) a = fmaf(net.W3[t * kHid + k], h2[k], a);
        scores[row * n_out + t] = a;
    }
}

// Forward pass of kBatchRows samples by one workgroup, and (BWD) their part of
// the backward pass: one launch where a launch per layer spent its time on
// launch gaps (a batch of 256 is 4 MFLOP).  The weights sit in LDS with rows
// padded to 65 (13) floats, so that neither the forward's walk along a row
// per lane nor the backward's walk along a column per lane meets a bank
// twice; a wave holds one sample, so activations are LDS broadcasts.
//
// BWD leaves h1, h2, the unscaled output residuals ds = mask (s - t), their
// images d2 and d1 at the two hidden layers (ReLU masked) and, per workgroup,
// the sum of ds^2 and the mask count; k_mlp_grad applies 2 / count to the
// finished sums, so no pass over the batch has to wait for the count.
// Measured, batch 256: forward, loss and input gradients 6 launches and
// 51 us -> one launch of 7 us (GPU time, MI355X).
constexpr int kBatchRows = 8;
constexpr int kMaxOut = SPMV_K_COUNT;
constexpr int kPadH = kHid + 1, kPadI = kIn + 1;

template <bool BWD>
__global__ __launch_bounds__(256) void k_mlp_rows(
    const float *__restrict__ params, int n_out, const float *__restrict__ x, int64_t B,
    float *__restrict__ scores, const float *__restrict__ target,
    const float *__restrict__ mask, float *__restrict__ gh1, float *__restrict__ gh2,
    float *__restrict__ gds, float *__restrict__ gd2, float *__restrict__ gd1,
    float *__restrict__ sums) {
    __shared__ float w1[kHid * kPadI], w2[kHid * kPadH], w3[kMaxOut * kPadH];
    __shared__ float xs[kBatchRows * kIn], h1[kBatchRows * kHid], h2[kBatchRows * kHid];
    __shared__ float ds[kBatchRows * kMaxOut], cs[kBatchRows * kMaxOut], d2[kBatchRows * kHid];
    const Net net = unpack(params, n_out);
    const int t = threadIdx.x;
    const int64_t row0 = (int64_t)blockIdx.x * kBatchRows;
    const int rows = (int)(B - row0 < kBatchRows ? B - row0 : kBatchRows);
#pragma unroll
    for (int q = 0; q < kHid * kHid / 256; ++q) {
        const int i = t + q * 256;
        w2[(i >> 6) * kPadH + (i & 63)] = net.W2[i];
    }
#pragma unroll
    for (int q = 0; q < kHid * kIn / 256; ++q) {
        const int i = t + q * 256;
        w1[i / kIn * kPadI + i % kIn] = net.W1[i];
    }
    for (int i = t; i < n_out * kHid; i += 256) w3[(i >> 6) * kPadH + (i & 63)] = net.W3[i];
    if (t < rows * kIn) xs[t] = x[row0 * kIn + t];
    const int j = t & (kHid - 1);
    const float b1 = net.b1[j], b2 = net.b2[j];
    __syncthreads();
    for (int r = t / kHid; r < rows; r += 256 / kHid) {
        float a = b1;
#pragma unroll
        for (int k = 0; k < kIn; ++k) a = fmaf(w1[j * kPadI + k], xs[r * kIn + k], a);
        a = fmaxf(a, 0.0f);
        h1[r * kHid + j] = a;
        if constexpr (BWD) gh1[(row0 + r) * kHid + j] = a;
    }
    __syncthreads();
    for (int r = t / kHid; r < rows; r += 256 / kHid) {
        float a = b2;
#pragma unroll
        for (int k = 0; k < kHid; ++k) a = fmaf(w2[j * kPadH + k], h1[r * kHid + k], a);
        a = fmaxf(a, 0.0f);
        h2[r * kHid + j] = a;
        if constexpr (BWD) gh2[(row0 + r) * kHid + j] = a;
    }
    __syncthreads();
    if (t < rows * n_out) {
        const int r = t / n_out, o = t - r * n_out;
        float a = net.b3[o];
#pragma unroll
        for (int k = 0; k < kHid; ++k) a = fmaf(w3[o * kPadH + k], h2[r * kHid + k], a);
        if constexpr (!BWD) {
            scores[row0 * n_out + t] = a;
        } else {
            const bool on = mask[row0 * n_out + t] > 0.0f;
            const float d = on ? a - target[row0 * n_out + t] : 0.0f;
            ds[t] = d;
            cs[t] = on ? 1.0f : 0.0f;
            gds[row0 * n_out + t] = d;
        }
    }
    if constexpr (BWD) {
        __syncthreads();
        if (t >= 192) {   // one wave, in a fixed order
            float l = 0.0f, c = 0.0f;
            for (int i = j; i < rows * n_out; i += 64) {
                l = fmaf(ds[i], ds[i], l);
                c += cs[i];
            }
            for (int off = 32; off > 0; off >>= 1) {
                l += __shfl_xor(l, off);
                c += __shfl_xor(c, off);
            }
            if (j == 0) {
                sums[2 * blockIdx.x] = l;
                sums[2 * blockIdx.x + 1] = c;
            }
        }
        for (int r = t / kHid; r < rows; r += 256 / kHid) {
            float a = 0.0f;
            for (int o = 0; o < n_out; ++o) a = fmaf(ds[r * n_out + o], w3[o * kPadH + j], a);
            a = h2[r * kHid + j] > 0.0f ? a : 0.0f;
            d2[r * kHid + j] = a;
            gd2[(row0 + r) * kHid + j] = a;
        }
        __syncthreads();
        for (int r = t / kHid; r < rows; r += 256 / kHid) {
            float a = 0.0f;
#pragma unroll
            for (int k = 0; k < kHid; ++k) a = fmaf(d2[r * kHid + k], w2[k * kPadH + j], a);
            gd1[(row0 + r) * kHid + j] = h1[r * kHid + j] > 0.0f ? a : 0.0f;
        }
    }
}

// Weight and bias gradients of all three layers in one launch:
//   gW[j, k] = scale sum_b d[b, j] in[b, k],  gb[j] = scale sum_b d[b, j],
// scale = 2 / max(1, mask count).  The sums over the batch are contractions,
// so they run on the matrix cores in float32 (v_mfma_f32_16x16x4_f32, four
// samples a step): a workgroup takes a 16 x 16 tile of one layer's gW, its
// 16 waves the samples in steps of four, 16 steps apart, kGradAhead steps of
// loads issued before any is used; the wave tiles are added in wave order.
// The bias is the same product with a column of ones.  The sums were one
// thread's serial walk over the batch, bound by one load's latency after
// the other: 57 us a layer at batch 256 (three launches, 171 us); with 8 loads
// in flight per lane on the vector units 4.6 us for all three but 125 us at
// batch 4096 (18 workgroups behind their scalar loads); so 4.0 and 20 us.
constexpr int kGradWaves = 16, kGradTile = 16, kGradStep = 4, kGradAhead = 4;

__global__ __launch_bounds__(64 * kGradWaves) void k_mlp_grad(
    int64_t B, int n_out, const float *__restrict__ x, const float *__restrict__ h1,
    const float *__restrict__ h2, const float *__restrict__ ds, const float *__restrict__ d2,
    const float *__restrict__ d1, const float *__restrict__ sums, int64_t nsums,
    float *__restrict__ grad, float *__restrict__ loss) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    __shared__ float red[kGradWaves][kGradTile * kGradTile];
    __shared__ float redb[kGradWaves][kGradTile];
    __shared__ float total[2];
    constexpr int T = kHid / kGradTile;   // tiles along a hidden dimension
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane % kGradTile, ls = lane / kGradTile;   // tile index, sample of the step
    const int blk = (int)blockIdx.x;
    const float *d, *in;
    float *gW, *gb;
    int nin, nout, j0, k0;
    Net g = unpack(grad, n_out);
    if (blk < T * T) {
        d = d2, in = h1, nin = kHid, nout = kHid, j0 = blk / T * kGradTile, k0 = blk % T * kGradTile;
        gW = (float *)g.W2, gb = (float *)g.b2;
    } else if (blk < T * T + T) {
        d = d1, in = x, nin = kIn, nout = kHid, j0 = (blk - T * T) * kGradTile, k0 = 0;
        gW = (float *)g.W1, gb = (float *)g.b1;
    } else {
        d = ds, in = h2, nin = kHid, nout = n_out, j0 = 0, k0 = (blk - T * T - T) * kGradTile;
        gW = (float *)g.W3, gb = (float *)g.b3;
    }
    const bool jon = j0 + li < nout, kon = k0 + li < nin;
    const float *dp = d + j0 + li, *ip = in + k0 + li;
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, accb = acc;
    for (int64_t b0 = (int64_t)wave * kGradStep + ls; b0 - ls < B;
         b0 += kGradWaves * kGradStep * kGradAhead) {
        float dv[kGradAhead], iv[kGradAhead];
#pragma unroll
        for (int u = 0; u < kGradAhead; ++u) {
            const int64_t b = b0 + u * (kGradWaves * kGradStep);
            dv[u] = b < B && jon ? dp[b * nout] : 0.0f;
            iv[u] = b < B && kon ? ip[b * nin] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kGradAhead; ++u) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[u], iv[u], acc, 0, 0, 0);
            accb = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[u], 1.0f, accb, 0, 0, 0);
        }
    }
    // accumulator r of a lane is tile row 4 (lane / 16) + r, column lane % 16
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        red[wave][(4 * ls + r) * kGradTile + li] = acc[r];
        if (li == 0) redb[wave][4 * ls + r] = accb[r];
    }
    // squared residuals and mask count over the workgroups of k_mlp_rows, in
    // a fixed order (the count is a whole number, exact below 2^24)
    if (wave < 2) {
        float s = 0.0f;
        for (int64_t i = lane; i < nsums; i += 64) s += sums[2 * i + wave];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) total[wave] = s;
    }
    __syncthreads();
    const float cnt = fmaxf(total[1], 1.0f);
    if (blk == 0 && threadIdx.x == 0) *loss = total[0] / cnt;
    const int t = threadIdx.x;
    if (t < kGradTile * kGradTile) {
        const int j = j0 + t / kGradTile, k = k0 + t % kGradTile;
        if (j < nout && k < nin) {
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < kGradWaves; ++w) s += red[w][t];
            gW[j * nin + k] = 2.0f * s / cnt;
        }
    } else if (t < kGradTile * kGradTile + kGradTile && k0 == 0) {
        const int c = t - kGradTile * kGradTile;
        if (j0 + c < nout) {
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < kGradWaves; ++w) s += redb[w][c];
            gb[j0 + c] = 2.0f * s / cnt;
        }
    }
}
static_assert(kMaxOut <= kGradTile && kIn <= kGradTile, "one tile of outputs, one of inputs");

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float beta1, float beta2,
                       float eps, float c1, float c2) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    float gi = g[i];
    float mi = beta1 * m[i] + (1.0f - beta1) * gi;
    float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    float mhat = mi / c1, vhat = vi / c2;
    p[i] -= lr * mhat / (sqrtf(vhat) + eps);
}

inline unsigned blocks(int64_t work, int bs) { return (unsigned)((work + bs - 1) / bs); }

// The caller's workspace: activations and residuals of every sample, then
// the per-workgroup sums (two floats for every kBatchRows samples, where
// spmv_mlp_workspace_floats leaves SPMV_K_COUNT floats per sample).
struct Work {
    float *h1, *h2, *ds, *d2, *d1, *sums;
};

inline Work carve(float *ws, int64_t B, int n_out) {
    Work w;
    w.h1 = ws;
    w.h2 = w.h1 + B * kHid;
    w.ds = w.h2 + B * kHid;
    w.d2 = w.ds + B * n_out;
    w.d1 = w.d2 + B * kHid;
    w.sums = w.d1 + B * kHid;
    return w;
}

}  // namespace

spmv_status run_mlp_infer(const float *params, int n_out, const float *mean, const float *stdv,
                          const float *raw, int64_t rows, float *scores, hipStream_t s) {
    if (rows == 0) return SPMV_OK;
    k_mlp_infer<<<(unsigned)rows, 64, 0, s>>>(params, n_out, mean, stdv, raw, scores);
    SMAT_LAUNCHED("mlp_infer");
    return SPMV_OK;
}

}  // namespace smat

using namespace smat;

extern "C" int64_t spmv_mlp_param_count(int32_t n_out) {
    return (int64_t)kHid * kIn + kHid + (int64_t)kHid * kHid + kHid + (int64_t)n_out * kHid + n_out;
}

extern "C" int64_t spmv_mlp_workspace_floats(int64_t batch) {
    return batch * (4 * kHid + 2 * SPMV_K_COUNT) + 64;
}

extern "C" spmv_status spmv_mlp_forward(const float *params_dev, int32_t n_out, const float *x_dev,
                                        int64_t batch, float *scores_dev, float *workspace_dev,
                                        void *stream) {
    if (!params_dev || !x_dev || !scores_dev || !workspace_dev || batch < 0 || n_out <= 0 ||
        n_out > SPMV_K_COUNT) {
        set_error("spmv_mlp_forward: bad argument");
        return SPMV_EINVAL;
    }
    if (batch == 0) return SPMV_OK;
    k_mlp_rows<false><<<blocks(batch, kBatchRows), 256, 0, (hipStream_t)stream>>>(
        params_dev, n_out, x_dev, batch, scores_dev, nullptr, nullptr, nullptr, nullptr, nullptr,
        nullptr, nullptr, nullptr);
    SMAT_LAUNCHED("mlp_forward");
    return SPMV_OK;
}

extern "C" spmv_status spmv_mlp_backward(const float *params_dev, int32_t n_out, const float *x_dev,
                                         const float *target_dev, const float *mask_dev,
                                         int64_t batch, float *grad_dev, float *loss_dev,
                                         float *workspace_dev, void *stream) {
    if (!params_dev || !x_dev || !target_dev || !mask_dev || !grad_dev || !loss_dev ||
        !workspace_dev || batch <= 0 || n_out <= 0 || n_out > SPMV_K_COUNT) {
        set_error("spmv_mlp_backward: bad argument");
        return SPMV_EINVAL;
    }
    hipStream_t s = (hipStream_t)stream;
    Work w = carve(workspace_dev, batch, n_out);
    const unsigned nrows = blocks(batch, kBatchRows);
    k_mlp_rows<true><<<nrows, 256, 0, s>>>(params_dev, n_out, x_dev, batch, nullptr, target_dev,
                                           mask_dev, w.h1, w.h2, w.ds, w.d2, w.d1, w.sums);
    SMAT_LAUNCHED("mlp_rows");
    constexpr unsigned kT = kHid / kGradTile;
    const unsigned ngrad = kT * kT + 2 * kT;   // tiles of gW2, gW1 and gW3
    k_mlp_grad<<<ngrad, 64 * kGradWaves, 0, s>>>(batch, n_out, x_dev, w.h1, w.h2, w.ds, w.d2,
                                                 w.d1, w.sums, nrows, grad_dev, loss_dev);
    SMAT_LAUNCHED("mlp_backward");
    return SPMV_OK;
}

extern "C" spmv_status spmv_mlp_adam(float *params_dev, const float *grad_dev, float *adam_m_dev,
                                     float *adam_v_dev, int64_t n_params, int32_t step, float lr,
                                     float beta1, float beta2, float eps, void *stream) {
    if (!params_dev || !grad_dev || !adam_m_dev || !adam_v_dev || n_params < 0 || step < 1) {
        set_error("spmv_mlp_adam: bad argument");
        return SPMV_EINVAL;
    }
    if (n_params == 0) return SPMV_OK;
    float c1 = (float)(1.0 - pow((double)beta1, (double)step));
    float c2 = (float)(1.0 - pow((double)beta2, (double)step));
    k_adam<<<blocks(n_params, 256), 256, 0, (hipStream_t)stream>>>(
        params_dev, grad_dev, adam_m_dev, adam_v_dev, n_params, lr, beta1, beta2, eps, c1, c2);
    SMAT_LAUNCHED("mlp_adam");
    return SPMV_OK;
}
