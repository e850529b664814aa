// mlp.hip -- the linking-length proposer: a 24 -> 64 -> 64 -> 1 ReLU network
// that predicts ln(l) of a node from 24 summary features.  Training kernels
// (fp32 forward, backward, Adam) and the node inference kernel (bf16 weights
// and activations, fp32 accumulation) are all here; nothing in this file
// decides a result of the method: a proposal only chooses the bracket that
// the exact counting step then verifies.
//
// Parameter layout (fp32, 5825 values): W1[64][24], b1[64], W2[64][64],
// b2[64], W3[64], b3[1].  Features are standardised with a per-feature mean
// and standard deviation kept beside the parameters.
#include "common.h"
#include "phase_common.h"

namespace rs {

constexpr int NIN = RS_NFEAT, NH = 64;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NH * NIN, OFF_W2 = OFF_B1 + NH,
              OFF_B2 = OFF_W2 + NH * NH, OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH,
              NPARAM = OFF_B3 + 1;
static_assert(NPARAM == 5825, "parameter count");

// Forward, and with GRAD the backward to every parameter, of a minibatch.
// What bounds it: 15552 multiply-adds per sample are little work (0.13 GFLOP
// at 4096 samples), so the time is the chain of layers and the launches.  A
// workgroup takes 32 samples, so that 4096 of them still spread over 128
// CUs; the layers and the weight gradients are fp32 matrix products
// (16x16x4 tiles, wavefront w owns hidden units 16w..16w+15), activations
// stay in LDS, each wavefront's weights in registers.  The parameter
// gradients are summed in the accumulators over a workgroup's samples and
// written once as a partial vector; k_mlp_reduce sums the partials in a
// fixed order in fp64, so the result does not depend on timing.  At 4096
// samples one training step took 1.23 ms with one thread per parameter
// summing the whole batch, and takes 17.6 us this way.
constexpr int MT = 32;             // samples per workgroup and pass
constexpr int SH = NH + 4;         // LDS strides: operand reads spread over the banks
constexpr int SX = NIN + 12;       // columns 24.. : 1 (bias gradient), then zeros
constexpr int MLP_MAX_BLOCKS = 512;

template <bool GRAD>
__global__ void __launch_bounds__(256)
k_mlp_batch(const float* __restrict__ p, const float* __restrict__ X,
            const float* __restrict__ T, int64_t n, float* __restrict__ Y,
            float* __restrict__ part, double* __restrict__ lpart) {
    __shared__ float sx[MT * SX], h1[MT * SH], h2[MT * SH], dh1[GRAD ? MT * SH : 1];
    __shared__ float w3[NH], sdy[MT];
    __shared__ double red[MT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lm = lane & 15, lk = lane >> 4;       // tile row or column, k offset
    const int n0 = 16 * wave;
    float w1r[NIN / 4], w2r[NH / 4], w2t[GRAD ? NH / 4 : 1];
#pragma unroll
    for (int k = 0; k < NIN / 4; k++) w1r[k] = p[OFF_W1 + (n0 + lm) * NIN + 4 * k + lk];
#pragma unroll
    for (int k = 0; k < NH / 4; k++) w2r[k] = p[OFF_W2 + (n0 + lm) * NH + 4 * k + lk];
    if constexpr (GRAD) {
#pragma unroll
        for (int k = 0; k < NH / 4; k++) w2t[k] = p[OFF_W2 + (4 * k + lk) * NH + n0 + lm];
    }
    const float bias1 = p[OFF_B1 + n0 + lm], bias2 = p[OFF_B2 + n0 + lm], bias3 = p[OFF_B3];
    if (tid < NH) w3[tid] = p[OFF_W3 + tid];
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 g1[2] = {zero, zero}, g2[4] = {zero, zero, zero, zero};
    float gw3 = 0.0f, gb2 = 0.0f, gb3 = 0.0f;       // lane = hidden unit (gw3, gb2)
    double lsum = 0.0;

    const int64_t tiles = (n + MT - 1) / MT;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t s0 = t * MT;
        const int rows = (int)(n - s0 < MT ? n - s0 : MT);
        __syncthreads();
        for (int q = tid; q < MT * SX; q += 256) {
            const int r = q / SX, c = q % SX;
            sx[q] = r >= rows ? 0.0f
                    : c < NIN ? X[(s0 + r) * NIN + c] : c == NIN ? 1.0f : 0.0f;
        }
        __syncthreads();
        // rows past the batch hold zero activations, so they add nothing
        for (int mt = 0; mt < MT / 16; mt++) {
            f32x4 acc = {bias1, bias1, bias1, bias1};
#pragma unroll
            for (int k = 0; k < NIN / 4; k++)
                acc = mfma_16x16x4(sx[(16 * mt + lm) * SX + 4 * k + lk], w1r[k], acc);
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int row = 16 * mt + 4 * lk + r;
                h1[row * SH + n0 + lm] = row < rows && acc[r] > 0.0f ? acc[r] : 0.0f;
            }
        }
        __syncthreads();
        for (int mt = 0; mt < MT / 16; mt++) {
            f32x4 acc = {bias2, bias2, bias2, bias2};
#pragma unroll
            for (int k = 0; k < NH / 4; k++)
                acc = mfma_16x16x4(h1[(16 * mt + lm) * SH + 4 * k + lk], w2r[k], acc);
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int row = 16 * mt + 4 * lk + r;
                h2[row * SH + n0 + lm] = row < rows && acc[r] > 0.0f ? acc[r] : 0.0f;
            }
        }
        __syncthreads();
        {   // output, eight lanes a sample
            const int s = tid >> 3, q = tid & 7;
            float y = 0.0f;
#pragma unroll
            for (int i = 0; i < NH / 8; i++) y = fmaf(w3[8 * i + q], h2[s * SH + 8 * i + q], y);
#pragma unroll
            for (int o = 1; o < 8; o <<= 1) y += __shfl_xor(y, o, 64);
            y += bias3;
            if (q == 0) {
                const bool in = s < rows;
                if constexpr (GRAD) {
                    const float d = in ? y - T[s0 + s] : 0.0f;
                    sdy[s] = 2.0f * d / (float)n;
                    red[s] = (double)d * (double)d;
                } else if (in) {
                    Y[s0 + s] = y;
                }
            }
        }
        if constexpr (GRAD) {
            __syncthreads();
            if (tid == 0)
                for (int s = 0; s < MT; s++) lsum += red[s];
            // gradients of the output layer, and h2 becomes its own gradient
#pragma unroll
            for (int i = 0; i < MT / 4; i++) {
                const int s = wave * (MT / 4) + i;
                const float dy = sdy[s], a = h2[s * SH + lane];
                const float d = a > 0.0f ? dy * w3[lane] : 0.0f;
                gw3 = fmaf(dy, a, gw3);
                gb2 += d;
                gb3 += dy;
                h2[s * SH + lane] = d;
            }
            __syncthreads();
            for (int mt = 0; mt < MT / 16; mt++) {
                f32x4 acc = zero;
#pragma unroll
                for (int k = 0; k < NH / 4; k++)
                    acc = mfma_16x16x4(h2[(16 * mt + lm) * SH + 4 * k + lk], w2t[k], acc);
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int o = (16 * mt + 4 * lk + r) * SH + n0 + lm;
                    dh1[o] = h1[o] > 0.0f ? acc[r] : 0.0f;
                }
            }
            // W2: rows of the gradient are output units, columns hidden ones
#pragma unroll
            for (int k = 0; k < MT / 4; k++) {
                const float b = h1[(4 * k + lk) * SH + n0 + lm];
#pragma unroll
                for (int mt = 0; mt < 4; mt++)
                    g2[mt] = mfma_16x16x4(h2[(4 * k + lk) * SH + 16 * mt + lm], b, g2[mt]);
            }
            __syncthreads();
            // W1 and b1 (the column of ones)
#pragma unroll
            for (int k = 0; k < MT / 4; k++) {
                const float a = dh1[(4 * k + lk) * SH + n0 + lm];
#pragma unroll
                for (int nt = 0; nt < 2; nt++)
                    g1[nt] = mfma_16x16x4(a, sx[(4 * k + lk) * SX + 16 * nt + lm], g1[nt]);
            }
        }
    }
    if constexpr (GRAD) {
        float* g = part + (int64_t)blockIdx.x * NPARAM;
#pragma unroll
        for (int nt = 0; nt < 2; nt++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int j = n0 + 4 * lk + r, i = 16 * nt + lm;
                if (i < NIN) g[OFF_W1 + j * NIN + i] = g1[nt][r];
                else if (i == NIN) g[OFF_B1 + j] = g1[nt][r];
            }
#pragma unroll
        for (int mt = 0; mt < 4; mt++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                g[OFF_W2 + (16 * mt + 4 * lk + r) * NH + n0 + lm] = g2[mt][r];
        __syncthreads();
        h1[tid] = gw3;                    // [wave][unit]
        h2[tid] = gb2;
        if (lane == 0) dh1[wave] = gb3;   // every lane holds its wavefront's sum
        __syncthreads();
        if (tid < NH) {
            g[OFF_W3 + tid] = (h1[tid] + h1[64 + tid]) + (h1[128 + tid] + h1[192 + tid]);
            g[OFF_B2 + tid] = (h2[tid] + h2[64 + tid]) + (h2[128 + tid] + h2[192 + tid]);
        }
        if (tid == 0) {
            g[OFF_B3] = (dh1[0] + dh1[1]) + (dh1[2] + dh1[3]);
            lpart[blockIdx.x] = lsum;
        }
    }
}

// Sum of the workgroups' partial gradients (fixed order, fp64), the loss, and
// with ADAM the parameter update.  64 parameters a workgroup, four lanes
// each: reading the partials is a chain of loads per lane, so it is cut in
// four and spread over 92 workgroups.
template <bool ADAM>
__global__ void __launch_bounds__(256)
k_mlp_reduce(const float* __restrict__ part, const double* __restrict__ lpart, int nb, int64_t n,
             float* __restrict__ grad, float* __restrict__ loss, float* __restrict__ p,
             float* __restrict__ m, float* __restrict__ v, float lr, float b1, float b2,
             float eps, float c1, float c2) {
    __shared__ double red[256];
    const int q = blockIdx.x * 64 + (threadIdx.x & 63), sl = threadIdx.x >> 6;
    double a = 0.0;
    if (q < NPARAM) {
#pragma unroll 8
        for (int b = sl; b < nb; b += 4) a += (double)part[(int64_t)b * NPARAM + q];
    }
    red[threadIdx.x] = a;
    __syncthreads();
    if (sl == 0 && q < NPARAM) {
        const int t = threadIdx.x;
        const float gq = (float)((red[t] + red[64 + t]) + (red[128 + t] + red[192 + t]));
        if constexpr (ADAM) {
            const float mq = b1 * m[q] + (1.0f - b1) * gq;
            const float vq = b2 * v[q] + (1.0f - b2) * gq * gq;
            m[q] = mq;
            v[q] = vq;
            const float mh = mq / c1, vh = vq / c2;
            p[q] -= lr * mh / (sqrtf(vh) + eps);
        } else {
            grad[q] = gq;
        }
    }
    if (blockIdx.x == 0) {
        __syncthreads();
        double l = 0.0;
        for (int b = threadIdx.x; b < nb; b += 256) l += lpart[b];
        red[threadIdx.x] = l;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss = (float)(red[0] / (double)n);
    }
}

// per-feature mean and standard deviation (one thread per feature)
__global__ void k_mlp_stats(const float* __restrict__ X, int64_t n, float* __restrict__ mean,
                            float* __restrict__ stdv) {
    int i = threadIdx.x;
    if (i >= NIN) return;
    double s = 0.0, s2 = 0.0;
    for (int64_t k = 0; k < n; k++) {
        double v = X[k * NIN + i];
        s += v;
        s2 += v * v;
    }
    double mu = n > 0 ? s / (double)n : 0.0;
    double var = n > 0 ? s2 / (double)n - mu * mu : 0.0;
    mean[i] = (float)mu;
    stdv[i] = var > 1e-12 ? (float)sqrt(var) : 1.0f;
}

__global__ void k_mlp_standardize(float* __restrict__ X, int64_t n, const float* __restrict__ mean,
                                  const float* __restrict__ stdv) {
    int64_t q = blockIdx.x * 256ll + threadIdx.x;
    if (q >= n * NIN) return;
    int i = (int)(q % NIN);
    X[q] = (X[q] - mean[i]) / stdv[i];
}

// ---------------------------------------------------------------------------
// node inference: bf16 weights and activations, fp32 accumulation
// ---------------------------------------------------------------------------

RS_DEV float bf16_round(float x) {
    // round to nearest even at 8 mantissa bits (finite inputs)
    uint32_t u = __float_as_uint(x);
    uint32_t lsb = (u >> 16) & 1u;
    u += 0x7fffu + lsb;
    return __uint_as_float(u & 0xffff0000u);
}

__global__ void __launch_bounds__(256)
k_mlp_infer(const float* __restrict__ model, int nv, const float* __restrict__ feat,
            float* __restrict__ out_ln_l) {
    __shared__ float w[NPARAM];
    __shared__ float mu[NIN], sd[NIN];
    const float* p = model + 2 * NIN;
    for (int i = threadIdx.x; i < NPARAM; i += 256) w[i] = bf16_round(p[i]);
    for (int i = threadIdx.x; i < NIN; i += 256) {
        mu[i] = model[i];
        sd[i] = model[NIN + i];
    }
    __syncthreads();
    int v = blockIdx.x * 256 + threadIdx.x;
    if (v >= nv) return;
    float x[NIN], h1[NH];
#pragma unroll
    for (int i = 0; i < NIN; i++) x[i] = bf16_round((feat[(int64_t)v * NIN + i] - mu[i]) / sd[i]);
    for (int j = 0; j < NH; j++) {
        float a = w[OFF_B1 + j];
#pragma unroll
        for (int i = 0; i < NIN; i++) a += w[OFF_W1 + j * NIN + i] * x[i];
        h1[j] = bf16_round(a > 0.0f ? a : 0.0f);
    }
    float y = w[OFF_B3];
    for (int j = 0; j < NH; j++) {
        float a = w[OFF_B2 + j];
        for (int i = 0; i < NH; i++) a += w[OFF_W2 + j * NH + i] * h1[i];
        y += w[OFF_W3 + j] * bf16_round(a > 0.0f ? a : 0.0f);
    }
    out_ln_l[v] = y;
}

int mlp_infer(const float* model_dev, int nv, const float* feat, float* out, hipStream_t st) {
    if (nv <= 0) return RS_OK;
    k_mlp_infer<<<(nv + 255) / 256, 256, 0, st>>>(model_dev, nv, feat, out);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// per-workgroup partial gradients and losses of one minibatch
static int mlp_partials(const float* params, const float* X, const float* T, int64_t n,
                        float** part, double** lpart, int* nb, hipStream_t st) {
    const int64_t tiles = (n + MT - 1) / MT;
    *nb = (int)(tiles < MLP_MAX_BLOCKS ? tiles : MLP_MAX_BLOCKS);
    Arena* ar;
    RS_TRY(arena_call_begin(1u << AR_MLP));   // only the standalone proposer entry points get here
    RS_TRY(arena_reserve(AR_MLP, arena_round(4 * (size_t)NPARAM * *nb) + arena_round(8 * *nb),
                         &ar));
    *part = take<float>(ar, (size_t)NPARAM * *nb);
    *lpart = take<double>(ar, *nb);
    if (!*lpart) return RS_EINTERNAL;
    k_mlp_batch<true><<<*nb, 256, 0, st>>>(params, X, T, n, nullptr, *part, *lpart);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

}  // namespace rs

extern "C" {

int rs_mlp_forward(const float* params, const float* X, int64_t n, float* y, void* stream) {
    if (!params || (n > 0 && (!X || !y)) || n < 0) return RS_EINVAL;
    if (n == 0) return RS_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t tiles = (n + rs::MT - 1) / rs::MT;
    rs::k_mlp_batch<false><<<(unsigned)(tiles < 4096 ? tiles : 4096), 256, 0, st>>>(
        params, X, nullptr, n, y, nullptr, nullptr);
    RS_HIP(hipGetLastError());
    RS_HIP(hipStreamSynchronize(st));
    return RS_OK;
}

int rs_mlp_grad(const float* params, const float* X, const float* T, int64_t n, float* grad,
                float* loss, void* stream) {
    if (!params || !X || !T || !grad || !loss || n <= 0) return RS_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float* part;
    double* lpart;
    int nb;
    std::unique_lock<std::mutex> lk;
    RS_TRY(rs::call_lock(&lk));
    RS_TRY(rs::mlp_partials(params, X, T, n, &part, &lpart, &nb, st));
    rs::k_mlp_reduce<false><<<(rs::NPARAM + 63) / 64, 256, 0, st>>>(
        part, lpart, nb, n, grad, loss, nullptr, nullptr, nullptr, 0.0f, 0.0f, 0.0f, 0.0f, 1.0f,
        1.0f);
    RS_HIP(hipGetLastError());
    RS_HIP(hipStreamSynchronize(st));
    return RS_OK;
}

int rs_mlp_train_step(float* params, float* m, float* v, int64_t step, const float* X,
                      const float* T, int64_t n, float lr, float* loss, void* stream) {
    if (!params || !m || !v || !X || !T || !loss || n <= 0 || step < 1 || !(lr > 0.0f))
        return RS_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float* part;
    double* lpart;
    int nb;
    std::unique_lock<std::mutex> lk;
    RS_TRY(rs::call_lock(&lk));
    RS_TRY(rs::mlp_partials(params, X, T, n, &part, &lpart, &nb, st));
    const float b1 = 0.9f, b2 = 0.999f;
    float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    rs::k_mlp_reduce<true><<<(rs::NPARAM + 63) / 64, 256, 0, st>>>(
        part, lpart, nb, n, nullptr, loss, params, m, v, lr, b1, b2, 1e-8f, c1, c2);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

int rs_mlp_standardize(float* X, int64_t n, float* mean, float* stdv, int compute, void* stream) {
    if (!X || !mean || !stdv || n < 0) return RS_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (compute) rs::k_mlp_stats<<<1, 64, 0, st>>>(X, n, mean, stdv);
    if (n > 0)
        rs::k_mlp_standardize<<<(unsigned)((n * rs::NIN + 255) / 256), 256, 0, st>>>(X, n, mean,
                                                                                  stdv);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

int rs_mlp_infer(const float* model, int64_t n, const float* feat, float* out, void* stream) {
    if (!model || n < 0 || (n > 0 && (!feat || !out))) return RS_EINVAL;
    RS_TRY(rs::mlp_infer(model, (int)n, feat, out, static_cast<hipStream_t>(stream)));
    RS_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
    return RS_OK;
}

}  // extern "C"
