// Training of the block-feature selector network on the device: targets,
// feature standardisation, forward pass, backpropagation and Adam (Kingma
// and Ba).  Not part of compression or decompression; the network it
// produces is used by the selector mode of the compressor.  Activations,
// gradients of 16 samples and Adam are fp32; the sums over a minibatch's
// workgroups, the losses and the feature statistics are double.  All run in a
// fixed order, so a run is repeatable on one device, but training is not meant
// to be bit-exact across machines (a given parameter set is).
#include "fz_common.h"
#include "fz_kernels.h"

namespace fz {

namespace {
constexpr int kW1 = 2 * kNFeat, kB1 = kW1 + kNHid * kNFeat, kW2 = kB1 + kNHid, kB2 = kW2 + kNHid * kNHid,
              kW3 = kB2 + kNHid, kB3 = kW3 + kNOut * kNHid;
static_assert(kB3 + kNOut == kSelectorParams, "selector layout");
}  // namespace

// t = log2(1 + bits) per sample and predictor
__global__ void k_targets(const uint32_t* __restrict__ costs, uint64_t n, float* __restrict__ t) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 3 * n; i += (uint64_t)gridDim.x * blockDim.x)
        t[i] = log2f(1.0f + (float)costs[i]);
}

// Mean and standard deviation of each feature over the samples: mu and
// rs = 1 / std (1 where the feature is constant) to w.  Memory-latency
// bound (64 B per sample, a few MB): every workgroup sums a strided share
// of whole rows (thread = feature t % 16 of a row, so a wave reads 256
// contiguous bytes), in double, and leaves its 32 sums to the one workgroup
// of k_feature_stats, which adds them in a fixed order.  32768 samples:
// 7.4 us for both (60 us with one workgroup per feature, each reading every
// row).
__global__ __launch_bounds__(256) void k_feature_sums(const float* __restrict__ feat, uint64_t n,
                                                      double* __restrict__ part) {
    __shared__ double s1[256], s2[256];
    const uint32_t t = threadIdx.x, f = t & (kNFeat - 1);
    double a = 0.0, b = 0.0;
    for (uint64_t i = (uint64_t)blockIdx.x * 16 + (t >> 4); i < n; i += (uint64_t)gridDim.x * 16) {
        const double v = feat[i * kNFeat + f];
        a += v;
        b += v * v;
    }
    s1[t] = a;
    s2[t] = b;
    __syncthreads();
    for (uint32_t h = 128; h >= (uint32_t)kNFeat; h >>= 1) {
        if (t < h) {
            s1[t] += s1[t + h];
            s2[t] += s2[t + h];
        }
        __syncthreads();
    }
    if (t < (uint32_t)kNFeat) {
        part[blockIdx.x * 2 * kNFeat + t] = s1[t];
        part[blockIdx.x * 2 * kNFeat + kNFeat + t] = s2[t];
    }
}

__global__ __launch_bounds__(256) void k_feature_stats(const double* __restrict__ part, uint32_t parts, uint64_t n,
                                                       float* __restrict__ w) {
    __shared__ double r[256];
    const uint32_t t = threadIdx.x, f = t % (2 * kNFeat);
    double a = 0.0;
#pragma unroll 4
    for (uint32_t k = t / (2 * kNFeat); k < parts; k += 8) a += part[k * 2 * kNFeat + f];
    r[t] = a;
    __syncthreads();
    for (uint32_t h = 128; h >= (uint32_t)(2 * kNFeat); h >>= 1) {
        if (t < h) r[t] += r[t + h];
        __syncthreads();
    }
    if (t >= (uint32_t)kNFeat) return;
    const double m = r[t] / (double)n;
    double var = r[kNFeat + t] / (double)n - m * m;
    if (var < 0.0) var = 0.0;
    const double sd = sqrt(var);
    w[t] = (float)m;
    w[kNFeat + t] = sd > 1e-12 ? (float)(1.0 / sd) : 1.0f;
}

// Forward pass, backpropagation and weight gradients of a minibatch in one
// kernel.  A workgroup of four waves takes 16 samples at a time; every
// product of a layer with those samples is a 16 x 16 tile per wave (wave =
// 16 units) on the fp32 matrix instruction 16x16x4, whose operands are
// fp32 and whose sums are fp32 chains.  The network sits in registers in
// operand layout, loaded once per workgroup together with the first
// samples; the activations and deltas pass through LDS (rows of 68 floats:
// 16-byte reads of consecutive rows fall into different banks).  The
// gradient of the workgroup's samples stays in the accumulators and goes to
// its own row of `part`; k_train_reduce adds the rows.
//
// At a batch of 1024 the step is latency-bound (64 workgroups, 15 k
// multiply-adds per sample), hence 16 samples per workgroup, one tile.
// Measured per step of 1024: one thread per sample and then one thread per
// parameter over the whole batch 580 us (weight gradients 491, forward 54,
// backward 35: 4 to 22 workgroups); this split with vector instructions
// and the weights in LDS 16.3 us; this kernel 6.4 us.
//
// Operand layouts (lane l, q = l / 16, u = l % 16): A[row u][k], B[k][column
// u] with one k per q; D[row 4 q + r][column u] in register r.  Which k a
// lane group takes in which of the products is free as long as A and B
// agree: k = 16 q + i where a row is read along k (16 bytes at a time),
// k = 4 i + q otherwise.
typedef float f32x4v __attribute__((ext_vector_type(4)));
constexpr int kRow = kNHid + 4, kZRow = kNFeat + 4;

__device__ __forceinline__ f32x4v mfma4(float a, float b, f32x4v c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__global__ __launch_bounds__(256) void k_train_step(const float* __restrict__ w, const float* __restrict__ feat,
                                                    const float* __restrict__ tgt, const uint32_t* __restrict__ idx,
                                                    uint32_t B, float* __restrict__ part) {
    __shared__ __align__(16) float Z[kTrainTile * kZRow], H1[kTrainTile * kRow], H2[kTrainTile * kRow],
        D1[kTrainTile * kRow], D2[kTrainTile * kRow];
    __shared__ __align__(16) float DY[kTrainTile * 4];
    __shared__ float SE[4];
    const uint32_t t = threadIdx.x, wv = t >> 6, q = (t >> 4) & 3, u = t & 15;
    const uint32_t j = 16 * wv + u;  // this lane's unit (column of D)
    // sample and feature this thread standardises; sample and four units of
    // the output layer
    const uint32_t sl = t >> 4, fi = t & 15;
    const float mu = w[fi], rs = w[kNFeat + fi];
    float w1[4], w2f[16], w2b[16], w3[kNOut];
#pragma unroll
    for (int i = 0; i < 4; i++) w1[i] = w[kW1 + j * kNFeat + 4 * q + i];
#pragma unroll
    for (int i = 0; i < 16; i++) {
        w2f[i] = w[kW2 + j * kNHid + 16 * q + i];    // row of unit j
        w2b[i] = w[kW2 + (16 * q + i) * kNHid + j];  // column of unit j
    }
    float4 w3o[kNOut];
    float b3[kNOut];
#pragma unroll
    for (int o = 0; o < kNOut; o++) {
        w3[o] = w[kW3 + o * kNHid + j];
        const float* r = w + kW3 + o * kNHid + 4 * fi;
        w3o[o] = make_float4(r[0], r[1], r[2], r[3]);
        b3[o] = w[kB3 + o];
    }
    const float b1 = w[kB1 + j], b2 = w[kB2 + j];

    const f32x4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4v g2[4] = {zero, zero, zero, zero}, g1 = zero;
    float g3[kNOut] = {}, gb1 = 0.0f, gb2 = 0.0f, gb3 = 0.0f, se = 0.0f;
    const uint32_t ntiles = (B + kTrainTile - 1) / kTrainTile;
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        // a sample past the batch is all zero and gets no delta
        const uint32_t s = tile * kTrainTile + sl;
        const bool in = s < B;
        const uint64_t k = in ? (idx ? idx[s] : s) : 0;
        const float zf = in ? (feat[k * kNFeat + fi] - mu) * rs : 0.0f;
        float tg[kNOut];
#pragma unroll
        for (int o = 0; o < kNOut; o++) tg[o] = in ? tgt[k * kNOut + o] : 0.0f;
        __syncthreads();  // the previous tile's reads are done
        Z[sl * kZRow + fi] = zf;
        __syncthreads();
        // hidden layers: D[sample 4 q + r][unit j]
        f32x4v h1 = {b1, b1, b1, b1}, h2 = {b2, b2, b2, b2};
        {
            const float4 x = *reinterpret_cast<const float4*>(&Z[u * kZRow + 4 * q]);
            h1 = mfma4(x.x, w1[0], h1);
            h1 = mfma4(x.y, w1[1], h1);
            h1 = mfma4(x.z, w1[2], h1);
            h1 = mfma4(x.w, w1[3], h1);
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {
            h1[r] = h1[r] > 0.0f ? h1[r] : 0.0f;
            H1[(4 * q + r) * kRow + j] = h1[r];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float4 x = *reinterpret_cast<const float4*>(&H1[u * kRow + 16 * q + 4 * i]);
            h2 = mfma4(x.x, w2f[4 * i], h2);
            h2 = mfma4(x.y, w2f[4 * i + 1], h2);
            h2 = mfma4(x.z, w2f[4 * i + 2], h2);
            h2 = mfma4(x.w, w2f[4 * i + 3], h2);
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {
            h2[r] = h2[r] > 0.0f ? h2[r] : 0.0f;
            H2[(4 * q + r) * kRow + j] = h2[r];
        }
        __syncthreads();
        {
            // outputs: 16 lanes per sample, 4 units each
            const float4 h = *reinterpret_cast<const float4*>(&H2[sl * kRow + 4 * fi]);
#pragma unroll
            for (int o = 0; o < kNOut; o++) {
                float r = w3o[o].x * h.x;
                r = __builtin_fmaf(w3o[o].y, h.y, r);
                r = __builtin_fmaf(w3o[o].z, h.z, r);
                r = __builtin_fmaf(w3o[o].w, h.w, r);
#pragma unroll
                for (int d = 8; d > 0; d >>= 1) r += __shfl_xor(r, d, 16);
                const float e = in ? r + b3[o] - tg[o] : 0.0f;
                if (fi == 0) {
                    se = __builtin_fmaf(e, e, se);
                    DY[sl * 4 + o] = 2.0f * e / (3.0f * (float)B);
                }
            }
            if (fi == 0) DY[sl * 4 + 3] = 0.0f;
        }
        __syncthreads();
        // dh2 = (dy W3) where h2 > 0
        f32x4v d2, d1 = zero;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const float4 dy = *reinterpret_cast<const float4*>(&DY[(4 * q + r) * 4]);
            float d = dy.x * w3[0];
            d = __builtin_fmaf(dy.y, w3[1], d);
            d = __builtin_fmaf(dy.z, w3[2], d);
            d2[r] = h2[r] > 0.0f ? d : 0.0f;
            D2[(4 * q + r) * kRow + j] = d2[r];
            gb2 += d2[r];
            // (a sample past the batch has activations too, of the biases
            // alone: where they overflow, 0 times them would be no number)
            const float a2 = tile * kTrainTile + 4 * q + r < B ? h2[r] : 0.0f;
            g3[0] = __builtin_fmaf(dy.x, a2, g3[0]);
            g3[1] = __builtin_fmaf(dy.y, a2, g3[1]);
            g3[2] = __builtin_fmaf(dy.z, a2, g3[2]);
            // lanes 0..2 of wave 0's groups: the output biases
            gb3 += u == 0 ? dy.x : (u == 1 ? dy.y : dy.z);
        }
        __syncthreads();
        // dh1 = (dh2 W2) where h1 > 0
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float4 x = *reinterpret_cast<const float4*>(&D2[u * kRow + 16 * q + 4 * i]);
            d1 = mfma4(x.x, w2b[4 * i], d1);
            d1 = mfma4(x.y, w2b[4 * i + 1], d1);
            d1 = mfma4(x.z, w2b[4 * i + 2], d1);
            d1 = mfma4(x.w, w2b[4 * i + 3], d1);
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {
            d1[r] = h1[r] > 0.0f ? d1[r] : 0.0f;
            D1[(4 * q + r) * kRow + j] = d1[r];
            gb1 += d1[r];
        }
        // dW2 rows 16 wv .., all columns: A = delta^T, B = activations,
        // k = sample
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float x = D2[(4 * i + q) * kRow + j];
#pragma unroll
            for (int c = 0; c < 4; c++) g2[c] = mfma4(x, H1[(4 * i + q) * kRow + 16 * c + u], g2[c]);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; i++) g1 = mfma4(D1[(4 * i + q) * kRow + j], Z[(4 * i + q) * kZRow + u], g1);
    }
    // sums over the lane groups (each holds 4 of a tile's 16 samples)
    auto over_q = [](float v) {
        v += __shfl_xor(v, 16, 64);
        return v + __shfl_xor(v, 32, 64);
    };
    gb1 = over_q(gb1);
    gb2 = over_q(gb2);
    gb3 = over_q(gb3);
#pragma unroll
    for (int o = 0; o < kNOut; o++) g3[o] = over_q(g3[o]);
    float* P = part + (uint64_t)blockIdx.x * kTrainRow;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const uint32_t row = 16 * wv + 4 * q + r;
#pragma unroll
        for (int c = 0; c < 4; c++) P[kW2 + row * kNHid + 16 * c + u] = g2[c][r];
        P[kW1 + row * kNFeat + u] = g1[r];
    }
    if (q == 0) {
        P[kB1 + j] = gb1;
        P[kB2 + j] = gb2;
#pragma unroll
        for (int o = 0; o < kNOut; o++) P[kW3 + o * kNHid + j] = g3[o];
        if (wv == 0 && u < (uint32_t)kNOut) P[kB3 + u] = gb3;
    }
    if (t < (uint32_t)kW1) P[t] = 0.0f;  // mu, rs: set from the data, not learned
    // squared errors of the workgroup's samples
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) se += __shfl_xor(se, d, 64);
    if ((t & 63) == 0) SE[wv] = se;
    __syncthreads();
    if (t == 0) P[kSelectorParams] = (SE[0] + SE[1]) + (SE[2] + SE[3]);
}

// Adam on one learned parameter.
__device__ __forceinline__ void adam_update(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                                            uint32_t p, float gp, float lr, float b1, float b2, float eps, float c1,
                                            float c2) {
    const float mp = b1 * m[p] + (1.0f - b1) * gp;
    const float vp = b2 * v[p] + (1.0f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    w[p] -= lr * (mp / c1) / (sqrtf(vp / c2) + eps);
}

// Sums of the workgroups' gradient rows, in double, in row order within
// eight slices and then over the slices; the loss (sum of the squared errors / (3 B));
// with A.m also the Adam step.  Thread = (parameter, slice), so that a row
// of 64 workgroups is eight loads per thread, all in flight: latency-bound
// (2.9 us).
constexpr int kRedParams = 32, kRedSlices = 8;
__global__ __launch_bounds__(256) void k_train_reduce(const float* __restrict__ part, uint32_t rows, uint32_t B,
                                                      float* __restrict__ grad, float* __restrict__ loss,
                                                      double* __restrict__ loss_sum, TrainAdam A, float c1, float c2) {
    __shared__ double r[kRedSlices][kRedParams];
    const uint32_t t = threadIdx.x, q = t % kRedParams, sl = t / kRedParams;
    const uint32_t p = blockIdx.x * kRedParams + q;
    double acc = 0.0;
    if (p <= (uint32_t)kSelectorParams) {
        const uint32_t per = (rows + kRedSlices - 1) / kRedSlices;
        const uint32_t k0 = sl * per, k1 = min(rows, k0 + per);
#pragma unroll 8
        for (uint32_t k = k0; k < k1; k++) acc += part[(uint64_t)k * kTrainRow + p];
    }
    r[sl][q] = acc;
    __syncthreads();
    if (sl != 0 || p > (uint32_t)kSelectorParams) return;
    acc = ((r[0][q] + r[1][q]) + (r[2][q] + r[3][q])) + ((r[4][q] + r[5][q]) + (r[6][q] + r[7][q]));
    if (p == (uint32_t)kSelectorParams) {
        const double l = acc / (3.0 * (double)B);
        if (loss) *loss = (float)l;
        if (loss_sum) *loss_sum += l;
        return;
    }
    const float gp = (float)acc;
    grad[p] = gp;
    if (A.m && p >= (uint32_t)kW1) adam_update(A.w, A.m, A.v, p, gp, A.lr, A.b1, A.b2, A.eps, c1, c2);
}

// Adam on the learned parameters; step number t >= 1.
__global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, float lr, float b1, float b2, float eps, float c1, float c2) {
    const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < (uint32_t)kW1 || p >= (uint32_t)kSelectorParams) return;
    adam_update(w, m, v, p, g[p], lr, b1, b2, eps, c1, c2);
}

void launch_targets(hipStream_t st, const uint32_t* costs, uint64_t n, float* t) {
    uint64_t grid = (3 * n + 255) / 256;
    if (grid > 4096) grid = 4096;
    if (grid) hipLaunchKernelGGL(k_targets, dim3((uint32_t)grid), dim3(256), 0, st, costs, n, t);
}

// w is followed by the scratch of the partial sums (kTrainWBytes).
void launch_feature_stats(hipStream_t st, const float* feat, uint64_t n, float* w) {
    uint64_t parts = (n + 127) / 128;
    if (parts > kFeatureParts) parts = kFeatureParts;
    double* part = reinterpret_cast<double*>(w + kTrainRow);
    hipLaunchKernelGGL(k_feature_sums, dim3((uint32_t)parts), dim3(256), 0, st, feat, n, part);
    hipLaunchKernelGGL(k_feature_stats, dim3(1), dim3(256), 0, st, part, (uint32_t)parts, n, w);
}

void launch_train_batch(hipStream_t st, const float* w, const float* feat, const float* tgt, const uint32_t* idx,
                        uint32_t B, TrainScratch& s, float* loss_out) {
    const uint32_t rows = train_rows(B);
    float c1 = 1.0f, c2 = 1.0f;
    if (s.adam.m) {
        c1 = 1.0f - powf(s.adam.b1, (float)s.adam.t);
        c2 = 1.0f - powf(s.adam.b2, (float)s.adam.t);
    }
    hipLaunchKernelGGL(k_train_step, dim3(rows), dim3(256), 0, st, w, feat, tgt, idx, B, s.Z);
    hipLaunchKernelGGL(k_train_reduce, dim3((kSelectorParams + kRedParams) / kRedParams), dim3(256), 0, st, s.Z, rows,
                       B, s.grad, loss_out, s.loss_sum, s.adam, c1, c2);
}

void launch_adam(hipStream_t st, float* w, float* m, float* v, const float* g, int t, float lr, float b1, float b2,
                 float eps) {
    const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3((kSelectorParams + 255) / 256), dim3(256), 0, st, w, m, v, g, lr, b1, b2, eps,
                       c1, c2);
}

}  // namespace fz
