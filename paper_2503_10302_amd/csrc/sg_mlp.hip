// sg_mlp.hip -- FP32 kernels of the ladder-predictor network
// (4 -> 64 -> 64 -> 33, ReLU; outputs: log beta_0, softplus increments of
// log beta_1..31, log ICM cutoff).  Tiny dense layers: plain VALU arithmetic, one
// 64-lane work-group per sample, no matrix cores.  A training step of 64 samples is two
// launches, 73 -> 12 us (before: one lane summed the outputs, every work-group wrote a whole
// gradient to memory, and the host waited for each step's loss).
#include <algorithm>
#include <mutex>

#include "sg_internal.h"

namespace sg {

constexpr int NI = 4, NH = 64, NO = 33;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NH * NI, OFF_W2 = OFF_B1 + NH;
constexpr int OFF_B2 = OFF_W2 + NH * NH, OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NO * NH;
constexpr int NPARAM = OFF_B3 + NO;   // 6625; then mean[4], std[4]

__device__ __forceinline__ float softplus_f(float x) { return x > 20.f ? x : log1pf(expf(x)); }
__device__ __forceinline__ float sigmoid_f(float x) { return 1.f / (1.f + expf(-x)); }

// What the gradient needs of one sample, in floats: a one (the biases' activation), the
// standardised features, the activations, the deltas and the squared errors.
constexpr int R_ONE = 0, R_XS = 1, R_A1 = 8, R_A2 = R_A1 + NH, R_DZ1 = R_A2 + NH, R_DZ2 = R_DZ1 + NH;
constexpr int R_DO = R_DZ2 + NH, R_D2 = R_DO + 40;
static_assert(R_D2 + NO <= kMlpRecFloats, "record size");

// The values v of lanes 0 .. N - 1 of a one-wave work-group in every lane (through LDS, read four
// at a time).
template <int N>
__device__ __forceinline__ void share(float *buf, float v, float (&o)[N])
{
    __syncthreads();
    buf[threadIdx.x] = v;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; k += 4) {
        const float4 r = *(const float4 *)(buf + k);
        o[k] = r.x;
        if (k + 1 < N) o[k + 1] = r.y;
        if (k + 2 < N) o[k + 2] = r.z;
        if (k + 3 < N) o[k + 3] = r.w;
    }
}

// Forward (and, with y != null, backward to the deltas) over samples [s0, s1) of a batch of
// `batch`, one wave per sample in turn; the weights, both their rows and columns, are loaded
// once into registers, so a sample is one chain of dependent multiplies and adds (what bounds
// it).  rec: [s1 - s0] records (with y), out: [.][NO]
// network outputs.  Every sum runs in the order of its index (the values do not depend on how
// the samples are spread over work-groups).
__global__ __launch_bounds__(64) void mlp_sample_kernel(const float *P, const float *x, const float *y,
                                                        const int *idx, int batch, int s0, int s1,
                                                        float *rec, float *out)
{
    __shared__ __align__(16) float buf[NH];
    const int i = threadIdx.x;
    const int io = min(i, NO - 1);   // lanes past the outputs repeat the last one
    // the first sample's loads go ahead of the weights'
    int sm = s0 + blockIdx.x;
    int b = sm < s1 ? (idx ? idx[sm] : sm) : 0;
    float xin = x[(size_t)b * NI + (i & 3)], t = y ? y[(size_t)b * NO + io] : 0.f;
    float w1[NI], w2[NH], w3[NH], w2c[NH], w3c[NO];
#pragma unroll
    for (int k = 0; k < NI; ++k) w1[k] = P[OFF_W1 + i * NI + k];
#pragma unroll
    for (int k = 0; k < NH; k += 4) {
        const float4 r = *(const float4 *)(P + OFF_W2 + i * NH + k);
        const float4 q = *(const float4 *)(P + OFF_W3 + io * NH + k);
        w2[k] = r.x; w2[k + 1] = r.y; w2[k + 2] = r.z; w2[k + 3] = r.w;
        w3[k] = q.x; w3[k + 1] = q.y; w3[k + 2] = q.z; w3[k + 3] = q.w;
    }
    if (y) {
#pragma unroll
        for (int o = 0; o < NO; ++o) w3c[o] = P[OFF_W3 + o * NH + i];
#pragma unroll
        for (int o = 0; o < NH; ++o) w2c[o] = P[OFF_W2 + o * NH + i];
    }
    const float b1 = P[OFF_B1 + i], b2 = P[OFF_B2 + i], b3 = P[OFF_B3 + io];
    const float mean = P[NPARAM + (i & 3)], sd = P[NPARAM + NI + (i & 3)];
    for (; sm < s1; sm += gridDim.x) {
        if (sm != s0 + (int)blockIdx.x) {
            b = idx ? idx[sm] : sm;
            xin = x[(size_t)b * NI + (i & 3)];
            if (y) t = y[(size_t)b * NO + io];
        }
        const float xs = (xin - mean) / sd;
        float xv[NI], h[NH], ov[NO];
        share(buf, xs, xv);
        float z1 = b1;
#pragma unroll
        for (int k = 0; k < NI; ++k) z1 += w1[k] * xv[k];
        const float a1 = z1 > 0.f ? z1 : 0.f;
        share(buf, a1, h);
        float z2 = b2;
#pragma unroll
        for (int k = 0; k < NH; ++k) z2 += w2[k] * h[k];
        const float a2 = z2 > 0.f ? z2 : 0.f;
        share(buf, a2, h);
        float os = b3;
#pragma unroll
        for (int k = 0; k < NH; ++k) os += w3[k] * h[k];
        // log betas: the running sum of the first output and the softplus increments
        const float inc = i >= 1 && i < 32 ? softplus_f(os) : os;
        share(buf, inc, ov);
        float ys = ov[0];
#pragma unroll
        for (int k = 1; k < 32; ++k) {
            const float v = ys + ov[k];
            ys = k <= i ? v : ys;
        }
        if (i >= 32) ys = os;
        if (out && i < NO) out[(size_t)b * NO + i] = ys;
        if (!y) continue;
        // dL/dy = 2 (y - t) / (B * 33); back through the cumulative softplus
        const float d = ys - t;
        const float dy = 2.f * d / (float)(batch * NO);
        share(buf, dy, ov);
        float suffix = 0.f;   // sum of dy_j over 31 >= j >= max(i, 1)
#pragma unroll
        for (int k = 31; k >= 1; --k) {
            const float v = suffix + ov[k];
            suffix = k >= i ? v : suffix;
        }
        float dO = i >= 1 && i < 32 ? sigmoid_f(os) * suffix : suffix + dy;
        if (i >= 32) dO = dy;
        share(buf, dO, ov);
        float da2 = 0.f;
#pragma unroll
        for (int o = 0; o < NO; ++o) da2 += ov[o] * w3c[o];
        const float dz2 = a2 > 0.f ? da2 : 0.f;
        share(buf, dz2, h);
        float da1 = 0.f;
#pragma unroll
        for (int o = 0; o < NH; ++o) da1 += h[o] * w2c[o];
        const float dz1 = a1 > 0.f ? da1 : 0.f;
        float *R = rec + (size_t)(sm - s0) * kMlpRecFloats;
        if (i == 0) R[R_ONE] = 1.f;
        if (i < NI) R[R_XS + i] = xs;
        R[R_A1 + i] = a1;
        R[R_A2 + i] = a2;
        R[R_DZ1 + i] = dz1;
        R[R_DZ2 + i] = dz2;
        if (i < NO) {
            R[R_DO + i] = dO;
            R[R_D2 + i] = d * d;
        }
    }
}

// Gradient of the samples [s0, s1) from their records, one parameter per thread: per group of
// `per` samples a sum in sample order, the groups' sums added in group order (acc[0], acc[1]: the
// present group's sum and the sum of those before, carried when a batch takes several launches).
// The last work-group sums the squared errors the same way, one group per thread.  At the end of
// the batch (s1 == batch) the gradient goes to grad (nullable) and, with lr > 0, into an Adam
// step (Kingma & Ba, bias correction c1, c2).  The records of a minibatch stay in L2: the kernel
// is bound by the latency of a few rounds of their loads (64 in flight per thread: 4.5 us per 64 samples; 7.4 us with 32).
__global__ __launch_bounds__(64) void mlp_grad_kernel(const float *rec, int batch, int per, int s0, int s1,
                                                      float *acc, float *loss, float *grad, float *P,
                                                      float *m, float *v, float lr, float b1, float b2,
                                                      float eps, float c1, float c2)
{
    constexpr int ST = kMlpRecFloats;
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x >= (unsigned)batch) return;   // at most one group per sample
        const int64_t g0 = (int64_t)threadIdx.x * per;
        if (g0 >= batch) {   // the last groups may be empty
            loss[threadIdx.x] = 0.f;
            return;
        }
        const int l0 = (int)g0, l1 = (int)min((int64_t)batch, g0 + per);
        float s = l0 >= s0 ? 0.f : loss[threadIdx.x];
        for (int sm = max(l0, s0); sm < min(l1, s1); ++sm)
#pragma unroll
            for (int k = 0; k < NO; ++k) s += rec[(size_t)(sm - s0) * ST + R_D2 + k];
        if (l0 < s1 && l1 > s0) loss[threadIdx.x] = s;
        return;
    }
    const int p = blockIdx.x * 64 + threadIdx.x;
    if (p >= NPARAM) return;
    int od, oa;   // places of the parameter's delta and activation in a record
    if (p < OFF_B1) { od = R_DZ1 + p / NI; oa = R_XS + p % NI; }
    else if (p < OFF_W2) { od = R_DZ1 + (p - OFF_B1); oa = R_ONE; }
    else if (p < OFF_B2) { od = R_DZ2 + (p - OFF_W2) / NH; oa = R_A1 + (p - OFF_W2) % NH; }
    else if (p < OFF_W3) { od = R_DZ2 + (p - OFF_B2); oa = R_ONE; }
    else if (p < OFF_B3) { od = R_DO + (p - OFF_W3) / NH; oa = R_A2 + (p - OFF_W3) % NH; }
    else { od = R_DO + (p - OFF_B3); oa = R_ONE; }
    float g = 0.f, s = 0.f;
    if (s0 > 0) {
        g = acc[p];
        s = acc[NPARAM + p];
    }
    // the optimiser's state goes ahead of the records
    const float P0 = lr > 0.f ? P[p] : 0.f, m0 = lr > 0.f ? m[p] : 0.f, v0 = lr > 0.f ? v[p] : 0.f;
    int left = per - s0 % per;   // samples until the present group ends
    constexpr int U = 32;
    const float *R = rec;
    for (int sm = s0; sm < s1; sm += U, R += U * ST) {
        float d[U], f[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = min(u, s1 - 1 - sm);   // past the end: the last record again
            d[u] = R[q * ST + od];
            f[u] = R[q * ST + oa];
        }
        if (per == 1) {   // a group is one sample
#pragma unroll
            for (int u = 0; u < U; ++u) s = sm + u < s1 ? s + (0.f + d[u] * f[u]) : s;
            continue;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (sm + u >= s1) break;
            g += d[u] * f[u];
            if (--left == 0) {
                s += g;
                g = 0.f;
                left = per;
            }
        }
    }
    if (s1 < batch) {
        acc[p] = g;
        acc[NPARAM + p] = s;
        return;
    }
    if (left != per) s += g;   // the last, shorter group
    if (grad) grad[p] = s;
    if (lr > 0.f) {
        const float mp = b1 * m0 + (1.f - b1) * s;
        const float vp = b2 * v0 + (1.f - b2) * s * s;
        m[p] = mp;
        v[p] = vp;
        P[p] = P0 - lr * (mp / c1) / (sqrtf(vp / c2) + eps);
    }
}

hipError_t launch_mlp_forward(const float *P, const float *x, int n, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(mlp_sample_kernel, dim3(n < 1024 ? n : 1024), dim3(64), 0, s, P, x,
                       (const float *)nullptr, (const int *)nullptr, n, 0, n, (float *)nullptr, out);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(float *P, const float *x, const float *y, const int *idx, int batch,
                           const MlpWork &w, float *loss, float *grad, const MlpAdam *adam, hipStream_t s)
{
    const int nblk = batch < kMlpGroups ? batch : kMlpGroups;
    const int per = (int)(((int64_t)batch + nblk - 1) / nblk);
    MlpAdam a{};
    float c1 = 1.f, c2 = 1.f;
    if (adam) {
        a = *adam;
        c1 = 1.f - powf(a.b1, (float)a.step);
        c2 = 1.f - powf(a.b2, (float)a.step);
    }
    // records of at most w.chunk samples at a time
    for (int s0 = 0; s0 < batch;) {
        const int s1 = (int)std::min<int64_t>(batch, (int64_t)s0 + w.chunk), n = s1 - s0;
        hipLaunchKernelGGL(mlp_sample_kernel, dim3(n < 1024 ? n : 1024), dim3(64), 0, s, P, x, y, idx, batch,
                           s0, s1, w.rec, (float *)nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(mlp_grad_kernel, dim3((NPARAM + 63) / 64 + 1), dim3(64), 0, s, w.rec, batch, per,
                           s0, s1, w.acc, loss, grad, P, a.m, a.v, a.lr, a.b1, a.b2, a.eps, c1, c2);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        s0 = s1;
    }
    return hipSuccess;
}

// Device memory of the allocation-free prediction entry point: the staging area of the
// network inputs (raw features, [kPredictMax][NI]) followed by the network outputs
// ([kPredictMax][NO]).  One copy per GPU, held until the process ends.  In host code the
// name below is only a stand-in: every host-side use goes through the address that
// hipGetSymbolAddress returns for the current device (mlp_scratch).
static __device__ __align__(256) float scratch[kPredictMax * (NI + NO)];
static_assert(kPredictScratchFloats == kPredictMax * (NI + NO), "scratch layout");

namespace {
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t mlp_scratch(float **p)
{
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *a = nullptr;
        e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = (float *)a;
    }
    *p = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace sg
