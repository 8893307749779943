// mlp.hip -- the per-pair degree model on the GPU: inference with the
// (type, degree) choice, and the forward/backward/Adam kernels that train it.
//
// Model: 4 -> 64 -> 64 -> 11 (tanh hidden layers, linear output = predicted
// log10 pair error at degrees 2..12), FP32.  Parameter layout in degree.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <string>

#include "degree.hpp"
#include "engine.hpp"

namespace bldtt {
namespace {

constexpr int kBlock = 256;

[[noreturn]] void throw_launch(hipError_t e, const char* where) {
    throw Error(-3, std::string("HIP launch failed in ") + where + ": " + hipGetErrorString(e));
}
#define CHECK_LAUNCH()                                      \
    do {                                                    \
        hipError_t e_ = hipGetLastError();                  \
        if (e_ != hipSuccess) throw_launch(e_, __func__);   \
    } while (0)

__device__ __forceinline__ void normalise(const float* __restrict__ M, const float* f, float* x) {
    const float* mean = M + kNParams;
    const float* scale = mean + kNIn;
#pragma unroll
    for (int k = 0; k < kNIn; ++k) x[k] = (f[k] - mean[k]) * scale[k];
}

// tanh(s) = sign(s) (1 - e^{-2|s|}) / (1 + e^{-2|s|}), branch free from the
// hardware 2^x and reciprocal (absolute error ~1e-7; exactly +-1 once e^{-2|s|}
// underflows).
__device__ __forceinline__ float fast_tanh(float s) {
    const float t = __builtin_amdgcn_exp2f(-2.8853900817779268f * fabsf(s));
    return copysignf((1.0f - t) * __builtin_amdgcn_rcpf(1.0f + t), s);
}

// The model in LDS: all lanes read the same weight at once (a broadcast), and
// the 20 KB of weights would not stay in the scalar cache.
__device__ __forceinline__ const float* stage_model(const float* __restrict__ M, float* sM) {
    for (int k = threadIdx.x; k < kNModel; k += kBlock) sM[k] = M[k];
    __syncthreads();
    return sM;
}

// Forward pass of one sample.
__device__ __forceinline__ void forward(const float* __restrict__ M, const float* x, float* y) {
    float h1[kNHid];
#pragma unroll
    for (int o = 0; o < kNHid; ++o) {
        float s = M[kOffB1 + o];
#pragma unroll
        for (int k = 0; k < kNIn; ++k) s = fmaf(M[kOffW1 + o * kNIn + k], x[k], s);
        h1[o] = fast_tanh(s);
    }
#pragma unroll
    for (int k = 0; k < kNOut; ++k) y[k] = M[kOffB3 + k];
    for (int j = 0; j < kNHid; ++j) {
        float s = M[kOffB2 + j];
#pragma unroll
        for (int i = 0; i < kNHid; ++i) s = fmaf(M[kOffW2 + j * kNHid + i], h1[i], s);
        float a = fast_tanh(s);
#pragma unroll
        for (int k = 0; k < kNOut; ++k) y[k] = fmaf(M[kOffW3 + k * kNHid + j], a, y[k]);
    }
}

// Separated-pair type for degree d (Algorithm 2): CC when both clusters hold
// more than (d+1)^3 particles, CP / PC when only the target / source does, PP otherwise.
__device__ __forceinline__ int sep_type(int64_t ct, int64_t cs, int d, int pp_cc_only) {
    const int64_t np = (int64_t)(d + 1) * (d + 1) * (d + 1);
    if (ct > np && cs > np) return 3;
    if (pp_cc_only) return 0;
    if (ct > np) return 2;
    if (cs > np) return 1;
    return 0;
}

__device__ __forceinline__ double pair_cost(int type, int64_t ct, int64_t cs, int d) {
    const double np = (double)(d + 1) * (d + 1) * (d + 1);
    if (type == 3) return np * np;
    if (type == 2) return np * (double)cs;
    if (type == 1) return (double)ct * np;
    return (double)ct * (double)cs;
}

// Inference and choice: the cheapest (type, degree) whose predicted error is at
// most tau, with direct evaluation (PP) always a candidate.  Pairs whose
// geometric features fall outside the training range use the fallback degree.
__global__ __launch_bounds__(kBlock) void k_mlp_select(const float* __restrict__ M, const float* __restrict__ feats,
                                                       const int64_t* __restrict__ counts, int64_t n, float log_tau,
                                                       int fallback, int pp_cc_only, uint8_t* __restrict__ choice) {
    __shared__ float sM[kNModel];
    M = stage_model(M, sM);
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    const int64_t ct = counts[2 * p], cs = counts[2 * p + 1];
    float f[kNIn];
#pragma unroll
    for (int k = 0; k < kNIn; ++k) f[k] = feats[kNIn * p + k];
    const float* lo = M + kNParams + 2 * kNIn;
    const float* hi = lo + kNIn;
    bool in_range = true;
#pragma unroll
    for (int k = 0; k < 2; ++k) in_range = in_range && f[k] >= lo[k] && f[k] <= hi[k];
#pragma unroll
    for (int k = 2; k < kNIn; ++k) f[k] = fminf(fmaxf(f[k], lo[k]), hi[k]);   // counts: clamp
    if (!in_range) {
        choice[p] = (uint8_t)(sep_type(ct, cs, fallback, pp_cc_only) << 4 | fallback);
        return;
    }
    float x[kNIn], y[kNOut];
    normalise(M, f, x);
    forward(M, x, y);
    int best_t = 0, best_d = 0;
    double best = pair_cost(0, ct, cs, 0);
    for (int d = kDegMin; d <= kDegMax; ++d) {
        if (!(y[d - kDegMin] <= log_tau)) continue;
        int t = sep_type(ct, cs, d, pp_cc_only);
        double c = pair_cost(t, ct, cs, d);
        if (c < best) {
            best = c;
            best_t = t;
            best_d = d;
        }
    }
    choice[p] = (uint8_t)(best_t << 4 | best_d);
}

__global__ __launch_bounds__(kBlock) void k_mlp_forward(const float* __restrict__ M, const float* __restrict__ feats,
                                                        int64_t n, float* __restrict__ out) {
    __shared__ float sM[kNModel];
    M = stage_model(M, sM);
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    float f[kNIn], x[kNIn], y[kNOut];
#pragma unroll
    for (int k = 0; k < kNIn; ++k) f[k] = feats[kNIn * p + k];
    normalise(M, f, x);
    forward(M, x, y);
#pragma unroll
    for (int k = 0; k < kNOut; ++k) out[kNOut * p + k] = y[k];
}

// ---------------------------------------------------------------------------
// Loss and gradient of a batch in two launches.
//
// k_grad_part: a work group runs forward and backward of kGradSamples samples at
// a time with the weights and every activation in LDS, and adds the samples'
// contributions to the 5195 parameters' gradients in its registers (thread
// (wave w, lane i) owns dW2[16 w .. 16 w + 15][i]), which it writes once at its
// end.  Wave w holds samples 2 w, 2 w + 1, lane j the hidden unit j; W2 rows are
// padded to 65 floats, so a row read across lanes and a column read both touch
// every bank.  k_grad_finish adds the groups' partials in group order and
// divides by the number of valid targets (and takes the Adam step when asked).
//
// Bound by latency: 10 MFLOP at 1024 samples, a few us of dependent LDS reads and
// barriers per group.  Five kernels before (activations through memory, one
// thread per parameter over every sample in turn, 260 us of it at 1024
// samples) took 330 us, these two 15 us: a call 382 -> 49 us.
// ---------------------------------------------------------------------------
constexpr int kGradSamples = 8;                        // samples per round of a work group
constexpr int kGradGroups = 208;                       // work groups at most
constexpr int kGradPart = kNParams + 2;                // gradient sums, squared errors, valid targets (bits)
constexpr int kW2Pitch = kNHid + 1;

__global__ __launch_bounds__(kBlock) void k_grad_part(const float* __restrict__ M, const float* __restrict__ feats,
                                                      const float* __restrict__ tgt, int64_t n,
                                                      float* __restrict__ part) {
    constexpr int S = kGradSamples;
    static_assert(kBlock == 4 * kNHid && S == 8 && kNOut * S <= kBlock, "one wave per two samples, one lane per unit");
    __shared__ float W1[kNHid * kNIn], B1[kNHid], W2[kNHid * kW2Pitch], B2[kNHid], W3[kNOut * kNHid], B3[kNOut];
    __shared__ float X[S][kNIn];
    __shared__ float A1[kNHid][S], A2[kNHid][S], Z2[kNHid][S], Z1[kNHid][S], dY[kNOut][S];
    __shared__ float red[kBlock];
    __shared__ unsigned redn[kBlock];
    const int t = threadIdx.x, wave = t >> 6, j = t & 63;
    for (int k = t; k < kNHid * kNIn; k += kBlock) W1[k] = M[kOffW1 + k];
    for (int k = t; k < kNHid * kNHid; k += kBlock) W2[(k >> 6) * kW2Pitch + (k & 63)] = M[kOffW2 + k];
    for (int k = t; k < kNOut * kNHid; k += kBlock) W3[k] = M[kOffW3 + k];
    if (t < kNHid) {
        B1[t] = M[kOffB1 + t];
        B2[t] = M[kOffB2 + t];
    }
    if (t < kNOut) B3[t] = M[kOffB3 + t];
    float g2[16], g3[3], g1 = 0.f, gb = 0.f, sq = 0.f;
    unsigned valid = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) g2[k] = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) g3[k] = 0.f;
    const int s0 = 2 * wave;
    for (int64_t b = (int64_t)blockIdx.x * S; b < n; b += (int64_t)gridDim.x * S) {
        __syncthreads();                                   // the last round's readers are done
        if (t < S) {
            float x[kNIn] = {0.f, 0.f, 0.f, 0.f};          // past the last sample: any finite value
            if (b + t < n) {
                float f[kNIn];
#pragma unroll
                for (int k = 0; k < kNIn; ++k) f[k] = feats[kNIn * (b + t) + k];
                normalise(M, f, x);
            }
#pragma unroll
            for (int k = 0; k < kNIn; ++k) X[t][k] = x[k];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float s = B1[j];
#pragma unroll
            for (int k = 0; k < kNIn; ++k) s = fmaf(W1[j * kNIn + k], X[s0 + q][k], s);
            A1[j][s0 + q] = fast_tanh(s);
        }
        __syncthreads();
        {
            float u = B2[j], v = u;
#pragma unroll 16
            for (int i = 0; i < kNHid; ++i) {
                const float w = W2[j * kW2Pitch + i];
                u = fmaf(w, A1[i][s0], u);
                v = fmaf(w, A1[i][s0 + 1], v);
            }
            A2[j][s0] = fast_tanh(u);
            A2[j][s0 + 1] = fast_tanh(v);
        }
        __syncthreads();
        if (t < kNOut * S) {                               // output o of sample c; twice its error, 0 for NaN targets
            const int o = t >> 3, c = t & 7;
            float y = B3[o];
#pragma unroll 16
            for (int i = 0; i < kNHid; ++i) y = fmaf(W3[o * kNHid + i], A2[i][c], y);
            float d = 0.f;
            if (b + c < n) {
                const float want = tgt[kNOut * (b + c) + o];
                if (!isnan(want)) {
                    d = y - want;
                    ++valid;
                }
            }
            sq = fmaf(d, d, sq);
            dY[o][c] = 2.f * d;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {                      // dZ2 = (W3^T dY) (1 - A2^2)
            float s = 0.f;
#pragma unroll
            for (int o = 0; o < kNOut; ++o) s = fmaf(W3[o * kNHid + j], dY[o][s0 + q], s);
            const float a = A2[j][s0 + q];
            Z2[j][s0 + q] = s * (1.f - a * a);
        }
        __syncthreads();
        {                                                  // dZ1 = (W2^T dZ2) (1 - A1^2), lane j the unit of layer 1
            float u = 0.f, v = 0.f;
#pragma unroll 16
            for (int i = 0; i < kNHid; ++i) {
                const float w = W2[i * kW2Pitch + j];
                u = fmaf(w, Z2[i][s0], u);
                v = fmaf(w, Z2[i][s0 + 1], v);
            }
            const float a = A1[j][s0], c = A1[j][s0 + 1];
            Z1[j][s0] = u * (1.f - a * a);
            Z1[j][s0 + 1] = v * (1.f - c * c);
        }
        __syncthreads();
        // the samples' products, in sample order
        float a1[S];
#pragma unroll
        for (int c = 0; c < S; ++c) a1[c] = A1[j][c];
#pragma unroll
        for (int k = 0; k < 16; ++k)
#pragma unroll
            for (int c = 0; c < S; ++c) g2[k] = fmaf(Z2[16 * wave + k][c], a1[c], g2[k]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int o = wave + 4 * k;                    // row o of W3, lane j its column
            if (o < kNOut)
#pragma unroll
                for (int c = 0; c < S; ++c) g3[k] = fmaf(dY[o][c], A2[j][c], g3[k]);
        }
#pragma unroll
        for (int c = 0; c < S; ++c) g1 = fmaf(Z1[t >> 2][c], X[c][t & 3], g1);
#pragma unroll
        for (int c = 0; c < S; ++c)
            gb += wave == 0 ? Z1[j][c] : (wave == 1 ? Z2[j][c] : (wave == 2 && j < kNOut ? dY[j < kNOut ? j : 0][c] : 0.f));
    }
    float* out = part + (int64_t)blockIdx.x * kGradPart;
    out[kOffW1 + t] = g1;
#pragma unroll
    for (int k = 0; k < 16; ++k) out[kOffW2 + (16 * wave + k) * kNHid + j] = g2[k];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (wave + 4 * k < kNOut) out[kOffW3 + (wave + 4 * k) * kNHid + j] = g3[k];
    if (wave == 0) out[kOffB1 + j] = gb;
    if (wave == 1) out[kOffB2 + j] = gb;
    if (wave == 2 && j < kNOut) out[kOffB3 + j] = gb;
    red[t] = sq;
    redn[t] = valid;
    __syncthreads();
    for (int k = kBlock / 2; k > 0; k >>= 1) {
        if (t < k) {
            red[t] += red[t + k];
            redn[t] += redn[t + k];
        }
        __syncthreads();
    }
    if (t == 0) {
        out[kNParams] = red[0];
        out[kNParams + 1] = __uint_as_float(redn[0]);
    }
}

// Adam state and constants of a training step (null parameters: gradient only).
struct AdamStep {
    float *p, *m, *v;
    float lr, b1, b2, eps, c1, c2;
};

// grad = the groups' sums in group order / valid targets (0 when none is valid), 64
// parameters per work group, each wave every fourth group; group 0 also writes
// the loss.
__global__ __launch_bounds__(kBlock) void k_grad_finish(const float* __restrict__ part, int groups,
                                                        float* __restrict__ grad, float* __restrict__ loss, AdamStep a) {
    __shared__ float red[4][kNHid];
    __shared__ float rsq[kBlock];
    __shared__ unsigned long long rn[kBlock];
    const int t = threadIdx.x, wave = t >> 6, q = blockIdx.x * 64 + (t & 63);
    rn[t] = t < groups ? __float_as_uint(part[(int64_t)t * kGradPart + kNParams + 1]) : 0u;
    rsq[t] = t < groups ? part[(int64_t)t * kGradPart + kNParams] : 0.f;
    float s = 0.f;
    if (q < kNParams)
#pragma unroll 8
        for (int b = wave; b < groups; b += 4) s += part[(int64_t)b * kGradPart + q];
    red[wave][t & 63] = s;
    __syncthreads();
    for (int k = kBlock / 2; k > 0; k >>= 1) {
        if (t < k) {
            rn[t] += rn[t + k];
            rsq[t] += rsq[t + k];
        }
        __syncthreads();
    }
    const float inv = rn[0] > 0 ? __fdiv_rn(1.0f, (float)rn[0]) : 0.0f;
    if (blockIdx.x == 0 && t == 0) *loss = rsq[0] * inv;
    if (wave > 0 || q >= kNParams) return;
    const float g = (((red[0][t] + red[1][t]) + red[2][t]) + red[3][t]) * inv;
    if (grad) grad[q] = g;
    if (a.p) {
        const float mi = a.b1 * a.m[q] + (1.f - a.b1) * g;
        const float vi = a.b2 * a.v[q] + (1.f - a.b2) * g * g;
        a.m[q] = mi;
        a.v[q] = vi;
        a.p[q] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
    }
}

// Work memory of bldtt_mlp_loss_grad_noalloc, one copy per GPU for the life of
// the process: the partial gradients of every work group.  Host code reaches
// it only through the address that hipGetSymbolAddress returns on each device.
constexpr int64_t kNoAllocSamples = 4096;
static __device__ __align__(256) float scratch[(int64_t)kGradGroups * kGradPart];

inline unsigned blocks(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

namespace {
int grad_groups(int64_t n) { return (int)std::min<int64_t>(kGradGroups, (n + kGradSamples - 1) / kGradSamples); }
}  // namespace

int64_t mlp_work_floats(int64_t batch) { return (int64_t)grad_groups(batch) * kGradPart; }

void launch_mlp_select(const float* model, const float* feats, const int64_t* counts, int64_t n, float log_tau,
                       int fallback, int pp_cc_only, uint8_t* choice, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_mlp_select, dim3(blocks(n)), dim3(kBlock), 0, st, model, feats, counts, n, log_tau, fallback,
                       pp_cc_only, choice);
    CHECK_LAUNCH();
}

void launch_mlp_forward(const float* model, const float* feats, int64_t n, float* out, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_mlp_forward, dim3(blocks(n)), dim3(kBlock), 0, st, model, feats, n, out);
    CHECK_LAUNCH();
}

namespace {
void enqueue_loss_grad(const float* model, const float* feats, const float* targets, int64_t n, float* work, float* grad,
                       float* loss, const AdamStep& step, hipStream_t st) {
    const int groups = grad_groups(n);
    hipLaunchKernelGGL(k_grad_part, dim3(groups), dim3(kBlock), 0, st, model, feats, targets, n, work);
    hipLaunchKernelGGL(k_grad_finish, dim3((kNParams + 63) / 64), dim3(kBlock), 0, st, (const float*)work, groups, grad,
                       loss, step);
    CHECK_LAUNCH();
}

// Device address of `scratch` per device, looked up once per device with that
// device current (each GPU holds its own copy at its own address).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch[kMaxDevices] = {};

float* scratch_on_current_device() {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) throw Error(-3, std::string("hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) throw Error(-5, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            throw Error(-3, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch[dev] = static_cast<float*>(ptr);
    }
    return g_scratch[dev];
}
}  // namespace

void launch_mlp_loss_grad(const float* model, const float* feats, const float* targets, int64_t n, float* work,
                          float* grad, float* loss, hipStream_t st) {
    if (n <= 0) return;
    enqueue_loss_grad(model, feats, targets, n, work, grad, loss, AdamStep{}, st);
}

void launch_mlp_step(float* model, const float* feats, const float* targets, int64_t n, float* work, float* loss, float* m,
                     float* v, float lr, float b1, float b2, float eps, int step, hipStream_t st) {
    if (n <= 0) return;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    enqueue_loss_grad(model, feats, targets, n, work, nullptr, loss, AdamStep{model, m, v, lr, b1, b2, eps, c1, c2}, st);
}

int64_t mlp_noalloc_max_samples() { return kNoAllocSamples; }

void launch_mlp_loss_grad_noalloc(const float* model, const float* feats, const float* targets, int64_t n, float* grad,
                                  float* loss, hipStream_t st) {
    if (n < 1 || n > kNoAllocSamples) throw Error(-1, "bldtt_mlp_loss_grad_noalloc: n must lie in [1, 4096]");
    enqueue_loss_grad(model, feats, targets, n, scratch_on_current_device(), grad, loss, AdamStep{}, st);
}

}  // namespace bldtt
