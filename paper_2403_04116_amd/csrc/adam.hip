// Radiation intensity response (Eq. 3) and the fused optimiser step.
//
// RIRF: intensity = sigmoid(w . f) per Gaussian, one thread per Gaussian.
//
// Adam: gradients of the activated parameters -> raw gradients (chain rule
// through exp / sigmoid / the response) -> Adam (bias-corrected moments,
// Kingma & Ba Algorithm 1) -> new raw parameters and the activated copies
// the next rendering reads.  HBM bound: about 28 bytes read and 16-20 written
// per scalar.
#include "common.h"

#include <math.h>

#include <algorithm>

namespace xg {

namespace {

__device__ __forceinline__ float sigmoidf(float x) { return 1.0f / (1.0f + expf(-x)); }

// Weights staged in LDS (at most XG_MAX_FEATURES).
__device__ __forceinline__ void load_weights(const float *w, int nf, float *s_w) {
    for (int k = threadIdx.x; k < nf; k += blockDim.x) s_w[k] = w[k];
    __syncthreads();
}

__device__ __forceinline__ float rirf_dot(const float *f, const float *s_w, int nf) {
    float acc = 0.0f;
    for (int k = 0; k < nf; ++k) acc = fmaf(s_w[k], f[k], acc);
    return acc;
}

__global__ __launch_bounds__(256) void k_rirf_fwd(const float *features, const float *weights,
                                                  int64_t n, int nf, float *intensity) {
    __shared__ float s_w[XG_MAX_FEATURES];
    load_weights(weights, nf, s_w);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    intensity[i] = sigmoidf(rirf_dot(features + i * nf, s_w, nf));
}

__global__ __launch_bounds__(256) void k_rirf_bwd(const float *features, const float *weights,
                                                  int64_t n, int nf, const float *dl_di,
                                                  float *grad_f) {
    __shared__ float s_w[XG_MAX_FEATURES];
    load_weights(weights, nf, s_w);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float s = sigmoidf(rirf_dot(features + i * nf, s_w, nf));
    const float g = dl_di[i] * s * (1.0f - s);
    float *gf = grad_f + i * nf;
    for (int k = 0; k < nf; ++k) gf[k] += g * s_w[k];
}

constexpr int64_t kAdamBlocks = 4096;   // 16 per CU (2048: 149 us where this takes 145)

struct AdamArgs {
    xg_params p;
    xg_grads g;
    float *m, *v;
    const int32_t *step;
    const int32_t *gate;    // nullable: nonzero skips the step
    xg_adam c;
    float b1, c1, b2, c2;   // beta and 1 - beta, each rounded once from double
    float *scales, *opacity, *intensity;
    int64_t n;
};

// Per-block step coefficients (bias corrections, position rate) in double
// from the device step counter; false when the gate skips the step.
__device__ __forceinline__ bool step_coefficients(const AdamArgs &a, float coef[3]) {
    __shared__ float s_coef[3];
    __shared__ int s_skip;
    if (threadIdx.x == 0) {
        s_skip = a.gate != nullptr && *a.gate != 0;
        const int t = *a.step + 1;
        const double f = (double)min(t - 1, a.c.lr_means_steps) / (double)max(a.c.lr_means_steps, 1);
        s_coef[0] = (float)(1.0 - pow(a.c.beta1, (double)t));
        s_coef[1] = (float)(1.0 - pow(a.c.beta2, (double)t));
        s_coef[2] = (float)exp((1.0 - f) * log((double)a.c.lr_means_start) +
                               f * log((double)a.c.lr_means_end));
    }
    __syncthreads();
    coef[0] = s_coef[0];
    coef[1] = s_coef[1];
    coef[2] = s_coef[2];
    return !s_skip;
}

// One scalar's new value; its moments are updated in place.
__device__ __forceinline__ float adam_value(const AdamArgs &a, float x, float grad, float lr, float bias1,
                                            float bias2, float &m, float &v) {
    m = a.b1 * m + a.c1 * grad;
    v = a.b2 * v + a.c2 * grad * grad;
    const float mhat = m / bias1;
    const float vhat = v / bias2;
    return x - lr * mhat / (sqrtf(vhat) + a.c.eps);
}

// Four consecutive floats at any 4-byte boundary: one 16-byte access (the
// moments of a group start at a multiple of n, of any parity).
struct __attribute__((packed, aligned(4))) Quad {
    float v[4];
};

// Quads of the scalar part: [means | log_scales | quats | opacity_logit],
// each group rounded up to whole quads.
struct AdamQuads {
    int64_t end[4];   // running quad counts
    __host__ __device__ AdamQuads(int64_t n) {
        end[0] = (3 * n + 3) / 4;
        end[1] = end[0] + (3 * n + 3) / 4;
        end[2] = end[1] + n;
        end[3] = end[2] + (n + 3) / 4;
    }
};

// `cnt` (1..4) consecutive scalars of one group.  KIND: 0 identity, 1 exp
// (scales), 2 sigmoid (opacity); k0: index of the first in the moments.
template <int KIND>
__device__ __forceinline__ void adam_quad(const AdamArgs &a, float *param, const float *grad, float *act, int64_t k0,
                                          int cnt, float lr, float bias1, float bias2) {
    Quad x, g, m, v, o;
    if (cnt == 4) {
        x = *reinterpret_cast<const Quad *>(param);
        g = *reinterpret_cast<const Quad *>(grad);
        m = *reinterpret_cast<const Quad *>(a.m + k0);
        v = *reinterpret_cast<const Quad *>(a.v + k0);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = i < cnt ? i : 0;
            x.v[i] = param[c];
            g.v[i] = grad[c];
            m.v[i] = a.m[k0 + c];
            v.v[i] = a.v[k0 + c];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // chain rule at the value the renderer used
        float gr = g.v[i];
        if (KIND == 1) {
            gr *= expf(x.v[i]);
        } else if (KIND == 2) {
            const float s = sigmoidf(x.v[i]);
            gr *= s * (1.0f - s);
        }
        x.v[i] = adam_value(a, x.v[i], gr, lr, bias1, bias2, m.v[i], v.v[i]);
        if (KIND == 1) o.v[i] = expf(x.v[i]);
        if (KIND == 2) o.v[i] = sigmoidf(x.v[i]);
    }
    if (cnt == 4) {
        *reinterpret_cast<Quad *>(param) = x;
        *reinterpret_cast<Quad *>(a.m + k0) = m;
        *reinterpret_cast<Quad *>(a.v + k0) = v;
        if (KIND) *reinterpret_cast<Quad *>(act) = o;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < cnt) {
                param[i] = x.v[i];
                a.m[k0 + i] = m.v[i];
                a.v[k0 + i] = v.v[i];
                if (KIND) act[i] = o.v[i];
            }
    }
}

// Sum over the G consecutive lanes of a group (G <= 16, in every lane).
template <int G>
__device__ __forceinline__ float group_sum(float x) {
#define XG_LANE_ADD(ctrl)                                                                                   \
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, true))
    if (G > 1) XG_LANE_ADD(0xB1);    // quad_perm: lane ^ 1
    if (G > 2) XG_LANE_ADD(0x4E);    // quad_perm: lane ^ 2
    if (G > 4) XG_LANE_ADD(0x141);   // row_half_mirror (the quads are even by now)
    if (G > 8) XG_LANE_ADD(0x128);   // row_ror:8
#undef XG_LANE_ADD
    return x;
}

// One launch for all raw parameters: the first `scalar_blocks` workgroups
// take the scalars of means, scales, quaternions and opacity, the others
// the feature vectors.  HBM bound; every lane moves quads of 16 bytes, so
// that few wavefronts keep enough bytes in flight, and a feature vector's
// inner products need G / 4 lanes and no LDS (G: its length rounded up to a
// power of two).  1M Gaussians, 16 features, 716 MB: 78 + 136 us as two
// launches of one scalar per lane -> 145 us.
//
// Features: lane k of a group owns features 4 k .. 4 k + 3; the response's
// chain rule at the current features, Adam on each, then the new intensity
// from the updated features.
template <int G>
__global__ __launch_bounds__(256) void k_adam(AdamArgs a, int scalar_blocks) {
    __shared__ float s_w[XG_MAX_FEATURES];
    const int nf = a.p.n_features;
    load_weights(a.p.weights, nf, s_w);
    float coef[3];
    if (!step_coefficients(a, coef)) return;
    const float bias1 = coef[0], bias2 = coef[1], lr_means = coef[2];
    const int64_t n = a.n;
    if ((int)blockIdx.x < scalar_blocks) {
        const AdamQuads q(n);
        for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < q.end[3];
             t += (int64_t)scalar_blocks * blockDim.x) {
            if (t < q.end[0]) {
                const int64_t e = 4 * t;
                adam_quad<0>(a, a.p.means + e, a.g.means + e, nullptr, e, (int)min((int64_t)4, 3 * n - e), lr_means,
                             bias1, bias2);
            } else if (t < q.end[1]) {
                const int64_t e = 4 * (t - q.end[0]);
                adam_quad<1>(a, a.p.log_scales + e, a.g.scales + e, a.scales + e, 3 * n + e,
                             (int)min((int64_t)4, 3 * n - e), a.c.lr_scales, bias1, bias2);
            } else if (t < q.end[2]) {
                const int64_t e = 4 * (t - q.end[1]);
                adam_quad<0>(a, a.p.quats + e, a.g.quats + e, nullptr, 6 * n + e, 4, a.c.lr_quats, bias1, bias2);
            } else {
                const int64_t e = 4 * (t - q.end[2]);
                adam_quad<2>(a, a.p.opacity_logit + e, a.g.opacity + e, a.opacity + e, 10 * n + e,
                             (int)min((int64_t)4, n - e), a.c.lr_opacity, bias1, bias2);
            }
        }
        return;
    }
    constexpr int L = G > 4 ? G / 4 : 1;    // lanes per Gaussian
    const int k = 4 * (int)(threadIdx.x % L);   // the stride is a multiple of L
    const int cnt = min(4, nf - k);             // this lane's features (may be < 1)
    float w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = i < cnt ? s_w[k + i] : 0.0f;
    for (int64_t t = (int64_t)(blockIdx.x - scalar_blocks) * blockDim.x + threadIdx.x; t < n * L;
         t += (int64_t)(gridDim.x - scalar_blocks) * blockDim.x) {
        const int64_t i = t / L;
        float *f = a.p.features + i * nf + k;
        const int64_t k0 = 11 * n + i * nf + k;
        Quad x = {}, m = {}, v = {};
        if (cnt == 4) {
            x = *reinterpret_cast<const Quad *>(f);
            m = *reinterpret_cast<const Quad *>(a.m + k0);
            v = *reinterpret_cast<const Quad *>(a.v + k0);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < cnt) {
                    x.v[j] = f[j];
                    m.v[j] = a.m[k0 + j];
                    v.v[j] = a.v[k0 + j];
                }
        }
        float dot = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) dot = fmaf(w[j], x.v[j], dot);
        const float s = sigmoidf(group_sum<L>(dot));
        const float gs = a.g.intensity[i] * s * (1.0f - s);
        float dn = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x.v[j] = adam_value(a, x.v[j], gs * w[j], a.c.lr_feature, bias1, bias2, m.v[j], v.v[j]);
            dn = j < cnt ? fmaf(w[j], x.v[j], dn) : dn;
        }
        if (cnt == 4) {
            *reinterpret_cast<Quad *>(f) = x;
            *reinterpret_cast<Quad *>(a.m + k0) = m;
            *reinterpret_cast<Quad *>(a.v + k0) = v;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < cnt) {
                    f[j] = x.v[j];
                    a.m[k0 + j] = m.v[j];
                    a.v[k0 + j] = v.v[j];
                }
        }
        dn = group_sum<L>(dn);
        if (k == 0) a.intensity[i] = sigmoidf(dn);
    }
}

__global__ void k_step_advance(int32_t *step, const int32_t *gate) {
    if (threadIdx.x == 0 && (gate == nullptr || *gate == 0)) *step += 1;
}

// Workgroups of 256 threads of a grid-stride launch over n work items, at
// most `most`: the per-workgroup set-up (step coefficients in double, the
// response weights) then runs a few thousand times rather than once per 256
// items.
int64_t grid_of(int64_t n, int64_t most) { return std::min(std::max<int64_t>((n + 255) / 256, 1), most); }

}  // namespace

hipError_t launch_rirf_fwd(const float *features, const float *weights, int64_t n, int nf,
                           float *intensity, hipStream_t s) {
    const int64_t nb = (n + 255) / 256;
    if (nb > 0)
        hipLaunchKernelGGL(k_rirf_fwd, dim3((unsigned)nb), dim3(256), 0, s, features, weights, n, nf,
                           intensity);
    return hipGetLastError();
}

hipError_t launch_rirf_bwd(const float *features, const float *weights, int64_t n, int nf,
                           const float *dl_di, float *grad_f, hipStream_t s) {
    const int64_t nb = (n + 255) / 256;
    if (nb > 0)
        hipLaunchKernelGGL(k_rirf_bwd, dim3((unsigned)nb), dim3(256), 0, s, features, weights, n, nf,
                           dl_di, grad_f);
    return hipGetLastError();
}

hipError_t launch_adam(const xg_params &p, const xg_grads &g, float *m, float *v, int32_t *step,
                       const xg_adam &c, float *scales, float *opacity, float *intensity,
                       const int32_t *gate, hipStream_t s) {
    AdamArgs a{p, g, m, v, step, gate, c,
               (float)c.beta1, (float)(1.0 - c.beta1), (float)c.beta2, (float)(1.0 - c.beta2),
               scales, opacity, intensity, (int64_t)p.n};
    int G = 1;
    while (G < p.n_features) G *= 2;
    const int64_t n = p.n, L = G > 4 ? G / 4 : 1;
    // kAdamBlocks workgroups shared out by the bytes of the two parts
    const int64_t sb = grid_of(AdamQuads(n).end[3], kAdamBlocks * 11 / (11 + p.n_features) + 1);
    const int64_t fb = grid_of(n * L, kAdamBlocks * p.n_features / (11 + p.n_features) + 1);
    const dim3 grid((unsigned)(sb + fb)), block(256);
    switch (G) {
        case 1: hipLaunchKernelGGL(k_adam<1>, grid, block, 0, s, a, (int)sb); break;
        case 2: hipLaunchKernelGGL(k_adam<2>, grid, block, 0, s, a, (int)sb); break;
        case 4: hipLaunchKernelGGL(k_adam<4>, grid, block, 0, s, a, (int)sb); break;
        case 8: hipLaunchKernelGGL(k_adam<8>, grid, block, 0, s, a, (int)sb); break;
        case 16: hipLaunchKernelGGL(k_adam<16>, grid, block, 0, s, a, (int)sb); break;
        case 32: hipLaunchKernelGGL(k_adam<32>, grid, block, 0, s, a, (int)sb); break;
        case 64: hipLaunchKernelGGL(k_adam<64>, grid, block, 0, s, a, (int)sb); break;
        default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_step_advance, dim3(1), dim3(64), 0, s, step, gate);
    return hipGetLastError();
}

}  // namespace xg
