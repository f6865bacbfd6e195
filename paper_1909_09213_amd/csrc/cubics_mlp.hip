// Training and evaluation kernels of the branching-policy network (forward
// with BF16 MFMA / FP32 accumulation, backward with wave reductions, Adam on
// FP32 master weights, BF16 re-rounding of the weights the MFMAs read).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "cubics_internal.h"
#include "cubics_mlp.h"

namespace cubics {

// bf16 copies of W1 (padded to 16 inputs) and w2 of hidden unit h from the fp32
// master theta
__device__ __forceinline__ void round_weights(const float *theta, uint16_t *w1b, uint16_t *w2b, int h) {
    if (h >= POLICY_H) return;
    for (int k = 0; k < MLP_FPAD; ++k)
        w1b[h * MLP_FPAD + k] = k < POLICY_F ? f2bf(theta[OFF_W1 + h * POLICY_F + k]) : (uint16_t)0;
    w2b[h] = f2bf(theta[OFF_W2 + h]);
}
__global__ void policy_round_kernel(const float *theta, uint16_t *w1b, uint16_t *w2b) {
    round_weights(theta, w1b, w2b, threadIdx.x);
}

// bf16 B operand of layer 1 for row s of X (fp32 rows of stride ld, features
// in columns 0..POLICY_F-1): lane holds features 4 (lane / 16) + j
__device__ __forceinline__ bf16x4 load_xT(const float *X, int ld, long long s, long long N, int kq) {
    bf16x4 xT;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = 4 * kq + j;
        xT[j] = (short)((s < N && k < POLICY_F) ? f2bf(X[s * ld + k]) : (uint16_t)0);
    }
    return xT;
}

// y[s] for N rows of X
__global__ __launch_bounds__(256) void mlp_forward_kernel(PolicyDev P, const float *X, int ld, long long N, float *y) {
    const int lane = __lane_id();
    const int wave = threadIdx.x >> 6;
    const int row = lane & 15, kq = lane >> 4;
    for (long long tile = (long long)blockIdx.x * 4 + wave; tile * 16 < N; tile += (long long)gridDim.x * 4) {
        const long long s = tile * 16 + row;
        const bf16x4 xT = load_xT(X, ld, s, N, kq);
        const f32x4 acc = mlp_tile(P, xT, lane, nullptr);
        if (row == 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const long long ss = tile * 16 + 4 * kq + r;
                if (ss < N) y[ss] = acc[r] + *P.b2;
            }
        }
    }
}

// Sum over the 16 lanes of a row, in its lane 15.
__device__ __forceinline__ float row_sum(float v) {
    const auto up = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v += up(v, std::integral_constant<int, 0x111>{});  // row_shr:1
    v += up(v, std::integral_constant<int, 0x112>{});
    v += up(v, std::integral_constant<int, 0x114>{});
    v += up(v, std::integral_constant<int, 0x118>{});
    return v;
}

// Gradient of the mean squared error over N rows and, with Adam arguments, the
// training step.  The rounding of weights and activations to bf16 is treated
// as the identity in the backward pass (straight-through).
//
// A wave keeps its sums over all its 16-row tiles in registers: lane (row,
// kq) sums for its row's share of the 16 hidden units 16 t + 4 kq + r that the
// forward pass leaves it, seven sums each, and only at the end are lanes,
// waves and workgroups added up.  (Reducing every tile over its 16 rows by
// shuffles and LDS atomics took 7 x 16 reductions a tile.)  With w2 taken out
// of the sum, d loss / d W1[h][k] = w2[h] sum_s [p_sh > 0] dy_s x_sk.
// Layer 2 runs as w2 (in every row) times the hidden tile, so that each lane
// receives the output of its own row.  The workgroup that ends last (ticket)
// writes the results or takes Adam's step, and clears the sums for the next
// launch: one launch where there were five.  Workgroups add to one of
// GRAD_COPIES copies of the sums: additions to one line are served in turn.
// 135,797 rows: 89 -> 39 us for the gradient, 100 -> 38 us for a step (both
// with the host's wait); 4,000,000 rows 1.77 ms -> 0.16 ms.
__global__ __launch_bounds__(256) void mlp_grad_kernel(PolicyDev P, const float *X, int ld, const float *T, int ldt,
                                                       long long N, float *sums, uint32_t *ticket, float *grad,
                                                       float *loss, AdamArgs A) {
    __shared__ float g[POLICY_NP + 1];
    __shared__ int is_last;
    const int lane = __lane_id();
    const int wave = threadIdx.x >> 6;
    const int row = lane & 15, kq = lane >> 4;
    for (int i = threadIdx.x; i <= POLICY_NP; i += blockDim.x) g[i] = 0.f;
    const float invN = 1.0f / (float)N, bias2 = *P.b2;
    // the network's operands of this lane (see mlp_tile)
    bf16x4 a1[4], a2[4];
    float b1[16];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a1[t][j] = (short)P.w1[(size_t)(16 * t + row) * MLP_FPAD + 4 * kq + j];
            a2[t][j] = (short)P.w2[16 * t + 4 * kq + j];
            b1[4 * t + j] = P.b1[16 * t + 4 * kq + j];
        }
    float gx[16][POLICY_F + 1], gw2[16], gb2 = 0.f, lsum = 0.f;  // gx[.][POLICY_F]: b1
#pragma unroll
    for (int h = 0; h < 16; ++h) {
        gw2[h] = 0.f;
#pragma unroll
        for (int k = 0; k <= POLICY_F; ++k) gx[h][k] = 0.f;
    }
    const long long stride = (long long)gridDim.x * 4;
    long long tile = (long long)blockIdx.x * 4 + wave;
    // the row's inputs and target, loaded a tile ahead
    float xin[POLICY_F], tin = 0.f;
    const auto fetch = [&](long long t) {
        const long long s = t * 16 + row;
        const bool in = s < N;
#pragma unroll
        for (int k = 0; k < POLICY_F; ++k) xin[k] = in ? X[s * ld + k] : 0.f;
        tin = in ? T[s * ldt] : 0.f;
    };
    if (tile * 16 < N) fetch(tile);
    for (; tile * 16 < N; tile += stride) {
        const bool valid = tile * 16 + row < N;
        uint16_t xb[POLICY_F];
        float x[POLICY_F];
#pragma unroll
        for (int k = 0; k < POLICY_F; ++k) {
            xb[k] = f2bf(xin[k]);
            x[k] = bf2f(xb[k]);
        }
        const float target = tin;
        if ((tile + stride) * 16 < N) fetch(tile + stride);
        bf16x4 xT;  // features 4 kq + j
#pragma unroll
        for (int j = 0; j < 4; ++j) xT[j] = (short)(kq == 0 ? xb[j] : (kq == 1 && j == 0 ? xb[4] : (uint16_t)0));
        float pre[16], hid[16];
        f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            const f32x4 d1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1[t], xT, zero, 0, 0, 0);
            bf16x4 hb;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float p = d1[r] + b1[4 * t + r];
                pre[4 * t + r] = p;
                const uint16_t b = f2bf(p > 0.f ? p : 0.f);
                hid[4 * t + r] = bf2f(b);
                hb[r] = (short)b;
            }
            y = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a2[t], hb, y, 0, 0, 0);
        }
        const float e = valid ? y[0] + bias2 - target : 0.f;
        const float dy = 2.f * e * invN;
        if (kq == 0) {
            lsum += e * e * invN;
            gb2 += dy;
        }
#pragma unroll
        for (int h = 0; h < 16; ++h) {
            gw2[h] += dy * hid[h];
            const float d = pre[h] > 0.f ? dy : 0.f;
#pragma unroll
            for (int k = 0; k < POLICY_F; ++k) gx[h][k] += d * x[k];
            gx[h][POLICY_F] += d;
        }
    }
    __syncthreads();  // g is zero
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * t + r, h = 16 * t + 4 * kq + r;
            const float w2 = bf2f((uint16_t)a2[t][r]);
            const float s2 = row_sum(gw2[i]);
            float s1[POLICY_F + 1];
#pragma unroll
            for (int k = 0; k <= POLICY_F; ++k) s1[k] = row_sum(gx[i][k]);
            if (row == 15) {
                atomicAdd(&g[OFF_W2 + h], s2);
                atomicAdd(&g[OFF_B1 + h], w2 * s1[POLICY_F]);
#pragma unroll
                for (int k = 0; k < POLICY_F; ++k) atomicAdd(&g[OFF_W1 + h * POLICY_F + k], w2 * s1[k]);
            }
        }
    const float sb2 = row_sum(gb2), sl = row_sum(lsum);
    if (lane == 15) {
        atomicAdd(&g[OFF_B2], sb2);
        atomicAdd(&g[POLICY_NP], sl);
    }
    __syncthreads();
    float *mine = sums + (blockIdx.x % GRAD_COPIES) * GRAD_STRIDE;
    for (int i = threadIdx.x; i <= POLICY_NP; i += blockDim.x)
        __hip_atomic_fetch_add(&mine[i], g[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // every thread's additions are done before the workgroup takes its ticket
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (threadIdx.x == 0)
        is_last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!is_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    for (int i = threadIdx.x; i <= POLICY_NP; i += blockDim.x) {
        float part[GRAD_COPIES], gi = 0.f;
#pragma unroll
        for (int c = 0; c < GRAD_COPIES; ++c)
            part[c] = __hip_atomic_load(&sums[c * GRAD_STRIDE + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int c = 0; c < GRAD_COPIES; ++c) {
            gi += part[c];
            __hip_atomic_store(&sums[c * GRAD_STRIDE + i], 0.f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (i == POLICY_NP) {
            *loss = gi;
            if (A.theta) *A.loss_host = gi;
            continue;
        }
        grad[i] = gi;
        if (A.theta) {
            // Adam (Kingma & Ba) on the fp32 master parameters
            const float mi = A.beta1 * A.m[i] + (1.f - A.beta1) * gi;
            const float vi = A.beta2 * A.v[i] + (1.f - A.beta2) * gi * gi;
            A.m[i] = mi;
            A.v[i] = vi;
            const float mh = mi / (1.f - powf(A.beta1, (float)A.step));
            const float vh = vi / (1.f - powf(A.beta2, (float)A.step));
            const float th = A.theta[i] - A.lr * mh / (sqrtf(vh) + A.eps);
            A.theta[i] = th;
            A.theta_host[i] = th;
            g[i] = th;
        }
    }
    if (threadIdx.x == 0) *ticket = 0u;
    if (A.theta) {
        __syncthreads();
        round_weights(g, A.w1b, A.w2b, threadIdx.x);
    }
}

__global__ void fill_kernel(float *p, int n, float v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t launch_policy_round(const float *theta, uint16_t *w1b, uint16_t *w2b, hipStream_t st) {
    hipLaunchKernelGGL(policy_round_kernel, dim3(1), dim3(64), 0, st, theta, w1b, w2b);
    return hipGetLastError();
}
hipError_t launch_mlp_forward(const PolicyDev &P, const float *X, int ld, long long N, float *y, hipStream_t st) {
    long long tiles = (N + 15) / 16;
    int blocks = (int)((tiles + 3) / 4);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(mlp_forward_kernel, dim3(blocks), dim3(256), 0, st, P, X, ld, N, y);
    return hipGetLastError();
}
// sums: GRAD_COPIES x GRAD_STRIDE floats and then the ticket, zero before the
// first launch and left zero by every launch.  adam == nullptr: gradient only.
hipError_t launch_mlp_grad(const PolicyDev &P, const float *X, int ld, const float *T, int ldt, long long N,
                           float *sums, float *grad, float *loss, const AdamArgs *adam, hipStream_t st) {
    const AdamArgs none = {};
    // four tiles a wave up to 64 workgroups, then eight, up to the two
    // workgroups per CU that their registers allow: every workgroup costs the
    // additions of its sums, every tile of a wave about a microsecond
    const long long tiles = (N + 15) / 16;
    const long long want = tiles <= 1024 ? (tiles + 15) / 16 : std::max<long long>(64, (tiles + 31) / 32);
    const int blocks = (int)std::min<long long>(512, want);
    hipLaunchKernelGGL(mlp_grad_kernel, dim3(blocks), dim3(256), 0, st, P, X, ld, T, ldt, N, sums,
                       (uint32_t *)(sums + GRAD_COPIES * GRAD_STRIDE), grad, loss, adam ? *adam : none);
    return hipGetLastError();
}
hipError_t launch_fill(float *p, int n, float v, hipStream_t st) {
    hipLaunchKernelGGL(fill_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

}  // namespace cubics
