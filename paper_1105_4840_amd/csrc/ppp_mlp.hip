// Surrogate F(lambda) for learned window placement: a 1 -> 64 -> 64 -> 1 tanh
// network y(t) with its input derivative dy/dt (the slope the protocol
// measures as k (lambda_i - <x_i>), Eq. 14), trained on value and slope
// targets.  Parameters are used through their bf16 values; the activations
// entering a product (h1, u1, h2, u2 and the layer-2 error signals) are bf16;
// all arithmetic and accumulation is fp32.  The three dense contractions per
// tile of 16 points,
//   [a2 | v2]         = W2   [h1 | u1]          (forward, value and slope path)
//   [g_h1 | g_u1]     = W2^T [g_a2 | g_v2]      (backward)
//   dW2              += [g_a2 | g_v2] [h1 | u1]^T
// run on the matrix cores (v_mfma_f32_16x16x32_bf16, wave64).
#include <hip/hip_runtime.h>

#include "ppp_launch.hpp"

namespace ppp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int MH = 64;        // hidden width
constexpr int MT = 16;        // batch points per tile
constexpr int MC = 2 * MT;    // GEMM columns per tile: value path then slope path
constexpr int NP = MH + MH + MH * MH + MH + MH + 1;
constexpr int OFF_W1 = 0, OFF_B1 = MH, OFF_W2 = 2 * MH, OFF_B2 = 2 * MH + MH * MH, OFF_W3 = OFF_B2 + MH,
              OFF_B3 = OFF_W3 + MH;

// bf16 by round-to-nearest-even of the fp32 bit pattern
__device__ __forceinline__ uint16_t bf16_bits(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_val(float x) { return __uint_as_float((uint32_t)bf16_bits(x) << 16); }

// Row strides in LDS: padded so that a wavefront's 64 units (or 16 rows of a
// matrix operand) fall into different banks; unpadded rows of 32 floats put all
// 64 units of a column into two banks.
constexpr int LW = MH + 8;    // rows of 64 bf16 (16-byte aligned)
constexpr int LC = MC + 8;    // rows of 32 bf16
constexpr int LY = MC + 1;    // rows of 32 floats
constexpr int LR = MH + 4;    // rows of 64 floats read four at a time
constexpr int kStage = 1024;  // training points held in LDS

struct MlpShared {
    alignas(16) uint16_t w2[MH * LW];    // [out][in]
    alignas(16) uint16_t w2t[MH * LW];   // [in][out]
    alignas(16) uint16_t xc[MC * LW];    // [column][unit]   (h1 | u1), point-major
    alignas(16) uint16_t xm[MH * LC];    // [unit][column]
    alignas(16) uint16_t gc[MC * LW];    // (g_a2 | g_v2), point-major
    alignas(16) uint16_t gm[MH * LC];
    float y2[MH * LY];       // W2 [h1 | u1]
    float b2g[MH * LY];      // W2^T [g_a2 | g_v2]
    alignas(16) float red_y[MT * LR];
    alignas(16) float red_dy[MT * LR];
    float acc[4][256];
    float vec[4][MH];        // bf16 values of w1, b1, b2, w3
    float pt[MT][4];         // -, ey, ed, -
    float b3;
    float data[5][kStage];   // t, yv, wv, ys, wsl
};

// One 16x16 output tile: acc += A[16 rows][K] * B[K][16 cols], A row-major with
// row stride lda, B given transposed (column-major, stride ldb), K a multiple of 32.
__device__ __forceinline__ f32x4 mfma_tile(const uint16_t *A, int lda, const uint16_t *Bt, int ldb, int K, f32x4 acc) {
    const int l = __lane_id();
    const int r = l & 15, kq = (l >> 4) * 8;
    for (int k0 = 0; k0 < K; k0 += 32) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(A + r * lda + k0 + kq);
        const bf16x8 b = *reinterpret_cast<const bf16x8 *>(Bt + r * ldb + k0 + kq);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
    return acc;
}
// D layout of the 16x16 tile: lane l holds column l & 15, rows 4 (l >> 4) + i.
__device__ __forceinline__ void store_tile(float *D, int ldd, int r0, int c0, f32x4 acc) {
    const int l = __lane_id();
    for (int i = 0; i < 4; ++i) D[(r0 + 4 * (l >> 4) + i) * ldd + c0 + (l & 15)] = acc[i];
}

// Adam (Kingma and Ba, beta1 = 0.9, beta2 = 0.999) on one parameter; mh, vh turn
// the new moments into their bias-corrected values.
template <typename Mh, typename Vh>
__device__ __forceinline__ void adam_update(float &p, float &m, float &v, float g, float lr, Mh &&mh, Vh &&vh) {
    // fused by name, so that every kernel rounds alike
    const float mi = fmaf(0.1f, g, 0.9f * m);
    const float vi = fmaf(g, 0.001f * g, 0.999f * v);
    m = mi; v = vi;
    p -= lr * mh(mi) / (sqrtf(vh(vi)) + 1e-8f);
}

// Bias corrections of the steps of one training launch, as reciprocals.  The
// quotient of two floats lies at least 2^-49 of itself from every point half way
// between floats, so the fp64 product with the reciprocal, 2^-52 off at most,
// rounds to the same float as the division.
constexpr int kTrainSteps = 128;
struct TrainSteps { double inv_c1[kTrainSteps], inv_c2[kTrainSteps]; };

enum MlpMode { MLP_FORWARD, MLP_GRAD, MLP_TRAIN };

// MLP_FORWARD: y and dy/dt of the points, 16-point tiles spread over workgroups.
// MLP_GRAD: loss and gradient, one workgroup (its sums keep the order of the points).
// MLP_TRAIN: `iters` gradient steps with Adam in one launch.
//
// Thread (wave q, lane j) works on unit j and the points q, q + 4, q + 8, q + 12
// of a tile.  Bound: the latency of a tile's chain (two tanh layers, three
// barriers forward and four back, 64 ordered additions), not arithmetic: training
// runs a few tiles a step.  A training step took 24.6 us for the gradient, 4.6
// for Adam and 2 launches; in one launch the parameters and moments stay in
// registers (W2's in the layout its gradient tiles leave the matrix cores in),
// the tanh of the forward pass are kept for the backward one, and the points in LDS.
template <MlpMode MODE>
__global__ __launch_bounds__(256) void mlp_kernel(float *__restrict__ params, const float *__restrict__ t,
                                                  const float *__restrict__ yv, const float *__restrict__ wv,
                                                  const float *__restrict__ ys, const float *__restrict__ wsl, int n,
                                                  float *__restrict__ y_out, float *__restrict__ dy_out,
                                                  float *__restrict__ grad, float *__restrict__ loss,
                                                  float *__restrict__ am, float *__restrict__ av, float lr, int iters,
                                                  const TrainSteps steps) {
    __shared__ MlpShared S;
    constexpr bool BACK = MODE != MLP_FORWARD;
    const int tid = threadIdx.x, j = tid & 63, w = tid >> 6;
    const int mrow = 16 * w + 4 * (j >> 4), mcol = j & 15;   // W2 element [mrow + i][16 nt + mcol]
    float p2[4][4], m2[4][4], v2m[4][4];                     // training: W2 and its moments
    float pv = 0.f, mv = 0.f, vv = 0.f;                      // entry j of vector w (W1, b1, b2, w3)
    float p3 = 0.f, m3 = 0.f, v3 = 0.f;                      // b3 (thread 0)
    const int vec_off[4] = {OFF_W1, OFF_B1, OFF_B2, OFF_W3};
    const int vo = vec_off[w] + j;
    for (int nt = 0; nt < 4; ++nt)
        for (int i = 0; i < 4; ++i) {
            const int m = mrow + i, k = 16 * nt + mcol, o = OFF_W2 + m * MH + k;
            const float p = params[o];
            if (MODE == MLP_TRAIN) { p2[nt][i] = p; m2[nt][i] = am[o]; v2m[nt][i] = av[o]; }
            const uint16_t b = bf16_bits(p);
            S.w2[m * LW + k] = b;
            S.w2t[k * LW + m] = b;
        }
    pv = params[vo];
    S.vec[w][j] = bf16_val(pv);
    if (MODE == MLP_TRAIN) { mv = am[vo]; vv = av[vo]; }
    if (tid == 0) {
        p3 = params[OFF_B3];
        S.b3 = bf16_val(p3);
        if (MODE == MLP_TRAIN) { m3 = am[OFF_B3]; v3 = av[OFF_B3]; }
    }
    const bool staged = BACK && n <= kStage;
    if (staged)
        for (int i = tid; i < n; i += 256) {
            S.data[0][i] = t[i]; S.data[1][i] = yv[i]; S.data[2][i] = wv[i]; S.data[3][i] = ys[i]; S.data[4][i] = wsl[i];
        }
    const int tiles = (n + MT - 1) / MT;
    const int t_begin = BACK ? 0 : blockIdx.x;
    const int t_step = BACK ? 1 : gridDim.x;
    __syncthreads();
    for (int it = 0; it < (MODE == MLP_TRAIN ? iters : 1); ++it) {
        const float w1 = S.vec[0][j], b1 = S.vec[1][j], b2 = S.vec[2][j], w3 = S.vec[3][j];
        // per-thread accumulators for the unit j
        float aW1 = 0.f, aB1 = 0.f, aB2 = 0.f, aW3 = 0.f, aB3 = 0.f, aL = 0.f;
        f32x4 dW2[4];
        for (int q = 0; q < 4; ++q) dW2[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int tile = t_begin; tile < tiles; tile += t_step) {
            const int base = tile * MT;
            // layer 1: h1 and u1 = (1 - h1^2) W1 into the bf16 matrix operands
            float tp[4], h1[4], h2[4], v2[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = w + 4 * i, P = base + p;
                const bool valid = P < n;
                tp[i] = valid ? (staged ? S.data[0][P] : t[P]) : 0.f;
                h1[i] = tanhf(w1 * tp[i] + b1);
                const float u1 = (1.f - h1[i] * h1[i]) * w1;
                const uint16_t bh = valid ? bf16_bits(h1[i]) : 0, bu = valid ? bf16_bits(u1) : 0;
                S.xc[p * LW + j] = bh; S.xc[(MT + p) * LW + j] = bu;
                if (BACK) { S.xm[j * LC + p] = bh; S.xm[j * LC + MT + p] = bu; }
            }
            __syncthreads();
            // [a2 - b2 | v2] = W2 [h1 | u1]: 4 x 2 output tiles, wave w takes row tile w
            for (int nt = 0; nt < 2; ++nt) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma_tile(S.w2 + 16 * w * LW, LW, S.xc + 16 * nt * LW, LW, MH, acc);
                store_tile(S.y2, LY, 16 * w, 16 * nt, acc);
            }
            __syncthreads();
            // layer 2 and the output
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = w + 4 * i;
                v2[i] = S.y2[j * LY + MT + p];
                h2[i] = tanhf(S.y2[j * LY + p] + b2);
                const float u2 = (1.f - h2[i] * h2[i]) * v2[i];
                S.red_y[p * LR + j] = w3 * bf16_val(h2[i]);
                S.red_dy[p * LR + j] = w3 * bf16_val(u2);
            }
            __syncthreads();
            if (tid < 2 * MT) {
                // lanes 0-15 add up y of their point over the units in order, lanes 16-31 dy/dt
                const int p = tid & (MT - 1), P = base + p;
                const float4 *r = reinterpret_cast<const float4 *>((tid < MT ? S.red_y : S.red_dy) + p * LR);
                float y = 0.f;
#pragma unroll
                for (int q = 0; q < MH / 4; ++q) {
                    const float4 a = r[q];
                    y += a.x; y += a.y; y += a.z; y += a.w;
                }
                const float dy = __shfl(y, p + MT);
                if (tid < MT) {
                    y += S.b3;
                    float ey = 0.f, ed = 0.f;
                    if (P < n) {
                        if (!BACK) { y_out[P] = y; if (dy_out) dy_out[P] = dy; }
                        else {
                            const float wy = staged ? S.data[2][P] : wv[P], wd = staged ? S.data[4][P] : wsl[P];
                            const float ry = y - (staged ? S.data[1][P] : yv[P]), rd = dy - (staged ? S.data[3][P] : ys[P]);
                            ey = 2.f * wy * ry; ed = 2.f * wd * rd;
                            aL += wy * ry * ry + wd * rd * rd;
                            aB3 += ey;
                        }
                    }
                    S.pt[p][1] = ey; S.pt[p][2] = ed;
                }
            }
            __syncthreads();
            if (!BACK) continue;
            // backward through layer 2 (both paths)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = w + 4 * i;
                const float s2 = 1.f - h2[i] * h2[i];
                const float u2 = s2 * v2[i];
                const float ey = S.pt[p][1], ed = S.pt[p][2];
                aW3 += ey * bf16_val(h2[i]) + ed * bf16_val(u2);
                const float g_u2 = ed * w3;
                const float g_h2 = ey * w3 + g_u2 * (-2.f * h2[i] * v2[i]);
                const float g_v2 = g_u2 * s2;
                const float g_a2 = g_h2 * s2;
                aB2 = fmaf(s2, g_h2, aB2);
                const uint16_t ba = bf16_bits(g_a2), bv = bf16_bits(g_v2);
                S.gc[p * LW + j] = ba; S.gc[(MT + p) * LW + j] = bv;
                S.gm[j * LC + p] = ba; S.gm[j * LC + MT + p] = bv;
            }
            __syncthreads();
            // [g_h1 | g_u1] = W2^T [g_a2 | g_v2]
            for (int nt = 0; nt < 2; ++nt) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma_tile(S.w2t + 16 * w * LW, LW, S.gc + 16 * nt * LW, LW, MH, acc);
                store_tile(S.b2g, LY, 16 * w, 16 * nt, acc);
            }
            // dW2[m][k] += sum_c G[m][c] X[k][c]
            for (int nt = 0; nt < 4; ++nt)
                dW2[nt] = mfma_tile(S.gm + 16 * w * LC, LC, S.xm + 16 * nt * LC, LC, MC, dW2[nt]);
            __syncthreads();
            // backward through layer 1
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = w + 4 * i;
                if (base + p >= n) continue;
                const float s1 = 1.f - h1[i] * h1[i];
                const float g_u1 = S.b2g[j * LY + MT + p];
                const float g_h1 = S.b2g[j * LY + p] + g_u1 * (-2.f * h1[i] * w1);
                const float g_a1 = g_h1 * s1;
                aW1 += g_u1 * s1 + g_a1 * tp[i];
                aB1 += g_a1;
            }
            // (the next tile writes xc and xm, last read before the barrier above)
        }
        if (!BACK) return;
        // fixed-order reductions of the per-thread accumulators: wave w adds up vector w
        S.acc[0][tid] = aW1; S.acc[1][tid] = aB1; S.acc[2][tid] = aB2; S.acc[3][tid] = aW3;
        if (tid < MT) { S.pt[tid][0] = aB3; S.pt[tid][3] = aL; }
        __syncthreads();
        float g = 0.f;
        for (int q = 0; q < 4; ++q) g += S.acc[w][q * MH + j];
        float g3 = 0.f, L = 0.f;
        if (tid == 0)
            for (int i = 0; i < MT; ++i) { g3 += S.pt[i][0]; L += S.pt[i][3]; }
        if (MODE == MLP_GRAD) {
            for (int nt = 0; nt < 4; ++nt) store_tile(grad + OFF_W2, MH, 16 * w, 16 * nt, dW2[nt]);
            grad[vo] = g;
            if (tid == 0) { grad[OFF_B3] = g3; if (loss) loss[0] = L; }
            return;
        }
        const double i1 = steps.inv_c1[it], i2 = steps.inv_c2[it];
        auto mh = [&](float x) { return (float)((double)x * i1); };
        auto vh = [&](float x) { return (float)((double)x * i2); };
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                adam_update(p2[nt][i], m2[nt][i], v2m[nt][i], dW2[nt][i], lr, mh, vh);
                const int m = mrow + i, k = 16 * nt + mcol;
                const uint16_t b = bf16_bits(p2[nt][i]);
                S.w2[m * LW + k] = b;
                S.w2t[k * LW + m] = b;
            }
        adam_update(pv, mv, vv, g, lr, mh, vh);
        S.vec[w][j] = bf16_val(pv);
        if (tid == 0) {
            adam_update(p3, m3, v3, g3, lr, mh, vh);
            S.b3 = bf16_val(p3);
            if (it == iters - 1) loss[0] = L;
        }
        __syncthreads();
    }
    if (MODE != MLP_TRAIN) return;
    for (int nt = 0; nt < 4; ++nt)
        for (int i = 0; i < 4; ++i) {
            const int o = OFF_W2 + (mrow + i) * MH + 16 * nt + mcol;
            params[o] = p2[nt][i]; am[o] = m2[nt][i]; av[o] = v2m[nt][i];
        }
    params[vo] = pv; am[vo] = mv; av[vo] = vv;
    if (tid == 0) { params[OFF_B3] = p3; am[OFF_B3] = m3; av[OFF_B3] = v3; }
}

__global__ void adam_kernel(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, float lr, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NP) return;
    adam_update(p[i], m[i], v[i], g[i], lr, [&](float x) { return x / c1; }, [&](float x) { return x / c2; });
}

hipError_t launch_mlp_forward(const float *params, const float *t, int n, float *y, float *dy, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int tiles = (n + MT - 1) / MT;
    hipLaunchKernelGGL(mlp_kernel<MLP_FORWARD>, dim3(tiles < 1024 ? tiles : 1024), dim3(256), 0, stream,
                       const_cast<float *>(params), t, nullptr, nullptr, nullptr, nullptr, n, y, dy, nullptr, nullptr,
                       nullptr, nullptr, 0.f, 1, TrainSteps{});
    return hipGetLastError();
}

hipError_t launch_mlp_grad(const float *params, const float *t, const float *yv, const float *wv, const float *ys,
                           const float *wsl, int n, float *grad, float *loss, hipStream_t stream) {
    hipLaunchKernelGGL(mlp_kernel<MLP_GRAD>, dim3(1), dim3(256), 0, stream, const_cast<float *>(params), t, yv, wv, ys,
                       wsl, n, nullptr, nullptr, grad, loss, nullptr, nullptr, 0.f, 1, TrainSteps{});
    return hipGetLastError();
}

hipError_t launch_mlp_train(float *params, const float *t, const float *yv, const float *wv, const float *ys,
                            const float *wsl, int n, float *m, float *v, float *loss, float lr, int first_step,
                            int iters, hipStream_t stream) {
    for (int done = 0; done < iters; done += kTrainSteps) {
        const int k = iters - done < kTrainSteps ? iters - done : kTrainSteps;
        TrainSteps steps{};
        for (int i = 0; i < k; ++i) {
            const float step = (float)(first_step + done + i);
            steps.inv_c1[i] = 1.0 / (double)(1.f - powf(0.9f, step));
            steps.inv_c2[i] = 1.0 / (double)(1.f - powf(0.999f, step));
        }
        hipLaunchKernelGGL(mlp_kernel<MLP_TRAIN>, dim3(1), dim3(256), 0, stream, params, t, yv, wv, ys, wsl, n, nullptr,
                           nullptr, nullptr, loss, m, v, lr, k, steps);
    }
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float *params, const float *grad, float *m, float *v, float lr, int step,
                           hipStream_t stream) {
    const float c1 = 1.f - powf(0.9f, (float)step), c2 = 1.f - powf(0.999f, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3((NP + 255) / 256), dim3(256), 0, stream, params, grad, m, v, lr, c1, c2);
    return hipGetLastError();
}

}  // namespace ppp
