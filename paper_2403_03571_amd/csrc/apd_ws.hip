// apd_ws.hip -- the learned warm start: a per-seed network that predicts the
// initial weights of Algorithm 2 (arXiv 2403.03571 starts from W_0 = 0).
//
// Features (2D), per seed i: its own (x_i, upper triangle of A_i, N v_i),
// the mean over its 16 nearest seeds (Euclidean, ties to the lower index)
// of (sqrt(N)(x_j - x_i), upper triangle of A_j, N v_j, N |x_j - x_i|^2_{A_i},
// N |x_j - x_i|^2_{A_j}), its distance to the box boundary along each axis
// scaled by sqrt(N / |Omega|), the volume deficit d_i = N (v_i - |C_i|) of
// its cell at W = 0 (the gradient (2.8) of one pass at zero weights), and the
// 1-, 2- and 3-fold repeated 16-neighbour means of d: 20 numbers.  The
// optimal weights respond to the deficit like the inverse of a graph
// Laplacian, which the repeated means reach beyond the nearest seeds.
// Network: 20 -> 128 -> 128 -> 128 -> 1, ReLU between layers, parameters
// one flat FP32 vector (per layer W [in][out] row-major, then b).
// Training: mean squared error against t_i = N (w*_i - mean w*), Adam.
// Prediction: w_i = (y_i - mean y) / N.
#include "../../include/apd.h"
#include "apd_internal.h"

#include <math.h>
#include <stdarg.h>
#include <stdio.h>

#include <algorithm>
#include <string>

namespace apd {
namespace ws {

constexpr int kFeat = 20;
constexpr int kPoolHops = 3;
constexpr int kHid = 128;
constexpr int kNeigh = 16;
constexpr int64_t kParams = (int64_t)kFeat * kHid + kHid + 2 * ((int64_t)kHid * kHid + kHid) + kHid + 1;

const int64_t kParamCount = kParams;

// offsets of the layers in the flat vector
constexpr int64_t oW1 = 0, ob1 = oW1 + kFeat * kHid;
constexpr int64_t oW2 = ob1 + kHid, ob2 = oW2 + kHid * kHid;
constexpr int64_t oW3 = ob2 + kHid, ob3 = oW3 + kHid * kHid;
constexpr int64_t oW4 = ob3 + kHid, ob4 = oW4 + kHid;

namespace {

// ------------------------------------------------------------- features

// (distance, index) order: the nearer seed, the lower index on equal ones.
__device__ inline bool nearer(double d, int j, double e, int k) { return d < e || (d == e && j < k); }

// The wave's least (d, j), in every lane: DPP steps within the rows of 16
// lanes (rotations by 8 and 4, then within quads), then the rows' results.
template <int CTRL>
__device__ inline void nearest_step(double &d, int &j) {
    const long long b = __double_as_longlong(d);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    const int oj = __builtin_amdgcn_update_dpp(0, j, CTRL, 0xF, 0xF, false);
    const double od = __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
    if (nearer(od, oj, d, j)) {
        d = od;
        j = oj;
    }
}
__device__ inline void wave_nearest(double &d, int &j) {
    nearest_step<0x128>(d, j);  // row_ror 8
    nearest_step<0x124>(d, j);  // row_ror 4
    nearest_step<0x4E>(d, j);   // quad_perm 2,3,0,1
    nearest_step<0xB1>(d, j);   // quad_perm 1,0,3,2
    const long long b = __double_as_longlong(d);
    double rd = INFINITY;
    int rj = 0x7fffffff;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), 16 * r);
        const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 16 * r);
        const int oj = __builtin_amdgcn_readlane(j, 16 * r);
        const double od = __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
        if (r == 0 || nearer(od, oj, rd, rj)) {
            rd = od;
            rj = oj;
        }
    }
    d = rd;
    j = rj;
}

constexpr int kTop = 4;  // nearest seeds a lane keeps

// One wave per seed.  A lane takes the seeds lane, lane + 64, ... and keeps
// its kTop nearest in order; then the wave's nearest head is taken 16 times
// (ties to the lower index).  A lane whose kTop are all taken (4 of the 16
// nearest among its 64th of the seeds, about one wave in 10^4) looks through
// its seeds again for the next ones.  The neighbours' terms are formed by 16
// lanes at once and summed in the order of the neighbours.  (16 rounds over
// all seeds and 16 dependent loads of a neighbour took 53 us for 700 seeds;
// this takes 14.)
__global__ __launch_bounds__(256) void kw_features(int n, const double *__restrict__ x,
                                                   const double *__restrict__ A,
                                                   const double *__restrict__ v, double lo0,
                                                   double lo1, double hi0, double hi1, float *F,
                                                   int *nb) {
    __shared__ double s_t[4][kNeigh][9];
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 4 + wave;
    if (i >= n) return;  // whole waves leave together
    const double xi0 = x[2 * i], xi1 = x[2 * i + 1];
    const int k = min(kNeigh, n - 1);
    double td[kTop];
    int tj[kTop];
    // the lane's kTop nearest after (pd, pj)
    auto collect = [&](double pd, int pj) {
#pragma unroll
        for (int q = 0; q < kTop; ++q) {
            td[q] = INFINITY;
            tj[q] = 0x7fffffff;
        }
#pragma unroll 4
        for (int j = lane; j < n; j += 64) {
            const double d0 = xi0 - x[2 * j], d1 = xi1 - x[2 * j + 1];
            double d = d0 * d0 + d1 * d1;
            int c = j;
            if (j == i || !nearer(pd, pj, d, j)) continue;
#pragma unroll
            for (int q = 0; q < kTop; ++q)
                if (nearer(d, c, td[q], tj[q])) {
                    const double t = td[q];
                    const int u = tj[q];
                    td[q] = d;
                    tj[q] = c;
                    d = t;
                    c = u;
                }
        }
    };
    collect(-1.0, -1);
    int mine = 0;  // lane r < k: neighbour r
    int used = 0;
    for (int r = 0; r < k; ++r) {
        double d = td[0];
        int j = tj[0];
        wave_nearest(d, j);
        if (lane == r) mine = j;
        if ((j & 63) == lane && tj[0] == j) {
            // taken: the next of this lane
#pragma unroll
            for (int q = 0; q + 1 < kTop; ++q) {
                td[q] = td[q + 1];
                tj[q] = tj[q + 1];
            }
            td[kTop - 1] = INFINITY;
            tj[kTop - 1] = 0x7fffffff;
            if (++used == kTop) {
                collect(d, j);
                used = 0;
            }
        }
    }
    const double N = (double)n;
    const double *ai = A + 4 * i;
    if (lane < k) {
        nb[(size_t)i * kNeigh + lane] = mine;
        const int j = mine;
        const double dx0 = x[2 * j] - xi0, dx1 = x[2 * j + 1] - xi1;
        const double *aj = A + 4 * j;
        double *t = s_t[wave][lane];
        t[0] = dx0;
        t[1] = dx1;
        t[2] = aj[0];
        t[3] = aj[1];
        t[4] = aj[3];
        t[5] = N * v[j];
        t[6] = N * (dx0 * (ai[0] * dx0 + ai[1] * dx1) + dx1 * (ai[1] * dx0 + ai[3] * dx1));
        t[7] = N * (dx0 * (aj[0] * dx0 + aj[1] * dx1) + dx1 * (aj[1] * dx0 + aj[3] * dx1));
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane >= 16) return;
    const double area = (hi0 - lo0) * (hi1 - lo1);
    const double sc = sqrt(N / area);
    // lane q writes feature q
    double f;
    if (lane < 6) {
        f = lane == 0 ? xi0 : lane == 1 ? xi1 : lane == 2 ? ai[0] : lane == 3 ? ai[1] : lane == 4 ? ai[3] : N * v[i];
    } else if (lane < 14) {
        double s = 0.0;
        for (int r = 0; r < k; ++r) s += s_t[wave][r][lane - 6];
        const double c = (double)k;
        f = k == 0 ? 0.0 : lane < 8 ? sqrt(N) * s / c : s / c;
    } else {
        f = lane == 14 ? sc * fmin(xi0 - lo0, hi0 - xi0) : sc * fmin(xi1 - lo1, hi1 - xi1);
    }
    F[(size_t)i * kFeat + lane] = (float)f;
}

// The deficit d_i = N grad_i at W = 0 (feature 16) and its 1-, 2- and 3-fold
// repeated means over the 16 nearest seeds of each seed, in neighbour order
// (features 17 to 19; zero for a lone seed).  Up to kPoolSeeds seeds one block
// does it all with the values in LDS (four launches of 4.7 us each before);
// more seeds take a launch per hop, in and out in global memory.
constexpr int kPoolSeeds = 4096;

__device__ inline double pool_mean(int n, const int *nb, const double *in, int i) {
    const int k = min(kNeigh, n - 1);
    double s = 0.0;
    if (k == kNeigh) {
        const int4 *q = reinterpret_cast<const int4 *>(nb + (size_t)i * kNeigh);
        const int4 a = q[0], b = q[1], c = q[2], d = q[3];
        const int id[kNeigh] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w, d.x, d.y, d.z, d.w};
#pragma unroll
        for (int r = 0; r < kNeigh; ++r) s += in[id[r]];
    } else {
        for (int r = 0; r < k; ++r) s += in[nb[(size_t)i * kNeigh + r]];
    }
    return k > 0 ? s / (double)k : 0.0;
}

__global__ __launch_bounds__(1024) void kw_pool_all(int n, const int *nb, const double *grad, float *F) {
    __shared__ double d[2][kPoolSeeds];
    for (int i = threadIdx.x; i < n; i += 1024) {
        const double t = (double)n * grad[i];
        d[0][i] = t;
        F[(size_t)i * kFeat + 16] = (float)t;
    }
    for (int h = 0; h < kPoolHops; ++h) {
        __syncthreads();
        for (int i = threadIdx.x; i < n; i += 1024) {
            const double m = pool_mean(n, nb, d[h & 1], i);
            d[(h + 1) & 1][i] = m;
            F[(size_t)i * kFeat + 17 + h] = (float)m;
        }
    }
}

__global__ __launch_bounds__(256) void kw_deficit(int n, const double *grad, double *out, float *F) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double d = (double)n * grad[i];
    out[i] = d;
    F[(size_t)i * kFeat + 16] = (float)d;
}

__global__ __launch_bounds__(256) void kw_pool(int n, const int *nb, const double *in, double *out,
                                               float *F, int col) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double m = pool_mean(n, nb, in, i);
    out[i] = m;
    F[(size_t)i * kFeat + col] = (float)m;
}

// ------------------------------------------------- training on the matrix cores

// Forward and backward in three launches (one for the forward alone), all
// products on the FP32 matrix cores: v_mfma_f32_16x16x4_f32 and _32x32x2_f32
// multiply and accumulate in FP32, at the rate of the vector ALU but without
// its operand traffic.  The path is bound by latency, not by arithmetic
// (0.85 GFLOP for 4096 samples, 5.6 us at the matrix cores' 153 TFLOP/s): one
// product per launch through LDS took 21 launches and 272 us of kernels,
// these three 34 us (kw_net 17, kw_grad 13, kw_reduce 4).
//   kw_net       a block per 16 samples keeps their activations in LDS through
//                the layers and back: y, the loss terms and the layers'
//                inputs H and output gradients dZ in global memory
//   kw_grad      the weight and bias gradients, split over the samples
//   kw_reduce    the splits added in order (deterministic), the loss, and
//                for a training step Adam's update

typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));

constexpr int kTS = 16;         // samples per block of kw_net: 256 blocks for 4096
constexpr int kNetThreads = 512; // its 8 waves, one per 16 columns of a layer
constexpr int kRowF = kHid + 4; // LDS row of activations (the 16 rows of a column on distinct banks)

// The contraction index of the 16x16x4 products runs over k = 16 t + 4 g + c
// at step 4 t + c for the lanes of group g = lane / 16, on both operands, so
// that a lane reads its activations (and, where they are contiguous in k, its
// weights) four at a time.

// out = act W (W [K][128] row-major): the wave's 16 columns n0 .. n0 + 15; rows
// k >= KV of W and columns of act past KV are zero.
template <int KT>
__device__ inline floatx4_t net_tile(const float (&w)[KT][4], const float *act, int lane) {
    const int row = lane & 15, g = lane >> 4;
    floatx4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        const floatx4_t a = *reinterpret_cast<const floatx4_t *>(act + row * kRowF + 16 * t + 4 * g);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c], w[t][c], acc, 0, 0, 0);
    }
    return acc;
}
template <int KT, int KV>
__device__ inline void fwd_weights(const float *W, int n0, int lane, float (&w)[KT][4]) {
    const int col = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int k = 16 * t + 4 * g + c;
            w[t][c] = (KV == 16 * KT || k < KV) ? W[(size_t)k * kHid + n0 + col] : 0.0f;
        }
}
// The same for out = dZ W^T (the contraction over W's columns).
__device__ inline void bwd_weights(const float *W, int n0, int lane, float (&w)[kHid / 16][4]) {
    const int col = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < kHid / 16; ++t) {
        const floatx4_t v = *reinterpret_cast<const floatx4_t *>(W + (size_t)(n0 + col) * kHid + 16 * t + 4 * g);
#pragma unroll
        for (int c = 0; c < 4; ++c) w[t][c] = v[c];
    }
}

// The global activations of one pass: H1, H2, H3 and dZ1, dZ2, dZ3 [S][128],
// dy [S], one loss term per block.
struct NetBufs {
    float *H[3];
    float *dZ[3];
    float *dy;
    double *lossp;
};

// Samples 16 b .. of block b through the network (and, with BWD, back):
// wave w holds the output columns 16 w .. 16 w + 15 of every layer.
// The weights of all layers are loaded first (loads behind stores would wait
// for them layer by layer), and each layer's H and dZ leave LDS past the
// caches while the next one is computed: the next kernel reads them on other
// XCDs, and the write-back of 12.6 MB of them at the kernel's end took longer
// than the products (4096 samples: 7 us for the forward pass alone).
template <bool BWD>
__global__ __launch_bounds__(kNetThreads) void kw_net(const float *__restrict__ P, const float *__restrict__ X,
                                                      const float *__restrict__ tgt, int S, float *__restrict__ y,
                                                      NetBufs nb) {
    // X, H1, H2, H3, dZ3, dZ2, dZ1
    __shared__ __attribute__((aligned(16))) float act[BWD ? 7 : 4][kTS * kRowF];
    __shared__ float s_r[kTS];
    const int lane = __lane_id(), tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = 16 * wave, s0 = blockIdx.x * kTS;
    const int col = lane & 15, g = lane >> 4, n = n0 + col;
    float w1[2][4], w2[kHid / 16][4], w3[kHid / 16][4], w3t[kHid / 16][4], w2t[kHid / 16][4];
    {
        const int r = tid >> 5, k = tid & 31;
        act[0][r * kRowF + k] = (k < kFeat && s0 + r < S) ? X[(size_t)(s0 + r) * kFeat + k] : 0.0f;
    }
    fwd_weights<2, kFeat>(P + oW1, n0, lane, w1);
    const float b1 = P[ob1 + n], b2 = P[ob2 + n], b3 = P[ob3 + n];
    fwd_weights<kHid / 16, kHid>(P + oW2, n0, lane, w2);
    fwd_weights<kHid / 16, kHid>(P + oW3, n0, lane, w3);
    if constexpr (BWD) {
        bwd_weights(P + oW3, n0, lane, w3t);
        bwd_weights(P + oW2, n0, lane, w2t);
    }
    // bias and ReLU of a layer's tile
    auto store = [&](const floatx4_t acc, float bn, float *dst) {
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[(4 * g + r) * kRowF + n] = fmaxf(acc[r] + bn, 0.0f);
    };
    // a thread writes 4 columns of one sample
    auto put = [&](const float *src, float *glob) {
        const int m = tid >> 5, c = 4 * (tid & 31);
        if (s0 + m < S)
            __builtin_nontemporal_store(*reinterpret_cast<const floatx4_t *>(&src[m * kRowF + c]),
                                        reinterpret_cast<floatx4_t *>(glob + (size_t)(s0 + m) * kHid + c));
    };
    __syncthreads();
    store(net_tile<2>(w1, act[0], lane), b1, act[1]);
    __syncthreads();
    if (BWD) put(act[1], nb.H[0]);
    store(net_tile<kHid / 16>(w2, act[1], lane), b2, act[2]);
    __syncthreads();
    if (BWD) put(act[2], nb.H[1]);
    store(net_tile<kHid / 16>(w3, act[2], lane), b3, act[3]);
    __syncthreads();
    if (BWD) put(act[3], nb.H[2]);
    // the output: 32 threads per sample, 4 columns each
    {
        const int m = tid >> 5, q = tid & 31;
        float v = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) v = fmaf(act[3][m * kRowF + q + 32 * k], P[oW4 + q + 32 * k], v);
#pragma unroll
        for (int o = 16; o >= 1; o >>= 1) v += __shfl_xor(v, o);
        v += P[ob4];
        const bool in = s0 + m < S;
        if (q == 0 && in && y) y[s0 + m] = v;
        if constexpr (BWD) {
            // r, dy = 2 r / S, and dZ3 = dy W4^T where H3 > 0 (every thread of the
            // sample holds v)
            const float r = in ? v - tgt[s0 + m] : 0.0f;
            const float dy = 2.0f * r / (float)S;
            if (q == 0) {
                s_r[m] = r;
                if (in) nb.dy[s0 + m] = dy;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = q + 32 * k;
                act[4][m * kRowF + c] = act[3][m * kRowF + c] > 0.0f ? dy * P[oW4 + c] : 0.0f;
            }
        }
    }
    if constexpr (BWD) {
        // dZ = (dZ_next W^T) where H > 0
        auto back = [&](const floatx4_t acc, const float *H, float *dst) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = 4 * g + r;
                dst[m * kRowF + n] = H[m * kRowF + n] > 0.0f ? acc[r] : 0.0f;
            }
        };
        __syncthreads();
        if (tid == 0) {
            double l = 0.0;
            for (int m = 0; m < kTS; ++m) l += (double)s_r[m] * (double)s_r[m];
            nb.lossp[blockIdx.x] = l;
        }
        put(act[4], nb.dZ[2]);
        back(net_tile<kHid / 16>(w3t, act[4], lane), act[2], act[5]);
        __syncthreads();
        put(act[5], nb.dZ[1]);
        back(net_tile<kHid / 16>(w2t, act[5], lane), act[1], act[6]);
        __syncthreads();
        put(act[6], nb.dZ[0]);
    }
}

// Gradients of one slice of the samples, into part[slice][kParams].  Block
// job 0-3 and 4-7: the 64 x 64 quarters of dW3 = H2^T dZ3 and dW2 = H1^T dZ2, a
// wave per 32 x 32 tile; 8, 9: the halves of dW1 = X^T dZ1 (rows past 20 are
// empty; waves 0 and 1); 10, 11: the bias gradients and the output layer's.
// The samples come through LDS 128 at a time, every load of a chunk in flight
// at once: the arrays were written from other XCDs, so each load goes past the
// L2 (read straight into the products' operands 16 samples at a time the
// kernel took 12 to 14 us for 4096 samples).
constexpr int kGradChunk = 128;
constexpr int kGradJobs = 12;

__global__ __launch_bounds__(256) void kw_grad(const float *__restrict__ X, int S, int kslice, NetBufs nb,
                                               float *__restrict__ part) {
    __shared__ __attribute__((aligned(16))) float sm[2][kGradChunk][64];
    const int job = blockIdx.x, tid = threadIdx.x, lane = __lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ka = blockIdx.y * kslice, kb = min(S, ka + kslice);
    float *out = part + (size_t)blockIdx.y * kParams;
    if (job >= 10) {
        // column n over half of the slice per thread: dW4, db3 and db4 (job
        // 10) or db1 and db2 (11); the halves are added in LDS
        const int n = tid & 127, half = tid >> 7;
        const bool last = job == 10;
        const float *U = last ? nb.H[2] : nb.dZ[0], *V = last ? nb.dZ[2] : nb.dZ[1];
        const int mid = ka + (kb - ka + 1) / 2, k1 = half ? kb : mid;
        float s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
        constexpr int C = 32;  // samples whose values are loaded together
        for (int k0 = half ? mid : ka; k0 < k1; k0 += C) {
            float u[C], v[C], d[C];
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const bool in = k0 + q < k1;
                u[q] = in ? U[(size_t)(k0 + q) * kHid + n] : 0.0f;
                v[q] = in ? V[(size_t)(k0 + q) * kHid + n] : 0.0f;
                d[q] = in && last ? nb.dy[k0 + q] : 0.0f;
            }
#pragma unroll
            for (int q = 0; q < C; ++q) {
                s1 = fmaf(u[q], last ? d[q] : 1.0f, s1);
                s2 += v[q];
                s3 += d[q];
            }
        }
        float *red = &sm[0][0][0];
        if (half) {
            red[n] = s1;
            red[128 + n] = s2;
            if (n == 0) red[256] = s3;
        }
        __syncthreads();
        if (!half) {
            out[(last ? oW4 : ob1) + n] = s1 + red[n];
            out[(last ? ob3 : ob2) + n] = s2 + red[128 + n];
            if (last && n == 0) out[ob4] = s3 + red[256];
        }
        return;
    }
    const bool first = job >= 8;  // the first layer
    const int q = job & 3;
    const float *A = first ? X : job < 4 ? nb.H[1] : nb.H[0];
    const float *B = first ? nb.dZ[0] : job < 4 ? nb.dZ[2] : nb.dZ[1];
    const int lda = first ? kFeat : kHid, rows = first ? kFeat : kHid;
    const int m0 = first ? 0 : 64 * (q >> 1), n0 = 64 * (first ? job - 8 : q & 1);
    const int64_t o = first ? oW1 : job < 4 ? oW3 : oW2;
    const int c = lane & 31, h = lane >> 5;
    const int mt = first ? 0 : 32 * (wave >> 1), nt = 32 * (wave & 1);  // the wave's tile in the block's
    floatx16_t acc{}, odd{};  // two chains: half the roundings, and no wait between products
    for (int k0 = ka; k0 < kb; k0 += kGradChunk) {
        // 16 threads per sample row, 4 columns each
        constexpr int R = kGradChunk / 16;
        floatx4_t va[R], vb[R];
        const int e = 4 * (tid & 15);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int k = k0 + (tid >> 4) + 16 * r;
            const bool in = k < kb;
            va[r] = floatx4_t{};
            if (in && m0 + e < rows) {
                const float *src = A + (size_t)k * lda + m0 + e;
                if (!first) va[r] = *reinterpret_cast<const floatx4_t *>(src);
                else  // the caller's array may lie at any float
                    va[r] = floatx4_t{src[0], src[1], src[2], src[3]};
            }
            vb[r] = in ? *reinterpret_cast<const floatx4_t *>(B + (size_t)k * kHid + n0 + e) : floatx4_t{};
        }
        __syncthreads();  // the previous chunk's reads
#pragma unroll
        for (int r = 0; r < R; ++r) {
            *reinterpret_cast<floatx4_t *>(&sm[0][(tid >> 4) + 16 * r][e]) = va[r];
            *reinterpret_cast<floatx4_t *>(&sm[1][(tid >> 4) + 16 * r][e]) = vb[r];
        }
        __syncthreads();
        const int cnt = min(kGradChunk, kb - k0);
        if (!first || wave < 2)
            for (int k = 0; k < cnt; k += 4) {  // rows past the slice are zero
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(sm[0][k + h][mt + c], sm[1][k + h][nt + c], acc, 0, 0, 0);
                odd = __builtin_amdgcn_mfma_f32_32x32x2f32(sm[0][k + 2 + h][mt + c], sm[1][k + 2 + h][nt + c], odd, 0, 0,
                                                           0);
            }
    }
    if (first && wave >= 2) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int m = m0 + mt + 8 * (r >> 2) + 4 * h + (r & 3);
        if (m < rows) out[o + (int64_t)m * kHid + n0 + nt + c] = acc[r] + odd[r];
    }
}

// Parameter i's gradient: the sum of its ns slices in order, into G, or with
// ADAM applied (beta 0.9 / 0.999, bias correction c1, c2).  Block 0 also
// takes the loss: the mean of the samples' squares from nl terms (double,
// fixed order), to a device or a pinned host address.
template <bool ADAM>
__global__ __launch_bounds__(256) void kw_reduce(int ns, const float *__restrict__ part, float *__restrict__ G,
                                                 float *__restrict__ p, float *__restrict__ mo, float *__restrict__ ve,
                                                 float lr, float c1, float c2, int64_t nl, const double *lossp, int S,
                                                 double *loss) {
    __shared__ double red[256];
    if (blockIdx.x == 0 && loss) {
        double l = 0.0;
        for (int64_t k = threadIdx.x; k < nl; k += 256) l += lossp[k];
        red[threadIdx.x] = l;
        __syncthreads();
        for (int o = 128; o >= 1; o >>= 1) {
            if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss = red[0] / (double)S;
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= kParams) return;
    // in double: it costs nothing beside the loads
    double sum = 0.0;
#pragma unroll 8
    for (int q = 0; q < ns; ++q) sum += (double)part[(size_t)q * kParams + i];
    const float gi = (float)sum;
    if constexpr (ADAM) {
        const float mi = 0.9f * mo[i] + 0.1f * gi;
        const float vi = 0.999f * ve[i] + 0.001f * gi * gi;
        mo[i] = mi;
        ve[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
    } else {
        G[i] = gi;
    }
}

// w_i = (y_i - mean y) / N in double (one block, fixed order)
__global__ __launch_bounds__(1024) void kw_center(int n, const float *y, double *w) {
    __shared__ double red[1024];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) s += (double)y[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 512; o >= 1; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    const double mean = red[0] / (double)n;
    for (int i = threadIdx.x; i < n; i += 1024) w[i] = ((double)y[i] - mean) / (double)n;
}

// t_i = N (w_i - mean w) in float (one block, fixed order)
__global__ __launch_bounds__(1024) void kw_targets(int n, const double *w, float *t) {
    __shared__ double red[1024];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) s += w[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 512; o >= 1; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    const double mean = red[0] / (double)n;
    for (int i = threadIdx.x; i < n; i += 1024) t[i] = (float)((double)n * (w[i] - mean));
}

// ------------------------------------------------------- BF16 inference

// Inference in BF16 on the matrix cores with FP32 accumulation
// (v_mfma_f32_32x32x16_bf16): the weights are kept as transposed BF16 copies
// (layer 1 padded from 20 to 32 inputs), activations are rounded to BF16
// between layers, biases and the ReLU are applied in FP32.
constexpr int kK1 = 32;                                  // layer-1 inputs, padded
constexpr int64_t kBfW1 = 0;                             // [128][32]
constexpr int64_t kBfW2 = kBfW1 + (int64_t)kHid * kK1;   // [128][128]
constexpr int64_t kBfW3 = kBfW2 + (int64_t)kHid * kHid;  // [128][128]
constexpr int64_t kBfW4 = kBfW3 + (int64_t)kHid * kHid;  // [128]
constexpr int64_t kBfCount = kBfW4 + kHid;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned short ushort8_t __attribute__((ext_vector_type(8)));

// round to nearest even (the values are finite)
__device__ inline unsigned short to_bf16(float v) {
    const unsigned u = __float_as_uint(v);
    return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ inline float from_bf16(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

__global__ __launch_bounds__(256) void kw_to_bf16(const float *P, unsigned short *Wb) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= kBfCount) return;
    float v;
    if (e < kBfW2) {
        const int o = (int)(e / kK1), k = (int)(e % kK1);
        v = k < kFeat ? P[oW1 + (int64_t)k * kHid + o] : 0.0f;
    } else if (e < kBfW4) {
        const int64_t base = e < kBfW3 ? kBfW2 : kBfW3;
        const int64_t src = e < kBfW3 ? oW2 : oW3;
        const int o = (int)((e - base) / kHid), k = (int)((e - base) % kHid);
        v = P[src + (int64_t)k * kHid + o];
    } else {
        v = P[oW4 + (e - kBfW4)];
    }
    Wb[e] = to_bf16(v);
}

// A block per 32 samples, wave w the outputs 32 w .. 32 w + 31 of every layer,
// the weights of all layers loaded before the first product; y[s] for s < S.
// (A wave per 32 samples doing all 128 columns left 22 waves on the chip for
// 700 samples and waited for the weights product by product: 17.5 us.)
__global__ __launch_bounds__(256) void kw_infer_bf16(const float *P, const unsigned short *Wb,
                                                     const float *X, int S, float *y) {
    constexpr int kRow = kHid + 8;  // padded LDS row
    __shared__ __attribute__((aligned(16))) unsigned short act[2][32 * kRow];
    const int lane = __lane_id(), tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    const int s0 = blockIdx.x * 32, o = 32 * wave + col;
    bf16x8_t w1[kK1 / 16], w2[kHid / 16], w3[kHid / 16];
    auto load = [&](const unsigned short *Wt, int kin, int k0) {
        return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const ushort8_t *>(Wt + (int64_t)o * kin + k0 + 8 * half));
    };
#pragma unroll
    for (int k = 0; k < kK1 / 16; ++k) w1[k] = load(Wb + kBfW1, kK1, 16 * k);
#pragma unroll
    for (int k = 0; k < kHid / 16; ++k) w2[k] = load(Wb + kBfW2, kHid, 16 * k);
#pragma unroll
    for (int k = 0; k < kHid / 16; ++k) w3[k] = load(Wb + kBfW3, kHid, 16 * k);
    const float b1 = P[ob1 + o], b2 = P[ob2 + o], b3 = P[ob3 + o];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int e = tid + 256 * q, r = e / kK1, k = e % kK1;
        const float v = (s0 + r < S && k < kFeat) ? X[(int64_t)(s0 + r) * kFeat + k] : 0.0f;
        act[0][r * kRow + k] = to_bf16(v);
    }
    auto put = [&](const floatx16_t &acc, float bo, unsigned short *dst) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = 8 * (r / 4) + 4 * half + (r % 4);
            dst[row * kRow + o] = to_bf16(fmaxf(acc[r] + bo, 0.0f));
        }
    };
    auto mul = [&](const unsigned short *src, int k, const bf16x8_t &w, floatx16_t acc) {
        const bf16x8_t a = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const ushort8_t *>(src + col * kRow + 16 * k + 8 * half));
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, w, acc, 0, 0, 0);
    };
    __syncthreads();
    floatx16_t acc{};
#pragma unroll
    for (int k = 0; k < kK1 / 16; ++k) acc = mul(act[0], k, w1[k], acc);
    put(acc, b1, act[1]);
    __syncthreads();
    acc = floatx16_t{};
#pragma unroll
    for (int k = 0; k < kHid / 16; ++k) acc = mul(act[1], k, w2[k], acc);
    put(acc, b2, act[0]);
    __syncthreads();
    acc = floatx16_t{};
#pragma unroll
    for (int k = 0; k < kHid / 16; ++k) acc = mul(act[0], k, w3[k], acc);
    put(acc, b3, act[1]);
    __syncthreads();
    // output layer: y = b4 + sum_o h3[o] w4[o] (BF16 operands, FP32 sums), a lane
    // per half row
    if (wave != 0) return;
    float part = 0.0f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const ushort8_t h = *reinterpret_cast<const ushort8_t *>(&act[1][col * kRow + 64 * half + 8 * q]);
        const ushort8_t w = *reinterpret_cast<const ushort8_t *>(Wb + kBfW4 + 64 * half + 8 * q);
#pragma unroll
        for (int e = 0; e < 8; ++e) part = fmaf(from_bf16(h[e]), from_bf16(w[e]), part);
    }
    part += __shfl_xor(part, 32);
    if (half == 0 && s0 + col < S) y[s0 + col] = part + P[ob4];
}

// Slices of the samples for the weight gradients: at most kSplitMax, a
// multiple of 16 samples each.
int grad_slice(int S) { return std::max(16, ((S + kSplitMax - 1) / kSplitMax + 15) & ~15); }

// The activations of S samples in buf (act_floats(S) floats): six [S][128]
// arrays, dy, the loss terms, the slices of the gradients.
NetBufs net_bufs(float *buf, int S, float **part) {
    NetBufs nb;
    const size_t n = (size_t)S * kHid;
    for (int k = 0; k < 3; ++k) {
        nb.H[k] = buf + k * n;
        nb.dZ[k] = buf + (3 + k) * n;
    }
    // doubles at an even offset of the (256-byte aligned) buffer
    nb.lossp = reinterpret_cast<double *>(buf + 6 * n);
    float *rest = buf + 6 * n + 2 * (size_t)((S + kTS - 1) / kTS);
    nb.dy = rest;
    *part = rest + S;
    return nb;
}

// Forward, backward and the slices of the gradients.
hipError_t gradients(hipStream_t s, const float *P, const float *X, const float *t, int S, const NetBufs &nb,
                     float *part, int *ns) {
    const int slice = grad_slice(S);
    *ns = (S + slice - 1) / slice;
    kw_net<true><<<(unsigned)((S + kTS - 1) / kTS), kNetThreads, 0, s>>>(P, X, t, S, nullptr, nb);
    kw_grad<<<dim3(kGradJobs, (unsigned)*ns), 256, 0, s>>>(X, S, slice, nb, part);
    return hipGetLastError();
}

}  // namespace

// Floats of activations and gradient slices for S samples.
int64_t act_floats(int64_t S) {
    return S * (6 * kHid + 1) + 2 * ((S + kTS - 1) / kTS) + (int64_t)kSplitMax * kParams;
}

// y [S] of S samples.
hipError_t forward(hipStream_t s, const float *P, const float *X, int S, float *y) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    kw_net<false><<<(unsigned)((S + kTS - 1) / kTS), kNetThreads, 0, s>>>(P, X, nullptr, S, y, NetBufs{});
    return hipGetLastError();
}

const int64_t kBf16Count = kBfCount;

hipError_t to_bf16_weights(hipStream_t s, const float *P, unsigned short *Wb) {
    (void)hipGetLastError();
    kw_to_bf16<<<(unsigned)((kBfCount + 255) / 256), 256, 0, s>>>(P, Wb);
    return hipGetLastError();
}

hipError_t infer_bf16(hipStream_t s, const float *P, const unsigned short *Wb, const float *X, int S,
                      float *y) {
    (void)hipGetLastError();
    kw_infer_bf16<<<(unsigned)((S + 31) / 32), 256, 0, s>>>(P, Wb, X, S, y);
    return hipGetLastError();
}

// Loss (if not null, written by the device: pinned or device memory) and its
// gradient with respect to the flat parameters (into G).
hipError_t backward(hipStream_t s, const float *P, const float *X, const float *t, int S, float *buf, float *G,
                    double *loss) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    float *part;
    int ns;
    const NetBufs nb = net_bufs(buf, S, &part);
    const hipError_t e = gradients(s, P, X, t, S, nb, part, &ns);
    if (e != hipSuccess) return e;
    kw_reduce<false><<<(unsigned)((kParams + 255) / 256), 256, 0, s>>>(ns, part, G, nullptr, nullptr, nullptr, 0.0f,
                                                                       1.0f, 1.0f, (S + kTS - 1) / kTS, nb.lossp, S, loss);
    return hipGetLastError();
}

// The gradient and Adam's step number `step` on the parameters P and the
// moments M, V.
hipError_t train_step(hipStream_t s, float *P, float *M, float *V, const float *X, const float *t, int S, float *buf,
                      float lr, int64_t step, double *loss) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    float *part;
    int ns;
    const NetBufs nb = net_bufs(buf, S, &part);
    const hipError_t e = gradients(s, P, X, t, S, nb, part, &ns);
    if (e != hipSuccess) return e;
    const float c1 = 1.0f - powf(0.9f, (float)step), c2 = 1.0f - powf(0.999f, (float)step);
    kw_reduce<true><<<(unsigned)((kParams + 255) / 256), 256, 0, s>>>(ns, part, nullptr, P, M, V, lr, c1, c2,
                                                                      (S + kTS - 1) / kTS, nb.lossp, S, loss);
    return hipGetLastError();
}

hipError_t features(hipStream_t s, int n, const double *x, const double *A, const double *v,
                    const double *lo, const double *hi, const double *grad0, int *nb, double *tmp,
                    float *F) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    kw_features<<<(n + 3) / 4, 256, 0, s>>>(n, x, A, v, lo[0], lo[1], hi[0], hi[1], F, nb);
    if (n <= kPoolSeeds) {
        kw_pool_all<<<1, 1024, 0, s>>>(n, nb, grad0, F);
        return hipGetLastError();
    }
    const unsigned nb1 = (unsigned)((n + 255) / 256);
    kw_deficit<<<nb1, 256, 0, s>>>(n, grad0, tmp, F);
    for (int h = 0; h < kPoolHops; ++h) {
        const double *in = tmp + (size_t)(h & 1) * n;
        double *out = tmp + (size_t)((h + 1) & 1) * n;
        kw_pool<<<nb1, 256, 0, s>>>(n, nb, in, out, F, 17 + h);
    }
    return hipGetLastError();
}

hipError_t targets(hipStream_t s, int n, const double *w, float *t) {
    (void)hipGetLastError();
    kw_targets<<<1, 1024, 0, s>>>(n, w, t);
    return hipGetLastError();
}

hipError_t center(hipStream_t s, int n, const float *y, double *w) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    kw_center<<<1, 1024, 0, s>>>(n, y, w);
    return hipGetLastError();
}

}  // namespace ws
}  // namespace apd
