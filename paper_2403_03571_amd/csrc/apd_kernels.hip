// apd_kernels.hip -- gfx950 kernels of the APD hot path.
//
// One evaluation of the discretised dual problem (Section 2.3 of
// arXiv 2403.03571) is a chain of kernels on one stream:
//
//   k_prep        blocks of seeds, the last to finish combining their
//                 partials: gauge max of w, Gershgorin bound and
//                 eigenvalue ranges of the anisotropy matrices, input
//                 validation, zeroed moments (in a fit's graph it also
//                 takes the trial weights from pinned host memory).
//   k_super_cull  candidate lists of super-tiles (passes with lists).
//   k_assign_*    the O(N J) part (Algorithm 1): every pixel of a tile
//                 scans every seed (or the tile's candidates), keeps the
//                 argmin, and the tile reduces the exact integer moments of
//                 each cell it touched.  _fp64 evaluates
//                 C_ij = |y_j - x_i|^2_{A_i} - w_i exactly as the definition
//                 is written; _vec (FP32 vector ALU), _mfma (FP32 matrix
//                 cores) and _bf16 (bf16 matrix cores) evaluate it in local
//                 coordinates and queue every pixel whose top-two gap is
//                 within their rounding bound.
//   k_recheck_staged  re-runs the scan of every queued pixel in double, in
//                 the definition's own expression order, so every label
//                 equals that of an exact double-precision argmin (passes
//                 over every seed; passes with lists re-check in the tile).
//   k_finalize    blocks of cells, the last to finish combining them:
//                 objective (2.7), gradient (2.8), maximum relative volume
//                 error, centroids, from the moments.
//
// The whole file is built with -ffp-contract=off: the double-precision
// costs are evaluated without fused multiply-adds, and the single-precision
// path fuses only where it says so (fmaf).
#include "apd_device.h"

#include <math.h>

#include <algorithm>

namespace apd {
namespace {

using namespace dev;

// ------------------------------------------------------------- k_prep

// Up to kOneBlock seeds the prep and finalize kernels are one block with a
// seed per thread; above, blocks of kRedThreads whose last one to finish
// combines the partials.  The exchange through memory (fences that reach the
// other XCDs, the ticket, the partials read back) costs more than what the
// blocks share: prep 8.2 us for 1000 seeds in four blocks, 4.7 in one.
constexpr int kRedThreads = 256;
constexpr int kOneBlock = 1024;

// Groups for n seeds: one seed per thread of kRedThreads up to kMaxParts
// groups (blocks, above kOneBlock seeds).
__host__ __device__ inline int red_groups(int n) {
    const int k = n / kRedThreads + (n % kRedThreads ? 1 : 0);
    return k < 1 ? 1 : k > kMaxParts ? kMaxParts : k;
}

// Seeds [lo, hi) of block b when n seeds are split over gridDim.x blocks.
__device__ inline void block_range(int n, int *lo, int *hi) {
    const int per = (n + (int)gridDim.x - 1) / (int)gridDim.x;
    *lo = min(n, (int)blockIdx.x * per);
    *hi = min(n, *lo + per);
}

// True in the last block to finish; its partials and those of every other
// block (written by the blocks' threads 0) are then visible to it.
__device__ inline bool last_block(unsigned *ticket) {
    __shared__ bool s_last;
    if (threadIdx.x == 0) {
        __threadfence();
        s_last = atomicAdd(ticket, 1u) == gridDim.x - 1;
        __threadfence();
    }
    __syncthreads();
    return s_last;
}

// Validation, max_i w_i, sum_i v_i, the Gershgorin bound of the largest
// eigenvalue, the eigenvalue ranges (culling) and the zeroed moments, over
// blocks of T seeds (a single block for T = kOneBlock).  With w_only (the
// later evaluations of a fit) only what depends on the weights is formed
// again; the rest stays as the fit's first evaluation left it.
template <int D, int T>
__global__ __launch_bounds__(T) void k_prep(Geo g, Seeds sd, Scalars *sc, uint64_t *mom, double *eig, BlockParts *bp,
                                            const double *w_src, bool w_only) {
    constexpr int K = moments_per_cell(D);
    constexpr int kRedWaves = T / 64;
    __shared__ double s_w[kRedWaves];
    __shared__ double s_v[kRedWaves];
    __shared__ float s_l[kRedWaves];
    __shared__ float s_k[kRedWaves];
    __shared__ int s_b[kRedWaves];
    const int tid = threadIdx.x;
    int i0, i1;
    block_range(g.n, &i0, &i1);
    double wm = -INFINITY, vs = 0.0;
    float lam = 0.0f, kap = 0.0f;
    int bad = 0;
    for (int i = i0 + tid; i < i1; i += T) {
        double wi;
        if (w_src) {
            // the pass's weights, from the host; later kernels read sd.w
            wi = w_src[i];
            const_cast<double *>(sd.w)[i] = wi;
        } else {
            wi = sd.w[i];
        }
        if (!isfinite(wi)) bad |= kBadW;
        wm = fmax(wm, wi);
        if (w_only) continue;
        for (int d = 0; d < D; ++d)
            if (!isfinite(sd.x[(size_t)i * D + d])) bad |= kBadX;
        const double *a = sd.A + (size_t)i * D * D;
        double u[3][3];
        for (int r = 0; r < D; ++r)
            for (int c = 0; c < D; ++c) {
                u[r][c] = (r <= c) ? a[r * D + c] : a[c * D + r];
                if (!isfinite(u[r][c])) bad |= kBadA;
            }
        // Sylvester: leading principal minors positive
        bool spd = u[0][0] > 0.0;
        const double m2 = u[0][0] * u[1][1] - u[0][1] * u[0][1];
        spd = spd && m2 > 0.0;
        double det = m2;
        if (D == 3) {
            det = u[0][0] * (u[1][1] * u[2][2] - u[1][2] * u[1][2]) -
                  u[0][1] * (u[0][1] * u[2][2] - u[1][2] * u[0][2]) +
                  u[0][2] * (u[0][1] * u[1][2] - u[1][1] * u[0][2]);
            spd = spd && det > 0.0;
        }
        if (!spd) bad |= kBadSPD;
        if (eig) {
            double lo, hi;
            eig_range<D>(u, &lo, &hi);
            eig[2 * (size_t)i] = lo;
            eig[2 * (size_t)i + 1] = hi;
        }
        // Gershgorin: lambda_max <= max_r sum_c |a_rc|
        double lg = 0.0;
        for (int r = 0; r < D; ++r) {
            double rs = 0.0;
            for (int c = 0; c < D; ++c) rs += fabs(u[r][c]);
            lg = fmax(lg, rs);
        }
        lam = fmaxf(lam, (float)lg);
        if (spd) kap = fmaxf(kap, (float)cond_bound(D, lg, det));
        if (sd.v) {
            const double vi = sd.v[i];
            if (!(vi > 0.0) || !isfinite(vi)) bad |= kBadV;
            vs += vi;
        }
    }
    if (mom)
        for (size_t t = (size_t)blockIdx.x * T + tid; t < (size_t)g.n * K; t += (size_t)gridDim.x * T) mom[t] = 0ull;
    // block reduction: a butterfly inside each wave, then the wave results
    // in wave order by thread 0 (whose slots 0 then hold the block's values)
    auto reduce = [&](double a, double v, float l, float kk, int b) {
        a = wave_max(a);
        int any = 0;
#pragma unroll
        for (int bit = 1; bit <= kBadAll; bit <<= 1) any |= __ballot((b & bit) != 0) ? bit : 0;
        b = any;
        if (!w_only) {
            v = wave_sum(v);
            l = (float)wave_max((double)l);
            kk = (float)wave_max((double)kk);
        }
        __syncthreads();  // earlier readers of the slots are done
        if (__lane_id() == 0) {
            const int wv = tid >> 6;
            s_w[wv] = a;
            s_v[wv] = v;
            s_l[wv] = l;
            s_k[wv] = kk;
            s_b[wv] = b;
        }
        __syncthreads();
        if (tid == 0)
            for (int k = 1; k < kRedWaves; ++k) {
                s_w[0] = fmax(s_w[0], s_w[k]);
                s_v[0] = s_v[0] + s_v[k];
                s_l[0] = fmaxf(s_l[0], s_l[k]);
                s_k[0] = fmaxf(s_k[0], s_k[k]);
                s_b[0] = s_b[0] | s_b[k];
            }
    };
    reduce(wm, vs, lam, kap, bad);
    if constexpr (T != kOneBlock) {
        if (tid == 0) {
            bp->a[blockIdx.x] = s_w[0];
            bp->b[blockIdx.x] = s_v[0];
            bp->l[blockIdx.x] = s_l[0];
            bp->k[blockIdx.x] = s_k[0];
            bp->bad[blockIdx.x] = s_b[0];
        }
        if (!last_block(&bp->ticket)) return;
        const bool have = tid < (int)gridDim.x;
        reduce(have ? bp->a[tid] : -INFINITY, have ? bp->b[tid] : 0.0, have ? bp->l[tid] : 0.0f,
               have ? bp->k[tid] : 0.0f, have ? bp->bad[tid] : 0);
    }
    if (tid == 0) {
        float lm = s_l[0] * 1.0001f;
        if (w_only) {
            lm = sc->lam;
        } else {
            sc->vsum = s_v[0];
            sc->lam = lm;
            sc->kap = s_k[0] * 1.0001f;
        }
        sc->wmax = s_w[0];
        sc->sab = dslack_abs(g, s_w[0], lm);
        sc->lsl = list_slack(g, sc->sab, lm);
        sc->bad = s_b[0];
        sc->qcount = 0u;
        sc->credited = 0u;
        sc->gpix = 0.0;
        sc->g = 0.0;
        sc->maxrel = 0.0;
        if (!w_only) sc->qtotal = 0ull;
        if constexpr (T != kOneBlock) bp->ticket = 0u;
    }
}

// Zero n 32-bit words (a kernel rather than a memset, so that the call can
// sit inside a captured graph).
__global__ __launch_bounds__(256) void k_zero_words(unsigned *p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

// sc->gpix = sum of part[0, n) in a fixed order: thread t sums t, t + 256, ...
// in order, then a tree over the threads (one block).
__global__ __launch_bounds__(256) void k_sum_parts(const double *part, int64_t n, Scalars *sc) {
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) sc->gpix = red[0];
}

// sum_j mass[j] into sc->qtotal (after k_prep has zeroed it).
__global__ __launch_bounds__(256) void k_mass_total(int64_t J, const uint8_t *mass, Scalars *sc) {
    __shared__ unsigned long long red[256];
    unsigned long long s = 0;
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < J; j += (int64_t)gridDim.x * 256)
        s += mass[j];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(&sc->qtotal, red[0]);
}

// Seeds above which a super-tile's list is built by 512 threads.
constexpr int kSuperWideSeeds = 2048;

// ------------------------------------------------------ k_assign_fp64

// One block per tile (dev::fp64_tile): the tile's candidate seeds or every
// seed.
template <int D, bool CULL>
__global__ __launch_bounds__(kThreads) void k_assign_fp64(Geo g, Seeds sd, const Scalars *sc, const double *eig,
                                                         PassOut out) {
    __shared__ Fp64Smem<D, CULL> sm;
    const int b0 = D == 2 ? blockIdx.y : blockIdx.z;
    const int b1 = D == 2 ? blockIdx.x : blockIdx.y;
    const int b2 = D == 2 ? 0 : blockIdx.x;
    double *part = nullptr;
    if (out.cost_part) part = out.cost_part + ((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    fp64_tile<D, CULL>(g, sd, sc->wmax, Cert{sc->lam, sc->kap, sc->sab, sc->lsl}, eig, b0, b1, b2, sm, out, part);
}

// ------------------------------------------------ k_assign_fp32 / _cull

// One block per tile of the vector single-precision kernel: every seed
// (dev::vec_tile), or the tile's candidate seeds (dev::list_tile).
template <int D, int P>
__global__ __launch_bounds__(kThreads, 4) void k_assign_vec(Geo g, Seeds sd, Scalars *sc, PassOut out) {
    __shared__ VecSmem<D> sm;
    const Cert ct{sc->lam, sc->kap, sc->sab, sc->lsl};
    if constexpr (D == 2) vec_tile<2, P>(g, sd, sc->wmax, ct, blockIdx.y, blockIdx.x, 0, sm, out, &sc->qcount);
    else vec_tile<3, P>(g, sd, sc->wmax, ct, blockIdx.z, blockIdx.y, blockIdx.x, sm, out, &sc->qcount);
}

template <int D, int P, bool GAP, bool W>
__global__ __launch_bounds__(kThreads, (P <= 4 && !GAP) ? 5 : 4) void k_assign_list(Geo g, Seeds sd, Scalars *sc,
                                                                                    const double *eig, PassOut out) {
    __shared__ ListSmem<D, P, GAP, W> sm;
    const Cert ct{sc->lam, sc->kap, sc->sab, sc->lsl};
    if constexpr (D == 2)
        list_tile<2, P, GAP, W>(g, sd, sc->wmax, ct, eig, blockIdx.y, blockIdx.x, 0, sm, out, &sc->qcount);
    else
        list_tile<3, P, GAP, W>(g, sd, sc->wmax, ct, eig, blockIdx.z, blockIdx.y, blockIdx.x, sm, out, &sc->qcount);
}

// ------------------------------------------------------ k_assign_mfma

// One block per tile; the tile body (dev::mfma_tile) is shared with the
// batched persistent kernel.
template <int D>
__global__ __launch_bounds__(kThreads) void k_assign_mfma(Geo g, Seeds sd, Scalars *sc,
                                                         PassOut out) {
    __shared__ __attribute__((aligned(16))) float sC[kMfmaLds];
    if (D == 2)
        dev::mfma_tile<2>(g, sd, sc->wmax, Cert{sc->lam, sc->kap, sc->sab, sc->lsl}, blockIdx.y, blockIdx.x, 0, sC, out, &sc->qcount);
    else
        dev::mfma_tile<3>(g, sd, sc->wmax, Cert{sc->lam, sc->kap, sc->sab, sc->lsl}, blockIdx.z, blockIdx.y, blockIdx.x, sC, out,
                          &sc->qcount);
}

// ------------------------------------------------------ k_seed_order

// The seeds sorted by the Morton code of the box cell that holds them (16^3
// cells in 3D, 64^2 in 2D), by one block: counts per cell, an exclusive
// scan, then each seed's slot.  The hybrid kernel scans the seeds in this
// order, so that its super-blocks of 64 consecutive seeds cover compact
// regions and a wave's pixels fall in few of them (its winner search takes
// one round per distinct winning super-block).  Seeds of one cell take
// their slots in any order: the pass's labels, certificates and moments do
// not depend on it (an unflagged pixel's winner is the unique FP32 minimum;
// a flagged one is re-evaluated in double over every seed).
constexpr int kOrderThreads = 1024;
constexpr int kOrderBins = 4096;

template <int D>
__device__ inline int seed_bin(const Geo &g, const Seeds &sd, int i) {
    constexpr int B = D == 3 ? 16 : 64;  // cells per axis
    constexpr int BITS = D == 3 ? 4 : 6;
    int q[3] = {0, 0, 0};
    for (int d = 0; d < D; ++d) {
        const double t = (sd.x[(size_t)i * D + d] - g.lo[d]) / (g.s[d] * (double)g.grid[d]);
        q[d] = t >= 0.0 ? (int)fmin(t * B, (double)(B - 1)) : 0;  // seeds outside the box clamp
    }
    int code = 0;
    for (int b = 0; b < BITS; ++b)
        for (int d = 0; d < D; ++d) code |= ((q[d] >> b) & 1) << (D * b + d);
    return code;
}

template <int D>
__global__ __launch_bounds__(kOrderThreads) void k_seed_order(Geo g, Seeds sd, int *ord) {
    __shared__ int cnt[kOrderBins];
    __shared__ int wex[kOrderThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int b = tid; b < kOrderBins; b += kOrderThreads) cnt[b] = 0;
    __syncthreads();
    for (int i = tid; i < g.n; i += kOrderThreads) atomicAdd(&cnt[seed_bin<D>(g, sd, i)], 1);
    __syncthreads();
    // exclusive scan: thread t holds cells 4t .. 4t + 3
    constexpr int PER = kOrderBins / kOrderThreads;
    int c[PER], sum = 0;
    for (int k = 0; k < PER; ++k) {
        c[k] = cnt[PER * tid + k];
        sum += c[k];
    }
    int inc = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) wex[wave] = inc;
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int w = 0; w < kOrderThreads / 64; ++w) {
            const int t = wex[w];
            wex[w] = run;
            run += t;
        }
    }
    __syncthreads();
    int off = wex[wave] + inc - sum;
    for (int k = 0; k < PER; ++k) {
        cnt[PER * tid + k] = off;
        off += c[k];
    }
    __syncthreads();
    for (int i = tid; i < g.n; i += kOrderThreads) ord[atomicAdd(&cnt[seed_bin<D>(g, sd, i)], 1)] = i;
}

// ------------------------------------------------------ k_assign_hyb

// One block per tile (dev::hyb_tile): 16 x 16 x 8 in 3D at three blocks per
// CU, so that the scan keeps its registers (at four, spills in the scan add
// about 4 GB of scratch traffic per launch on the 3D workload for the same
// time); 32 x 32 in 2D at four.
template <int D>
__global__ __launch_bounds__(kThreads, D == 3 ? 3 : 4) void k_assign_hyb(Geo g, Seeds sd, Scalars *sc,
                                                                          PassOut out) {
    __shared__ __attribute__((aligned(16))) HybSmem<D> sm;
    if constexpr (D == 3)
        hyb_tile<3>(g, sd, sc->wmax, Cert{sc->lam, sc->kap, sc->sab, sc->lsl}, blockIdx.z, blockIdx.y, blockIdx.x, sm, out,
                    &sc->qcount);
    else
        hyb_tile<2>(g, sd, sc->wmax, Cert{sc->lam, sc->kap, sc->sab, sc->lsl}, blockIdx.y, blockIdx.x, 0, sm, out, &sc->qcount);
}

// ------------------------------------------------------ k_assign_bf16

// One block per tile of the vector kernel's shape with P pixels per lane
// (dev::bf16_tile), over every seed, staged C at a time.
template <int D, int P, int C>
__global__ __launch_bounds__(kThreads) void k_assign_bf16(Geo g, Seeds sd, Scalars *sc, PassOut out) {
    __shared__ dev::Bf16Smem<D, C> sm;
    const int b0 = D == 2 ? blockIdx.y : blockIdx.z;
    const int b1 = D == 2 ? blockIdx.x : blockIdx.y;
    const int b2 = D == 2 ? 0 : blockIdx.x;
    dev::bf16_tile<D, P, C>(g, sd, sc->wmax, Cert{sc->lam, sc->kap, sc->sab, sc->lsl}, b0, b1, b2, sm, out, &sc->qcount);
}

// --------------------------------------------------------- k_super_cull

// One block of T threads per super-tile (dev::super_tile_list).
template <int D, int T>
__global__ __launch_bounds__(T) void k_super_cull(Geo g, Seeds sd, const Scalars *sc, const double *eig, PassOut out,
                                                  Regions rg, float4 *list, int *ids, int *count) {
    __shared__ SuperSmem<D, T> sm;
    const int st = blockIdx.x;
    const size_t at = (size_t)st * (size_t)out.super_cap;
    super_tile_list<D, T>(g, sd, sc->wmax, Cert{sc->lam, sc->kap, sc->sab, sc->lsl}, eig, out, rg, st,
                          list + at * rec_vec(D), ids ? ids + at : nullptr, count + st, out.super_cap, sm);
}

// One block per region (dev::region_list).
constexpr int kRegionThreads = 1024;
template <int D>
__global__ __launch_bounds__(kRegionThreads) void k_region_cull(Geo g, Seeds sd, const Scalars *sc, const double *eig,
                                                                PassOut out, Regions rg) {
    __shared__ int s_list[kRegionCap];
    __shared__ float s_red[kRegionThreads / 64];
    __shared__ int s_cnt;
    region_list<D, kRegionThreads>(g, sd, sc->wmax, Cert{sc->lam, sc->kap, sc->sab, sc->lsl}, eig, out, rg,
                                   blockIdx.x, s_list, s_cnt, s_red);
}

// ---------------------------------------------------------- k_recheck

// Seeds per staged chunk of the re-check kernels.
template <int D> struct RecheckChunk { static constexpr int value = D == 2 ? 1024 : 512; };

// Re-check over every seed (passes without candidate lists): the seeds are
// staged in LDS chunk by chunk and a group of G lanes takes one queued
// pixel, G the largest power of two that still covers the whole queue in
// one round of the grid's waves (short queues spread each pixel over many
// lanes, long ones give every lane its own pixel); lane r of a group scans
// the staged seeds r, r + G, ... in increasing order, then the group takes
// the (value, lowest index) minimum.  The double cost is evaluated in the
// expression order of dev::exact_cost, so the labels are those of an exact
// double-precision argmin with ties to the lowest index.
template <int D>
__global__ __launch_bounds__(kThreads) void k_recheck_staged(Geo g, Seeds sd, const Scalars *sc,
                                                            PassOut out) {
    constexpr int S = RecheckChunk<D>::value;
    __shared__ StagedSeeds<D, S> sm;
    const unsigned nq = sc->qcount;
    const unsigned wslots = gridDim.x * kWaves;
    int G = 64;
    while (G > 1 && (unsigned long long)wslots * (unsigned)(64 / G) < nq) G >>= 1;
    const unsigned per_wave = 64u / (unsigned)G;
    const int lane = __lane_id();
    const int wave = threadIdx.x >> 6;
    const int n = g.n;
    for (unsigned base = 0; base < nq; base += wslots * per_wave) {
        // the whole block skips a round with none of its pixels
        const unsigned first = base + (unsigned)blockIdx.x * kWaves * per_wave;
        if (first >= nq) break;
        const unsigned pix = first + (unsigned)wave * per_wave + (unsigned)(lane / G);
        const bool valid = pix < nq;
        const uint32_t j = valid ? out.queue[pix] : 0u;
        int k[3];
        double y[D];
        pixel_of<D>(g, j, k, y);
        double b = INFINITY, s2 = INFINITY;
        int bi = 0x7fffffff;
        for (int c0 = 0; c0 < n; c0 += S) {
            const int cnt = min(S, n - c0);
            __syncthreads();
            for (int i = threadIdx.x; i < cnt; i += kThreads) stage_seed<D, S>(sm, sd, i, c0 + i);
            __syncthreads();
            for (int i = lane % G; i < cnt; i += G) {
                const double c = staged_cost<D, S>(sm, i, y);
                if (c < b) {
                    s2 = b;
                    b = c;
                    bi = c0 + i;
                } else {
                    s2 = fmin(s2, c);
                }
            }
        }
        if (out.rel_gap) group_min2(b, bi, s2, G);
        else group_min(b, bi, G);
        if (bi >= n) bi = 0;  // no finite cost (non-finite input, reported by the prep step)
        if (valid && lane % G == 0) {
            if (out.labels) out.labels[j] = bi;
            if (out.mom) dev::pixel_moments_add<D>(out.mom, bi, k, dev::pixel_weight(g, j));
            if (out.rel_gap) out.rel_gap[j] = dev::gap_exact(b, s2, sc->wmax);
        }
    }
}

// Waits for this wave's stores, so that after a barrier one thread's fence
// covers those of the whole block.  A system fence writes back the L2, and one
// by each wave of the block took most of the kernel: 8.0 -> 4.8 us for one block
// of 1024 threads, 9.4 -> 7.8 for 40 blocks (N = 10^4); a fit's evaluation at
// 1024^2, N = 1000, 53 -> 47 us.
__device__ inline void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// -------------------------------------------------------- k_finalize

// Every cell's term of eq. (2.7) (dev::cell_final) and its relative volume
// error, over blocks of cells; the terms are summed in a fixed order (a
// butterfly in each wave, the waves of 256 cells in order, then a butterfly
// over these groups), the same in one block (T = kOneBlock: four groups) and
// in several, so the objective is deterministic.
template <int D, int T>
__global__ __launch_bounds__(T) void k_finalize(Geo g, Seeds sd, const uint64_t *mom, Scalars *sc, FinalOut out,
                                                BlockParts *bp) {
    constexpr int K = moments_per_cell(D);
    constexpr int kGroupWaves = kRedThreads / 64;
    __shared__ double s_g[T / 64];
    __shared__ double s_m[T / 64];
    const int tid = threadIdx.x;
    const int groups = red_groups(g.n);  // of at most kRedThreads cells when T is kOneBlock
    const int per = (g.n + groups - 1) / groups;
    const int grp = T == kOneBlock ? tid / kRedThreads : (int)blockIdx.x;
    const int i0 = min(g.n, grp * per), i1 = min(g.n, i0 + per);
    // the scalars of the earlier kernels, loaded ahead of their use
    Scalars pass = Scalars{};
    unsigned published = 0u;
    if (tid == 0) {
        pass = *sc;
        published = bp->published;
    }
    double gs = 0.0, mr = 0.0;
    for (int i = i0 + tid % kRedThreads; i < i1; i += kRedThreads) {
        double gi, rel, ybar[3];
        gs += dev::cell_final<D>(g, sd, mom + (size_t)i * K, i, &gi, &rel, ybar);
        mr = fmax(mr, rel);
        if (out.grad) out.grad[i] = gi;
        if (out.counts) out.counts[i] = (int64_t)mom[(size_t)i * K];
        if (out.centroids)
            for (int d = 0; d < D; ++d) out.centroids[(size_t)i * D + d] = ybar[d];
    }
    auto reduce = [&](double a, double m) {
        a = wave_sum(a);
        m = wave_max(m);
        __syncthreads();
        if (__lane_id() == 0) {
            s_g[tid >> 6] = a;
            s_m[tid >> 6] = m;
        }
        __syncthreads();
        // thread 0 of each group (of the block, when it is one group)
        if (tid % kRedThreads == 0)
            for (int k = 1; k < kGroupWaves; ++k) {
                s_g[tid >> 6] = s_g[tid >> 6] + s_g[(tid >> 6) + k];
                s_m[tid >> 6] = fmax(s_m[tid >> 6], s_m[(tid >> 6) + k]);
            }
    };
    reduce(gs, mr);
    // thread 0's scalars for the host, all but seq
    auto put = [&](double gt, double mx) {
        sc->g = gt;
        sc->maxrel = mx;
        if (!out.host_sc) return;
        Scalars *h = out.host_sc;
        h->wmax = pass.wmax;
        h->vsum = pass.vsum;
        h->g = gt;
        h->maxrel = mx;
        h->qcount = pass.qcount;
        h->lam = pass.lam;
        h->bad = pass.bad;
        h->qtotal = pass.qtotal;
        h->credited = pass.credited;
        bp->published = published + 1u;
    };
    // the host waits for seq, so it goes last, after every other write of the
    // pass (each thread's, the gradient among them) has reached the host
    auto publish = [&] {
        __hip_atomic_store(&out.host_sc->seq, published + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    };
    const double gp = g.power != 2 ? g.munit * pass.gpix : 0.0;
    auto objective = [&](double sum) { return g.power != 2 ? sum + gp : sum; };
    if constexpr (T == kOneBlock) {
        // the butterfly over at most four groups; one fence covers the
        // gradient and the scalars
        if (out.host_sc) stores_done();
        __syncthreads();  // the groups' sums
        if (tid == 0) {
            double mx = s_m[0];
            for (int k = 1; k < 4; ++k) mx = fmax(mx, s_m[k * kGroupWaves]);
            put(objective((s_g[0] + s_g[2 * kGroupWaves]) + (s_g[kGroupWaves] + s_g[3 * kGroupWaves])), mx);
            if (out.host_sc) {
                __threadfence_system();
                publish();
            }
        }
    } else {
        if (tid == 0) {
            bp->a[blockIdx.x] = s_g[0];
            bp->b[blockIdx.x] = s_m[0];
        }
        if (out.host_sc) {
            stores_done();
            __syncthreads();
            if (tid == 0) __threadfence_system();
        }
        if (!last_block(&bp->ticket)) return;
        const bool have = tid < (int)gridDim.x;
        reduce(have ? bp->a[tid] : 0.0, have ? bp->b[tid] : 0.0);
        if (tid == 0) {
            put(objective(s_g[0]), s_m[0]);
            bp->ticket = 0u;
            if (out.host_sc) {
                __threadfence_system();
                publish();
            }
        }
    }
}


template <int D, int P = kP>
dim3 tile_grid(const Geo &g) {
    constexpr int E0 = tile_ext(D, P, 0), E1 = tile_ext(D, P, 1), E2 = tile_ext(D, P, 2);
    if (D == 2) return dim3((g.grid[1] + E1 - 1) / E1, (g.grid[0] + E0 - 1) / E0, 1);
    return dim3((g.grid[2] + E2 - 1) / E2, (g.grid[1] + E1 - 1) / E1, (g.grid[0] + E0 - 1) / E0);
}

// 8 pixels per lane halve the per-seed work of the lanes but give 2048-pixel
// tiles; below 1024 such tiles (4 waves per SIMD on 256 CUs) the 4-pixel
// form keeps the chip full.
template <int D>
hipError_t launch_vec(const Geo &g, const Seeds &sd, Scalars *sc, const PassOut &out, hipStream_t st) {
    if (vec_pixels_per_lane(g, false) == 8) k_assign_vec<D, 8><<<tile_grid<D, 8>(g), kThreads, 0, st>>>(g, sd, sc, out);
    else k_assign_vec<D, 4><<<tile_grid<D, 4>(g), kThreads, 0, st>>>(g, sd, sc, out);
    return hipGetLastError();
}

template <int D, bool GAP, bool W = false>
hipError_t launch_list(const Geo &g, const Seeds &sd, Scalars *sc, const double *eig, const PassOut &out,
                       hipStream_t st) {
    if (out.tp == 8) {
        k_assign_list<D, 8, GAP, W><<<tile_grid<D, 8>(g), kThreads, 0, st>>>(g, sd, sc, eig, out);
    } else if (out.tp == 4) {
        k_assign_list<D, 4, GAP, W><<<tile_grid<D, 4>(g), kThreads, 0, st>>>(g, sd, sc, eig, out);
    } else {
        if constexpr (D == 3)  // the rule takes 2 rows in 3D only
            k_assign_list<D, 2, GAP, W><<<tile_grid<D, 2>(g), kThreads, 0, st>>>(g, sd, sc, eig, out);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

int vec_pixels_per_lane(const Geo &g, bool cull, bool gap) {
    if (g.vec_p == 4 || g.vec_p == 8) return g.vec_p;
    int64_t J = 1;
    for (int d = 0; d < g.dim; ++d) J *= g.grid[d];
    // measured: with candidate lists the smaller wave boxes of 4 rows win
    // (fewer candidates per wave), except on large grids of large cells, whose
    // lists are short either way, so that halving the work per wave box pays.
    // Evaluation in us, 4 / 8 rows, at 1700 pixels per cell: 96^3 54.6 / 56.3,
    // 128^3 66.6 / 64.1, 200^3 113.8 / 100.8, 1024^2 50.2 / 50.0, 2048^2 64.9 /
    // 62.2, 4000^2 132.8 / 116.4; at 300 per cell: 128^3 109.4 / 112.5, 200^3
    // 352 / 375, 2048^2 120.7 / 136.1, 4000^2 262 / 305.
    // In 3D 2 rows (8^3 tiles) on small grids, where 16 x 8 x 8 tiles leave
    // compute units idle, and on small cells, whose wave lists they keep
    // short: 2 / 4 rows at 300 per cell 40^3 36.4 / 44.1, 64^3 53.5 / 62.3,
    // 128^3 96 / 106, 256^3 749 / 871; at 600 56^3 47.9 / 48.5, 80^3 55.1 / 60.4,
    // 128^3 78.2 / 74.3, 256^3 393 / 357; at 1700 48^3 35.3 / 36.1, 80^3 48.6 /
    // 48.7, 96^3 55.7 / 52.3.  (2D: 256^2 34.3 / 34.4, 512^2 41.4 / 42.5, 1024^2
    // 46.4 / 43.0: 4 rows.)
    if (cull && g.dim == 3) {
        const dim3 t = tile_grid<3, 4>(g);
        const int64_t tiles = (int64_t)t.x * t.y * t.z;
        if (J < (int64_t)1 << 19 && tiles < 1024) return 2;
        // not where the tiles stick out of a thin grid, whose wave boxes hold the
        // same pixels either way (600000 x 1 x 1, N = 2000: 2.6 / 1.4 ms), nor for the
        // relative gaps, whose lists come from separate bounds, which smaller
        // boxes shorten less than they multiply the tiles (256^3, N = 55924: 922 /
        // 681 us; 128^3, 6990: 102 / 97)
        if (J < (int64_t)450 * g.n && tiles * 1024 <= 2 * J && !gap) return 2;
    }
    // In 2D not from 8000 pixels per cell: the smaller tiles lie inside one cell
    // often enough to be credited whole, which the boundary-aware refinement is
    // for (4096^2 with 1000 cells: 5021 of 16384 tiles against 853 of 8192; the
    // pass itself would take 82 instead of 119 us with 8 rows).
    const bool large = J >= (int64_t)1 << (g.dim == 2 ? 22 : 21) && J >= (int64_t)1000 * g.n;
    if (cull) return large && (g.dim == 3 || J < (int64_t)8000 * g.n) ? 8 : 4;
    // over every seed, 8 rows halve the per-seed work of a lane once the grid
    // keeps the chip busy
    return J >= 1024 * 2048 ? 8 : 4;
}

template <int D>
static void launch_prep_d(const Geo &g, const Seeds &sd, Scalars *sc, uint64_t *mom, double *eig, BlockParts *bp,
                          hipStream_t st, const double *w_src, bool w_only) {
    if (g.n <= kOneBlock)
        k_prep<D, kOneBlock><<<1, kOneBlock, 0, st>>>(g, sd, sc, mom, eig, bp, w_src, w_only);
    else
        k_prep<D, kRedThreads><<<red_groups(g.n), kRedThreads, 0, st>>>(g, sd, sc, mom, eig, bp, w_src, w_only);
}

hipError_t launch_prep(const Geo &g, const Seeds &sd, Scalars *sc, uint64_t *mom, double *eig,
                       BlockParts *bp, hipStream_t st, const double *w_src, bool w_only) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    if (g.dim == 2) launch_prep_d<2>(g, sd, sc, mom, eig, bp, st, w_src, w_only);
    else launch_prep_d<3>(g, sd, sc, mom, eig, bp, st, w_src, w_only);
    return hipGetLastError();
}

int64_t fp64_blocks(const Geo &g) {
    const dim3 b = g.dim == 2 ? tile_grid<2>(g) : tile_grid<3>(g);
    return (int64_t)b.x * b.y * b.z;
}

hipError_t launch_assign_fp64(const Geo &g, const Seeds &sd, Scalars *sc, const double *eig, const PassOut &out,
                              hipStream_t st) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    if (g.dim == 2) {
        if (eig) k_assign_fp64<2, true><<<tile_grid<2>(g), kThreads, 0, st>>>(g, sd, sc, eig, out);
        else k_assign_fp64<2, false><<<tile_grid<2>(g), kThreads, 0, st>>>(g, sd, sc, eig, out);
    } else {
        if (eig) k_assign_fp64<3, true><<<tile_grid<3>(g), kThreads, 0, st>>>(g, sd, sc, eig, out);
        else k_assign_fp64<3, false><<<tile_grid<3>(g), kThreads, 0, st>>>(g, sd, sc, eig, out);
    }
    if (out.cost_part) k_sum_parts<<<1, 256, 0, st>>>(out.cost_part, fp64_blocks(g), sc);
    return hipGetLastError();
}

hipError_t launch_assign_fp32(const Geo &g, const Seeds &sd, Scalars *sc, const PassOut &out,
                              hipStream_t st) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    return g.dim == 2 ? launch_vec<2>(g, sd, sc, out, st) : launch_vec<3>(g, sd, sc, out, st);
}

template <int D>
static void launch_super(const Geo &g, const Seeds &sd, const Scalars *sc, const double *eig, const PassOut &out,
                         const Regions &rg, float4 *list, int *ids, int *count, hipStream_t st) {
    const int nb = out.nst[0] * out.nst[1] * out.nst[2];
    if (rg.rec) {
        k_region_cull<D><<<rg.nh[0] * rg.nh[1] * rg.nh[2], kRegionThreads, 0, st>>>(g, sd, sc, eig, out, rg);
        k_super_cull<D, 512><<<nb, 512, 0, st>>>(g, sd, sc, eig, out, rg, list, ids, count);
    } else if (g.n > kSuperWideSeeds) {
        // a block reads every seed: many seeds need many loads in flight
        k_super_cull<D, 512><<<nb, 512, 0, st>>>(g, sd, sc, eig, out, rg, list, ids, count);
    } else {
        k_super_cull<D, 256><<<nb, 256, 0, st>>>(g, sd, sc, eig, out, rg, list, ids, count);
    }
}

hipError_t launch_super_cull(const Geo &g, const Seeds &sd, const Scalars *sc, const double *eig,
                             const PassOut &out, const Regions &rg, float4 *list, int *ids, int *count,
                             hipStream_t st) {
    (void)hipGetLastError();
    if (g.dim == 2) launch_super<2>(g, sd, sc, eig, out, rg, list, ids, count, st);
    else launch_super<3>(g, sd, sc, eig, out, rg, list, ids, count, st);
    return hipGetLastError();
}

// Both single-precision tiers' passes over candidate lists.  The bf16 tier's
// lists are as short as the FP32 tier's (9 seeds per wave of 512 voxels), where
// blocks of 32 seeds on the matrix cores are mostly padding and their looser
// bound asks for FP32 costs all the same, so it scans them in FP32 as well:
// evaluation in us, bf16 blocks / FP32 scan, 1024^2 with 1000 cells 65.6 / 50.0,
// 2048^2 with 2467 127 / 62, 128^3 with 1233 120 / 62, 256^3 with 10^4 631 / 153.
hipError_t launch_assign_cull(const Geo &g, const Seeds &sd, Scalars *sc, const double *eig,
                              const PassOut &out, hipStream_t st) {
    (void)hipGetLastError();
    if (out.rel_gap)
        return g.dim == 2 ? launch_list<2, true>(g, sd, sc, eig, out, st)
                          : launch_list<3, true>(g, sd, sc, eig, out, st);
    if (g.mass && out.mom)
        return g.dim == 2 ? launch_list<2, false, true>(g, sd, sc, eig, out, st)
                          : launch_list<3, false, true>(g, sd, sc, eig, out, st);
    return g.dim == 2 ? launch_list<2, false>(g, sd, sc, eig, out, st)
                      : launch_list<3, false>(g, sd, sc, eig, out, st);
}

hipError_t launch_assign_mfma(const Geo &g, const Seeds &sd, Scalars *sc, const PassOut &out,
                              hipStream_t st) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    if (g.dim == 2) {
        dim3 grid((g.grid[1] + 31) / 32, (g.grid[0] + kExt0 - 1) / kExt0, 1);
        k_assign_mfma<2><<<grid, kThreads, 0, st>>>(g, sd, sc, out);
    } else {
        dim3 grid((g.grid[2] + 7) / 8, (g.grid[1] + 3) / 4, (g.grid[0] + kExt0 - 1) / kExt0);
        k_assign_mfma<3><<<grid, kThreads, 0, st>>>(g, sd, sc, out);
    }
    return hipGetLastError();
}

hipError_t launch_assign_hyb(const Geo &g, const Seeds &sd, Scalars *sc, const PassOut &out,
                             hipStream_t st) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    if (g.dim == 3) {
        dim3 grid((g.grid[2] + 7) / 8, (g.grid[1] + 15) / 16, (g.grid[0] + kHybRows3 - 1) / kHybRows3);
        k_assign_hyb<3><<<grid, kThreads, 0, st>>>(g, sd, sc, out);
    } else {
        dim3 grid((g.grid[1] + 31) / 32, (g.grid[0] + kHybRows2 - 1) / kHybRows2);
        k_assign_hyb<2><<<grid, kThreads, 0, st>>>(g, sd, sc, out);
    }
    return hipGetLastError();
}

hipError_t launch_seed_order(const Geo &g, const Seeds &sd, int *ord, hipStream_t st) {
    (void)hipGetLastError();
    if (g.dim == 3) k_seed_order<3><<<1, kOrderThreads, 0, st>>>(g, sd, ord);
    else k_seed_order<2><<<1, kOrderThreads, 0, st>>>(g, sd, ord);
    return hipGetLastError();
}

// Seeds per staged chunk of the bf16 tile: 1024 in 2D (N = 1000 is one chunk),
// 256 in 3D.
template <int D, int P>
static void launch_bf16(const Geo &g, Seeds sd, Scalars *sc, const PassOut &out, hipStream_t st) {
    k_assign_bf16<D, P, D == 2 ? 1024 : 256><<<tile_grid<D, P>(g), kThreads, 0, st>>>(g, sd, sc, out);
}

template <int D>
static void launch_bf16_rows(const Geo &g, Seeds sd, Scalars *sc, const PassOut &out, hipStream_t st) {
    if (bf16_pixels_per_lane(g) == 4) launch_bf16<D, 4>(g, sd, sc, out, st);
    else launch_bf16<D, 2>(g, sd, sc, out, st);
}

// Pixel rows per lane of the bf16 tile: 4 in 2D and 2 in 3D (where the
// tile's two matrix-core operands per block take twice the registers), or
// half the pixels per lane set for the vector kernel (4 or 8).
int bf16_pixels_per_lane(const Geo &g) {
    if (g.vec_p == 4 || g.vec_p == 8) return g.vec_p / 2;
    return g.dim == 2 ? 4 : 2;
}

hipError_t launch_assign_bf16(const Geo &g, const Seeds &sd, Scalars *sc, const PassOut &out, hipStream_t st) {
    (void)hipGetLastError();
    if (g.dim == 2) launch_bf16_rows<2>(g, sd, sc, out, st);
    else launch_bf16_rows<3>(g, sd, sc, out, st);
    return hipGetLastError();
}

hipError_t launch_recheck(const Geo &g, const Seeds &sd, const Scalars *sc, const PassOut &out,
                          hipStream_t st) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    // the seeds staged in LDS: three blocks of 48 KB or four of 40 KB per
    // compute unit
    if (g.dim == 2) k_recheck_staged<2><<<768, kThreads, 0, st>>>(g, sd, sc, out);
    else k_recheck_staged<3><<<1024, kThreads, 0, st>>>(g, sd, sc, out);
    return hipGetLastError();
}

hipError_t launch_zero(void *p, size_t bytes, hipStream_t st) {
    (void)hipGetLastError();
    const size_t n = bytes / 4;
    const unsigned nb = (unsigned)std::min<size_t>(256, (n + 255) / 256);
    if (n) k_zero_words<<<nb, 256, 0, st>>>(static_cast<unsigned *>(p), n);
    return hipGetLastError();
}

hipError_t launch_mass_total(const Geo &g, Scalars *sc, hipStream_t st) {
    (void)hipGetLastError();
    int64_t J = 1;
    for (int d = 0; d < g.dim; ++d) J *= g.grid[d];
    const unsigned nb = (unsigned)std::min<int64_t>(1024, (J + 255) / 256);
    k_mass_total<<<nb, 256, 0, st>>>(J, g.mass, sc);
    return hipGetLastError();
}

hipError_t launch_finalize(const Geo &g, const Seeds &sd, const uint64_t *mom, Scalars *sc,
                           const FinalOut &out, BlockParts *bp, hipStream_t st) {
    (void)hipGetLastError();  // clear a stale error left by an earlier call
    const int nb = red_groups(g.n);
    if (g.n <= kOneBlock) {
        if (g.dim == 2) k_finalize<2, kOneBlock><<<1, kOneBlock, 0, st>>>(g, sd, mom, sc, out, bp);
        else k_finalize<3, kOneBlock><<<1, kOneBlock, 0, st>>>(g, sd, mom, sc, out, bp);
    } else {
        if (g.dim == 2) k_finalize<2, kRedThreads><<<nb, kRedThreads, 0, st>>>(g, sd, mom, sc, out, bp);
        else k_finalize<3, kRedThreads><<<nb, kRedThreads, 0, st>>>(g, sd, mom, sc, out, bp);
    }
    return hipGetLastError();
}

}  // namespace apd
