// apd_device.h -- device building blocks shared by the single-instance and
// the batched kernels of libapd: tile layout, the exact double cost, the
// per-tile epilogue (labels, re-check queue, exact integer moments), the
// matrix-core assignment of one tile, the double re-check of one pixel and
// the finalize of one cell.  Included by the .hip sources only.
#pragma once

#include "apd_internal.h"

#include <math.h>

namespace apd {
namespace dev {

// ------------------------------------------------------------ tile layout

// A block covers a tile of pixels (tile_ext: 2D 8P x 32 as 2 x 2 waves of
// 4 x 16 lanes, 3D 16 x 16 x 8 as 2 x 2 waves of 8 x 8 lanes for P = 8, else
// 4P x 8 x 8 as 4 waves stacked along axis 0); each lane
// owns P consecutive pixels along axis 0 and a fixed position on the other
// axes, so consecutive lanes touch consecutive pixel indices along the
// last axis.

constexpr int kExt0 = kWaves * kP;  // extent along axis 0 of the matrix-core tile

template <int D>
struct Tile {
    int k0w;         // axis-0 index of this lane's first pixel
    int k[3];        // this lane's pixel indices (k[0] of p = 0)
    int org[3];      // origin of this wave's box of pixels
    int anc[3];      // tile anchor (centre) in index units
    int lane;
};

// Axis-0 index of the first pixel and the other indices of lane L of a wave
// whose box starts at org.
template <int D, int P>
__device__ inline void lane_pixel(const int *org, int L, int &k0, int &k1, int &k2) {
    if (D == 2) {
        k0 = org[0] + (L >> 4) * P;
        k1 = org[1] + (L & 15);
        k2 = 0;
    } else {
        k0 = org[0];
        k1 = org[1] + (L >> 3);
        k2 = org[2] + (L & 7);
    }
}

// Tile (b0, b1, b2): b0 along axis 0, b1 along axis 1, b2 along axis 2.
template <int D, int P = kP>
__device__ inline Tile<D> tile_at(int b0, int b1, int b2) {
    constexpr int E0 = tile_ext(D, P, 0), E1 = tile_ext(D, P, 1), E2 = tile_ext(D, P, 2);
    Tile<D> t;
    int lane = __lane_id();
    // keeps a kernel that loops over tiles from holding every value derived
    // from the lane in registers across the loop
    asm volatile("" : "+v"(lane));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    t.lane = lane;
    if (D == 2) {
        t.org[2] = 0;
    } else {
        t.org[2] = b2 * E2;
    }
    t.org[0] = b0 * E0 + wave_off(D, P, 0, wave);
    t.org[1] = b1 * E1 + wave_off(D, P, 1, wave);
    lane_pixel<D, P>(t.org, lane, t.k0w, t.k[1], t.k[2]);
    t.k[0] = t.k0w;
    t.anc[0] = b0 * E0 + E0 / 2;
    t.anc[1] = b1 * E1 + E1 / 2;
    t.anc[2] = D == 3 ? b2 * E2 + E2 / 2 : 0;
    return t;
}

// The tile of this block (grid x along the last axis).
template <int D, int P = kP>
__device__ inline Tile<D> tile_of(const Geo &g) {
    if (D == 2) return tile_at<D, P>(blockIdx.y, blockIdx.x, 0);
    return tile_at<D, P>(blockIdx.z, blockIdx.y, blockIdx.x);
}

template <int D>
__device__ inline bool lane_in_grid(const Geo &g, const Tile<D> &t) {
    bool ok = t.k[1] < g.grid[1];
    if (D == 3) ok = ok && t.k[2] < g.grid[2];
    return ok;
}

template <int D>
__device__ inline uint32_t pixel_index(const Geo &g, int k0, const Tile<D> &t) {
    if (D == 2) return (uint32_t)k0 * (uint32_t)g.grid[1] + (uint32_t)t.k[1];
    return ((uint32_t)k0 * (uint32_t)g.grid[1] + (uint32_t)t.k[1]) * (uint32_t)g.grid[2] +
           (uint32_t)t.k[2];
}

// ------------------------------------------------- exact double-precision

// Pixel centre y_d = lo_d + (k_d + 1/2) s_d (eq. (2.6)).
__device__ inline double centre(const Geo &g, int d, int k) {
    return g.lo[d] + ((double)k + 0.5) * g.s[d];
}

// |y - x|_A^power from the squared norm q, clamped at 0 for power != 2.
__device__ inline double power_of_norm(double q, int power) {
    if (power == 2) return q;
    const double qc = q > 0.0 ? q : 0.0;
    return power == 1 ? sqrt(qc) : power == 3 ? qc * sqrt(qc) : qc * qc;
}

// C_ij = (y - x_i)^T A_i (y - x_i) - w_i in the definition's order: d = y - x,
// each row of A d summed left to right, then sum_r d_r (A d)_r left to right.
// For power p != 2 the cost is |y - x_i|_{A_i}^p - w_i, from the squared
// norm q clamped at 0 as sqrt(q) (p = 1), q sqrt(q) (p = 3) or q q (p = 4).
template <int D>
__device__ inline double exact_cost(const double *__restrict__ x, const double *__restrict__ A,
                                    const double *__restrict__ w, int i, const double *y, int power = 2) {
    double d[D];
#pragma unroll
    for (int r = 0; r < D; ++r) d[r] = y[r] - x[(size_t)i * D + r];
    const double *a = A + (size_t)i * D * D;
    double q = 0.0;
#pragma unroll
    for (int r = 0; r < D; ++r) {
        double row = 0.0;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const double arc = (r <= c) ? a[r * D + c] : a[c * D + r];
            const double t = arc * d[c];
            row = (c == 0) ? t : row + t;
        }
        const double t = d[r] * row;
        q = (r == 0) ? t : q + t;
    }
    return power_of_norm(q, power) - w[i];
}

// The expanded cost of seed i about a tile anchor, for the single-precision
// tiers: with e = x_i - anchor and u = y - anchor,
//   C_i(u) = sum_{d<=e'} q_de' u_d u_e' + sum_d l_d u_d + c,
// q the upper triangle of A_i with the off-diagonal entries doubled (2D:
// a00, 2a01, a11; 3D: a00, 2a01, 2a02, a11, 2a12, a22), l = -2 A_i e and
// c = e^T A_i e - (w_i - w_max).  Computed in double, so that rounding each
// to FP32 once leaves it within 2^-24 of its own value, whatever the
// conditioning of A_i (in FP32 the cancellation in e^T A e could cost up to
// the condition number times that).
template <int D>
__device__ inline void seed_terms(const Seeds &sd, int i, const double *anc, double wmax, double *q,
                                  double *l, double *c, double *e, double *wp) {
    const double *xi = sd.x + (size_t)i * D;
    const double *a = sd.A + (size_t)i * D * D;
    for (int d = 0; d < D; ++d) e[d] = xi[d] - anc[d];
    *wp = sd.w[i] - wmax;
    double ee = 0.0;
    for (int r = 0; r < D; ++r) {
        double ae = 0.0;
        for (int k = 0; k < D; ++k) ae += a[(r <= k) ? r * D + k : k * D + r] * e[k];
        l[r] = -2.0 * ae;
        ee += e[r] * ae;
    }
    *c = ee - *wp;
    int t = 0;
    for (int r = 0; r < D; ++r)
        for (int k = r; k < D; ++k) q[t++] = (r == k ? 1.0 : 2.0) * a[r * D + k];
}

// Eigenvalue range of a symmetric 2x2 or 3x3 matrix (upper triangle u),
// closed form (the 3x3 case by the trigonometric solution of the
// characteristic cubic), widened by a relative 1e-6 for the rounding of the
// formulas.
template <int D>
__device__ inline void eig_range(const double (&u)[3][3], double *lmin, double *lmax) {
    if (D == 2) {
        const double m = 0.5 * (u[0][0] + u[1][1]);
        const double h = 0.5 * (u[0][0] - u[1][1]);
        const double r = sqrt(h * h + u[0][1] * u[0][1]);
        *lmin = m - r;
        *lmax = m + r;
    } else {
        const double p1 = u[0][1] * u[0][1] + u[0][2] * u[0][2] + u[1][2] * u[1][2];
        const double q = (u[0][0] + u[1][1] + u[2][2]) / 3.0;
        const double d0 = u[0][0] - q, d1 = u[1][1] - q, d2 = u[2][2] - q;
        const double p2 = d0 * d0 + d1 * d1 + d2 * d2 + 2.0 * p1;
        const double pp = sqrt(p2 / 6.0);
        if (pp <= 1e-300) {
            *lmin = *lmax = q;
        } else {
            const double b00 = d0 / pp, b11 = d1 / pp, b22 = d2 / pp;
            const double b01 = u[0][1] / pp, b02 = u[0][2] / pp, b12 = u[1][2] / pp;
            const double det = b00 * (b11 * b22 - b12 * b12) - b01 * (b01 * b22 - b12 * b02) +
                               b02 * (b01 * b12 - b11 * b02);
            const double rr = fmin(1.0, fmax(-1.0, 0.5 * det));
            const double phi = acos(rr) / 3.0;
            *lmax = q + 2.0 * pp * cos(phi);
            *lmin = q + 2.0 * pp * cos(phi + 2.0943951023931957);  // + 2 pi / 3
        }
    }
    const double span = fabs(*lmax) + fabs(*lmin);
    *lmin -= 1e-6 * span;
    *lmax += 1e-6 * span;
}

// --------------------------------------------------------- wave helpers

// The wave's total of v, wave-uniform, without LDS round trips: DPP adds
// within each row of 16 lanes (lane xor 1, xor 2, then the half-row and
// row mirrors), so that every lane of a row holds the row's sum, then the
// four row sums read from lanes 0, 16, 32, 48.  All lanes must be active.
__device__ inline unsigned wave_total(unsigned v) {
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);   // quad_perm 2,3,0,1
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);  // row_half_mirror
    v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false);  // row_mirror
    return (unsigned)__builtin_amdgcn_readlane((int)v, 0) + (unsigned)__builtin_amdgcn_readlane((int)v, 16) +
           (unsigned)__builtin_amdgcn_readlane((int)v, 32) + (unsigned)__builtin_amdgcn_readlane((int)v, 48);
}

// The wave's minimum, wave-uniform, the same way (float and double).
__device__ inline float wave_min(float v) {
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false)));
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false)));
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, false)));
    v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, false)));
    const int b = __float_as_int(v);
    return fminf(fminf(__int_as_float(__builtin_amdgcn_readlane(b, 0)), __int_as_float(__builtin_amdgcn_readlane(b, 16))),
                 fminf(__int_as_float(__builtin_amdgcn_readlane(b, 32)), __int_as_float(__builtin_amdgcn_readlane(b, 48))));
}
template <int CTRL>
__device__ inline double dpp_double(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ inline double lane_double(double x, int l) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ inline double wave_min(double v) {
    v = fmin(v, dpp_double<0xB1>(v));
    v = fmin(v, dpp_double<0x4E>(v));
    v = fmin(v, dpp_double<0x141>(v));
    v = fmin(v, dpp_double<0x140>(v));
    return fmin(fmin(lane_double(v, 0), lane_double(v, 16)), fmin(lane_double(v, 32), lane_double(v, 48)));
}

// The butterfly v = f(v, v of lane ^ o), o = 32, 16, 8, 4, 2, 1, for a
// commutative f, without the LDS round trips of __shfl_xor (two per step and
// double, about 100 cycles each): a half (row) swap leaves the pair's lower
// lane in one register and its upper lane in the other.  With it the prep and
// finalize of an evaluation in one block take 3.8 + 4.0 instead of 4.3 + 4.8 us.
template <class F>
__device__ inline double wave_butterfly(double v, F f) {
    auto swapped = [&](auto swap) {
        const long long b = __double_as_longlong(v);
        const auto lo = swap((unsigned)(b & 0xffffffffll)), hi = swap((unsigned)(b >> 32));
        auto join = [](unsigned l, unsigned h) { return __longlong_as_double(((long long)h << 32) | (long long)l); };
        return f(join(lo[0], hi[0]), join(lo[1], hi[1]));
    };
    v = swapped([](unsigned x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
    v = swapped([](unsigned x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
    v = f(v, dpp_double<0x128>(v));                    // row_ror:8
    v = f(v, dpp_double<0x1B>(dpp_double<0x141>(v)));  // ^ 7, then ^ 3
    v = f(v, dpp_double<0x4E>(v));
    return f(v, dpp_double<0xB1>(v));
}
__device__ inline double wave_sum(double v) {
    return wave_butterfly(v, [](double a, double b) { return a + b; });
}
__device__ inline double wave_max(double v) {
    return wave_butterfly(v, [](double a, double b) { return fmax(a, b); });
}

// ------------------------------------------------------ tile epilogue

// The labels of the settled pixels (a flagged pixel's is written by the
// re-check).
template <int D, int P>
__device__ inline void write_labels(const Geo &g, const Tile<D> &t, const bool (&act)[P], const int (&lab)[P],
                                    const bool (&flag)[P], const PassOut &out) {
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (act[p] && !flag[p]) out.labels[pixel_index<D>(g, t.k0w + p, t)] = lab[p];
}

// Labels, the re-check queue (where the pass has one), and the exact
// per-cell moments of every settled pixel.  For a cell the moments are the pixel count and the sums
// of o_d = 2 k_d + 1 and o_d o_e over its pixels (unsigned 64-bit atomics,
// so the result does not depend on the order of the additions).  Within a
// wave the pixels of one cell are first summed in 32 bits relative to the
// wave origin, then shifted to global coordinates once.
template <int D, int P = kP>
__device__ inline void tile_epilogue(const Geo &g, const Tile<D> &t, const bool (&act)[P],
                                     const int (&lab)[P], const bool (&flag)[P],
                                     const PassOut &out, unsigned *qcount) {
    constexpr int K = moments_per_cell(D);
    const int lane = t.lane;
    if (out.labels) write_labels<D, P>(g, t, act, lab, flag, out);
    // re-check queue: one atomic per block (the counter is a single address
    // shared by every block of the pass).  Every thread of the block comes
    // here (the queue pointers are uniform), so the barriers are safe.
    if (out.queue || out.queue64) {
        __shared__ unsigned s_q[kWaves + 1];
        const int wave = threadIdx.x >> 6;
        unsigned long long mk[P];
        unsigned tot = 0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            mk[p] = __ballot(act[p] && flag[p]);
            tot += (unsigned)__popcll(mk[p]);
        }
        if (lane == 0) s_q[wave] = tot;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned all = 0;
            for (int w = 0; w < kWaves; ++w) all += s_q[w];
            unsigned first = 0u;
            if (all && out.segs) {
                // pixels and segments with one atomic on the (pixels,
                // segments) pair
                const unsigned long long old =
                    atomicAdd(reinterpret_cast<unsigned long long *>(qcount), (1ull << 32) | all);
                first = (unsigned)old;
                out.segs[(unsigned)(old >> 32)] = QSeg{first, all, out.tile_id, (int32_t)out.tag};
            } else if (all) {
                first = atomicAdd(qcount, all);
            }
            s_q[kWaves] = first;
        }
        __syncthreads();
        if (tot) {
            unsigned base = s_q[kWaves];
            for (int w = 0; w < wave; ++w) base += s_q[w];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const unsigned long long m = mk[p];
                if (act[p] && flag[p]) {
                    const unsigned below = __builtin_amdgcn_mbcnt_hi(
                        (unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
                    const uint32_t j = pixel_index<D>(g, t.k0w + p, t);
                    if (out.queue64) out.queue64[base + below] = ((uint64_t)out.tag << 32) | j;
                    else out.queue[base + below] = j;
                }
                base += (unsigned)__popcll(m);
            }
        }
    }
    if (!out.mom) return;
    bool pend[P];
    unsigned qw[P];  // pixel weights (1 without them)
#pragma unroll
    for (int p = 0; p < P; ++p) {
        pend[p] = act[p] && !flag[p];
        qw[p] = (pend[p] && g.mass) ? (unsigned)g.mass[pixel_index<D>(g, t.k0w + p, t)] : 1u;
    }
    // the lane's position on axes 1, 2 is fixed: its pixels' monomials are
    // those of o0 (count, sum, sum of squares) times lane constants
    const unsigned o1 = 2u * (unsigned)(t.k[1] - t.org[1]) + 1u;
    const unsigned o2 = D == 3 ? 2u * (unsigned)(t.k[2] - t.org[2]) + 1u : 0u;
    const uint64_t G[3] = {2ull * (uint64_t)t.org[0], 2ull * (uint64_t)t.org[1],
                           2ull * (uint64_t)t.org[2]};
    for (;;) {
        int L = -1;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (L < 0) {
                const unsigned long long m = __ballot(pend[p]);
                if (m) L = __builtin_amdgcn_readlane(lab[p], __ffsll(m) - 1);
            }
        }
        if (L < 0) break;
        unsigned s0 = 0u, s1 = 0u, s2 = 0u;  // sum q, q o0, q o0^2 over this lane's pixels of L
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (pend[p] && lab[p] == L) {
                pend[p] = false;
                const unsigned o0 = 2u * (unsigned)(t.k0w - t.org[0] + p) + 1u;
                const unsigned q = qw[p];
                s0 += q;
                s1 += q * o0;
                s2 += q * o0 * o0;
            }
        }
        unsigned acc[K];
        if constexpr (D == 2) {
            // 1, o0, o1, o0^2, o0 o1, o1^2
            acc[0] = s0; acc[1] = s1; acc[2] = s0 * o1; acc[3] = s2; acc[4] = s1 * o1; acc[5] = s0 * (o1 * o1);
        } else {
            // 1, o0, o1, o2, o0^2, o0 o1, o0 o2, o1^2, o1 o2, o2^2
            acc[0] = s0; acc[1] = s1; acc[2] = s0 * o1; acc[3] = s0 * o2; acc[4] = s2; acc[5] = s1 * o1;
            acc[6] = s1 * o2; acc[7] = s0 * (o1 * o1); acc[8] = s0 * (o1 * o2); acc[9] = s0 * (o2 * o2);
        }
#pragma unroll
        for (int c = 0; c < K; ++c) acc[c] = wave_total(acc[c]);
        // global o = G + local o with G_d = 2 org_d; every lane forms the
        // cell's K sums, lane q adds the q-th: one instruction, K
        // consecutive 8-byte atomics in one or two 64-byte lines
        const uint64_t m = acc[0];
        uint64_t val[K];
        val[0] = m;
#pragma unroll
        for (int d = 0; d < D; ++d) val[1 + d] = m * G[d] + acc[1 + d];
        {
            int c = 0;
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int e = d; e < D; ++e, ++c)
                    val[1 + D + c] = m * G[d] * G[e] + G[d] * (uint64_t)acc[1 + e] +
                                     G[e] * (uint64_t)acc[1 + d] + (uint64_t)acc[1 + D + c];
        }
        uint64_t mine = 0;
#pragma unroll
        for (int q = 0; q < K; ++q) mine = lane == q ? val[q] : mine;
        if (lane < K)
            atomicAdd((unsigned long long *)out.mom + (size_t)L * K + lane, (unsigned long long)mine);
    }
}

// Moments of one pixel in global coordinates (re-check path).
template <int D>
__device__ inline void pixel_moments_add(uint64_t *mom, int L, const int *k, uint64_t q = 1) {
    constexpr int K = moments_per_cell(D);
    if (q == 0) return;
    unsigned long long *dst = (unsigned long long *)mom + (size_t)L * K;
    uint64_t o[3];
    for (int d = 0; d < D; ++d) o[d] = 2ull * (uint64_t)k[d] + 1ull;
    atomicAdd(dst, (unsigned long long)q);
    for (int d = 0; d < D; ++d) atomicAdd(dst + 1 + d, (unsigned long long)(q * o[d]));
    int c = 0;
    for (int d = 0; d < D; ++d)
        for (int e = d; e < D; ++e, ++c)
            atomicAdd(dst + 1 + D + c, (unsigned long long)(q * o[d] * o[e]));
}

// Moments of a whole box of pixels k_d in [a_d, b_d] in one go (closed
// forms of the sums of o = 2k + 1 and of its products): over an interval
// sum o = (b + 1)^2 - a^2 and sum o^2 = F(b + 1) - F(a), F(K) = K (4K^2 - 1) / 3
// (the sum of the first K odd squares), multiplied by the pixel counts of
// the other axes.  Exact in unsigned 64-bit arithmetic for the grids the
// moments allow.
template <int D>
__device__ inline void box_moments_add(uint64_t *mom, int L, const int *a, const int *b) {
    constexpr int K = moments_per_cell(D);
    uint64_t n[3] = {1, 1, 1}, s1[3] = {0, 0, 0}, s2[3] = {0, 0, 0};
    auto F = [](uint64_t k) { return k * (4ull * k * k - 1ull) / 3ull; };
    for (int d = 0; d < D; ++d) {
        const uint64_t lo = (uint64_t)a[d], hi = (uint64_t)b[d] + 1ull;
        n[d] = hi - lo;
        s1[d] = hi * hi - lo * lo;
        s2[d] = F(hi) - F(lo);
    }
    uint64_t m = 1;
    for (int d = 0; d < D; ++d) m *= n[d];
    unsigned long long *dst = (unsigned long long *)mom + (size_t)L * K;
    atomicAdd(dst, (unsigned long long)m);
    for (int d = 0; d < D; ++d) atomicAdd(dst + 1 + d, (unsigned long long)(m / n[d] * s1[d]));
    int c = 0;
    for (int d = 0; d < D; ++d)
        for (int e = d; e < D; ++e, ++c) {
            uint64_t v;
            if (d == e) {
                v = m / n[d] * s2[d];
            } else {
                uint64_t rest = 1;
                for (int f = 0; f < D; ++f)
                    if (f != d && f != e) rest *= n[f];
                v = rest * s1[d] * s1[e];
            }
            atomicAdd(dst + 1 + D + c, (unsigned long long)v);
        }
}

// Weight of pixel j in the moments: its q_j with pixel weights, else 1.
__device__ inline unsigned pixel_weight(const Geo &g, uint32_t j) {
    return g.mass ? (unsigned)g.mass[j] : 1u;
}

// ------------------------------------------- slack of the double costs

// The labels must agree with the double-precision evaluation of the
// definition (d = y - x, each row of A d, d^T (A d), minus w), whose own
// rounding is not zero.  For seed i with cost C <= B its error is at most
// 2^-48 ((kappa + 1) B + |w_max| + lambda_G sum_d Y_d^2): the products and
// sums of the form carry at most 12 roundings of 2^-53 each over terms
// summing to |d|^T |A| |d| <= lambda_G |d|^2 <= kappa |d|_A^2 <= kappa C,
// the subtraction of w over |w| <= |w_max| + C, and the rounding of y and d
// (|y_d| <= Y_d = |lo_d| + M_d s_d) adds 2 lambda_G |dd| |d| <= 2^-50
// (lambda_G sum Y_d^2 + 2 kappa C).  The certificates add twice that, with
// 2^-44 in place of 2^-48, to the required gap: the absolute part here, the
// part proportional to B as kslack() (B + r^2) (the r^2 covers the double
// rounding of the expansion's own coefficients, seed_terms, whose terms
// sum to at most lambda_G |e|^2 <= kappa (sqrt(B) + r)^2).
__device__ inline float dslack_abs(const Geo &g, double wmax, float lam) {
    double y2 = 0.0;
    for (int d = 0; d < g.dim; ++d) {
        const double y = fabs(g.lo[d]) + (double)g.grid[d] * g.s[d];
        y2 += y * y;
    }
    return (float)(0x1p-44 * (fabs(wmax) + (double)lam * y2));
}
// Slack of the owner-difference lists besides each seed's own: twice the
// double costs', plus 2^-20 of a pixel's scale lam s^2, above what underflow in
// FP32 can take from the terms.  Infinite (no lists) where the pixels' or the
// box's scale leaves the range in which that holds; the FP64 tier takes
// problems of any scale.
__device__ inline float list_slack(const Geo &g, float sab, float lam) {
    double smin = INFINITY, ext = 0.0;
    for (int d = 0; d < g.dim; ++d) {
        smin = fmin(smin, g.s[d]);
        ext = fmax(ext, g.s[d] * (double)g.grid[d]);
    }
    const double px = (double)lam * smin * smin, bx = (double)lam * ext * ext;
    const bool in = px >= 1e-31 && bx <= 1e31 && lam >= 1e-18f && lam <= 1e18f && smin >= 1e-18 && ext <= 1e18;
    return in ? 2.0f * sab + 0x1p-20f * (float)px : INFINITY;
}
__device__ inline float kslack(Cert ct) { return 0x1p-44f * (ct.kap + 1.0f); }

// Rounding bounds of the single-precision costs (derivations at vec_tile and
// bf16_tile) for any seed whose true cost, in the gauge w - w_max, is at
// most B, at a pixel at offset u from the tile anchor, r^2 = lambda_G |u|^2:
//   FP32 vector tile: gamma_9 S <= 2^-20 (B + 4 r sqrt(B) + 4 r^2)
//                     (gamma_9 = 0.5625 2^-20: a factor 1.78 to spare);
//   bf16 tile:        2^-15 (3 r^2 + 2 r sqrt(B)) + 2^-18 B
//                     (the proven 2^-15 (2.27 r^2 + 1.26 r sqrt(B)) +
//                     1.07 2^-19 B, with room).
__device__ inline float e32_bound(float B, float r, float r2) {
    return 0x1p-20f * (B + 4.0f * r * sqrtf(B) + 4.0f * r2);
}
__device__ inline float e16_bound(float B, float r, float r2) {
    return 0x1p-15f * (3.0f * r2 + 2.0f * r * sqrtf(B)) + 0x1p-18f * B;
}
// r^2 of a pixel at offset u (1.01 covers the FP32 rounding of this product)
__device__ inline float pixel_r2(Cert ct, float u0, float u1, float u2) {
    return ct.lam * fmaf(u0, u0, fmaf(u1, u1, u2 * u2)) * 1.01f;
}

// Certified lower bound of the relative top-two gap (C_(2) - C_(1)) / C_(2)
// (costs in the gauge w - w_max, so non-negative) of a settled pixel, from
// an upper bound c1u of the winner's true cost and a lower bound c2l of
// every other seed's: 1 - c1u / c2l, made smaller by 2^-20 for the FP32
// rounding of this expression; 0 when c2l <= 0, 1 when it is infinite.
// Costs of 1e37 and above are those of padding slots (1.7e38): pad_inf maps
// them to +infinity before any bound is formed, so nothing overflows.
__device__ inline float pad_inf(float c) { return c >= 1e37f ? INFINITY : c; }
__device__ inline float gap_lower(float c1u, float c2l) {
    if (c2l == INFINITY) return 1.0f;  // no other seed (only padding)
    if (!(c2l > 0.0f)) return 0.0f;
    const float g = (c2l - c1u) / c2l * (1.0f - 0x1p-20f);
    return g > 0.0f ? fminf(g, 1.0f) : 0.0f;
}
// The gap in double from the exact best and runner-up costs b <= s of the
// definition (weights not shifted): (s - b) / (s + w_max), rounded down to
// FP32; 1 for a single seed (s infinite).
__device__ inline float gap_exact(double b, double s, double wmax) {
    if (isinf(s) && s > 0.0) return 1.0f;
    const double den = s + wmax;
    if (!(den > 0.0)) return 0.0f;
    const double g = (s - b) / den;
    return g > 0.0 ? __double2float_rd(g) : 0.0f;
}

// Orders this wave's LDS writes before its lanes' later reads (and earlier
// reads before later writes): the wave's own barrier.
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------- moments on the matrix cores

// The moments of a tile whose pixels carry a small cell index (their
// position in the tile's candidate list) are a contraction: for each cell the
// sum over the pixels of (pixel in cell) times (monomials of the pixel), both
// small exact integers.  v_mfma_i32_16x16x64_i8 forms it for 16 cells x 64
// pixels x 16 columns: the cells' indicator on the rows, the pixels' monomials on the columns, from
// a constant table.  With o_d = 2 (k_d - anchor_d) + 1 the columns are 1, the
// o_d, and for each product o_d o_e its high and low part (o_d o_e = 32 h + l,
// 0 <= l < 32, so that both fit a signed byte up to tiles of 64 rows); the
// sums stay far below 2^31.  The waves add their cells' sums in LDS, one slot
// per cell of the tile's list, and the block writes each cell it holds once:
// m, S_d and S_de shifted from the anchor to global coordinates in 64 bits.
//
// Before, every wave reduced each of its cells by itself (10 wave totals of
// 11 instructions, the shift in 64 bits and 10 atomics to memory for each of
// about 4 cells per wave): half of the instructions of the 3D kernel, which
// went from 252 to 158 us (256^3, N = 10^4), the 2D one from 15.9 to 12.6 us
// (1024^2, N = 1000) and the batched one from 1.32 to 1.13 ms per evaluation
// (512 maps).
constexpr int kAccSlots = 64;  // cells of a tile (longer lists: tile_epilogue)

template <int D, int P>
struct MomTab {
    static constexpr int kSteps = P < 4 ? 4 : P;
    static constexpr int kProd = D * (D + 1) / 2;
    signed char v[kWaves][kSteps][64][16];
    int total[kWaves][16];  // each column's sum over the wave's pixels
    // step s, lane l, byte b: column l % 16 of pixel p = 4 (s / 4) + b % 4 of lane
    // 16 (l / 16) + 4 (s % 4) + b / 4 of the wave (the order in which the rows'
    // operand holds the pixels)
    constexpr MomTab() : v(), total() {
        constexpr int E[3] = {tile_ext(D, P, 0), tile_ext(D, P, 1), tile_ext(D, P, 2)};
        for (int w = 0; w < kWaves; ++w)
            for (int s = 0; s < kSteps; ++s)
                for (int q = 0; q < 64; ++q) {  // the pixels of the step: 4 groups of 16 bytes
                    const int L = 16 * (q / 16) + 4 * (s % 4) + (q % 16) / 4, p = 4 * (s / 4) + q % 4;
                    if (p >= P) continue;
                    const int k0 = wave_off(D, P, 0, w) + (D == 2 ? (L >> 4) * P : 0) + p;
                    const int k1 = wave_off(D, P, 1, w) + (D == 2 ? L & 15 : L >> 3);
                    const int o[3] = {2 * (k0 - E[0] / 2) + 1, 2 * (k1 - E[1] / 2) + 1,
                                      D == 3 ? 2 * ((L & 7) - E[2] / 2) + 1 : 0};
                    int col[16] = {};
                    col[0] = 1;
                    int c = 0;
                    for (int d = 0; d < D; ++d) {
                        col[1 + d] = o[d];
                        for (int e = d; e < D; ++e, ++c) {
                            const int t = o[d] * o[e];
                            col[1 + D + c] = t >> 5;
                            col[1 + D + kProd + c] = t & 31;
                        }
                    }
                    for (int n = 0; n < 16; ++n) {
                        v[w][s][16 * (q / 16) + n][q % 16] = (signed char)col[n];
                        total[w][n] += col[n];
                    }
                }
    }
};
template <int D, int P>
static __device__ const MomTab<D, P> mom_tab{};

typedef int intx4 __attribute__((ext_vector_type(4)));

// LDS of the moments: the cells' sums and each wave's byte selectors.
template <int P, bool W = false>
struct MomSmem {
    int acc[kAccSlots][16];
    alignas(16) unsigned sel[kWaves][2][(P + 3) / 4][64];
    alignas(16) unsigned wgt[W ? kWaves : 0][2][(P + 3) / 4][64];  // the weights' low and high 4 bits
};

// Zeroes the first n slots (a barrier must follow).
template <int P, bool W>
__device__ inline void moments_zero(MomSmem<P, W> &sm, int n) {
    for (int q = threadIdx.x; q < n * 16; q += kThreads) (&sm.acc[0][0])[q] = 0;
}

// Adds this wave's pixels: byte p % 4 of v[p / 4] the cell index of pixel p,
// below ncell (<= kAccSlots), or 127 (not counted); slot(j) the tile's slot of
// cell j.  Every lane of the wave must call it.
//
// The indicator operand holds 0 for a pixel of the row's cell and -1 for any
// other, and the sums start from the columns' totals, so each sum is the
// cell's own.  One byte permutation makes four entries: the pixels' indices
// relative to 8 consecutive cells are its selectors (bit 7 set, which selects
// 0xff, where the pixel is in none of them; each lane writes its own pixels'
// selectors once) and the lane's row is a table of 8 bytes.  A byte compare in
// the operand's layout took 3.4 instructions for four entries, 66 more per wave
// of 512 voxels.
//
// With pixel weights (W: mass, bytes; pix(p) the index of pixel p, below 0
// outside the grid) the entries of the row's cell are the weights' low and then
// their high 4 bits, in two products, and the sums start from zero (each wave
// reducing its cells by itself: 256^3, N = 10^4 270 us, so 193; 4000^2, N = 9411
// 182, 159).
template <int D, int P, bool W, class Slot, class Pix>
__device__ inline void moments_add(MomSmem<P, W> &sm, int lane, const unsigned (&v)[(P + 3) / 4], int ncell, Slot slot,
                                   const uint8_t *mass, Pix pix) {
    constexpr int S = MomTab<D, P>::kSteps, H = (P + 3) / 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane >> 4, col = lane & 15;
    intx4 tab[S];
#pragma unroll
    for (int k = 0; k < S; ++k) tab[k] = *reinterpret_cast<const intx4 *>(&mom_tab<D, P>.v[wave][k][lane][0]);
    const int total = mom_tab<D, P>.total[wave][col];
    const unsigned long long lut = ~(0xffull << (8 * (col & 7)));
    auto mask = [&](unsigned sel) { return __builtin_amdgcn_perm((unsigned)(lut >> 32), (unsigned)lut, sel); };
    if constexpr (W) {
#pragma unroll
        for (int hh = 0; hh < H; ++hh) {
            unsigned q[4], lo = 0u, hi = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t k = 4 * hh + j < P ? pix(4 * hh + j) : -1;
                q[j] = k >= 0 ? mass[k] : 0u;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lo |= (q[j] & 15u) << (8 * j);
                hi |= (q[j] >> 4) << (8 * j);
            }
            sm.wgt[wave][0][hh][lane] = lo;
            sm.wgt[wave][1][hh][lane] = hi;
        }
    }
    for (int j0 = 0; j0 < ncell; j0 += 16) {
        if (j0) wave_lds_sync();  // the selectors are read by other lanes
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int hh = 0; hh < H; ++hh) {
                // bytes are below 128, so no sum carries between them
                const unsigned y = v[hh] ^ ((unsigned)(j0 + 8 * h) * 0x01010101u);
                sm.sel[wave][h][hh][lane] = ((y + 0x78787878u) & 0x80808080u) | y;
            }
        wave_lds_sync();
        const int start = W ? 0 : total;
        intx4 sum = {start, start, start, start}, high = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const int at = 16 * row + 4 * (k % 4);
            intx4 a = *reinterpret_cast<const intx4 *>(&sm.sel[wave][col >> 3][k / 4][at]);
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = (int)mask((unsigned)a[e]);
            if constexpr (W) {
                intx4 lo = *reinterpret_cast<const intx4 *>(&sm.wgt[wave][0][k / 4][at]);
                intx4 hi = *reinterpret_cast<const intx4 *>(&sm.wgt[wave][1][k / 4][at]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    hi[e] &= ~a[e];
                    a[e] = lo[e] & ~a[e];
                }
                high = __builtin_amdgcn_mfma_i32_16x16x64_i8(hi, tab[k], high, 0, 0, 0);
            }
            sum = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, tab[k], sum, 0, 0, 0);
        }
        if constexpr (W) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] += 16 * high[r];
        }
        // register r: cell j0 + 4 row + r, column col
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = j0 + 4 * row + r;
            if (sum[r] != 0 && j < ncell) atomicAdd(&sm.acc[slot(j)][col], sum[r]);
        }
    }
}
// The same from an array of indices.
template <int D, int P, class Slot>
__device__ inline void moments_add(MomSmem<P> &sm, int lane, const int (&idx)[P], int ncell, Slot slot) {
    unsigned v[(P + 3) / 4];
#pragma unroll
    for (int hh = 0; hh < (P + 3) / 4; ++hh) {
        v[hh] = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            v[hh] |= (unsigned)(4 * hh + j < P ? idx[4 * hh + j < P ? 4 * hh + j : 0] : 127) << (8 * j);
    }
    moments_add<D, P, false>(sm, lane, v, ncell, slot, nullptr, [](int) { return (int64_t)-1; });
}

// Adds the tile's cells to the moments (after a barrier): list[k] the seed of
// slot k < n, anc the tile's anchor.
template <int D, int P, bool W>
__device__ inline void moments_flush(const MomSmem<P, W> &sm, const int *anc, const int *list, int n, uint64_t *mom) {
    constexpr int K = moments_per_cell(D);
    constexpr int NP = MomTab<D, P>::kProd;
    const int q = threadIdx.x & 15;
    // the pair (d, e) of this thread's product
    const int c = max(0, q - 1 - D);
    const int d = D == 2 ? (c == 2) : (c < 3 ? 0 : c < 5 ? 1 : 2);
    const int e = D == 2 ? (c >= 1) : (c < 3 ? c : c < 5 ? c - 2 : 2);
    auto G = [&](int k) { return (int64_t)(2u * (unsigned)(k == 0 ? anc[0] : k == 1 ? anc[1] : anc[2])); };
    for (int k = threadIdx.x >> 4; k < n; k += kThreads / 16) {
        const int *a = sm.acc[k];
        const int m = a[0];
        if (m == 0 || q >= K) continue;
        int64_t val = m;
        if (q > D) {
            const int64_t Gd = G(d), Ge = G(e);
            val = (int64_t)m * (Gd * Ge) + Gd * a[1 + e] + Ge * a[1 + d] + (int64_t)32 * a[1 + D + c] + a[1 + D + NP + c];
        } else if (q > 0) {
            val = (int64_t)m * G(q - 1) + a[q];
        }
        atomicAdd((unsigned long long *)mom + (size_t)list[k] * K + q, (unsigned long long)val);
    }
}

// ------------------------------------------- double re-check in the tile

// (value, seed) minimum over the G lanes of a group (G a power of two up to
// 64, groups aligned within the wave): the lowest seed among equal values.
__device__ inline void group_min(double &b, int &bi, int G) {
    for (int o = G / 2; o >= 1; o >>= 1) {
        const double ob = __shfl_xor(b, o);
        const int oi = __shfl_xor(bi, o);
        if (ob < b || (ob == b && oi < bi)) {
            b = ob;
            bi = oi;
        }
    }
}

// The same with the runner-up value s (the smallest value other than the
// winner's, ties included) carried along.
__device__ inline void group_min2(double &b, int &bi, double &s, int G) {
    for (int o = G / 2; o >= 1; o >>= 1) {
        const double ob = __shfl_xor(b, o);
        const int oi = __shfl_xor(bi, o);
        const double os = __shfl_xor(s, o);
        if (ob < b || (ob == b && oi < bi)) {
            s = fmin(os, b);
            b = ob;
            bi = oi;
        } else {
            s = fmin(s, ob);
        }
    }
}

// Double re-check of a wave's flagged pixels inside the tile's kernel (passes
// with candidate lists): all against the tile's list (list[0, nlist), seed
// numbers) or, without one, every seed 0 .. nlist - 1.  The list holds every
// seed that can attain the minimum anywhere in the tile, exact ties included,
// so the (value, lowest seed) minimum equals that of a scan over every seed
// in the definition's order.  A group of G lanes takes one pixel (G the
// largest power of two, up to 64, that leaves a group for every flagged pixel
// of the wave) and lane r of the group reads the seeds r, r + G, ... from
// global memory: a few pixels cost one round of loads and a reduction, and
// with many flagged every lane has its own.  About 2 in 10^4 pixels come
// here; a queue in global memory and a kernel of its own for them took 4.5 us
// per pass in 2D, 8.7 in 3D, and one list per tile to be written for it.
//
// scr: room of the wave for 64 P entries.  Writes the pixels' labels and
// moments, and with rel_gap their relative top-two gaps (gap_exact): the
// runner-up over the list, or, below it, the list's bound U (in the gauge
// w - w_max) under which no seed outside the list costs.  Every lane of the
// wave must call it.
template <int D, int P>
__device__ inline void recheck_flagged(const Geo &g, const Seeds &sd, const Tile<D> &t, const bool (&act)[P],
                                       const bool (&flag)[P], const int *list, int nlist, uint16_t *scr,
                                       const PassOut &out, unsigned *qcount, double wmax, double U) {
    static_assert(P <= 8, "a flagged pixel's code holds the lane and p");
    unsigned count = 0;
    unsigned long long mk[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        mk[p] = __ballot(act[p] && flag[p]);
        count += (unsigned)__popcll(mk[p]);
    }
    if (!count) return;
    const int lane = t.lane;
    wave_lds_sync();  // earlier reads of the room are done
    unsigned base = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const unsigned below = __builtin_amdgcn_mbcnt_hi((unsigned)(mk[p] >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((unsigned)mk[p], 0u));
        if (act[p] && flag[p]) scr[base + below] = (uint16_t)(lane | (p << 6));
        base += (unsigned)__popcll(mk[p]);
    }
    if (lane == 0 && qcount) atomicAdd(qcount, count);
    wave_lds_sync();
    int G = 64;
    while (G > 1 && (unsigned)(64 / G) < count) G >>= 1;
    const unsigned ngroups = (unsigned)(64 / G);
    const int grp = lane / G, r = lane % G;
    for (unsigned p0 = 0; p0 < count; p0 += ngroups) {
        const unsigned q = p0 + (unsigned)grp;
        const bool valid = q < count;
        const int code = valid ? scr[q] : 0;
        int k[3];
        lane_pixel<D, P>(t.org, code & 63, k[0], k[1], k[2]);
        k[0] += code >> 6;
        double y[D];
        for (int d = 0; d < D; ++d) y[d] = centre(g, d, k[d]);
        double b = INFINITY, s2 = INFINITY;
        int bi = 0x7fffffff;
        for (int z = r; z < nlist; z += G) {
            const int i = list ? list[z] : z;
            const double c = exact_cost<D>(sd.x, sd.A, sd.w, i, y);
            if (c < b || (c == b && i < bi)) {
                s2 = b;
                b = c;
                bi = i;
            } else {
                s2 = fmin(s2, c);
            }
        }
        if (out.rel_gap) group_min2(b, bi, s2, G);
        else group_min(b, bi, G);
        if (bi >= g.n) bi = 0;  // no finite cost (non-finite input, reported by the prep step)
        if (valid && r == 0) {
            uint32_t j = (uint32_t)k[0];
            for (int d = 1; d < D; ++d) j = j * (uint32_t)g.grid[d] + (uint32_t)k[d];
            if (out.labels) out.labels[j] = bi;
            if (out.mom) pixel_moments_add<D>(out.mom, bi, k, pixel_weight(g, j));
            if (out.rel_gap) {
                // a seed outside the list costs more than U - w_max (unshifted)
                const double su = U - wmax;
                out.rel_gap[j] = su < s2 ? gap_exact(b, su - 1e-9 * fabs(U), wmax) : gap_exact(b, s2, wmax);
            }
        }
    }
}

// ------------------------------------------------------ k_assign_mfma

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ inline int med3i(int a, int b, int c) { return max(min(a, b), min(max(a, b), c)); }
// (asm: next to med3i the compiler takes min(a, b) apart and makes two of it)
__device__ inline int min3i(int a, int b, int c) {
    int r;
    asm("v_min3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Single precision on the matrix cores.  The cost of seed i at pixel j in
// tile-local coordinates is a dot product of K = 6 (2D) or 10 (3D) terms,
//   C_ij = sum_k c_k(i) phi_k(u_j),
// c = (a00, 2a01, a11, -2(Ae)_0, -2(Ae)_1, e^T A e - w') and
// phi = (u0^2, u0 u1, u1^2, u0, u1, 1) in 2D (the 3D analogue has K = 10),
// so a 32-seed x 32-pixel block of costs is K/2 v_mfma_f32_32x32x2f32 with
// the seeds on the rows (operand A) and the pixels on the columns (operand
// B).  Each lane's 16 accumulators then hold one pixel against 16 seeds, and
// the running argmin stays inside the lane: the cost's float bits, whose low
// 4 mantissa bits are replaced by the accumulator number, order like the
// costs as signed integers, so min and med3 track the best and the
// runner-up in 3 ALU operations per pair.  The 32-seed block that last
// improved the best is recorded per pixel; the two half-waves, which hold
// the same pixels against the other 16 seeds, are merged at the end.
//
// Accumulator layout of the 32x32x2 f32 MFMA (one block): register r of
// lane l holds row 8 (r / 4) + 4 (l / 32) + (r % 4), column l % 32.
//
// Rounding bound as for k_assign_fp32, plus the 4 dropped mantissa bits
// (2^-19 relative of each compared cost).
// Tile (b0, b1, b2) of the grid: b0 along axis 0, b1 along axis 1, b2 along
// axis 2 (3D).  sC is the block's LDS staging area (kMfmaLds floats).
template <int D>
__device__ inline void mfma_tile(const Geo &g, const Seeds &sd, double wmax, Cert ct, int b0,
                                 int b1, int b2, float *sC, const PassOut &out,
                                 unsigned *qcount) {
    constexpr int KK = D == 2 ? 3 : 5;    // MFMA steps, K = 2 KK
    constexpr int SPS = D == 2 ? 8 : 16;  // floats per seed in LDS (two parity halves)
    constexpr int G = kP;                 // 32-pixel groups per wave, stacked on axis 0
    constexpr int E1 = D == 2 ? 32 : 4;   // group extent on axis 1
    constexpr int E2 = D == 2 ? 1 : 8;    // group extent on axis 2
    constexpr float kPad = 1.7e38f;       // cost of padding seeds

    const int lane = __lane_id();
    const int half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    Tile<D> t;
    t.lane = lane;
    if (D == 2) {
        t.org[0] = b0 * kExt0 + wave * G;
        t.org[1] = b1 * E1;
        t.org[2] = 0;
        t.k[1] = t.org[1] + col;
        t.k[2] = 0;
        t.anc[0] = b0 * kExt0 + kExt0 / 2;
        t.anc[1] = b1 * E1 + E1 / 2;
        t.anc[2] = 0;
    } else {
        t.org[0] = b0 * kExt0 + wave * G;
        t.org[1] = b1 * E1;
        t.org[2] = b2 * E2;
        t.k[1] = t.org[1] + col / E2;
        t.k[2] = t.org[2] + col % E2;
        t.anc[0] = b0 * kExt0 + kExt0 / 2;
        t.anc[1] = b1 * E1 + E1 / 2;
        t.anc[2] = b2 * E2 + E2 / 2;
    }
    t.k[0] = t.org[0];
    t.k0w = t.org[0];
    bool lane_ok = t.k[1] < g.grid[1];
    if (D == 3) lane_ok = lane_ok && t.k[2] < g.grid[2];

    float s[3];
    double anc[3];
    for (int d = 0; d < D; ++d) {
        s[d] = (float)g.s[d];
        anc[d] = g.lo[d] + (double)t.anc[d] * g.s[d];
    }
    // operand B: features of this lane's pixel in every group, parity = half
    float bf[G][KK];
    bool act[kP];
    {
        const float u1 = ((float)(t.k[1] - t.anc[1]) + 0.5f) * s[1];
        const float u2 = D == 3 ? ((float)(t.k[2] - t.anc[2]) + 0.5f) * s[2] : 0.0f;
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            act[gi] = lane_ok && half == 0 && (t.k0w + gi) < g.grid[0];
            const float u0 = ((float)(t.k0w + gi - t.anc[0]) + 0.5f) * s[0];
            if (D == 2) {
                const float ev[3] = {u0 * u0, u1 * u1, u1};
                const float od[3] = {u0 * u1, u0, 1.0f};
#pragma unroll
                for (int q = 0; q < KK; ++q) bf[gi][q] = half ? od[q] : ev[q];
            } else {
                const float ev[5] = {u0 * u0, u0 * u2, u1 * u2, u0, u2};
                const float od[5] = {u0 * u1, u1 * u1, u2 * u2, u1, 1.0f};
#pragma unroll
                for (int q = 0; q < KK; ++q) bf[gi][q] = half ? od[q] : ev[q];
            }
        }
    }

    int best[G], second[G], blk[G];
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
        best[gi] = 0x7fffffff;
        second[gi] = 0x7fffffff;
        blk[gi] = 0;
    }

    for (int base = 0; base < g.n; base += kChunk) {
        const int cnt = min(kChunk, g.n - base);
        const int padded = (cnt + 31) & ~31;
        __syncthreads();
        for (int q = threadIdx.x; q < padded; q += kThreads) {
            float *dst = sC + q * SPS;
            if (q >= cnt) {
                for (int z = 0; z < SPS; ++z) dst[z] = 0.0f;
                dst[SPS / 2 + KK - 1] = kPad;  // the constant term (odd parity, last step)
                continue;
            }
            const int i = base + q;
            double qd[6], ld[3], cd, ed[3], wpd;
            seed_terms<D>(sd, i, anc, wmax, qd, ld, &cd, ed, &wpd);
            if (D == 2) {
                // even k: a00, a11, -2(Ae)_1 ; odd k: 2a01, -2(Ae)_0, cc
                dst[0] = (float)qd[0]; dst[1] = (float)qd[2]; dst[2] = (float)ld[1]; dst[3] = 0.0f;
                dst[4] = (float)qd[1]; dst[5] = (float)ld[0]; dst[6] = (float)cd; dst[7] = 0.0f;
            } else {
                // even k: a00, 2a02, 2a12, -2(Ae)_0, -2(Ae)_2
                // odd k:  2a01, a11, a22, -2(Ae)_1, cc
                dst[0] = (float)qd[0]; dst[1] = (float)qd[2]; dst[2] = (float)qd[4]; dst[3] = (float)ld[0];
                dst[4] = (float)ld[2]; dst[5] = 0.0f; dst[6] = 0.0f; dst[7] = 0.0f;
                dst[8] = (float)qd[1]; dst[9] = (float)qd[3]; dst[10] = (float)qd[5]; dst[11] = (float)ld[1];
                dst[12] = (float)cd; dst[13] = 0.0f; dst[14] = 0.0f; dst[15] = 0.0f;
            }
        }
        __syncthreads();
        for (int cb = 0; cb < padded; cb += 32) {
            const float *src = sC + (cb + col) * SPS + half * (SPS / 2);
            float av[KK];
            {
                const float4 v0 = *reinterpret_cast<const float4 *>(src);
                av[0] = v0.x; av[1] = v0.y; av[2] = v0.z;
                if (D == 3) {
                    const float4 v1 = *reinterpret_cast<const float4 *>(src + 4);
                    av[3] = v0.w; av[4] = v1.x;
                }
            }
            const int sblk = base + cb;
            // all groups' products first, so the matrix cores run ahead of
            // the ALU work of the argmin
            floatx16 acc[G];
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
                acc[gi] = floatx16{};
#pragma unroll
                for (int q = 0; q < KK; ++q)
                    acc[gi] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[q], bf[gi][q], acc[gi], 0, 0, 0);
            }
#pragma unroll
            for (int gi = 0; gi < G; ++gi) {
                const int old = best[gi];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = (__float_as_int(acc[gi][r]) & ~15) | r;
                    second[gi] = med3i(best[gi], key, second[gi]);
                    best[gi] = min(best[gi], key);
                }
                blk[gi] = (best[gi] != old) ? sblk : blk[gi];
            }
        }
    }

    // merge the half-waves, decode the seed, certify
    float umax2;
    {
        const float h0 = (0.5f * kExt0 - 0.5f) * s[0];
        const float h1 = (0.5f * E1 - 0.5f) * s[1];
        umax2 = h0 * h0 + h1 * h1;
        if (D == 3) {
            const float h2 = (0.5f * E2 - 0.5f) * s[2];
            umax2 += h2 * h2;
        }
    }
    const float r2 = ct.lam * umax2 * 1.01f;
    const float sab = ct.sab, skb = kslack(ct);
    const float rr = sqrtf(r2);
    constexpr float rho = 0x1p-18f;
    int lab[kP];
    bool flag[kP];
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
        const int r = best[gi] & 15;
        const int seed = blk[gi] + 8 * (r >> 2) + 4 * half + (r & 3);
        const int ob = __shfl_xor(best[gi], 32);
        const int os = __shfl_xor(second[gi], 32);
        const int oseed = __shfl_xor(seed, 32);
        const bool other = ob < best[gi] || (ob == best[gi] && oseed < seed);
        const int nb = other ? ob : best[gi];
        const int ns = min(max(best[gi], ob), min(second[gi], os));
        lab[gi] = min(other ? oseed : seed, g.n - 1);
        const float fb = __int_as_float(nb), fs = __int_as_float(ns);
        const float bb = fmaxf(fb, 0.0f);
        const float B1 = bb + 0x1p-10f * (bb + r2);
        const float T = 2.0f * B1 + 4.0f * rr * sqrtf(B1) + 5.0f * r2;
        const float thr = 2.0f * rho * T + 0x1p-18f * fmaxf(fabsf(fb), fabsf(fs)) + sab + skb * (B1 + r2);
        flag[gi] = !((fs - fb) > thr);
        if (out.rel_gap && act[gi] && !flag[gi]) {
            const float c1u = (fb + 0x1p-19f * fabsf(fb) + rho * T + sab + skb * (B1 + r2)) * (1.0f + 0x1p-20f);
            const float f2 = pad_inf(fs);
            const float bs = fmaxf(f2, 0.0f);
            const float B2 = bs + 0x1p-10f * (bs + r2);
            const float eT2 = rho * (2.0f * B2 + 4.0f * rr * sqrtf(B2) + 5.0f * r2);
            const float c2l =
                f2 == INFINITY ? f2 : (f2 - 0x1p-19f * fabsf(f2) - eT2 - sab - skb * (B2 + r2)) * (1.0f - 0x1p-20f);
            out.rel_gap[pixel_index<D>(g, t.k0w + gi, t)] = fs > 0.0f ? gap_lower(c1u, c2l) : 0.0f;
        }
    }
    tile_epilogue<D>(g, t, act, lab, flag, out, qcount);
}

// ------------------------------------------------- vector fp32 tile

// Single precision on the vector ALU, with a certified margin.  For the tile
// anchor a (tile centre) and u = y - a, e_i = x_i - a:
//   C_ij = (u - e)^T A (u - e) - w_i' = u^T A u - 2 u^T A e + e^T A e - w_i'
// with w' = w - max w <= 0 (the argmin does not change under a common shift).
// The coefficients of the quadratic in u are formed per tile in LDS; each
// lane evaluates it for its kPv pixels along axis 0 as
//   C = (a00 u0 + beta) u0 + alpha,
// beta and alpha being the parts that depend only on the lane's other axes
// (3 FMA per seed and lane, 2 per pair).  The running argmin keeps the cost's
// float bits with the low 4 mantissa bits replaced by the seed's index within
// a group of 16 (signed-integer order is the cost order), so one and_or,
// one min and one med3 keep the best and the runner-up; the group that last
// improved the best is recorded once per 16 seeds.
//
// Rounding bound.  Write the cost as the sum of its monomials m: q_de u_d u_e,
// l_d u_d and c, and let S = sum |m|.  Each monomial reaches the computed
// cost through at most 9 roundings of relative size 2^-24 (3D; 8 in 2D):
// its FP32 coefficient (1; formed in double, seed_terms), its factors
// u_d = fl(fl(s_d) (k_d - a_d + 1/2)) (2 each, at most 2 factors) and the
// fused multiply-adds on its way (2 inside beta or alpha, then the 2 of
// the Horner step), so |C_fp32 - C| <= gamma_9 S, gamma_9 = 9u/(1 - 9u)
// < 2^-20 (u = 2^-24).  For a seed of true cost C: the quadratic part is at
// most |u|^T |A| |u| <= lambda_G |u|^2 <= r^2 (lambda_G the Gershgorin bound
// max_r sum_c |a_rc|, r^2 = lambda_G |u|max^2), the linear part
// 2 sum_d |(Ae)_d u_d| <= 2 |u| |Ae| <= 2 r sqrt(e^T A e), the constant
// e^T A e + w_max - w >= 0, and sqrt(e^T A e) <= sqrt(C) + r, so
// S <= C + 4 r sqrt(C) + 4 r^2, and T = 2B + 4 r sqrt(B) + 5 r^2 >= 1.13 S
// for every C <= B.  Hence |C_fp32 - C| <= rho T with rho = 2^-18 (4.5
// times gamma_9 / 1.13), for any symmetric positive definite A_i.
// A pixel is settled when C_(2) - C_(1) > 2 rho T(B1) + 2^-18 max|C| (the
// key bits dropped by the short scan) + the slack of the double costs
// (dslack_abs, kslack), B1 an upper bound of the true C_(1): any seed j
// with C_j <= B1 then has C_j >= C_(2) - rho T > C_(1) + rho T, one with
// C_j > B1 exceeds the winner's cost outright.  Every other pixel goes to
// the double re-check.
constexpr int kPv = 8;  // pixels per lane of the vector kernel (4 on small grids)


// Separate bounds of the costs, for the super-tiles and for the passes that
// return the relative gaps.  For the box B spanned by the tile's pixel centres,
//   min_{y in B} C_i(y) >= lmin_i dist(x_i, B)^2 - w_i'        = LB_i
//   max_{y in B} C_i(y) <= lmax_i maxdist(x_i, B)^2 - w_i'     = UB_i
// (lmin, lmax the eigenvalue range of A_i), so a seed with LB_i above
// U = min_k UB_k is beaten everywhere in the tile by the seed attaining U
// and cannot be the argmin (nor a near-tie) at any of its pixels.  The
// bounds are evaluated in double and widened by a relative 1e-9, far above
// the rounding of the double costs, so the candidate list contains every
// seed the exact double argmin could pick.  The argmin and its certificate
// are then those of k_assign_fp32 restricted to the candidates; the labels
// are unchanged.  Tiles with more than kCullCap candidates scan every seed.


// The box spanned by the pixel centres of the block of pixels starting at
// k0 with extents ext (clipped to the grid).
template <int D>
__device__ inline void cull_box(const Geo &g, const int *k0, const int *ext, double *blo, double *bhi) {
    for (int d = 0; d < D; ++d) {
        const int a = k0[d];
        const int b = min(a + ext[d], g.grid[d]) - 1;
        blo[d] = centre(g, d, a);
        bhi[d] = centre(g, d, max(b, a));
    }
}

template <class T> __device__ inline T tmin(T a, T b) { return a < b ? a : b; }
template <class T> __device__ inline T tmax(T a, T b) { return a > b ? a : b; }

// Range of the 2D quadratic form q(d) = a00 d0^2 + a01x2 d0 d1 + a11 d1^2
// (positive definite) over the box [p0, P0] x [p1, P1] of offsets d: the
// maximum is at a corner (q is convex); the minimum is 0 when the box holds
// d = 0, else it lies on an edge, where q is a 1D convex quadratic with its
// minimum at the stationary point clamped to the edge.
template <class T>
__device__ inline void quad_box_range2(T a00, T a01x2, T a11, T p0, T P0, T p1, T P1, T *qmin, T *qmax) {
    auto q = [&](T d0, T d1) { return a00 * d0 * d0 + a01x2 * d0 * d1 + a11 * d1 * d1; };
    auto clampv = [](T v, T lo, T hi) { return tmin(tmax(v, lo), hi); };
    *qmax = tmax(tmax(q(p0, p1), q(P0, p1)), tmax(q(p0, P1), q(P0, P1)));
    if (p0 <= T(0) && P0 >= T(0) && p1 <= T(0) && P1 >= T(0)) {
        *qmin = T(0);
        return;
    }
    T m = q(clampv(-a01x2 * p1 / (T(2) * a00), p0, P0), p1);
    m = tmin(m, q(clampv(-a01x2 * P1 / (T(2) * a00), p0, P0), P1));
    m = tmin(m, q(p0, clampv(-a01x2 * p0 / (T(2) * a11), p1, P1)));
    m = tmin(m, q(P0, clampv(-a01x2 * P0 / (T(2) * a11), p1, P1)));
    *qmin = m;
}

// Lower and upper bounds of seed i's cost C_i(y) - (w_i - wmax) over the box:
// in 2D with EXACT the exact range of the quadratic form (quad_box_range2),
// else the eigenvalue bounds lambda_min dist^2 and lambda_max maxdist^2.  The slack
// covers the rounding of either form: the absolute values of the form's
// terms sum to at most D lambda_max maxdist^2 (|2 a_rc d_r d_c| <=
// a_rr d_r^2 + a_cc d_c^2 for positive definite A).
//
// For costs of another power the range of the squared norm is taken to that
// power (both grow with it).  There the rounding of the double norm counts as
// its square root when the norm is near zero, sqrt(12 2^-53) sqrt(D lambda_max)
// maxdist < 1e-7 h for power 1 (less for 3 and 4): the slack is 1e-6 (h + |w'|),
// and that of an offset of the weights.
template <int D, bool EXACT = true>
__device__ inline void cull_bounds(const Seeds &sd, const double *eig, double wmax, const double *blo,
                                   const double *bhi, int i, double *lb, double *ub, int power = 2) {
    double dist2 = 0.0, far2 = 0.0;
    for (int d = 0; d < D; ++d) {
        const double xd = sd.x[(size_t)i * D + d];
        const double dd = fmax(0.0, fmax(blo[d] - xd, xd - bhi[d]));
        const double fd = fmax(xd - blo[d], bhi[d] - xd);
        dist2 += dd * dd;
        far2 += fd * fd;
    }
    const double wp = sd.w[i] - wmax;
    double l = eig[2 * (size_t)i] * dist2, h = eig[2 * (size_t)i + 1] * far2;
    const double slack = 1e-9 * (fabs(l) + (double)D * fabs(h) + fabs(wp));
    if constexpr (D == 2 && EXACT) {
        const double *a = sd.A + (size_t)i * 4;
        const double x0 = sd.x[(size_t)i * 2], x1 = sd.x[(size_t)i * 2 + 1];
        quad_box_range2<double>(a[0], 2.0 * a[1], a[3], blo[0] - x0, bhi[0] - x0, blo[1] - x1, bhi[1] - x1,
                                &l, &h);
    }
    if (power != 2) {
        l = power_of_norm(l, power);
        h = power_of_norm(h, power);
        const double sp = 1e-6 * (h + fabs(wp)) + 0x1p-44 * fabs(wmax);
        *lb = l - wp - sp;
        *ub = h - wp + sp;
        return;
    }
    *lb = l - wp - slack;
    *ub = h - wp + slack;
}

// Block-wide: of the seeds id(0) .. id(nsrc - 1) those whose lower bound
// does not exceed the smallest upper bound U, written to dst (at most cap of
// them, in any order); returns their number (which may exceed cap) and U in
// *Uout: every seed left out costs more than U everywhere in the box (what a
// pass that returns the relative gaps needs).  All threads of the block call
// it.  Up to kReg seeds per thread keep their bounds in registers between the
// two passes, as each takes about ten scattered loads: 256^3 with relative
// gaps, N = 27962 590 -> 440 us.
template <int D, class Id>
__device__ inline int build_candidates(const Seeds &sd, const double *eig, double wmax,
                                       const double *blo, const double *bhi, Id id,
                                       int nsrc, int *dst, int cap, int &s_cnt, double *s_red,
                                       double *Uout, int power = 2) {
    const int lane = __lane_id();
    constexpr int kReg = 8;
    const bool in_regs = nsrc <= kReg * kThreads;
    double lbr[kReg];
    int ir[kReg];
    double umin = INFINITY;
    if (in_regs) {
#pragma unroll
        for (int r = 0; r < kReg; ++r) {
            const int q = threadIdx.x + r * kThreads;
            lbr[r] = INFINITY;
            ir[r] = 0;
            if (q < nsrc) {
                double ub;
                ir[r] = id(q);
                cull_bounds<D, true>(sd, eig, wmax, blo, bhi, ir[r], &lbr[r], &ub, power);
                umin = fmin(umin, ub);
            }
        }
    } else {
        for (int q = threadIdx.x; q < nsrc; q += kThreads) {
            double lb, ub;
            cull_bounds<D, true>(sd, eig, wmax, blo, bhi, id(q), &lb, &ub, power);
            umin = fmin(umin, ub);
        }
    }
    umin = wave_min(umin);
    __syncthreads();  // s_cnt and s_red may still be read by an earlier use
    if (threadIdx.x == 0) s_cnt = 0;
    if (lane == 0) s_red[threadIdx.x >> 6] = umin;
    __syncthreads();
    const double U = fmin(fmin(s_red[0], s_red[1]), fmin(s_red[2], s_red[3]));
    *Uout = U;
    auto emit = [&](bool cand, int i) {
        const unsigned long long m = __ballot(cand);
        int base = 0;
        if (lane == 0 && m) base = atomicAdd(&s_cnt, (int)__popcll(m));
        base = __builtin_amdgcn_readlane(base, 0);
        const int below = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
        if (cand && base + below < cap) dst[base + below] = i;
    };
    if (in_regs) {
#pragma unroll
        for (int r = 0; r < kReg; ++r)
            if (r * kThreads < nsrc) emit((int)threadIdx.x + r * kThreads < nsrc && lbr[r] <= U, ir[r]);
    } else {
        for (int q0 = 0; q0 < nsrc; q0 += kThreads) {
            const int q = q0 + threadIdx.x;
            bool cand = false;
            int i = 0;
            if (q < nsrc) {
                i = id(q);
                double lb, ub;
                cull_bounds<D, true>(sd, eig, wmax, blo, bhi, i, &lb, &ub, power);
                cand = lb <= U;
            }
            emit(cand, i);
        }
    }
    __syncthreads();
    return s_cnt;
}

// ---- owner-difference lists
//
// The lists of the super-tiles, tiles and waves keep a seed only if it can
// beat the box's owner somewhere in the box.  The owner o is the candidate of least cost at
// the box centre; for any other candidate j the difference C_j - C_o is a
// quadratic in the offset d from the centre, so over |d_k| <= h_k
//   C_j - C_o >= (C_j - C_o)(0) - sum_k |g_k| h_k
//                + sum_k min(0, m_kk) h_k^2 - sum_{r<k} |m_rk| h_r h_k,
// g the difference of the gradients at the centre, m that of the matrices
// (off-diagonals doubled).  A seed whose bound is above the slack costs more
// than the owner at every point of the box, so it is not the argmin there
// (ties included).  This is much tighter than comparing separate bounds of
// the costs, whose ranges over the box are wide and move together: on the 3D
// workload (256^3, N = 10^4) a 16 x 8 x 8 tile keeps 17 seeds instead of 40
// and a wave 5.8 instead of 11.9, of which 3.8 win somewhere (2D 1024^2,
// N = 1000: 11 instead of 20, and 3.8 instead of 8.2).
//
// A seed about a box centre: the offset e = x - centre (formed in double),
// the upper triangle of A and w - w_max, in FP32.
template <int D>
struct SeedRec {
    static constexpr int kTri = D * (D + 1) / 2;
    float e[D];
    float a[kTri];
    float wp;
};

template <int D>
__device__ inline SeedRec<D> seed_rec(const Seeds &sd, double wmax, const double *ctr, int i) {
    const double *xi = sd.x + (size_t)i * D;
    const double *ai = sd.A + (size_t)i * D * D;
    SeedRec<D> r;
    int t = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        r.e[d] = (float)(xi[d] - ctr[d]);
#pragma unroll
        for (int k = d; k < D; ++k) r.a[t++] = (float)ai[d * D + k];
    }
    r.wp = (float)(sd.w[i] - wmax);
    return r;
}

// Its cost and gradient at the centre and its matrix (off-diagonals
// doubled); s is its share of the slack.
template <int D>
struct CellQuad {
    static constexpr int kTri = D * (D + 1) / 2;
    float c;
    float s;
    float g[D];
    float a[kTri];
};

// Cost e^T A e - w', gradient -2 A e; hh = |h|^2.  Slack: with E = |e| + |h|
// and S = lambda_G E^2 + |w'| the terms of the bound above sum to at most S in
// magnitude and reach it through fewer than 24 roundings of 2^-24, less than
// 2^-18 S per seed; s = 2^-15 (lam (|e|^2 + |h|^2) + |w'|) >= 2^-16 S, four times
// that.  An offset that is shifted from another centre (shift_slack) carries
// that shift's error besides.
template <int D>
__device__ inline CellQuad<D> cell_quad(const SeedRec<D> &r, float lam, float hh) {
    CellQuad<D> q;
    float e2 = hh, c = 0.0f;
    int t = 0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        float ae = 0.0f;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const int lo = j < k ? j : k, hi = j < k ? k : j;
            ae = fmaf(r.a[lo * D - lo * (lo - 1) / 2 + hi - lo], r.e[k], ae);
        }
        q.g[j] = -2.0f * ae;
        c = fmaf(r.e[j], ae, c);
        e2 = fmaf(r.e[j], r.e[j], e2);
#pragma unroll
        for (int k = j; k < D; ++k, ++t) q.a[t] = k > j ? 2.0f * r.a[t] : r.a[t];
    }
    q.c = c - r.wp;
    q.s = 0x1p-15f * fmaf(lam, e2, fabsf(r.wp));
    return q;
}

// What hh grows by for offsets formed from those about another centre, `shift`
// away, by an addition in FP32.  The stored offset, the shift and their sum leave
// at most t = 2^-22 |shift| in e besides relative roundings of e itself, and
// |shift| can be many times E: a last tile of one pixel under a super-tile of
// eight has h = 0.  The terms are then off by at most 2 lambda_G t E + lambda_G t^2
// more.  With 2^-10 |shift|^2 added to hh, the three quarters of s that the
// roundings leave hold 2^-15 lambda_G (3/8 E^2 + 2^-10 |shift|^2) >= 2^-19.7 lambda_G
// E |shift|, against 2^-21 lambda_G E |shift| (1 + 2^-20).
template <int D>
__device__ inline float shift_slack(const float *shift, float hh) {
#pragma unroll
    for (int d = 0; d < D; ++d) hh = fmaf(0x1p-10f * shift[d], shift[d], hh);
    return hh;
}

// Whether q can cost as little as the owner o somewhere in the box of half
// extents h (NaN counts as yes).
template <int D>
__device__ inline bool can_beat(const CellQuad<D> &q, const CellQuad<D> &o, const float *h, float slack) {
    float lb = q.c - o.c;
#pragma unroll
    for (int d = 0; d < D; ++d) lb = fmaf(-fabsf(q.g[d] - o.g[d]), h[d], lb);
    int t = 0;
#pragma unroll
    for (int r = 0; r < D; ++r)
#pragma unroll
        for (int k = r; k < D; ++k, ++t) {
            const float m = q.a[t] - o.a[t];
            lb = fmaf(r == k ? fminf(m, 0.0f) : -fabsf(m), h[r] * h[k], lb);
        }
    return !(lb > q.s + o.s + slack);
}

// Lane l's quadratic, wave-uniform.
template <int D>
__device__ inline CellQuad<D> lane_quad(const CellQuad<D> &q, int l) {
    auto get = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    CellQuad<D> r;
    r.c = get(q.c);
    r.s = get(q.s);
#pragma unroll
    for (int d = 0; d < D; ++d) r.g[d] = get(q.g[d]);
#pragma unroll
    for (int t = 0; t < CellQuad<D>::kTri; ++t) r.a[t] = get(q.a[t]);
    return r;
}

// Centre (double) and half extents (rounded up) of a box.
template <int D>
__device__ inline float box_centre(const double *blo, const double *bhi, double *ctr, float *h) {
    float hh = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        ctr[d] = 0.5 * (blo[d] + bhi[d]);
        h[d] = (float)(0.5 * (bhi[d] - blo[d])) * (1.0f + 0x1p-20f);
        hh = fmaf(h[d], h[d], hh);
    }
    return hh;
}

// Block-wide (T threads): of the seeds load(0) .. load(nsrc - 1), SeedRec
// about the centre of a box of half extents h, those that can beat the
// owner of the box somewhere in it, the owner included; keep(q, rec, pos) is
// called for each with its position in the list (in any order).  Returns
// their number.  slack: of the double costs (twice dslack_abs).
template <int D, int T, class Load, class Keep>
__device__ inline int owner_filter(int nsrc, Load load, const float *h, float hh, float lam, float slack, int &s_cnt,
                                   CellQuad<D> *s_own, Keep keep) {
    const int lane = __lane_id();
    // a short source keeps each thread's records in registers between the
    // two passes; a long one is read twice
    constexpr int kReg = 2;
    const bool in_regs = nsrc <= kReg * T;
    SeedRec<D> rc[kReg];
    CellQuad<D> cq[kReg], mine;
    mine.c = INFINITY;
    if (in_regs) {
#pragma unroll
        for (int r = 0; r < kReg; ++r) {
            const int q = threadIdx.x + r * T;
            if (q < nsrc) rc[r] = load(q);
        }
#pragma unroll
        for (int r = 0; r < kReg; ++r) {
            const int q = threadIdx.x + r * T;
            if (q < nsrc) {
                cq[r] = cell_quad<D>(rc[r], lam, hh);
                if (cq[r].c < mine.c) mine = cq[r];
            }
        }
    } else {
        for (int q = threadIdx.x; q < nsrc; q += T) {
            const CellQuad<D> c = cell_quad<D>(load(q), lam, hh);
            if (c.c < mine.c) mine = c;
        }
    }
    const unsigned long long lead = __ballot(mine.c == wave_min(mine.c));
    __syncthreads();  // s_cnt and s_own may still be read by an earlier use
    if (threadIdx.x == 0) s_cnt = 0;
    if (lane == max(0, __ffsll(lead) - 1)) s_own[threadIdx.x >> 6] = mine;
    __syncthreads();
    int ow = 0;
    float oc = s_own[0].c;
#pragma unroll
    for (int w = 1; w < T / 64; ++w) {
        const float c = s_own[w].c;
        ow = c < oc ? w : ow;
        oc = fminf(oc, c);
    }
    const CellQuad<D> own = s_own[ow];
    auto emit = [&](bool cand, int q, const SeedRec<D> &rec) {
        const unsigned long long m = __ballot(cand);
        if (!m) return;
        int base = 0;
        if (lane == 0) base = atomicAdd(&s_cnt, (int)__popcll(m));
        base = __builtin_amdgcn_readfirstlane(base);
        const int below = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
        if (cand) keep(q, rec, base + below);
    };
    if (in_regs) {
#pragma unroll
        for (int r = 0; r < kReg; ++r) {
            const int q = threadIdx.x + r * T;
            if (r * T < nsrc)
                emit(q < nsrc && can_beat<D>(cq[r], own, h, slack), q, rc[r]);
        }
    } else {
        for (int q0 = 0; q0 < nsrc; q0 += T) {
            const int q = q0 + threadIdx.x;
            SeedRec<D> rec = load(min(q, nsrc - 1));
            emit(q < nsrc && can_beat<D>(cell_quad<D>(rec, lam, hh), own, h, slack), q, rec);
        }
    }
    __syncthreads();
    return s_cnt;
}

// A super-tile's list in global memory: for each seed its record about the
// super-tile's centre and its number, packed in kRecVec float4 (16-byte pieces
// stored piece by piece, so that consecutive lanes read consecutive pieces).
// The tiles read their source seeds from it: gathered from the caller's
// double arrays each candidate took 10 scattered loads, which made the short
// lists a net loss in 3D.
template <int D>
__device__ inline void store_rec(float4 *list, int cap, int pos, const SeedRec<D> &r, int i) {
    const float id = __int_as_float(i);
    if constexpr (D == 2) {
        list[pos] = make_float4(r.e[0], r.e[1], r.wp, id);
        list[cap + pos] = make_float4(r.a[0], r.a[1], r.a[2], 0.0f);
    } else {
        list[pos] = make_float4(r.e[0], r.e[1], r.e[D - 1], id);
        list[cap + pos] = make_float4(r.a[0], r.a[1], r.a[2], r.wp);
        list[2 * (size_t)cap + pos] = make_float4(r.a[3 % SeedRec<D>::kTri], r.a[4 % SeedRec<D>::kTri], r.a[5 % SeedRec<D>::kTri], 0.0f);
    }
}
template <int D>
__device__ inline SeedRec<D> load_rec(const float4 *list, int cap, int pos, const float *shift, int &i) {
    SeedRec<D> r;
    const float4 v0 = list[pos], v1 = list[cap + pos];
    i = __float_as_int(v0.w);
    r.e[0] = v0.x + shift[0];
    r.e[1] = v0.y + shift[1];
    r.a[0] = v1.x;
    r.a[1] = v1.y;
    r.a[2] = v1.z;
    if constexpr (D == 2) {
        r.wp = v0.z;
    } else {
        const float4 v2 = list[2 * (size_t)cap + pos];
        r.e[D - 1] = v0.z + shift[2];
        r.wp = v1.w;
        r.a[3 % SeedRec<D>::kTri] = v2.x;
        r.a[4 % SeedRec<D>::kTri] = v2.y;
        r.a[5 % SeedRec<D>::kTri] = v2.z;
    }
    return r;
}

// The box (c0, c1, c2) of f[0] x f[1] x f[2] super-tiles each.
template <int D>
__device__ inline void super_box(const Geo &g, const PassOut &out, const int *f, const int *c, double *blo,
                                 double *bhi) {
    int ext[3], k0[3];
    for (int d = 0; d < 3; ++d) {
        ext[d] = tile_ext(D, out.tp, d) * out.sf[d] * f[d];
        k0[d] = c[d] * ext[d];
    }
    cull_box<D>(g, k0, ext, blo, bhi);
}

// Block-wide (T threads): of the seeds 0 .. nsrc - 1 (of rec's nsrc records,
// when given) those that the eigenvalue bounds
//   lambda_min dist(x, box)^2 - w' <= U = min_k lambda_max maxdist(x_k, box)^2 - w_k'
// leave a chance somewhere in the box, their numbers into list (room for cap,
// in any order); returns how many there are.
//
// Bound by the reads of every seed's 48 bytes by every block.  The bounds of
// squared norms are formed in FP32 from offsets taken in double: dist and far
// are off by at most 2^-22 far each, so the bounds by less than 2^-19
// (lambda_max far^2 + |w'|); twice that, and the lists' own slack (underflow),
// widens them.  A thread takes the seeds four at a time without a branch
// between, so that their loads are in flight together, and a wave reserves the
// places of all its seeds at once.  Over 512 super-tiles of 256^3, N = 10^4 (246
// MB from the L2s), against bounds in double taken one by one: 32.5 -> 24.5 us
// with 512 threads (one round of blocks; 1024 threads 28); 6.9 -> 4.8 on
// 1024^2, N = 1000.
template <int D, int T>
__device__ inline int box_survivors(const Geo &g, const Seeds &sd, double wmax, Cert ct, const double *eig,
                                    const double *blo, const double *bhi, const double *ctr, const float *h,
                                    const float4 *rec, int rec_cap, const float *shift, int nsrc, int *list, int cap,
                                    int &s_cnt, float *s_red) {
    const int lane = __lane_id();
    auto bounds_power = [&](int i, float &lb, float &ub) {
        double l, u;
        cull_bounds<D, false>(sd, eig, wmax, blo, bhi, i, &l, &u, g.power);
        lb = __double2float_rd(l);
        ub = __double2float_ru(u);
    };
    auto bounds_square = [&](int i, float &lb, float &ub) {
        float dist2 = 0.0f, far2 = 0.0f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const float e = fabsf((float)(sd.x[(size_t)i * D + d] - ctr[d]));
            const float dd = fmaxf(0.0f, e - h[d]), fd = e + h[d];
            dist2 = fmaf(dd, dd, dist2);
            far2 = fmaf(fd, fd, far2);
        }
        const float wp = (float)(sd.w[i] - wmax);
        // (one load of 16 bytes, at 8-byte addresses in the batched solver)
        const float lmin = (float)eig[2 * (size_t)i], lmax = (float)eig[2 * (size_t)i + 1];
        const float u = lmax * far2, slack = fmaf(0x1p-18f, u + fabsf(wp), ct.lsl);
        lb = fmaf(lmin, dist2, -wp) - slack;
        ub = (u - wp) + slack;
    };
    // from a region's record: x about its centre, w - w_max, the eigenvalue
    // range.  The offset's rounding is at most 2^-22 of its size, covered like
    // that of the others, and 2^-22 of the shift, which widens the box
    float hr[D];
#pragma unroll
    for (int d = 0; d < D; ++d) hr[d] = rec ? fmaf(0x1p-22f, fabsf(shift[d]), h[d]) * (1.0f + 0x1p-20f) : h[d];
    auto bounds_rec = [&](int q, float &lb, float &ub) {
        const float4 r = rec[q], v = rec[rec_cap + q];
        const float e[3] = {r.x + shift[0], r.y + shift[1], r.z + shift[2]};
        float dist2 = 0.0f, far2 = 0.0f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const float dd = fmaxf(0.0f, fabsf(e[d]) - hr[d]), fd = fabsf(e[d]) + hr[d];
            dist2 = fmaf(dd, dd, dist2);
            far2 = fmaf(fd, fd, far2);
        }
        const float u = v.y * far2, slack = fmaf(0x1p-18f, u + fabsf(r.w), ct.lsl);
        lb = fmaf(v.x, dist2, -r.w) - slack;
        ub = (u - r.w) + slack;
    };
    auto seed_at = [&](int q) { return rec ? __float_as_int(rec[rec_cap + q].z) : q; };
    constexpr int kUnroll = 4;
    constexpr int kKeep = T > kThreads ? 20 : 8;  // a thread's lower bounds kept in registers
    const bool in_regs = nsrc <= kKeep * T;
    float lbr[kKeep], umin = INFINITY;
    auto scan = [&](auto bounds) {
        if (in_regs) {
#pragma unroll
            for (int r0 = 0; r0 < kKeep; r0 += kUnroll) {
#pragma unroll
                for (int r = r0; r < r0 + kUnroll; ++r) lbr[r] = INFINITY;
                if (r0 * T >= nsrc) continue;
#pragma unroll
                for (int r = r0; r < r0 + kUnroll; ++r) {
                    // past the end the last seed again (no branch between the loads)
                    const int i = threadIdx.x + r * T;
                    float lb, ub;
                    bounds(min(i, nsrc - 1), lb, ub);
                    lbr[r] = i < nsrc ? lb : INFINITY;
                    umin = fminf(umin, ub);
                }
            }
        } else {
#pragma unroll kUnroll
            for (int i = threadIdx.x; i < nsrc; i += T) {
                float lb, ub;
                bounds(i, lb, ub);
                umin = fminf(umin, ub);
            }
        }
    };
    const bool square = g.power == 2;
    if (rec) scan(bounds_rec);
    else if (square) scan(bounds_square);
    else scan(bounds_power);
    umin = wave_min(umin);
    if (lane == 0) s_red[threadIdx.x >> 6] = umin;
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    float U = s_red[0];
#pragma unroll
    for (int w = 1; w < T / 64; ++w) U = fminf(U, s_red[w]);
    auto rank = [&](unsigned long long m) {
        return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    };
    auto reserve = [&](int n) {
        int base = 0;
        if (lane == 0) base = atomicAdd(&s_cnt, n);
        return __builtin_amdgcn_readfirstlane(base);
    };
    if (in_regs) {
        // one reservation for all of a wave's seeds
        unsigned long long keep[kKeep];
        int n = 0;
#pragma unroll
        for (int r = 0; r < kKeep; ++r) {
            keep[r] = __ballot((int)threadIdx.x + r * T < nsrc && !(lbr[r] > U));
            n += (int)__popcll(keep[r]);
        }
        if (n) {
            int base = reserve(n);
#pragma unroll
            for (int r = 0; r < kKeep; ++r) {
                if (!keep[r]) continue;
                const int pos = base + rank(keep[r]);
                if ((keep[r] >> lane & 1ull) && pos < cap) list[pos] = seed_at(threadIdx.x + r * T);
                base += (int)__popcll(keep[r]);
            }
        }
    } else {
        for (int i0 = 0; i0 < nsrc; i0 += T) {
            const int i = i0 + threadIdx.x;
            float lb = INFINITY, ub;
            if (i < nsrc) {
                if (rec) bounds_rec(i, lb, ub);
                else if (square) bounds_square(i, lb, ub);
                else bounds_power(i, lb, ub);
            }
            const bool cand = i < nsrc && !(lb > U);
            const unsigned long long m = __ballot(cand);
            if (!m) continue;
            const int pos = reserve((int)__popcll(m)) + rank(m);
            if (cand && pos < cap) list[pos] = seed_at(i);
        }
    }
    __syncthreads();
    return s_cnt;
}

// The seeds of region rg (a box of hf[0] x hf[1] x hf[2] super-tiles) that its
// super-tiles start from: with many of both, the super-tiles' reads of every
// seed would outweigh the rest of the pass (4000^2, N = 53333: 650 of 832 us; the
// regions take 58 and the super-tiles then 67).  Packed about the region's centre
// (box_survivors' bounds_rec).  All T threads of the block call it.
template <int D, int T>
__device__ inline void region_list(const Geo &g, const Seeds &sd, double wmax, Cert ct, const double *eig,
                                   const PassOut &out, const Regions &rg, int id, int *s_list, int &s_cnt,
                                   float *s_red) {
    float4 *rec = rg.rec + (size_t)id * 2 * rg.cap;
    int *count = rg.count + id;
    if (ct.lsl == INFINITY) {
        if (threadIdx.x == 0) *count = rg.cap + 1;
        return;
    }
    const int c[3] = {id / (rg.nh[2] * rg.nh[1]), id / rg.nh[2] % rg.nh[1], id % rg.nh[2]};
    double blo[3], bhi[3], ctr[D];
    float h[D];
    super_box<D>(g, out, rg.hf, c, blo, bhi);
    box_centre<D>(blo, bhi, ctr, h);
    const int m = box_survivors<D, T>(g, sd, wmax, ct, eig, blo, bhi, ctr, h, nullptr, 0, nullptr, g.n, s_list,
                                      rg.cap, s_cnt, s_red);
    if (threadIdx.x == 0) *count = m;
    if (m > rg.cap) return;
    for (int q = threadIdx.x; q < m; q += T) {
        const int i = s_list[q];
        const double *x = sd.x + (size_t)i * D;
        rec[q] = make_float4((float)(x[0] - ctr[0]), (float)(x[1] - ctr[1]), D == 3 ? (float)(x[D - 1] - ctr[D - 1]) : 0.0f,
                             (float)(sd.w[i] - wmax));
        rec[rg.cap + q] = make_float4((float)eig[2 * (size_t)i], (float)eig[2 * (size_t)i + 1], __int_as_float(i), 0.0f);
    }
}

// LDS of super_tile_list with T threads.
template <int D, int T>
struct SuperSmem {
    int list[kSuperCap];
    CellQuad<D> own[T / 64];
    float red[T / 64];
    int cnt;
};

// The candidate list of super-tile st (a box of sf[0] x sf[1] x sf[2] tiles of
// out.tp pixels per lane) into list (room for cap) or, where ids is given, the
// seeds' numbers alone into ids, how many there are into *count (above cap: every
// seed): the survivors of its box (box_survivors, from its
// region's list where the pass has regions), then, unless the pass returns the
// relative gaps (whose tiles need lists that bound the cost of every seed left
// out) or its costs are of another power, of these by the owner's difference.
// A seed that cannot win anywhere in the super-tile cannot win in any of its
// tiles.  All T threads of the block call it.
template <int D, int T>
__device__ inline void super_tile_list(const Geo &g, const Seeds &sd, double wmax, Cert ct, const double *eig,
                                       const PassOut &out, const Regions &rg, int st, float4 *list, int *ids,
                                       int *count, int cap, SuperSmem<D, T> &sm) {
    int c[3];
    c[2] = st % out.nst[2];
    c[1] = (st / out.nst[2]) % out.nst[1];
    c[0] = st / (out.nst[2] * out.nst[1]);
    if (ct.lsl == INFINITY) {
        if (threadIdx.x == 0) *count = cap + 1;
        return;
    }
    constexpr int kOne[3] = {1, 1, 1};
    double blo[3], bhi[3], ctr[D];
    float h[D];
    super_box<D>(g, out, kOne, c, blo, bhi);
    const float hh = box_centre<D>(blo, bhi, ctr, h);
    const float4 *rec = nullptr;
    int nsrc = g.n;
    float shift[3] = {0.0f, 0.0f, 0.0f};
    if (rg.rec) {
        const int rc[3] = {c[0] / rg.hf[0], c[1] / rg.hf[1], c[2] / rg.hf[2]};
        const int id = (rc[0] * rg.nh[1] + rc[1]) * rg.nh[2] + rc[2];
        if (rg.count[id] <= rg.cap) {
            rec = rg.rec + (size_t)id * 2 * rg.cap;
            nsrc = rg.count[id];
            double rlo[3], rhi[3], rctr[D];
            float rh[D];
            super_box<D>(g, out, rg.hf, rc, rlo, rhi);
            box_centre<D>(rlo, rhi, rctr, rh);
            for (int d = 0; d < D; ++d) shift[d] = (float)(rctr[d] - ctr[d]);
        }
    }
    const int m = box_survivors<D, T>(g, sd, wmax, ct, eig, blo, bhi, ctr, h, rec, rg.cap, shift, nsrc, sm.list,
                                      kSuperCap, sm.cnt, sm.red);
    if (m > kSuperCap) {
        if (threadIdx.x == 0) *count = cap + 1;
        return;
    }
    int n;
    if (out.rel_gap || g.power != 2) {
        for (int q = threadIdx.x; q < min(m, cap); q += T) {
            if (ids) ids[q] = sm.list[q];
            else store_rec<D>(list, cap, q, seed_rec<D>(sd, wmax, ctr, sm.list[q]), sm.list[q]);
        }
        n = m;
    } else {
        n = owner_filter<D, T>(
            m, [&](int q) { return seed_rec<D>(sd, wmax, ctr, sm.list[q]); }, h, hh, ct.lam,
            ct.lsl, sm.cnt, sm.own, [&](int q, const SeedRec<D> &r, int pos) {
                if (pos >= cap) return;
                if (ids) ids[pos] = sm.list[q];
                else store_rec<D>(list, cap, pos, r, sm.list[q]);
            });
    }
    if (threadIdx.x == 0) *count = n;
}

// Two scans of the staged seeds, with the same costs and certificate:
//  * short scans (fewer than kGroupScan seeds) keep the index of the best
//    seed in the low 4 bits of its cost (integer min / med3 on the keys:
//    3 operations per pixel and seed besides the 2 fused multiply-adds);
//  * long scans (over every seed) take the minimum of each group of 16 seeds with 3-input
//    minima (about half an operation per pixel and seed), keep the top two
//    group minima and the group of the best, and at the end of each staged
//    chunk re-evaluate the 16 costs of the winning group -- bit-identical
//    values, same operations on the same operands -- to find the winning
//    seed and the second-smallest cost inside that group.  The top two of
//    all costs are then (best, min(second group minimum, second inside the
//    winning group)).
constexpr int kGroupScan = 96;   // scans at least this long use group minima

// The candidate list of a tile's box, from its super-tile's list when it has
// one (else from every seed): into sm.list, at most kCullCap seeds; returns
// their number.  BOUNDS: by separate bounds of each seed's cost (a pass that
// returns the relative gaps, costs of another power); *U then bounds the cost
// of every seed left out.
template <int D, int P, bool BOUNDS, class Smem>
__device__ inline int tile_candidates(const Geo &g, const Seeds &sd, double wmax, Cert ct, const double *eig,
                                      const PassOut &out, int b0, int b1, int b2, Smem &sm, double *U) {
    if (ct.lsl == INFINITY) return kCullCap + 1;
    int *dst = sm.list;
    auto tile_box = [&](double *blo, double *bhi) {
        const int ext[3] = {tile_ext(D, P, 0), tile_ext(D, P, 1), tile_ext(D, P, 2)};
        const int k0[3] = {b0 * ext[0], b1 * ext[1], b2 * ext[2]};
        cull_box<D>(g, k0, ext, blo, bhi);
    };
    const float4 *src = nullptr;
    const int *ids = nullptr;
    int nsrc = g.n, cap = out.super_cap;
    const int sc[3] = {b0 / out.sf[0], b1 / out.sf[1], b2 / out.sf[2]};
    if (out.super_count) {
        const int st = (sc[0] * out.nst[1] + sc[1]) * out.nst[2] + sc[2];
        const int c = out.super_count[st];
        if (c <= cap) {
            if (out.super_ids) ids = out.super_ids + (size_t)st * (size_t)cap;
            else src = out.super_list + (size_t)st * (size_t)cap * rec_vec(D);
            nsrc = c;
        }
    }
    if constexpr (BOUNDS) {
        double blo[3], bhi[3];
        tile_box(blo, bhi);
        return build_candidates<D>(sd, eig, wmax, blo, bhi,
                                   [&](int q) { return src ? __float_as_int(src[q].w) : ids ? ids[q] : q; }, nsrc, dst,
                                   kCullCap,
                                   sm.cnt, sm.red, U, g.power);
    } else {
        float h[D], hh = 0.0f, shift[3] = {0.0f, 0.0f, 0.0f};
        const float slack = ct.lsl;
        if (src) {
            // the boxes' centres differ by a multiple of half a pixel
            const int tb[3] = {b0, b1, b2};
            for (int d = 0; d < D; ++d) {
                const int E = tile_ext(D, P, d), a = tb[d] * E, b = min(a + E, g.grid[d]) - 1;
                const int sa = sc[d] * out.sf[d] * E, sb = min(sa + out.sf[d] * E, g.grid[d]) - 1;
                const float s = (float)g.s[d];
                h[d] = 0.5f * (float)(b - a) * s * (1.0f + 0x1p-20f);
                hh = fmaf(h[d], h[d], hh);
                shift[d] = 0.5f * (float)((sa - a) + (sb - b)) * s;
            }
            return owner_filter<D, kThreads>(
                nsrc,
                [&](int q) {
                    int i;
                    return load_rec<D>(src, cap, q, shift, i);
                },
                h, shift_slack<D>(shift, hh), ct.lam, slack, sm.cnt, sm.own, [&](int q, const SeedRec<D> &, int pos) {
                    if (pos < kCullCap) dst[pos] = __float_as_int(src[q].w);
                });
        }
        double blo[3], bhi[3], ctr[D];
        tile_box(blo, bhi);
        hh = box_centre<D>(blo, bhi, ctr, h);
        return owner_filter<D, kThreads>(
            nsrc, [&](int q) { return seed_rec<D>(sd, wmax, ctr, ids ? ids[q] : q); }, h, hh, ct.lam, slack, sm.cnt,
            sm.own, [&](int q, const SeedRec<D> &, int pos) {
                if (pos < kCullCap) dst[pos] = ids ? ids[q] : q;
            });
    }
}

// Boundary-aware refinement: a tile whose list holds L alone (it beats every
// other seed everywhere in the tile) lies inside L's cell, so its pixels are
// labelled L and its moments
// are added in closed form (box_moments_add) -- the pixel-level scan, the
// certificate and the re-check are skipped; the labels and moments are
// those of the full evaluation.  All threads of the block call it (with the
// same L).
template <int D, int P>
__device__ inline void credit_tile(const Geo &g, const Tile<D> &t, int b0, int b1, int b2, int L,
                                   const PassOut &out) {
    constexpr int E0 = tile_ext(D, P, 0), E1 = tile_ext(D, P, 1), E2 = tile_ext(D, P, 2);
    if (out.labels && lane_in_grid<D>(g, t)) {
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (t.k0w + p < g.grid[0]) out.labels[pixel_index<D>(g, t.k0w + p, t)] = L;
    }
    if (threadIdx.x == 0) {
        const int base[3] = {b0 * E0, b1 * E1, b2 * E2};
        const int ext[3] = {E0, E1, E2};
        int a[3], b[3];
        for (int d = 0; d < D; ++d) {
            a[d] = base[d];
            b[d] = min(base[d] + ext[d], g.grid[d]) - 1;
        }
        if (out.mom) box_moments_add<D>(out.mom, L, a, b);
        if (out.credited) atomicAdd(out.credited, 1u);
    }
}

// A threshold that needs no square root, holds for every pixel of a tile and is
// linear in the best cost: 4 r sqrt(B) <= 2 B + 2 r^2 and r at the tile's corner
// (r2t), so vec_settle's is at most 2^-20 (6 B1 + 12 r^2) + ... + kbits max(|fb|,
// |fs|), and max(|fb|, |fs|) <= |fb| + (fs - fb).  Nearly every wave settles all
// of its pixels by it (3 instructions per pixel instead of about 45 with two
// square roots).
struct LooseCert {
    float k1, k2;
    __device__ inline LooseCert(Cert ct, float r2t, float kbits) {
        const float skb = kslack(ct);
        k1 = (0x1.8p-18f + skb + kbits) * (1.0f + 0x1p-7f);
        k2 = ((0x1.8p-17f + skb + 0x1p-9f * (0x1.8p-18f + skb)) * r2t + ct.sab) * (1.0f + 0x1p-7f);
    }
    __device__ inline bool settled(float fb, float fs) const { return (fs - fb) > fmaf(fabsf(fb), k1, k2); }
};

// The certificate of one pixel from its two smallest computed costs (fb, fs)
// and, where the pass returns it (GAP, or a pass over every seed), its relative
// gap; U bounds the cost of the seeds left out of the lists.  True: not
// settled.
template <int D, bool GAP>
__device__ inline bool vec_settle(const Geo &g, const Tile<D> &t, Cert ct, const float *s, float u0, float u1,
                                  float u2, float fb, float fs, float kbits, float U, bool act, int p,
                                  const PassOut &out) {
    const float sab = ct.sab, skb = kslack(ct);
    const float r2 = pixel_r2(ct, u0, u1, u2);
    const float bb = fmaxf(fb, 0.0f);
    const float B1 = bb + 0x1p-10f * (bb + r2);
    const float e1 = e32_bound(B1, sqrtf(r2), r2);
    const float thr = 2.0f * e1 + kbits * fmaxf(fabsf(fb), fabsf(fs)) + sab + skb * (B1 + r2);
    const bool flag = !((fs - fb) > thr);
    if (out.rel_gap && act && !flag) {
        // the winner costs at most c1u; a scanned seed at least fs minus its
        // bound, one left out of the lists more than their U
        const float c1u = (fb + 0x1p-19f * fabsf(fb) + e1 + sab + skb * (B1 + r2)) * (1.0f + 0x1p-20f);
        const float f2 = pad_inf(fs);
        const float bs = fmaxf(f2, 0.0f);
        const float B2 = bs + 0x1p-10f * (bs + r2);
        float c2l = f2 == INFINITY ? f2 : f2 - 0x1p-19f * fabsf(f2) - e32_bound(B2, sqrtf(r2), r2) - sab - skb * (B2 + r2);
        c2l = fminf(c2l, (U == INFINITY ? U : U - 0x1p-20f * fabsf(U))) * (1.0f - 0x1p-20f);
        out.rel_gap[pixel_index<D>(g, t.k0w + p, t)] = fs > 0.0f ? gap_lower(c1u, c2l) : 0.0f;
    }
    return flag;
}

// The coefficients of staged seed q along axis 0 at a lane's other
// coordinates: its cost at u0 is (a00 u0 + beta) u0 + alpha (2 fused
// multiply-adds per pixel after 3 (2D) or 7 (3D) per seed).  The staged rows of
// a seed: a00, 2a01, (a11 | 2a02), l0; then in 2D l1, c and in 3D a11, 2a12,
// a22, l1 and l2, c.
template <int D, int R>
__device__ inline void staged_coef(const float4 (&sC)[D][R], int q, float u1, float u2, float &a00, float &beta,
                                   float &alpha) {
    const float4 c0 = sC[0][q];
    const float4 c1 = sC[1][q];
    a00 = c0.x;
    if constexpr (D == 2) {
        beta = fmaf(c0.y, u1, c0.w);
        alpha = fmaf(fmaf(c0.z, u1, c1.x), u1, c1.y);
    } else {
        const float4 c2 = sC[2][q];
        beta = fmaf(c0.y, u1, fmaf(c0.z, u2, c0.w));
        alpha = fmaf(fmaf(c1.x, u1, fmaf(c1.y, u2, c1.w)), u1, fmaf(fmaf(c1.z, u2, c2.x), u2, c2.y));
    }
}

// Stages seed i at position q; z, w ride in the last row's free lanes.
template <int D, int R>
__device__ inline void stage_coef(float4 (&sC)[D][R], int q, const double *qd, const double *ld, double cd, float z,
                                  float w) {
    sC[0][q] = make_float4((float)qd[0], (float)qd[1], (float)qd[2], (float)ld[0]);
    if constexpr (D == 2) {
        sC[1][q] = make_float4((float)ld[1], (float)cd, z, w);
    } else {
        sC[1][q] = make_float4((float)qd[3], (float)qd[4], (float)qd[5], (float)ld[1]);
        sC[2][q] = make_float4((float)ld[2], (float)cd, z, w);
    }
}
// A padding seed: 1.7e38 everywhere.
template <int D, int R>
__device__ inline void stage_pad(float4 (&sC)[D][R], int q) {
    for (int r = 0; r < D - 1; ++r) sC[r][q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    sC[D - 1][q] = make_float4(0.0f, 1.7e38f, 0.0f, 0.0f);
}

// The cost's bits with the low 4 replaced by r (wave-uniform): integer order
// is the costs' order (one instruction, which the compiler splits in two).
__device__ inline int cost_key(float c, int r) {
    int k;
    asm("v_and_or_b32 %0, %1, -16, %2" : "=v"(k) : "v"(__float_as_int(c)), "s"(r));
    return k;
}

// Short scan of the staged positions pair(j) = idx(j) | idx(j + 1) << 16 (j
// even) below c2 (even): per pixel the best and second key so far, and in blk
// the block of 16 positions where the best was last lowered.
template <int D, int R, int P, class Pair>
__device__ inline void key_scan(const float4 (&sC)[D][R], int c2, Pair pair, const float (&u0)[P], float u1, float u2,
                                int (&best)[P], int (&second)[P], int (&blk)[P]) {
    unsigned next = pair(0);
    for (int q0 = 0; q0 < c2; q0 += 16) {
        int old[P];
#pragma unroll
        for (int p = 0; p < P; ++p) old[p] = best[p];
        for (int r2 = 0; r2 < 16 && q0 + r2 < c2; r2 += 2) {
            const unsigned two = next;
            next = pair(q0 + r2 + 2);  // the room is padded by a pair
            float a00, beta, alpha, b00, betb, alphb;
            staged_coef<D>(sC, (int)(two & 0xffffu), u1, u2, a00, beta, alpha);
            staged_coef<D>(sC, (int)(two >> 16), u1, u2, b00, betb, alphb);
#pragma unroll
            for (int p = 0; p < P; ++p) {
                // two candidates at a time: 3 instructions for the pair's top two
                const int ka = cost_key(fmaf(fmaf(a00, u0[p], beta), u0[p], alpha), r2);
                const int kb = cost_key(fmaf(fmaf(b00, u0[p], betb), u0[p], alphb), r2 + 1);
                second[p] = min(second[p], med3i(best[p], ka, kb));
                best[p] = min3i(best[p], ka, kb);
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) blk[p] = (best[p] != old[p]) ? q0 : blk[p];
    }
}

// Seeds per staged chunk of the vector tile over every seed (in 2D N = 1000 is
// one chunk).
template <int D> struct VecCfg { static constexpr int kChunk = D == 2 ? 1024 : 512; };

template <int D>
struct VecSmem {
    float4 sC[D][VecCfg<D>::kChunk];  // seed coefficients of one chunk
};

// The vector tile over every seed.
template <int D, int P = kPv>
__device__ inline void vec_tile(const Geo &g, const Seeds &sd, double wmax, Cert ct, int b0, int b1, int b2,
                                VecSmem<D> &sm, const PassOut &out, unsigned *qcount) {
    constexpr int E0 = tile_ext(D, P, 0), E1 = tile_ext(D, P, 1), E2 = tile_ext(D, P, 2);
    constexpr int kVecChunk = VecCfg<D>::kChunk;
    auto &sC = sm.sC;
    const Tile<D> t = tile_at<D, P>(b0, b1, b2);
    const bool lane_ok = lane_in_grid<D>(g, t);
    const int nscan = g.n;
    float s[3];
    double anc[3];
    for (int d = 0; d < D; ++d) {
        s[d] = (float)g.s[d];
        anc[d] = g.lo[d] + (double)t.anc[d] * g.s[d];
    }
    bool act[P];
    float u0[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        act[p] = lane_ok && (t.k0w + p) < g.grid[0];
        u0[p] = ((float)(t.k0w + p - t.anc[0]) + 0.5f) * s[0];
    }
    const float u1 = ((float)(t.k[1] - t.anc[1]) + 0.5f) * s[1];
    const float u2 = D == 3 ? ((float)(t.k[2] - t.anc[2]) + 0.5f) * s[2] : 0.0f;
    auto lane_coef = [&](int q, float &a00, float &beta, float &alpha) {
        staged_coef<D>(sC, q, u1, u2, a00, beta, alpha);
    };
    auto stage = [&](int base, int cnt, int padded) {
        for (int q = threadIdx.x; q < padded; q += kThreads) {
            if (q >= cnt) {
                stage_pad<D>(sC, q);
                continue;
            }
            double qd[6], ld[3], cd, ed[3], wpd;
            seed_terms<D>(sd, base + q, anc, wmax, qd, ld, &cd, ed, &wpd);
            stage_coef<D>(sC, q, qd, ld, cd, 0.0f, 0.0f);
        }
    };
    float fb[P], fs[P];  // the two smallest costs of each pixel
    int pos[P];          // the best seed
    bool lost[P];        // the winner was not found again (never expected)
#pragma unroll
    for (int p = 0; p < P; ++p) {
        fb[p] = INFINITY;
        fs[p] = INFINITY;
        pos[p] = 0;
        lost[p] = false;
    }
    // Long scan of one staged chunk (positions j < c16), merged into the
    // running top two; winners found here are seeds base + j.
    auto group_scan = [&](int c16, int base) {
        int blk[P];
#pragma unroll
        for (int p = 0; p < P; ++p) blk[p] = -1;
        for (int q0 = 0; q0 < c16; q0 += 16) {
            float m[P];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float a00, beta, alpha;
                lane_coef(q0 + r, a00, beta, alpha);
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const float c = fmaf(fmaf(a00, u0[p], beta), u0[p], alpha);
                    m[p] = r == 0 ? c : fminf(m[p], c);
                }
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                // top two of the group minima and the group of the best (a
                // select on the comparison, which needs no canonicalised
                // operand as a minimum would)
                fs[p] = __builtin_amdgcn_fmed3f(fb[p], m[p], fs[p]);
                const bool better = m[p] < fb[p];
                blk[p] = better ? q0 : blk[p];
                fb[p] = better ? m[p] : fb[p];
            }
        }
        // the winners found in this chunk: which seed of the group, and the
        // second-smallest cost inside the group
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (blk[p] < 0) continue;
            float s2 = INFINITY;
            int ix = -1;
            for (int r = 0; r < 16; ++r) {
                float a00, beta, alpha;
                lane_coef(blk[p] + r, a00, beta, alpha);
                const float c = fmaf(fmaf(a00, u0[p], beta), u0[p], alpha);
                const bool hit = ix < 0 && c == fb[p];
                ix = hit ? r : ix;
                s2 = hit ? s2 : fminf(s2, c);
            }
            lost[p] = ix < 0;
            pos[p] = base + blk[p] + max(ix, 0);
            fs[p] = fminf(fs[p], s2);
        }
    };
    const bool keyed = nscan < kGroupScan;  // the short scan's costs lose their low 4 bits
    if (!keyed) {
        for (int base = 0; base < nscan; base += kVecChunk) {
            const int cnt = min(kVecChunk, nscan - base);
            const int padded = (cnt + 15) & ~15;
            __syncthreads();
            stage(base, cnt, padded);
            __syncthreads();
            group_scan(padded, base);
        }
    } else {
        __syncthreads();
        stage(0, nscan, (nscan + 1) & ~1);
        __syncthreads();
        int best[P], second[P], blk[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            best[p] = 0x7fffffff;
            second[p] = 0x7fffffff;
            blk[p] = 0;
        }
        key_scan<D>(sC, (nscan + 1) & ~1, [](int j) { return (unsigned)j | (unsigned)(j + 1) << 16; }, u0, u1, u2,
                    best, second, blk);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            pos[p] = blk[p] + (best[p] & 15);
            fb[p] = __int_as_float(best[p]);
            fs[p] = __int_as_float(second[p]);
        }
    }
    const float kbits = keyed ? 0x1p-18f : 0.0f;
    bool flag[P];
    int lab[P];
    const LooseCert loose(ct, pixel_r2(ct, 0.5f * E0 * s[0], 0.5f * E1 * s[1], D == 3 ? 0.5f * E2 * s[2] : 0.0f), kbits);
    bool near = out.rel_gap != nullptr;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        flag[p] = lost[p] || !loose.settled(fb[p], fs[p]);
        near = near || flag[p];
        lab[p] = min(pos[p], nscan - 1);
    }
    if (__ballot(near)) {
#pragma unroll
        for (int p = 0; p < P; ++p)
            flag[p] = vec_settle<D, false>(g, t, ct, s, u0[p], u1, u2, fb[p], fs[p], kbits, INFINITY, act[p], p, out) ||
                      lost[p];
    }
    tile_epilogue<D, P>(g, t, act, lab, flag, out, qcount);
}

// LDS of the list tile (GAP: the pass also returns the relative gaps; W: it
// forms moments with pixel weights).
constexpr int kListChunk = 256;  // candidates staged at a time, one per thread

template <int D, int P, bool GAP, bool W = false>
struct ListSmem {
    // coefficients of the staged candidates, + a dummy (index kListChunk) whose
    // cost is never the minimum; with GAP the free lanes of the last row hold
    // the seed's eigenvalue range (FP32, rounded outwards)
    float4 sC[D][kListChunk + 1];
    float4 sB[GAP ? kListChunk : 1];  // (x - anchor, w - wmax) in FP32
    int list[kCullCap];               // candidate seeds of the tile
    // each wave's staged positions (and a pair of padding); then its flagged pixels
    alignas(4) uint16_t wl[kWaves][(64 * P > kListChunk ? 64 * P : kListChunk) + 4];
    MomSmem<P, W> mom[GAP ? 0 : 1];  // a pass that returns gaps forms no moments
    CellQuad<D> own[kWaves];
    double red[kWaves];
    int cnt;
};

// The vector tile over the seeds that can win somewhere in the tile: its
// candidates (tile_candidates; every seed when the list overflows) are staged
// in chunks of kListChunk, nearly always one; each wave narrows a chunk to the
// seeds that can win in its own box of pixels and scans those (key_scan).  A wave
// left with one candidate needs no scan.  A pass that returns the relative
// gaps (GAP) needs a bound of the cost of every seed it leaves out, so its lists
// come from separate bounds of each seed's cost, which give one.
//
// Bound by the issue of vector instructions: a wave of 512 voxels takes about
// 1330 of them on 256^3 with N = 10^4 (9 candidates, 45 each; the lists about
// 420), one per 5.7 clocks and SIMD.  So what every wave repeats is kept short
// (the settled / outside state of its pixels as bits of one register, a
// certificate of 3 instructions per pixel, the minima of two candidates at a
// time) and what is rare (several chunks, an unsettled pixel) shares its code.
// Against the form that shared the tile over every seed and its two scans
// (1694 instructions): 112 -> 96 us there, 12.0 -> 11.2 on 1024^2 with N = 1000,
// 429 -> 379 ms for a batched fit of 512 maps.
template <int D, int P, bool GAP = false, bool W = false>
__device__ inline void list_tile(const Geo &g, const Seeds &sd, double wmax, Cert ct, const double *eig, int b0,
                                 int b1, int b2, ListSmem<D, P, GAP, W> &sm, const PassOut &out, unsigned *qcount) {
    constexpr int E0 = tile_ext(D, P, 0), E1 = tile_ext(D, P, 1), E2 = tile_ext(D, P, 2);
    constexpr int kDummy = kListChunk;
    auto &sC = sm.sC;
    int *s_list = sm.list;
    const Tile<D> t = tile_at<D, P>(b0, b1, b2);
    const bool lane_ok = lane_in_grid<D>(g, t);
    double Utile = INFINITY;  // no seed left out of the tile's list costs less
    float Uwave = INFINITY;   // nor out of this wave's lists
    // ---- the candidate list, from the super-tile's list when it has one
    const int ncand = tile_candidates<D, P, GAP>(g, sd, wmax, ct, eig, out, b0, b1, b2, sm, &Utile);
    const bool full = ncand > kCullCap;
    const int nscan = full ? g.n : ncand;
    if (full || ncand >= g.n) Utile = INFINITY;  // no seed was left out
    if (!GAP && out.adaptive && ncand == 1 && !g.mass) {
        credit_tile<D, P>(g, t, b0, b1, b2, s_list[0], out);
        return;
    }
    const bool one = nscan <= kListChunk;
    // the pixels' positions in the tile's list index its moment slots
    const bool slots = one && !full && nscan <= kAccSlots;
    auto seed_at = [&](int q) { return full ? q : s_list[q]; };

    float s[3];
    double anc[3];
    for (int d = 0; d < D; ++d) {
        s[d] = (float)g.s[d];
        anc[d] = g.lo[d] + (double)t.anc[d] * g.s[d];
    }
    float u0[P];
    const float k0f = (float)(t.k0w - t.anc[0]);
#pragma unroll
    for (int p = 0; p < P; ++p) u0[p] = (k0f + ((float)p + 0.5f)) * s[0];
    const float u1 = ((float)(t.k[1] - t.anc[1]) + 0.5f) * s[1];
    const float u2 = D == 3 ? ((float)(t.k[2] - t.anc[2]) + 0.5f) * s[2] : 0.0f;
    // the wave's box: pixels ka .. kb along each axis
    int ka[3] = {0, 0, 0}, kb[3] = {0, 0, 0};
    for (int d = 0; d < D; ++d) {
        const int e = max(t.org[d], min(t.org[d] + wave_ext(D, P, d), g.grid[d]) - 1);
        ka[d] = t.org[d] - t.anc[d];
        kb[d] = e - t.anc[d];
    }
    const float r2t = pixel_r2(ct, 0.5f * E0 * s[0], 0.5f * E1 * s[1], D == 3 ? 0.5f * E2 * s[2] : 0.0f);
    uint16_t *wl = sm.wl[threadIdx.x >> 6];
    int best[P], second[P];  // the two smallest keys of each pixel
    int pos[P];              // the winner: its position in the wave's list (one chunk), else its seed
#pragma unroll
    for (int p = 0; p < P; ++p) {
        best[p] = 0x7fffffff;
        second[p] = 0x7fffffff;
        pos[p] = 0;
    }
    int c = 0;          // candidates of the wave in the last chunk
    bool sure = false;  // the wave has a single candidate
    for (int base = 0; base < nscan; base += kListChunk) {
        const int cnt = min(kListChunk, nscan - base);
        __syncthreads();
        if ((int)threadIdx.x < cnt) {
            const int q = threadIdx.x, i = seed_at(base + q);
            double qd[6], ld[3], cd, ed[3], wpd;
            seed_terms<D>(sd, i, anc, wmax, qd, ld, &cd, ed, &wpd);
            float lmn = 0.0f, lmx = 0.0f;
            if constexpr (GAP) {
                // rounded outwards: the FP32 bounds of the wave lists stay bounds
                lmn = (float)eig[2 * (size_t)i] * (1.0f - 0x1p-20f);
                lmx = (float)eig[2 * (size_t)i + 1] * (1.0f + 0x1p-20f);
                sm.sB[q] = make_float4((float)ed[0], (float)ed[1], D == 3 ? (float)ed[2] : 0.0f, (float)wpd);
            }
            stage_coef<D>(sC, q, qd, ld, cd, lmn, lmx);
        }
        if (threadIdx.x == kThreads - 1) stage_pad<D>(sC, kDummy);
        if constexpr (!GAP)
            if (slots && out.mom) moments_zero(sm.mom[0], nscan);
        __syncthreads();
        c = 0;
        auto append = [&](bool cand, int q) {
            const unsigned long long m = __ballot(cand);
            const int below = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            if (cand) wl[c + below] = (uint16_t)q;
            c += (int)__popcll(m);
        };
        if constexpr (GAP) {
            // FP32 bounds from the staged data, widened by a relative 1e-4 (far
            // above their rounding), so the wave list keeps every seed that
            // can win
            float wlo[3] = {0.0f, 0.0f, 0.0f}, whi[3] = {0.0f, 0.0f, 0.0f};
            for (int d = 0; d < D; ++d) {
                wlo[d] = ((float)ka[d] + 0.5f) * s[d];
                whi[d] = ((float)kb[d] + 0.5f) * s[d];
            }
            auto wbounds = [&](int q, float &lb, float &ub) {
                const float4 b = sm.sB[q];
                const float4 ce = sC[D - 1][q];  // .z, .w: eigenvalue range
                const float e[3] = {b.x, b.y, b.z};
                float dist2 = 0.0f, far2 = 0.0f;
                for (int d = 0; d < D; ++d) {
                    const float dd = fmaxf(0.0f, fmaxf(wlo[d] - e[d], e[d] - whi[d]));
                    const float fd = fmaxf(e[d] - wlo[d], whi[d] - e[d]);
                    dist2 = fmaf(dd, dd, dist2);
                    far2 = fmaf(fd, fd, far2);
                }
                float l = ce.z * dist2, h = ce.w * far2;
                const float slack = 1e-4f * (fabsf(l) + (float)D * fabsf(h) + fabsf(b.w)) + 1e-30f;
                if constexpr (D == 2) {
                    // the exact range of the quadratic form, as cull_bounds
                    const float4 c0 = sC[0][q];  // a00, 2 a01, a11
                    quad_box_range2<float>(c0.x, c0.y, c0.z, wlo[0] - e[0], whi[0] - e[0], wlo[1] - e[1],
                                           whi[1] - e[1], &l, &h);
                } else {
                    // the exact maximum: the form is convex, so at a corner
                    const float4 c0 = sC[0][q];  // a00, 2 a01, 2 a02
                    const float4 c1 = sC[1][q];  // a11, 2 a12, a22
                    float hm = 0.0f;
    #pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        const float d0 = ((v & 1) ? whi[0] : wlo[0]) - e[0];
                        const float d1 = ((v & 2) ? whi[1] : wlo[1]) - e[1];
                        const float d2 = ((v & 4) ? whi[2] : wlo[2]) - e[2];
                        const float qv = fmaf(fmaf(c0.x, d0, fmaf(c0.y, d1, c0.z * d2)), d0,
                                              fmaf(fmaf(c1.x, d1, c1.y * d2), d1, c1.z * d2 * d2));
                        hm = fmaxf(hm, qv);
                    }
                    h = hm;
                }
                lb = l - b.w - slack;
                ub = h - b.w + slack;
            };
            float um = INFINITY;
            for (int q = t.lane; q < cnt; q += 64) {
                float lb, ub;
                wbounds(q, lb, ub);
                um = fminf(um, ub);
            }
            um = wave_min(um);
            for (int q0 = 0; q0 < cnt; q0 += 64) {
                const int q = q0 + t.lane;
                bool cand = false;
                if (q < cnt) {
                    float lb, ub;
                    wbounds(q, lb, ub);
                    cand = lb <= um;
                }
                append(cand, q);
            }
            if (c < cnt) Uwave = fminf(Uwave, um);  // the chunk's candidates left out cost more
        } else {
            // the owner's differences from the staged quadratics.  Each
            // monomial of a cost reaches it, the gradient or the bound through
            // fewer than 24 roundings of 2^-24 and their magnitudes sum to at
            // most 3 C + 6 r^2 (the vector tile's bound), r^2 = lam |u|^2 at the
            // tile's corner: 2^-16 (|C| + 2 r^2) is more than twice that.  The
            // double rounding of the costs and of their coefficients is relative
            // to lam |d|^2, up to kappa times C: kslack (|C| + 2 r^2), four times
            // its 2^-46 (kappa + 1) (C + r^2), counts from kappa of about 2^30
            float uc[3], h[3];
            for (int d = 0; d < D; ++d) {
                uc[d] = (float)(ka[d] + kb[d] + 1) * (0.5f * s[d]);
                h[d] = (float)(kb[d] - ka[d]) * (0.5f * (1.0f + 0x1p-20f) * s[d]);
            }
            const float ks = 0x1p-16f + kslack(ct);
            auto staged_quad = [&](int q) {
                CellQuad<D> r;
                const float4 c0 = sC[0][q], c1 = sC[1][q];
                if constexpr (D == 2) {
                    r.a[0] = c0.x; r.a[1] = c0.y; r.a[2] = c0.z;
                    const float t0 = fmaf(c0.x, uc[0], fmaf(c0.y, uc[1], c0.w)), t1 = fmaf(c0.z, uc[1], c1.x);
                    r.c = fmaf(t0, uc[0], fmaf(t1, uc[1], c1.y));
                    r.g[0] = fmaf(c0.x, uc[0], t0);
                    r.g[1] = fmaf(c0.y, uc[0], fmaf(c0.z, uc[1], t1));
                } else {
                    const float4 c2 = sC[2][q];
                    r.a[0] = c0.x; r.a[1] = c0.y; r.a[2] = c0.z;
                    r.a[3] = c1.x; r.a[4] = c1.y; r.a[5] = c1.z;
                    const float t0 = fmaf(c0.x, uc[0], fmaf(c0.y, uc[1], fmaf(c0.z, uc[2], c0.w)));
                    const float t1 = fmaf(c1.x, uc[1], fmaf(c1.y, uc[2], c1.w));
                    const float t2 = fmaf(c1.z, uc[2], c2.x);
                    r.c = fmaf(t0, uc[0], fmaf(t1, uc[1], fmaf(t2, uc[2], c2.y)));
                    r.g[0] = fmaf(c0.x, uc[0], t0);
                    r.g[1] = fmaf(c0.y, uc[0], fmaf(c1.x, uc[1], t1));
                    r.g[D - 1] = fmaf(c0.z, uc[0], fmaf(c1.y, uc[1], fmaf(c1.z, uc[2], t2)));
                }
                r.s = ks * (fabsf(r.c) + 2.0f * r2t);
                return r;
            };
            const float sl = ct.lsl;
            // the owner: the wave's candidate of least cost at its centre
            CellQuad<D> mine;
            mine.c = INFINITY;
            if (t.lane < cnt) mine = staged_quad(t.lane);
            float best = mine.c;
            int bq = t.lane;
            for (int q = t.lane + 64; q < cnt; q += 64) {
                const float v = staged_quad(q).c;
                if (v < best) {
                    best = v;
                    bq = q;
                }
            }
            const int lead = max(0, __ffsll(__ballot(best == wave_min(best))) - 1);
            if (cnt <= 64) {
                append(t.lane < cnt && can_beat<D>(mine, lane_quad(mine, lead), h, sl), t.lane);
            } else {
                const CellQuad<D> own = staged_quad(__builtin_amdgcn_readlane(bq, lead));
                for (int q0 = 0; q0 < cnt; q0 += 64) {
                    const int q = q0 + t.lane;
                    append(q < cnt && can_beat<D>(staged_quad(min(q, cnt - 1)), own, h, sl), q);
                }
            }
        }
        if (t.lane < 3) wl[c + t.lane] = kDummy;
        wave_lds_sync();  // the list is read back by other lanes of the wave only
        sure = !GAP && one && c == 1;
        if (sure) break;
        const unsigned *pairs = reinterpret_cast<const unsigned *>(wl);
        auto pair = [&](int j) { return pairs[j >> 1]; };
        int blk[P];
#pragma unroll
        for (int p = 0; p < P; ++p) blk[p] = one ? 0 : -1;
        key_scan<D>(sC, (c + 1) & ~1, pair, u0, u1, u2, best, second, blk);
        if (one) {
#pragma unroll
            for (int p = 0; p < P; ++p) pos[p] = blk[p] + (best[p] & 15);
        } else {
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (blk[p] >= 0) pos[p] = seed_at(base + min((int)wl[blk[p] + (best[p] & 15)], cnt - 1));
        }
    }
    // bits of the lane's pixels: outside the grid, not settled
    const unsigned beyond = ~0u << (lane_ok ? max(0, min(P, g.grid[0] - t.k0w)) : 0);
    unsigned open = 0u;
    if (!sure) {
        constexpr float kbits = 0x1p-18f;  // the keys' low bits
        const LooseCert loose(ct, r2t, kbits);
        bool near = GAP;
#pragma unroll
        for (int p = 0; p < P; ++p)
            near = near || !loose.settled(__int_as_float(best[p]), __int_as_float(second[p]));
        if (__ballot(near)) {
            const float U = fminf((float)Utile, Uwave);
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const float fb = __int_as_float(best[p]), fs = __int_as_float(second[p]);
                if (GAP || __ballot(!loose.settled(fb, fs)))
                    open |= vec_settle<D, GAP>(g, t, ct, s, u0[p], u1, u2, fb, fs, kbits, U, !(beyond >> p & 1u), p,
                                               out)
                                ? 1u << p
                                : 0u;
            }
            open &= ~beyond;
        }
    }
    if constexpr (!GAP) {
        if (slots && out.mom) {
            unsigned v[(P + 3) / 4];
#pragma unroll
            for (int hh = 0; hh < (P + 3) / 4; ++hh) {
                v[hh] = 0u;
#pragma unroll
                for (int j = 0; j < 4; ++j) v[hh] |= (unsigned)(4 * hh + j < P ? pos[4 * hh + j < P ? 4 * hh + j : 0] : 0) << (8 * j);
            }
            const unsigned off = (beyond | open) & ((1u << P) - 1u);
            if (P % 4 != 0 || __ballot(off != 0u)) {
                // a bit of off into the low bit of its byte
#pragma unroll
                for (int hh = 0; hh < (P + 3) / 4; ++hh)
                    v[hh] |= (((beyond | open) >> (4 * hh) & 15u) * 0x00204081u & 0x01010101u) * 127u;
            }
            auto slot = [&](int j) { return (int)wl[j]; };
            auto pix = [&](int p) { return beyond >> p & 1u ? (int64_t)-1 : (int64_t)pixel_index<D>(g, t.k0w + p, t); };
            moments_add<D, P, W>(sm.mom[0], t.lane, v, c, slot, g.mass, pix);
        }
    }
    if (!slots || out.labels || __ballot(open != 0u)) {
        bool act[P], flag[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            act[p] = !(beyond >> p & 1u);
            flag[p] = open >> p & 1u;
        }
        if (!slots || out.labels) {
            int lab[P];
#pragma unroll
            for (int p = 0; p < P; ++p)
                lab[p] = !one ? pos[p] : c > 0 ? seed_at(wl[min(pos[p], c - 1)]) : 0;  // none: all flagged
            if (!slots) tile_epilogue<D, P>(g, t, act, lab, flag, out, nullptr);
            else write_labels<D, P>(g, t, act, lab, flag, out);
        }
        recheck_flagged<D, P>(g, sd, t, act, flag, full ? nullptr : s_list, nscan, wl, out, qcount, wmax, Utile);
    }
    if constexpr (!GAP) {
        if (slots && out.mom) {
            __syncthreads();
            moments_flush<D, P>(sm.mom[0], t.anc, s_list, nscan, out.mom);
        }
    }
}


// ------------------------------------------------------------ bf16 helpers

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short ushort8 __attribute__((ext_vector_type(8)));

// round to nearest even (finite inputs)
__device__ inline unsigned short bf16_bits(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
__device__ inline float bf16_value(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

// ------------------------------------------- hybrid matrix-core / vector tile

// Single precision over every seed, the work split between the two units.
// The cost of seed i at a pixel, in coordinates u about the tile anchor, is
// a quadratic in u0 whose coefficients depend on the pixel's other axes:
//   C = a00 u0^2 + beta u0 + alpha,
//   3D: beta  = 2a01 u1 + 2a02 u2 + l0,
//       alpha = a11 u1^2 + 2a12 u1 u2 + a22 u2^2 + l1 u1 + l2 u2 + c,
//   2D: beta  = 2a01 u1 + l0,  alpha = a11 u1^2 + l1 u1 + c
// (l = -2 A e, c = e^T A e - w', as seed_terms).  For 32 seeds x 32 positions
// (u1, u2) the matrix cores form beta and alpha, one
// v_mfma_f32_32x32x16_bf16 each: the coefficients split exactly into three
// bf16 parts against exact small-integer features (hyb_stage).  The vector
// ALU then evaluates the quadratic along axis 0 for rows placed
// symmetrically about the anchor, u0 = +-(j + 1/2) s0: a row pair shares
// q = a00 u0^2 + alpha and takes C = q +- beta u0, so 1.5 fused multiply-adds
// per pair and no per-seed coefficient work on the ALU.  The accumulator
// layout gives lane l the block rows 8 (r / 4) + 4 h + r % 4 (h = l / 32) at
// position l % 32: the two half-waves see the same pixels against the two
// halves of every block.  The seeds are scanned in the order of a
// space-filling curve (k_seed_order), and the running minimum is kept per
// kHybSB consecutive ones (a super-block, a compact region of the box),
// with the runner-up and that super-block's index.  At the
// end the two halves exchange their minima, so that only the pixel's true
// winning super-block is searched, once per distinct one in the wave: its
// products are formed again (the same operands, so the same bits) and the
// half holding the best cost finds the seed attaining it.
//
// Tiles (HybCfg): 3D 16 x 16 x 8 pixels, wave w covering the 8 row pairs
// and 4 x 8 positions (axis 1 from 4 w, axis 2); 2D 32 x 32 pixels, wave w
// covering row pairs 4 w .. 4 w + 3 and the tile's 32 positions.  After the
// half-waves are merged, lane l owns its pairs' rows below the anchor
// (h = 0) or above it (h = 1) at its position: NJ consecutive rows.
//
// Rounding bound (relative roundings of 2^-24 on each monomial's path to
// the computed cost, S the sum of the monomials' magnitudes, S <= C +
// 4 r sqrt(C) + 4 r^2 as for the vector tile): the coefficient's FP32
// rounding (1; the bf16 split, the integer features and their products are
// exact), the matrix-core sum (alpha: the start c - c_hi and its products,
// 16 in 3D and 10 in 2D, each addition possibly rounded), the two fused
// multiply-adds.  3D: at most 19 (beta's terms 11, a00 u0^2 5), so
// |C_fp32 - C| <= gamma_19 S < 1.19 2^-20 S, within hyb_bound (1.3125 2^-20
// S); 2D: at most 13, within e32_bound.
constexpr int kHybSB = 64;  // seeds per running-minimum group (super-block): one per lane

template <int D> struct HybCfg;
template <> struct HybCfg<3> {
    static constexpr int kRows = kHybRows3;  // tile rows along axis 0
    static constexpr int kPairs = 8;         // row pairs per lane
    static constexpr int kChunk = 512;       // seeds staged per chunk (a multiple of kHybSB)
};
template <> struct HybCfg<2> {
    static constexpr int kRows = kHybRows2;
    static constexpr int kPairs = 4;
    static constexpr int kChunk = 512;
};

// LDS of the hybrid tile: per staged seed its bf16 operand slots, group
// 2 m + h holding slots 8 h .. 8 h + 7 of product m (0: beta, 1: alpha), and
// its FP32 a00 and c - c_hi.  After the scan each wave re-stages one
// super-block at a time into its own 64 positions of the same arrays.
template <int D>
struct HybSmem {
    static constexpr int C = HybCfg<D>::kChunk;
    ushort8 a[4][C];
    float a00[C];
    float crest[C];
};

// An FP32 value as the exact sum of three bf16 parts (hi, mid, lo: 8
// significant bits each; each difference is exact in FP32).
__device__ inline void bf16_split3(float f, unsigned short *out) {
    const unsigned short hi = bf16_bits(f);
    const float r = f - bf16_value(hi);
    const unsigned short mid = bf16_bits(r);
    out[0] = hi;
    out[1] = mid;
    out[2] = bf16_bits(r - bf16_value(mid));
}

// The operand slots of one seed.  In tile-local half-pixel units
// o_d = 2 (k_d - anchor_d) + 1 (odd integers: 3D |o_1| <= 15, |o_2| <= 7;
// 2D |o_1| <= 31) the position's features are exact bf16 values (2D: o1^2,
// up to 961, as the sum of two, f2 = f2_hi + f2_lo) and the coefficients
// carry the half spacings h_d = s_d / 2:
//   3D beta  = (2a01 h1) o1 + (2a02 h2) o2 + l0,
//      alpha = (a11 h1^2) o1^2 + (2a12 h1 h2) o1 o2 + (a22 h2^2) o2^2
//              + (l1 h1) o1 + (l2 h2) o2 + c;
//   2D beta  = (2a01 h1) o1 + l0,  alpha = (a11 h1^2) o1^2 + (l1 h1) o1 + c.
// Each coefficient is rounded once to FP32 and split exactly into bf16 hi,
// mid and lo parts, one slot each (2D: a11's parts against f2_hi and again
// against f2_lo): 3D beta slots 0-8, alpha slots 0-14 and c_hi in 15; 2D
// beta slots 0-5, alpha slots 0-8 and c_hi in 9; the rest zero.  c - c_hi
// (exact in FP32) starts the alpha accumulator.  Padding seeds cost 1.7e38.
template <int D>
__device__ inline void hyb_stage(const Seeds &sd, int i, bool real, const double *anc, double wmax,
                                 double h1, double h2, ushort8 (&grp)[4], float &a00, float &crest) {
    constexpr int CHI = D == 3 ? 31 : 25;  // slot of c_hi (alpha's slots start at 16)
    unsigned short sl[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) sl[k] = 0;
    if (!real) {
        sl[CHI] = bf16_bits(1.7e38f);
        a00 = 0.0f;
        crest = 0.0f;
    } else {
        double qd[6], ld[3], cd, ed[3], wpd;
        seed_terms<D>(sd, i, anc, wmax, qd, ld, &cd, ed, &wpd);
        if constexpr (D == 3) {
            // qd = (a00, 2a01, 2a02, a11, 2a12, a22)
            const float cb[3] = {(float)(qd[1] * h1), (float)(qd[2] * h2), (float)ld[0]};
            const float ca[5] = {(float)(qd[3] * h1 * h1), (float)(qd[4] * h1 * h2), (float)(qd[5] * h2 * h2),
                                 (float)(ld[1] * h1), (float)(ld[2] * h2)};
#pragma unroll
            for (int k = 0; k < 3; ++k) bf16_split3(cb[k], sl + 3 * k);
#pragma unroll
            for (int k = 0; k < 5; ++k) bf16_split3(ca[k], sl + 16 + 3 * k);
        } else {
            // qd = (a00, 2a01, a11)
            bf16_split3((float)(qd[1] * h1), sl);
            bf16_split3((float)ld[0], sl + 3);
            bf16_split3((float)(qd[2] * h1 * h1), sl + 16);
            sl[19] = sl[16];
            sl[20] = sl[17];
            sl[21] = sl[18];
            bf16_split3((float)(ld[1] * h1), sl + 22);
        }
        const float cc = (float)cd;
        sl[CHI] = bf16_bits(cc);
        crest = cc - bf16_value(sl[CHI]);
        a00 = (float)qd[0];
    }
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
        ushort8 u;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) u[jj] = sl[8 * gq + jj];
        grp[gq] = u;
    }
}

// Rounding bound of the hybrid tile's costs: 2D that of the vector tile
// (e32_bound); 3D 1.3125 times it, for its longer matrix-core sum.
template <int D>
__device__ inline float hyb_bound(float B, float r, float r2) {
    return (D == 3 ? 0x1.5p-20f : 0x1p-20f) * (B + 4.0f * r * sqrtf(B) + 4.0f * r2);
}

// a wave-uniform float in a scalar register
__device__ inline float uniform_f(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

template <int D>
__device__ inline void hyb_tile(const Geo &g, const Seeds &sd, double wmax, Cert ct, int b0, int b1, int b2,
                                HybSmem<D> &sm, const PassOut &out, unsigned *qcount) {
    using Cfg = HybCfg<D>;
    constexpr int NJ = Cfg::kPairs;   // row pairs of a lane
    constexpr int NP = 2 * NJ;        // pixels a lane evaluates
    constexpr int CH = Cfg::kChunk;
    const int lane = __lane_id();
    const int half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    Tile<D> t;
    t.lane = lane;
    int j0;  // first row pair of this wave
    if constexpr (D == 3) {
        t.org[0] = b0 * Cfg::kRows;
        t.org[1] = b1 * 16 + wave * 4;
        t.org[2] = b2 * 8;
        t.anc[1] = b1 * 16 + 8;
        t.anc[2] = b2 * 8 + 4;
        t.k[1] = t.org[1] + (col >> 3);
        t.k[2] = t.org[2] + (col & 7);
        j0 = 0;
    } else {
        t.org[0] = b0 * Cfg::kRows;
        t.org[1] = b1 * 32;
        t.org[2] = 0;
        t.anc[1] = b1 * 32 + 16;
        t.anc[2] = 0;
        t.k[1] = t.org[1] + col;
        t.k[2] = 0;
        j0 = wave * NJ;
    }
    t.anc[0] = b0 * Cfg::kRows + Cfg::kRows / 2;
    t.k0w = half ? t.anc[0] + j0 : t.anc[0] - j0 - NJ;  // the rows this lane owns at the end
    t.k[0] = t.k0w;
    float s[3];
    double anc[3];
    for (int d = 0; d < D; ++d) {
        s[d] = (float)g.s[d];
        anc[d] = g.lo[d] + (double)t.anc[d] * g.s[d];
    }
    // rows: uj[j] = (j0 + j + 1/2) s0 above the anchor, -uj[j] below
    float uj[NJ], usq[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const float u = ((float)(j0 + j) + 0.5f) * s[0];
        uj[j] = uniform_f(u);
        usq[j] = uniform_f(u * u);
    }
    const float u1 = ((float)(t.k[1] - t.anc[1]) + 0.5f) * s[1];
    const float u2 = D == 3 ? ((float)(t.k[2] - t.anc[2]) + 0.5f) * s[2] : 0.0f;
    // operand B: the bf16 feature slots of this lane's position (half h
    // supplies slots 8 h .. 8 h + 7), as hyb_stage lays out the coefficients
    bf16x8 fbB, fbA;
    {
        float fB[16], fA[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) fB[k] = fA[k] = 0.0f;
        const float o1 = (float)(2 * (t.k[1] - t.anc[1]) + 1);
        if constexpr (D == 3) {
            const float o2 = (float)(2 * (t.k[2] - t.anc[2]) + 1);
            const float fb3[3] = {o1, o2, 1.0f}, fa3[5] = {o1 * o1, o1 * o2, o2 * o2, o1, o2};
#pragma unroll
            for (int k = 0; k < 9; ++k) fB[k] = fb3[k / 3];
#pragma unroll
            for (int k = 0; k < 15; ++k) fA[k] = fa3[k / 3];
            fA[15] = 1.0f;
        } else {
            const float f2 = o1 * o1, f2h = bf16_value(bf16_bits(f2)), f2l = f2 - f2h;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                fB[k] = o1;
                fB[3 + k] = 1.0f;
                fA[k] = f2h;
                fA[3 + k] = f2l;
                fA[6 + k] = o1;
            }
            fA[9] = 1.0f;
        }
        ushort8 uB, uA;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            uB[jj] = bf16_bits(half ? fB[8 + jj] : fB[jj]);
            uA[jj] = bf16_bits(half ? fA[8 + jj] : fA[jj]);
        }
        fbB = __builtin_bit_cast(bf16x8, uB);
        fbA = __builtin_bit_cast(bf16x8, uA);
    }
    const double h1 = 0.5 * g.s[1], h2 = D == 3 ? 0.5 * g.s[2] : 0.0;
    // the seed at scan position q (the scan follows out.seed_order)
    auto seed_at = [&](int q) { return out.seed_order ? out.seed_order[q] : q; };
    // seed i (padding unless real) into LDS position pos
    auto stage_at = [&](int pos, int i, bool real) {
        ushort8 gq[4];
        float a0, cr;
        hyb_stage<D>(sd, i, real, anc, wmax, h1, h2, gq, a0, cr);
#pragma unroll
        for (int k = 0; k < 4; ++k) sm.a[k][pos] = gq[k];
        sm.a00[pos] = a0;
        sm.crest[pos] = cr;
    };
    // beta and alpha of the 16 seeds (rows of this half) of the block staged
    // at positions pos .. pos + 31, at the lane's position: one
    // v_mfma_f32_32x32x16_bf16 each, alpha's accumulator starting from the
    // seeds' c - c_hi
    auto products = [&](int pos, floatx16 &bet, floatx16 &alp) {
        const bf16x8 ab = __builtin_bit_cast(bf16x8, sm.a[half][pos + col]);
        const bf16x8 aa = __builtin_bit_cast(bf16x8, sm.a[2 + half][pos + col]);
        floatx16 ci;
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            const float4 v = *reinterpret_cast<const float4 *>(&sm.crest[pos + 8 * qq + 4 * half]);
            ci[4 * qq] = v.x; ci[4 * qq + 1] = v.y; ci[4 * qq + 2] = v.z; ci[4 * qq + 3] = v.w;
        }
        bet = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ab, fbB, floatx16{}, 0, 0, 0);
        alp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aa, fbA, ci, 0, 0, 0);
    };
    // pixel 2 j + sgn: row anchor + j0 + j (sgn 0) or anchor - 1 - j0 - j (sgn 1)
    float fb[NP], fs[NP];
    int blk[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        fb[p] = INFINITY;
        fs[p] = INFINITY;
        blk[p] = 0;
    }

    for (int base = 0; base < g.n; base += CH) {
        const int cnt = min(CH, g.n - base);
        const int padded = (cnt + kHybSB - 1) & ~(kHybSB - 1);
        __syncthreads();
        for (int q = threadIdx.x; q < padded; q += kThreads)
            stage_at(q, q < cnt ? seed_at(base + q) : 0, q < cnt);
        __syncthreads();
        for (int sb = 0; sb < padded; sb += kHybSB) {
            float m[NP];
#pragma unroll
            for (int hb = 0; hb < kHybSB / 32; ++hb) {
                const int cb = sb + 32 * hb;
                floatx16 bet, alp;
                products(cb, bet, alp);
                float a0[16];
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    const float4 v = *reinterpret_cast<const float4 *>(&sm.a00[cb + 8 * qq + 4 * half]);
                    a0[4 * qq] = v.x; a0[4 * qq + 1] = v.y; a0[4 * qq + 2] = v.z; a0[4 * qq + 3] = v.w;
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const float q = fmaf(a0[r], usq[j], alp[r]);
                        const float cp = fmaf(bet[r], uj[j], q);
                        const float cm = fmaf(-bet[r], uj[j], q);
                        const bool first = hb == 0 && r == 0;
                        m[2 * j] = first ? cp : fminf(m[2 * j], cp);
                        m[2 * j + 1] = first ? cm : fminf(m[2 * j + 1], cm);
                    }
                }
            }
            const int gsb = (base + sb) / kHybSB;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                fs[p] = __builtin_amdgcn_fmed3f(fb[p], m[p], fs[p]);
                const bool better = m[p] < fb[p];
                blk[p] = better ? gsb : blk[p];
                fb[p] = better ? m[p] : fb[p];
            }
        }
    }

    // merge the half-waves' minima: lanes l and l ^ 32 hold the same pixels
    // against the two halves of every block, so after one exchange both know
    // each pixel's best cost, the super-block it lies in and the runner-up
    // among the super-block minima; bit p of `win` marks the pixels whose best
    // lies in this lane's half (both halves on equal costs in one super-block;
    // on equal costs in two, the lower super-block, and the certificate flags
    // the pixel either way)
    unsigned win = 0u;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const float ob = __shfl_xor(fb[p], 32);
        const float os = __shfl_xor(fs[p], 32);
        const int oi = __shfl_xor(blk[p], 32);
        const bool other = ob < fb[p] || (ob == fb[p] && oi < blk[p]);
        win |= (other ? 0u : 1u) << p;
        fs[p] = fminf(fmaxf(fb[p], ob), fminf(fs[p], os));
        fb[p] = fminf(fb[p], ob);
        blk[p] = other ? oi : blk[p];
    }

    // the seed inside each winning super-block: the wave forms the products
    // of one winning super-block at a time again (its smallest unresolved
    // one first) and each lane looks, among the costs of its half, for the
    // best of the pixels it won: the first seed attaining it and the smallest
    // of the other costs; a resolved pixel's blk holds its seed from then on
    unsigned done = 0u;  // bit p: resolved
    unsigned lostm = 0u; // bit p: the best cost was not found again (never expected)
    __syncthreads();     // every wave is done with the staged chunk
    for (;;) {
        int mine = 0x7fffffff;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (!(done >> p & 1u)) mine = min(mine, blk[p]);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) mine = min(mine, __shfl_xor(mine, o));
        const int wb = __builtin_amdgcn_readfirstlane(mine);
        if (wb == 0x7fffffff) break;
        unsigned want = 0u;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (!(done >> p & 1u) && blk[p] == wb) want |= 1u << p;
        done |= want;
        want &= win;
        // the super-block's 64 seeds, one per lane, in the wave's own 64
        // positions of the staging area
        {
            const int i = wb * kHybSB + lane;
            stage_at(64 * wave + lane, i < g.n ? seed_at(i) : 0, i < g.n);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // the lane's pixels in groups of 8 (4 row pairs), the products formed
        // again for each group, to bound the registers held; a group that no
        // lane of the wave wants is skipped
#pragma unroll
        for (int grp = 0; grp < NP / 8; ++grp) {
            if (!__ballot((want >> (8 * grp) & 0xffu) != 0u)) continue;
            float mn[8], s2[8];
            int ix[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                mn[e] = INFINITY;
                s2[e] = INFINITY;
                ix[e] = 0;
            }
#pragma unroll 1
            for (int hb = 0; hb < 2; ++hb) {
                const int pos = 64 * wave + 32 * hb;
                floatx16 bet, alp;
                products(pos, bet, alp);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float a0 = sm.a00[pos + 8 * (r >> 2) + 4 * half + (r & 3)];
                    const int k = 16 * hb + r;
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) {
                        const int j = 4 * grp + jj;
                        // the main scan's operations on the same operands
                        const float q = fmaf(a0, usq[j], alp[r]);
                        const float c2[2] = {fmaf(bet[r], uj[j], q), fmaf(-bet[r], uj[j], q)};
#pragma unroll
                        for (int sg = 0; sg < 2; ++sg) {
                            const int e = 2 * jj + sg;
                            const float c = c2[sg];
                            // best and second best so far, first index of the best
                            s2[e] = __builtin_amdgcn_fmed3f(mn[e], c, s2[e]);
                            ix[e] = c < mn[e] ? k : ix[e];
                            mn[e] = fminf(mn[e], c);
                        }
                    }
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int p = 8 * grp + e;
                if (!(want >> p & 1u)) continue;
                if (mn[e] != fb[p]) lostm |= 1u << p;
                // ix = 16 (block of 32 within the super-block) + r
                const int blk32 = ix[e] >> 4, r = ix[e] & 15;
                blk[p] = wb * kHybSB + 32 * blk32 + 8 * (r >> 2) + 4 * half + (r & 3);
                fs[p] = fminf(fs[p], s2[e]);
            }
        }
        // the area is rewritten by the next super-block
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // lane h keeps its pairs' rows below the anchor (h = 0) or above it
    // (h = 1), in row order p from t.k0w: h = 1 owns pixel (j = p, +), h = 0
    // pixel (j = NJ - 1 - p, -); the partner's seed and runner-up of those
    // pixels arrive by a swap across the half-waves
    const bool lane_ok = lane_in_grid<D>(g, t);
    // formed again rather than read: the scan has no register for it (8.67
    // instead of 8.63 ms at 256^3, N = 10^4)
    const float sab = dslack_abs(g, wmax, ct.lam), skb = kslack(ct);
    const unsigned owin = (unsigned)__shfl_xor((int)win, 32);
    const unsigned olost = (unsigned)__shfl_xor((int)lostm, 32);
    bool act[NJ], flag[NJ];
    int lab[NJ];
#pragma unroll
    for (int p = 0; p < NJ; ++p) {
        const int pa = 2 * p, pb = 2 * (NJ - 1 - p) + 1;  // (p, +) and (NJ - 1 - p, -)
        const int pm = half ? pa : pb;
        const float nb = fb[pm];  // equal in both halves
        const float ms = fs[pm];
        const int mi = blk[pm];
        const float os = __shfl_xor(half ? fs[pb] : fs[pa], 32);
        const int oi = __shfl_xor(half ? blk[pb] : blk[pa], 32);
        const bool mw = (win >> pm) & 1u, ow = (owin >> pm) & 1u;
        const float ns = fminf(ms, os);
        lab[p] = seed_at(min(mw && ow ? min(mi, oi) : mw ? mi : oi, g.n - 1));
        act[p] = lane_ok && t.k0w + p < g.grid[0];
        const float u0 = half ? uj[p] : -uj[NJ - 1 - p];
        const float r2 = pixel_r2(ct, u0, u1, u2);
        const float bb = fmaxf(nb, 0.0f);
        const float B1 = bb + 0x1p-10f * (bb + r2);
        const float e1 = hyb_bound<D>(B1, sqrtf(r2), r2);
        const float thr = 2.0f * e1 + sab + skb * (B1 + r2);
        flag[p] = ((lostm | olost) >> pm & 1u) || !((ns - nb) > thr);
        if (out.rel_gap && act[p] && !flag[p]) {
            const float c1u = (nb + 0x1p-19f * fabsf(nb) + e1 + sab + skb * (B1 + r2)) * (1.0f + 0x1p-20f);
            const float f2 = pad_inf(ns);
            const float bs = fmaxf(f2, 0.0f);
            const float B2 = bs + 0x1p-10f * (bs + r2);
            const float c2l = f2 == INFINITY ? f2
                              : (f2 - 0x1p-19f * fabsf(f2) - hyb_bound<D>(B2, sqrtf(r2), r2) - sab - skb * (B2 + r2)) *
                                    (1.0f - 0x1p-20f);
            out.rel_gap[pixel_index<D>(g, t.k0w + p, t)] = ns > 0.0f ? gap_lower(c1u, c2l) : 0.0f;
        }
    }
    tile_epilogue<D, NJ>(g, t, act, lab, flag, out, qcount);
}

// ------------------------------------------------------- bf16 matrix cores

// Slots of the bf16 dot product.  In tile-local half-pixel units
// v_d = 2 (k_d - anchor_d) + 1 (odd integers) the features are small
// integers, and every one of them is exactly a bf16 "hi" plus a bf16 "lo"
// part; each coefficient c is split as c_hi + c_lo (16 significant bits).
// A quadratic term c f takes three slots (c_hi f_hi, c_hi f_lo, c_lo f_hi),
// a linear one two (c_hi f, c_lo f), the constant three (c_hi + c_mid +
// c_lo, 24 significant bits: the constant carries the weight offset
// w_max - w, often the largest term).  2D: 3 x 3 + 2 x 2 + 3 = 16 slots (one
// 32x32x16 MFMA); 3D: 6 x 3 + 3 x 2 + 3 = 27 (two).
template <int D> struct Bf16Slots {
    static constexpr int NQ = D == 2 ? 3 : 6;   // quadratic features
    static constexpr int NL = D;                // linear features
    static constexpr int SLOTS = D == 2 ? 16 : 32;
    static constexpr int NM = SLOTS / 16;       // MFMAs per 32x32 block
    static_assert(3 * NQ + 2 * NL + 3 <= SLOTS, "bf16 slots");
};

// The coefficient side of the slots for one seed: c[0..NQ) quadratic,
// c[NQ..NQ+NL) linear, c[NQ+NL] constant.
template <int D>
__device__ inline void bf16_seed_slots(const float *c, unsigned short *out) {
    using SL = Bf16Slots<D>;
    int q = 0;
#pragma unroll
    for (int k = 0; k < SL::NQ + SL::NL + 1; ++k) {
        const unsigned short hi = bf16_bits(c[k]);
        const float rest = c[k] - bf16_value(hi);  // exact
        const unsigned short lo = bf16_bits(rest);
        out[q++] = hi;
        if (k < SL::NQ) out[q++] = hi;  // against f_lo
        if (k == SL::NQ + SL::NL) {
            // the constant: hi + mid + lo, each difference exact
            out[q++] = lo;
            out[q++] = bf16_bits(rest - bf16_value(lo));
        } else {
            out[q++] = lo;
        }
    }
#pragma unroll
    for (; q < SL::SLOTS; ++q) out[q] = 0;
}

// The feature side of the slots for one pixel: f as for the coefficients.
template <int D>
__device__ inline void bf16_pixel_slots(const float *f, unsigned short *out) {
    using SL = Bf16Slots<D>;
    int q = 0;
#pragma unroll
    for (int k = 0; k < SL::NQ + SL::NL + 1; ++k) {
        const unsigned short hi = bf16_bits(f[k]);
        if (k < SL::NQ) {
            const unsigned short lo = bf16_bits(f[k] - bf16_value(hi));
            out[q++] = hi;  // c_hi f_hi
            out[q++] = lo;  // c_hi f_lo
            out[q++] = hi;  // c_lo f_hi
        } else {
            out[q++] = hi;  // c_hi f (exact)
            out[q++] = hi;  // c_lo f
            if (k == SL::NQ + SL::NL) out[q++] = hi;  // the constant's third part
        }
    }
#pragma unroll
    for (; q < SL::SLOTS; ++q) out[q] = 0;
}

// LDS of the bf16 tile: per staged seed its bf16 slots (the matrix-core
// operand, seed-major so that a lane reads its 8 slots with one 16-byte
// load) and its FP32 coefficients in the layout of the vector tile
// (a00, 2a01, a11, -2(Ae)_0 | -2(Ae)_1, e^T A e - w' in 2D; the 3D rows
// hold a00, 2a01, 2a02, -2(Ae)_0 | a11, 2a12, a22, -2(Ae)_1 | -2(Ae)_2,
// e^T A e - w').
template <int D, int C>
struct Bf16Smem {
    static constexpr int kChunk = C;
    ushort8 sA[C * Bf16Slots<D>::SLOTS / 8];
    float4 sF4[D - 1][C];
    float2 sF2[C];
};

// Rows per lane of the bf16 tile: 4 in 2D, 2 in 3D (its two matrix-core
// operands per block need twice the registers).
template <int D> struct Bf16Rows { static constexpr int value = D == 2 ? 4 : 2; };

// The bf16 tier of one tile over every seed, in the vector tile's geometry
// (tile_at: P pixels per lane along axis 0).  A wave's pixels form 2P
// groups of 32: group 2r + c holds pixel r of lanes 32c .. 32c + 31, its
// column col that of lane 32c + col.  A 32-seed x 32-pixel block of costs
// is one (2D) or two (3D) v_mfma_f32_32x32x16_bf16 with the seeds on rows,
// so each lane holds 16 costs of one pixel (its column in the group)
// against 16 seeds (rows 8(r/4) + 4h + r%4 for the lane half h).  Those 16
// form a group:
//  * scan: per block and pixel group, the group minimum by 3-input integer
//    minima of the costs' bits (integer order is float order for the
//    non-negative costs; mixed-sign or negative near-ties fail the
//    certificate below), then the two smallest group minima and the group
//    of the best -- 12 operations per 16 pairs;
//  * at the end of each staged chunk the winning group of each pixel (over
//    both lane halves) is evaluated again in FP32 with the vector tile's
//    formulas, 8 seeds per lane half: this gives the label (the index is
//    kept in the low 4 bits of the FP32 cost) and the second-smallest cost
//    inside the group;
//  * certificate: with fb, fs the best and second FP32 costs of the winning
//    group and so the smallest bf16 group minimum of every other group, a
//    pixel is settled when fs - fb > 2 rho32 T + 2^-18 max|.| (as the FP32
//    tier) and so - fb > 2 rho16 T + 2^-18 max|.| (both plus the slack of
//    the double costs), rho32 = 2^-18 the bound of the FP32 costs and
//    rho16 = 2^-15 that of the bf16 costs.  Per monomial c f (c its FP32
//    coefficient in half-pixel units, f its integer feature): the
//    coefficient is within 2^-24 (1 + 2^-50) of its value; rounding to 8
//    significant bits gives |c - c_hi| <= 2^-8 |c| and |c - c_hi - c_lo|
//    <= 2^-16 |c|; f = f_hi + f_lo exactly (|v| < 64, so f < 2^12); the
//    slots hold c_hi f_hi + c_hi f_lo + c_lo f_hi = (c_hi + c_lo) f -
//    c_lo f_lo with |c_lo f_lo| <= 2^-16 (1 + 2^-8) |c f|; every product of
//    two bf16 numbers is exact in FP32; the accumulation of at most 31
//    products (two blocks of 16 slots in 3D, 15 in 2D) adds at most
//    gamma_31 < 2^-19 of sum |c f|.  So |C_bf16 - C| <= (2^-15 + 2^-19 +
//    2^-23) S (to first order) <= 1.07 2^-15 S, and S <= T / 1.13 as above: the
//    error is within rho16 T for any symmetric positive definite A_i.
//    Any seed that could beat the label would contradict one of the two
//    gaps, as in the single-tier argument; a negative bf16 minimum among
//    the other groups (integer order reversed) leaves so <= 0 < fb + the
//    gap, so such pixels are never settled.  Other pixels go to the double
//    re-check.
// The features are exact bf16 hi + lo pairs: in half-pixel units they are
// integers below 2^12 (|v| < 64).
template <int D, int P, int C>
__device__ inline void bf16_tile(const Geo &g, const Seeds &sd, double wmax, Cert ct, int b0, int b1, int b2,
                                 Bf16Smem<D, C> &sm, const PassOut &out, unsigned *qcount) {
    using SL = Bf16Slots<D>;
    static_assert(C % 32 == 0, "bf16 staging");
    constexpr int NG = 2 * P;  // 32-pixel groups per wave: gi = 2 r + c
    constexpr int kQ = SL::SLOTS / 8;  // 16-byte operand pieces per seed
    constexpr float kPad = 1.7e38f;

    const Tile<D> t = tile_at<D, P>(b0, b1, b2);
    const int lane = t.lane;
    const int half = lane >> 5, col = lane & 31;

    double ancd[3];
    float s[3];
    for (int d = 0; d < D; ++d) {
        ancd[d] = g.lo[d] + (double)t.anc[d] * g.s[d];
        s[d] = (float)g.s[d];
    }
    // the pixels of column col of each group: those of lane L = 32 c + col
    // of the wave (its first row k0c[c], its other indices), in FP32 and in
    // half-pixel units
    float u1c[2], u2c[2], v1c[2], v2c[2];
    int k0c[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        int k1, k2;
        lane_pixel<D, P>(t.org, 32 * c + col, k0c[c], k1, k2);
        u1c[c] = ((float)(k1 - t.anc[1]) + 0.5f) * s[1];
        u2c[c] = D == 3 ? ((float)(k2 - t.anc[2]) + 0.5f) * s[2] : 0.0f;
        v1c[c] = (float)(2 * (k1 - t.anc[1]) + 1);
        v2c[c] = D == 3 ? (float)(2 * (k2 - t.anc[2]) + 1) : 0.0f;
    }
    // matrix-core operand B (this lane's half of the pixel slots) per group
    bf16x8 bf[NG][SL::NM];
    float u0[NG];
#pragma unroll
    for (int r = 0; r < P; ++r) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int k0 = k0c[c] + r;
            u0[2 * r + c] = ((float)(k0 - t.anc[0]) + 0.5f) * s[0];
            const float v0 = (float)(2 * (k0 - t.anc[0]) + 1);
            const float v1 = v1c[c], v2 = v2c[c];
            float f[10];
            if (D == 2) {
                f[0] = v0 * v0; f[1] = v0 * v1; f[2] = v1 * v1;
                f[3] = v0; f[4] = v1; f[5] = 1.0f;
            } else {
                f[0] = v0 * v0; f[1] = v0 * v1; f[2] = v0 * v2;
                f[3] = v1 * v1; f[4] = v1 * v2; f[5] = v2 * v2;
                f[6] = v0; f[7] = v1; f[8] = v2; f[9] = 1.0f;
            }
            unsigned short sl[SL::SLOTS];
            bf16_pixel_slots<D>(f, sl);
#pragma unroll
            for (int m = 0; m < SL::NM; ++m) {
                ushort8 u;
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) u[jj] = half ? sl[16 * m + 8 + jj] : sl[16 * m + jj];
                bf[2 * r + c][m] = __builtin_bit_cast(bf16x8, u);
            }
        }
    }

    const int nscan = g.n;
    // staging of scan positions [base, base + cnt), padded to a multiple of
    // 32 with entries that cost 1.7e38 everywhere
    auto stage = [&](int base, int cnt, int padded) {
        for (int q = threadIdx.x; q < padded; q += kThreads) {
            float c[10];  // bf16-slot coefficients (half-pixel units)
            if (q >= cnt) {
#pragma unroll
                for (int z = 0; z < 10; ++z) c[z] = 0.0f;
                c[SL::NQ + SL::NL] = kPad;
                for (int r = 0; r < D - 1; ++r) sm.sF4[r][q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                sm.sF2[q] = make_float2(0.0f, kPad);
            } else {
                double qd[6], ld[3], cd, ed[3], wpd;
                seed_terms<D>(sd, base + q, ancd, wmax, qd, ld, &cd, ed, &wpd);
                const double h0 = 0.5 * g.s[0], h1 = 0.5 * g.s[1], h2 = D == 3 ? 0.5 * g.s[2] : 0.0;
                if (D == 2) {
                    sm.sF4[0][q] = make_float4((float)qd[0], (float)qd[1], (float)qd[2], (float)ld[0]);
                    sm.sF2[q] = make_float2((float)ld[1], (float)cd);
                    c[0] = (float)(qd[0] * h0 * h0); c[1] = (float)(qd[1] * h0 * h1);
                    c[2] = (float)(qd[2] * h1 * h1);
                    c[3] = (float)(ld[0] * h0); c[4] = (float)(ld[1] * h1); c[5] = (float)cd;
                } else {
                    sm.sF4[0][q] = make_float4((float)qd[0], (float)qd[1], (float)qd[2], (float)ld[0]);
                    sm.sF4[D - 2][q] = make_float4((float)qd[3], (float)qd[4], (float)qd[5], (float)ld[1]);
                    sm.sF2[q] = make_float2((float)ld[2], (float)cd);
                    c[0] = (float)(qd[0] * h0 * h0); c[1] = (float)(qd[1] * h0 * h1);
                    c[2] = (float)(qd[2] * h0 * h2); c[3] = (float)(qd[3] * h1 * h1);
                    c[4] = (float)(qd[4] * h1 * h2); c[5] = (float)(qd[5] * h2 * h2);
                    c[6] = (float)(ld[0] * h0); c[7] = (float)(ld[1] * h1); c[8] = (float)(ld[2] * h2);
                    c[9] = (float)cd;
                }
            }
            unsigned short sl[SL::SLOTS];
            bf16_seed_slots<D>(c, sl);
#pragma unroll
            for (int m = 0; m < kQ; ++m) {
                ushort8 u;
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) u[jj] = sl[8 * m + jj];
                sm.sA[q * kQ + m] = u;
            }
        }
    };
    // FP32 cost of staged seed q at the pixel (v0, v1, v2) (tile-local
    // coordinates; the vector tile's formulas)
    auto cost32 = [&](int q, float v0, float v1, float v2) {
        const float4 c0 = sm.sF4[0][q];
        const float2 cl = sm.sF2[q];
        float beta, alpha;
        if constexpr (D == 2) {
            beta = fmaf(c0.y, v1, c0.w);
            alpha = fmaf(fmaf(c0.z, v1, cl.x), v1, cl.y);
        } else {
            const float4 c1 = sm.sF4[D - 2][q];
            beta = fmaf(c0.y, v1, fmaf(c0.z, v2, c0.w));
            alpha = fmaf(fmaf(c1.x, v1, fmaf(c1.y, v2, c1.w)), v1, fmaf(fmaf(c1.z, v2, cl.x), v2, cl.y));
        }
        return fmaf(fmaf(c0.x, v0, beta), v0, alpha);
    };

    // group minima (bf16 costs as integers): best, second, block of the best
    int best[NG], second[NG], blk[NG];
    // the winning group evaluated in FP32: scan position, best and second keys
    int lab[NG], kb[NG], ks[NG];
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
        best[gi] = 0x7fffffff;
        second[gi] = 0x7fffffff;
        blk[gi] = -1;
        lab[gi] = 0;
        kb[gi] = 0x7fffffff;
        ks[gi] = 0x7fffffff;
    }
    for (int base = 0; base < nscan; base += C) {
        const int cnt = min(C, nscan - base);
        const int padded = (cnt + 31) & ~31;
        __syncthreads();
        stage(base, cnt, padded);
        __syncthreads();
        for (int cb = 0; cb < padded; cb += 32) {
            bf16x8 av[SL::NM];
#pragma unroll
            for (int m = 0; m < SL::NM; ++m)
                av[m] = __builtin_bit_cast(bf16x8, sm.sA[(cb + col) * kQ + 2 * m + half]);
            floatx16 acc[NG];
#pragma unroll
            for (int gi = 0; gi < NG; ++gi) {
                acc[gi] = floatx16{};
#pragma unroll
                for (int m = 0; m < SL::NM; ++m)
                    acc[gi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[m], bf[gi][m], acc[gi], 0, 0, 0);
            }
            const int gblk = base + cb;
#pragma unroll
            for (int gi = 0; gi < NG; ++gi) {
                int k[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) k[r] = __float_as_int(acc[gi][r]);
                const int t0 = min(min(k[0], k[1]), k[2]);
                const int t1 = min(min(k[3], k[4]), k[5]);
                const int t2 = min(min(k[6], k[7]), k[8]);
                const int t3 = min(min(k[9], k[10]), k[11]);
                const int t4 = min(min(k[12], k[13]), k[14]);
                const int m = min(min(min(t0, t1), t2), min(min(t3, t4), k[15]));
                second[gi] = med3i(best[gi], m, second[gi]);
                blk[gi] = m < best[gi] ? gblk : blk[gi];
                best[gi] = min(best[gi], m);
            }
        }
        // the pixel's winning group (ties to lane half 0); where it was
        // found in this chunk, evaluate it again in FP32
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
            const int pb = __shfl_xor(best[gi], 32);
            const int pblk = __shfl_xor(blk[gi], 32);
            const bool other = half == 0 ? pb < best[gi] : pb <= best[gi];
            const int wblk = other ? pblk : blk[gi];
            const int wh = other ? 1 - half : half;
            const bool need = wblk >= base;
            if (__ballot(need)) {
                // rows r = 8 half .. 8 half + 7 of the group: seeds
                // wblk + 8 (r / 4) + 4 wh + r % 4
                const int q0 = max(wblk - base, 0) + 4 * wh + 16 * half;
                int bk = 0x7fffffff, s2 = 0x7fffffff;
#pragma unroll
                for (int rr = 0; rr < 8; ++rr) {
                    const int q = q0 + 8 * (rr >> 2) + (rr & 3);
                    const float c = cost32(q, u0[gi], u1c[gi & 1], u2c[gi & 1]);
                    const int key = (__float_as_int(c) & ~15) | (8 * half + rr);
                    s2 = med3i(bk, key, s2);
                    bk = min(bk, key);
                }
                const int ob = __shfl_xor(bk, 32);
                const int os = __shfl_xor(s2, 32);
                const int nb = min(bk, ob);
                const int ns = min(max(bk, ob), min(s2, os));
                if (need) {
                    const int r = nb & 15;
                    lab[gi] = wblk + 8 * (r >> 2) + 4 * wh + (r & 3);
                    kb[gi] = nb;
                    ks[gi] = ns;
                }
            }
        }
    }

    const float sab = ct.sab, skb = kslack(ct);
    // lane l takes to the epilogue the groups of its own column half (the
    // pixels of column l % 32 of those groups are its own)
    const bool lane_ok = lane_in_grid<D>(g, t);
    bool act[P], flag[P];
    int labe[P];
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
        const int pb = __shfl_xor(best[gi], 32);
        const int ps = __shfl_xor(second[gi], 32);
        const int so = min(max(best[gi], pb), min(second[gi], ps));
        const float fb = __int_as_float(kb[gi]), fs = __int_as_float(ks[gi]);
        const float fo = __int_as_float(so);
        const float r2 = pixel_r2(ct, u0[gi], u1c[gi & 1], u2c[gi & 1]);
        const float rr = sqrtf(r2);
        const float bb = fmaxf(fb, 0.0f);
        const float B1 = bb + 0x1p-10f * (bb + r2);
        const float e32 = e32_bound(B1, rr, r2), e16 = e16_bound(B1, rr, r2);
        const float slack = sab + skb * (B1 + r2);
        const float thr32 = 2.0f * e32 + 0x1p-18f * fmaxf(fabsf(fb), fabsf(fs)) + slack;
        const float thr16 = e32 + e16 + 0x1p-18f * fmaxf(fabsf(fb), fabsf(fo)) + slack;
        const bool settled = (fs - fb) > thr32 && (fo - fb) > thr16;
        const int r = gi >> 1;
        if ((gi & 1) == half) {
            act[r] = lane_ok && (t.k0w + r) < g.grid[0];
            flag[r] = !settled;
            labe[r] = min(lab[gi], nscan - 1);
            if (out.rel_gap && act[r] && settled) {
                // the winner costs at most c1u; the rest of its group at
                // least fs, the other groups at least fo, each less its bound
                const float c1u = (fb + 0x1p-19f * fabsf(fb) + e32 + slack) * (1.0f + 0x1p-20f);
                const float f2 = pad_inf(fs), fo2 = pad_inf(fo);
                const float bs = fmaxf(f2, 0.0f), bo = fmaxf(fo2, 0.0f);
                const float Bs = bs + 0x1p-10f * (bs + r2), Bo = bo + 0x1p-10f * (bo + r2);
                const float cs = f2 == INFINITY
                                     ? f2
                                     : f2 - 0x1p-19f * fabsf(f2) - e32_bound(Bs, rr, r2) - sab - skb * (Bs + r2);
                const float co = fo2 == INFINITY ? fo2 : fo2 - e16_bound(Bo, rr, r2) - sab - skb * (Bo + r2);
                const float c2l = fminf(cs, co) * (1.0f - 0x1p-20f);
                out.rel_gap[pixel_index<D>(g, t.k0w + r, t)] =
                    (fs > 0.0f && fo > 0.0f) ? gap_lower(c1u, c2l) : 0.0f;
            }
        }
    }
    tile_epilogue<D, P>(g, t, act, labe, flag, out, qcount);
}

// ------------------------------------------------------- double re-check

// Seeds staged in LDS for the double re-check: x, the upper triangle of A
// (row by row) and w of up to S seeds.
template <int D, int S>
struct StagedSeeds {
    static constexpr int kSeeds = S;
    static constexpr int kTri = D * (D + 1) / 2;
    double x[D][S];
    double a[kTri][S];
    double w[S];
};

// Stage seed `i` at position q (every thread of the block calls it for its
// positions; a barrier must follow before the reads).
template <int D, int S>
__device__ inline void stage_seed(StagedSeeds<D, S> &sm, const Seeds &sd, int q, int i) {
    const double *xi = sd.x + (size_t)i * D;
    const double *ai = sd.A + (size_t)i * D * D;
    int t = 0;
    for (int r = 0; r < D; ++r) {
        sm.x[r][q] = xi[r];
        for (int c = r; c < D; ++c, ++t) sm.a[t][q] = ai[r * D + c];
    }
    sm.w[q] = sd.w[i];
}

// The double cost of the staged seed at position q at y, in the expression
// order of exact_cost (the same roundings, so the same value).
template <int D, int S>
__device__ inline double staged_cost(const StagedSeeds<D, S> &sm, int q, const double *y, int power = 2) {
    double dd[D];
#pragma unroll
    for (int e = 0; e < D; ++e) dd[e] = y[e] - sm.x[e][q];
    double qf = 0.0;
#pragma unroll
    for (int e = 0; e < D; ++e) {
        double row = 0.0;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const int lo = e < c ? e : c, hi = e < c ? c : e;
            const int tix = lo * D - lo * (lo - 1) / 2 + (hi - lo);  // (lo, hi) packed
            const double t = sm.a[tix][q] * dd[c];
            row = (c == 0) ? t : row + t;
        }
        const double t = dd[e] * row;
        qf = (e == 0) ? t : qf + t;
    }
    return power_of_norm(qf, power) - sm.w[q];
}

// ------------------------------------------------------- the FP64 tile

// LDS of the FP64 tile.
template <int D, bool CULL>
struct Fp64Smem {
    static constexpr int kChunk = 128;  // seeds staged at a time
    StagedSeeds<D, kChunk> seeds;
    int list[CULL ? kCullCap : 1];  // candidate seeds of the tile
    MomSmem<CULL ? kP : 1> mom[CULL ? 1 : 0];
    CellQuad<D> own[kWaves];
    double red[kWaves];
    double part[kWaves];
    int cnt;
};

// Every cost in double precision, in the order of the definition: a lane's kP
// pixels against the tile's candidate seeds (CULL) or every seed, staged in
// LDS.  The kernel over every seed, one at a time through scalar loads, took
// 190 us on 512^2 pixels with 500 seeds; with the lists 15 us (over every seed,
// staged, 145).  For costs
// other than the squared norm the block also sums its pixels' least costs,
// weighted by the pixel weights, in a fixed order (per lane, a butterfly in
// the wave, the waves in order) into *cost_part.
template <int D, bool CULL>
__device__ inline void fp64_tile(const Geo &g, const Seeds &sd, double wmax, Cert ct, const double *eig, int b0,
                                 int b1, int b2, Fp64Smem<D, CULL> &sm, const PassOut &out, double *cost_part) {
    constexpr int C = Fp64Smem<D, CULL>::kChunk;
    const Tile<D> t = tile_at<D>(b0, b1, b2);
    const bool lane_ok = lane_in_grid<D>(g, t);
    int nscan = g.n;
    bool full = true;
    if constexpr (CULL) {
        double U;
        const int ncand = g.power != 2 ? tile_candidates<D, kP, true>(g, sd, wmax, ct, eig, out, b0, b1, b2, sm, &U)
                                       : tile_candidates<D, kP, false>(g, sd, wmax, ct, eig, out, b0, b1, b2, sm, &U);
        full = ncand > kCullCap;
        nscan = full ? g.n : ncand;
        if (out.adaptive && ncand == 1 && !g.mass && !cost_part) {
            credit_tile<D, kP>(g, t, b0, b1, b2, sm.list[0], out);
            return;
        }
    }
    bool act[kP], flag[kP];
    double y[kP][D];
#pragma unroll
    for (int p = 0; p < kP; ++p) {
        act[p] = lane_ok && (t.k0w + p) < g.grid[0];
        flag[p] = false;
        y[p][0] = centre(g, 0, t.k0w + p);
        for (int d = 1; d < D; ++d) y[p][d] = centre(g, d, t.k[d]);
    }
    double best[kP], second[kP];
    int pos[kP];
#pragma unroll
    for (int p = 0; p < kP; ++p) {
        best[p] = INFINITY;
        second[p] = INFINITY;
        pos[p] = 0;
    }
    for (int c0 = 0; c0 < nscan; c0 += C) {
        const int cnt = min(C, nscan - c0);
        __syncthreads();
        if ((int)threadIdx.x < cnt)
            stage_seed<D, C>(sm.seeds, sd, threadIdx.x, full ? c0 + (int)threadIdx.x : sm.list[c0 + threadIdx.x]);
        if constexpr (CULL)
            if (c0 == 0 && out.mom) moments_zero(sm.mom[0], min(nscan, kAccSlots));
        __syncthreads();
#pragma unroll 2
        for (int q = 0; q < cnt; ++q) {
#pragma unroll
            for (int p = 0; p < kP; ++p) {
                const double c = staged_cost<D, C>(sm.seeds, q, y[p], g.power);
                // equal costs go to the lowest seed: a scan over every seed
                // meets it first, a list may hold it later
                bool better = c < best[p];
                if (CULL && !full && c == best[p]) better = sm.list[c0 + q] < sm.list[pos[p]];
                if (!CULL && out.rel_gap) second[p] = better ? best[p] : fmin(second[p], c);
                best[p] = better ? c : best[p];
                pos[p] = better ? c0 + q : pos[p];
            }
        }
    }
    int lab[kP];
#pragma unroll
    for (int p = 0; p < kP; ++p) {
        lab[p] = full ? pos[p] : nscan > 0 ? sm.list[pos[p]] : 0;
        if (!CULL && out.rel_gap && act[p])
            out.rel_gap[pixel_index<D>(g, t.k0w + p, t)] = gap_exact(best[p], second[p], wmax);
    }
    if (cost_part) {
        double sp = 0.0;
#pragma unroll
        for (int p = 0; p < kP; ++p)
            if (act[p]) sp += (double)pixel_weight(g, pixel_index<D>(g, t.k0w + p, t)) * best[p];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) sp += __shfl_xor(sp, o);
        if (t.lane == 0) sm.part[threadIdx.x >> 6] = sp;
        __syncthreads();
        if (threadIdx.x == 0) *cost_part = (sm.part[0] + sm.part[1]) + (sm.part[2] + sm.part[3]);
    }
    if constexpr (CULL) {
        if (nscan > 0 && nscan <= kAccSlots && !full && !g.mass) {
            if (out.labels) write_labels<D, kP>(g, t, act, lab, flag, out);
            if (out.mom) {
                int idx[kP];
#pragma unroll
                for (int p = 0; p < kP; ++p) idx[p] = act[p] ? pos[p] : 127;
                moments_add<D, kP>(sm.mom[0], t.lane, idx, nscan, [](int j) { return j; });
                __syncthreads();
                moments_flush<D, kP>(sm.mom[0], t.anc, sm.list, nscan, out.mom);
            }
            return;
        }
    }
    tile_epilogue<D>(g, t, act, lab, flag, out, nullptr);
}

// Grid index k and centre y of pixel j (eq. (2.6)).
template <int D>
__device__ inline void pixel_of(const Geo &g, uint32_t j, int *k, double *y) {
    uint32_t r = j;
    for (int d = D - 1; d >= 0; --d) {
        k[d] = (int)(r % (uint32_t)g.grid[d]);
        r /= (uint32_t)g.grid[d];
    }
    for (int d = 0; d < D; ++d) y[d] = centre(g, d, k[d]);
}

// Double re-check, by one wave, of the `count` queued pixels from queue
// position `start` against every seed (the batched passes without candidate
// lists).  The seeds are staged in the wave's own LDS (sm) chunk by chunk; a
// group of G lanes takes one pixel (G the largest power of two, up to 64,
// that leaves a group for every pixel of the segment), lane r of the group
// scans the staged positions r, r + G, ...  pixel_at(q) gives the pixel index
// at queue position q.  Every lane of the wave must call it.
template <int D, int S, class PixelAt>
__device__ inline void recheck_segment(const Geo &g, const Seeds &sd, unsigned start, unsigned count,
                                       PixelAt pixel_at, uint64_t *mom, StagedSeeds<D, S> &sm) {
    const int lane = __lane_id();
    int G = 64;
    while (G > 1 && (unsigned)(64 / G) < count) G >>= 1;
    const unsigned ngroups = (unsigned)(64 / G);
    const int grp = lane / G, r = lane % G;
    for (unsigned p0 = 0; p0 < count; p0 += ngroups) {
        const unsigned p = p0 + (unsigned)grp;
        const bool valid = p < count;
        const uint32_t j = valid ? pixel_at(start + p) : 0u;
        int k[3];
        double y[D];
        pixel_of<D>(g, j, k, y);
        double b = INFINITY;
        int bi = 0x7fffffff;
        for (int c0 = 0; c0 < g.n; c0 += S) {
            const int cnt = min(S, g.n - c0);
            wave_lds_sync();
            for (int q = lane; q < cnt; q += 64) stage_seed<D, S>(sm, sd, q, c0 + q);
            wave_lds_sync();
            for (int q = r; q < cnt; q += G) {
                const double c = staged_cost<D, S>(sm, q, y);
                if (c < b || (c == b && c0 + q < bi)) {
                    b = c;
                    bi = c0 + q;
                }
            }
        }
        group_min(b, bi, G);
        if (bi >= g.n) bi = 0;  // no finite cost (non-finite input, reported by the prep step)
        if (valid && r == 0) pixel_moments_add<D>(mom, bi, k, pixel_weight(g, j));
    }
}

// Finalize of one cell from its exact moments (o = 2k + 1, y = lo + h o,
// h = s/2):
//   m_i, grad_i = v_i - m_i |P|                                  eq. (2.8)
//   centroid ybar = lo + h S_d / m                                 Alg. 3
//   sum_{cell} |y - x_i|^2_A = m |ybar - x_i|^2_A
//                              + sum_de A_de h_d h_e (S_de - S_d S_e / m)
// returns the cell's term of eq. (2.7), (v_i - m_i |P|) w_i + |P| sum |y - x_i|^2_A,
// and its relative volume error.  For other costs (g.power != 2) the term is
// v_i w_i and the finalize adds |P| sum_j q_j C_{H_j j} (eq. (2.7) written
// over pixels), summed by the assignment kernel.
template <int D>
__device__ inline double cell_final(const Geo &g, const Seeds &sd, const uint64_t *M, int i,
                                   double *grad_i, double *rel_i, double *ybar) {
    const uint64_t m = M[0];
    const double md = (double)m;
    const double vi = sd.v[i], wi = sd.w[i];
    const double gi = vi - md * g.munit;
    *grad_i = gi;
    *rel_i = fabs(gi) / vi;
    const double *a = sd.A + (size_t)i * D * D;
    double h[3];
    for (int d = 0; d < D; ++d) h[d] = 0.5 * g.s[d];
    double integral = 0.0;
    if (m > 0 && g.power != 2) {
        // other costs: the cell's share of sum_j |P_j| C_{H_j j} is summed
        // pixel by pixel (Scalars::gpix); here only the centroid and v_i w_i
        for (int d = 0; d < D; ++d) ybar[d] = g.lo[d] + h[d] * ((double)M[1 + d] / md);
        return vi * wi;
    }
    if (m > 0) {
        double S1[3], dev[3];
        for (int d = 0; d < D; ++d) {
            S1[d] = (double)M[1 + d];
            ybar[d] = g.lo[d] + h[d] * (S1[d] / md);
            dev[d] = ybar[d] - sd.x[(size_t)i * D + d];
        }
        double q1 = 0.0, q2 = 0.0;
        int c = 0;
        for (int d = 0; d < D; ++d)
            for (int e = d; e < D; ++e, ++c) {
                const double ade = a[d * D + e] * (d == e ? 1.0 : 2.0);
                const double cov = (double)M[1 + D + c] - S1[d] * (S1[e] / md);
                q1 += ade * dev[d] * dev[e];
                q2 += ade * h[d] * h[e] * cov;
            }
        integral = g.munit * (md * q1 + q2);
    } else {
        for (int d = 0; d < D; ++d) ybar[d] = sd.x[(size_t)i * D + d];
        if (g.power != 2) return vi * wi;
    }
    return gi * wi + integral;
}

}  // namespace dev
}  // namespace apd
