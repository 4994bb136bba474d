// Leaf of the block-LU inversion, the method the paper compares SPIN with
// (Sec. 5, after Liu et al.): A = L U without pivoting, then L^-1 and U^-1.
// The block recursion around it (spin_api.cpp) uses the product kernels.
#include <hip/hip_runtime.h>

#include <cfloat>

#include "leaf_blocks.hpp"
#include "spin_kernels.hpp"

namespace spin {
namespace {

// One workgroup factors an order-L block (L <= kLuLeafMax) and inverts both
// factors in a single in-place pass.  Step k, with the pivot u_kk:
//   rows i > k   l_ik = x_ik / u_kk;  x_ij -= l_ik x_kj for every j != k (the
//                Schur complement right of k, L^-1 left of it);  x_ik = -l_ik
//   rows i < k   v_ik = x_ik / u_kk;  x_ij -= v_ik x_kj for j > k;  x_ik = v_ik
//                (row i of U^-1, from V U = I)
//   row k        x_kk = 1 / u_kk;  x_kj = -x_kj / u_kk for j > k
// Row k of U is used at step k only, so its place takes row k of U^-1 from
// then on, as the place of L's columns takes L^-1.
//
// Sixteen steps form a block step, as in the Gauss-Jordan leaves: one wave
// runs them on the diagonal block (the serial chain), one lane per row takes
// them through the block column (multipliers F) and one lane per column
// through the block row (R = rows of U and of L^-1 at their steps), and every
// other block takes four v_mfma_f64_16x16x4f64 with -F and R, except those
// above and left of the diagonal block, which step k leaves alone.  Wave w
// holds the 16 rows 16 w .. 16 w + 15 in accumulators; panels pass through LDS.
//
// Bound by the chains and panels, one after the other (7 us a block step of eight
// waves), against a column-at-a-time elimination and two substitution passes in
// LDS with two barriers per column before: order 128 731 -> 59 us.

// Pivots that are normal numbers with a normal reciprocal, which quotient
// needs.  Blocks with another one (subnormal, above 2^1022, zero or not
// finite) divide.
__device__ inline bool normal_pivot(double p) {
    const unsigned e = (unsigned)(__double_as_longlong(p) >> 52) & 0x7ffu;
    return e - 1u <= 2043u;
}

// The quotient f / p from its rounded reciprocal, with one correction step.
template <bool DIV>
__device__ inline double quotient(double f, double p, double pinv) {
    if constexpr (DIV) return f / p;
    const double q = f * pinv;
    return fma(fma(-q, p, f), pinv, q);
}

// Step K inside the diagonal block.  dr + 16 K gets row K as the step uses it,
// dm + 16 K the multipliers with the pivot itself at row K, iv[K] 1 / pivot.
template <bool DIV, int K>
__device__ __attribute__((always_inline)) inline void lu_step(d4_t &D, int rr, int g, double *dm, double *dr,
                                                              double *iv, double *dump) {
    constexpr int V = K / 4, G = K % 4;
    double *const st = dump + 256;  // the active column, passed to the other lane groups
    st[16 * g + rr] = D[V];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const double f = st[16 * G + rr];
    const double piv = readlane_f64(D[V], 16 * G + K);
    const double pinv = 1.0 / piv;
    const bool prow = rr == K;
    double *const pr = (prow ? dr : dump) + g;
#pragma unroll
    for (int v = 0; v < 4; ++v) pr[16 * K + 4 * v] = D[v];
    const double m = prow ? pinv : quotient<DIV>(f, piv, pinv);
    const double below = rr > K ? m : 0.0;  // multiplier left of column K
    if (g == 0) dm[16 * K + rr] = prow ? piv : m;
    if (g == 0 && prow) iv[K] = pinv;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const bool right = v > V || (v == V && g > G);
        const double u = row_bcast<K>(D[v]);
        const double base = (prow && right) ? 0.0 : D[v];
        D[v] = fma(-(right ? m : below), u, base);
    }
    if (g == G) D[V] = rr > K ? -m : m;
}

template <bool DIV, int... K>
__device__ __attribute__((always_inline)) inline void lu_chain(d4_t &D, int lane, double *dm, double *dr, double *iv,
                                                               double *dump, std::integer_sequence<int, K...>) {
    lane = opaque(lane);
    (lu_step<DIV, K>(D, lane & 15, lane >> 4, dm, dr, iv, dump), ...);
}

// The 16 steps on one row of the block column; the lane's group of 16 rows is
// above or below the diagonal block.  pv, iv: lane l % 16 holds pivot l % 16
// and its reciprocal.
template <bool DIV, int... K>
__device__ __attribute__((always_inline)) inline void lu_rows(double (&x)[16], const double *dr, int rr, bool above,
                                                              double pv, double iv, double *F, int ld,
                                                              std::integer_sequence<int, K...>) {
    double r[16] = {(above && rr < K ? 0.0 : dr[16 * K + rr])...};
    (
        [&] {
            const double m = quotient<DIV>(x[K], row_bcast<K>(pv), row_bcast<K>(iv));
            F[K * ld] = m;
            fmac_rows(x, r[K], m);
            x[K] = above ? m : -m;
        }(),
        ...);
}

// The 16 steps on one column of the block row; the lane's group of 16 columns
// is left or right of the diagonal block.
template <bool DIV, int... K>
__device__ __attribute__((always_inline)) inline void lu_cols(double (&y)[16], const double *dm, int rr, bool left,
                                                              double pv, double iv, double *R, int ld,
                                                              std::integer_sequence<int, K...>) {
    double m[16] = {(rr == K || (left && rr < K) ? 0.0 : dm[16 * K + rr])...};
    (
        [&] {
            const double u = y[K];
            R[K * ld] = u;
            fmac_rows(y, m[K], u);
            y[K] = left ? u : DIV ? -(u / row_bcast<K>(pv)) : -(u * row_bcast<K>(iv));
        }(),
        ...);
}

// N waves, orders up to 16 N.
template <int N>
__global__ void __launch_bounds__(64 * N)
    k_lu_leaf_inv(const double *__restrict__ A, int64_t lda, double *__restrict__ Li, int64_t ldl,
                  double *__restrict__ Ui, int64_t ldu, int L, int col0, int *status) {
    using S = BlkLds<N, 1, N>;
    constexpr int oIv = S::oDump + 320;  // the dump's first 256 + 12 doubles, then a column of 64
    __shared__ __attribute__((aligned(16))) double sm[oIv + 16];
    constexpr auto kSteps = std::make_integer_sequence<int, 16>{};
    const int t = threadIdx.x, lane0 = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    d4_t acc[N];
    {
        const int rr = lane0 & 15, g = lane0 >> 4, row = 16 * w + rr;
#pragma unroll
        for (int c = 0; c < N; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int col = 16 * c + 4 * v + g;
                // continued as the identity beyond the order
                acc[c][v] = (row < L && col < L) ? A[row + (int64_t)col * lda] : (row == col ? 1.0 : 0.0);
            }
    }
    const int nblk = (L + 15) >> 4;
    double *const F = sm + S::oF, *const R = sm + S::oR, *const dr = sm + S::oDr, *const dm = sm + S::oDm,
                 *const dump = sm + S::oDump, *const iv = sm + oIv;
    d4_t D{0.0, 0.0, 0.0, 0.0};
    int bad = 0;
    auto publish = [&](const int b, const int u) {
        const int ln = opaque(lane0), rr = ln & 15, g = ln >> 4;
        double *pc = sm + S::oPc + u * 16 * S::kFLd, *pr = sm + S::oPr + u * 16 * S::kPrLd;
        static_for<N>([&](auto c) {
            if (c == b) {
#pragma unroll
                for (int v = 0; v < 4; ++v) pc[(4 * v + g) * S::kFLd + 16 * w + rr] = acc[c][v];
                branch_end<c>();
            }
        });
        if (w == b) {
#pragma unroll
            for (int c = 0; c < N; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) pr[rr * S::kPrLd + 16 * c + 4 * v + g] = acc[c][v];
        }
    };
    publish(0, 0);
    if (w == 0) {
        D = acc[0];
        lu_chain<false>(D, lane0, dm, dr, iv, dump, kSteps);
    }
#pragma unroll 1
    for (int b = 0; b < nblk; ++b) {
        const int u = b & 1;
        const int lane = opaque(lane0), rr = lane & 15, g = lane >> 4;
        double *const pc = sm + S::oPc + u * 16 * S::kFLd, *const pr = sm + S::oPr + u * 16 * S::kPrLd;
        __syncthreads();
        const bool div = __any(!normal_pivot(dm[17 * rr]));  // the same in every wave
        if (div) {
            // the chain again, with divisions
            __syncthreads();
            if (w == b) {
#pragma unroll
                for (int v = 0; v < 4; ++v) D[v] = pr[rr * S::kPrLd + 16 * b + 4 * v + g];
                lu_chain<true>(D, lane, dm, dr, iv, dump, kSteps);
            }
            __syncthreads();
        }
        // ---- panels: one wave per 64 rows, one per 64 columns ----
        constexpr int CH = (16 * N + 63) / 64;
        if (w < CH) {
            const int row = 64 * w + lane;
            double x[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) x[j] = pc[j * S::kFLd + row];
            if (div)
                lu_rows<true>(x, dr, rr, (row >> 4) < b, dm[17 * rr], iv[rr], F + row, S::kFLd, kSteps);
            else
                lu_rows<false>(x, dr, rr, (row >> 4) < b, dm[17 * rr], iv[rr], F + row, S::kFLd, kSteps);
#pragma unroll
            for (int j = 0; j < 16; ++j) pc[j * S::kFLd + row] = x[j];
        } else if (w < 2 * CH) {
            const int col = 64 * (w - CH) + lane;
            double y[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) y[j] = pr[j * S::kPrLd + col];
            if (div)
                lu_cols<true>(y, dm, rr, (col >> 4) < b, dm[17 * rr], iv[rr], R + col, S::kRLd, kSteps);
            else
                lu_cols<false>(y, dm, rr, (col >> 4) < b, dm[17 * rr], iv[rr], R + col, S::kRLd, kSteps);
#pragma unroll
            for (int j = 0; j < 16; ++j) pr[j * S::kPrLd + col] = y[j];
        }
        if (w == 0) {
            // the first zero or non-finite pivot of the block
            const double p = dm[17 * rr];
            const unsigned long long m =
                __ballot(!(p != 0.0 && fabs(p) <= DBL_MAX) && 16 * b + rr < L) & 0xffffull;
            if (bad == 0 && m) bad = 16 * b + __builtin_ctzll(m) + 1;
        }
        __syncthreads();
        // ---- update ----
        if (w == b) {
            static_for<N>([&](auto c) {
                if (c == b) {
                    acc[c] = D;
                    branch_end<c>();
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[c][v] = pr[rr * S::kPrLd + 16 * c + 4 * v + g];
                    branch_end<c>();
                }
            });
        } else {
            double fa[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) fa[q] = -F[(4 * q + g) * S::kFLd + 16 * w + rr];
            static_for<N>([&](auto c) {
                if (c == b) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[c][v] = pc[(4 * v + g) * S::kFLd + 16 * w + rr];
                    branch_end<c>();
                }
            });
            auto update = [&](auto c) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(R[(4 * q + g) * S::kRLd + 16 * c + rr], fa[q],
                                                                  acc[c], 0, 0, 0);
            };
            const bool next = w == b + 1 && w < nblk;
            if (next) {
                // the next diagonal block first, and its chain
                __builtin_amdgcn_s_setprio(3);
                static_for<N>([&](auto c) {
                    if (c == w) {
                        update(c);
                        D = acc[c];
                        branch_end<c>();
                    }
                });
                lu_chain<false>(D, lane, dm, dr, iv, dump, kSteps);
                __builtin_amdgcn_s_setprio(0);
            }
            static_for<N>([&](auto c) {
                // rows above the diagonal block only right of it
                if (c != b && c < nblk && (w > b || c > b) && !(next && c == w)) {
                    update(c);
                    branch_end<c>();
                }
            });
        }
        if (b + 1 < nblk) publish(b + 1, (b + 1) & 1);
    }
    const int ln = opaque(lane0), sr = 16 * w + (ln & 15), sg = ln >> 4;
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int col = 16 * c + 4 * v + sg;
            if (sr < L && col < L) {
                const double f = acc[c][v];
                Li[sr + (int64_t)col * ldl] = sr > col ? f : (sr == col ? 1.0 : 0.0);
                Ui[sr + (int64_t)col * ldu] = sr <= col ? f : 0.0;
            }
        }
    if (t == 0 && bad) atomicMin(status, col0 + bad);
}

}  // namespace

hipError_t lu_leaf_launch(const double *A, int64_t lda, double *Li, int64_t ldl, double *Ui,
                          int64_t ldu, int64_t L, int64_t col0, int *status, hipStream_t s) {
    if (L < 1 || L > kLuLeafMax) return hipErrorInvalidValue;
    // four waves hold an order-64 block; eight would idle on it
    if (L <= 64)
        hipLaunchKernelGGL(k_lu_leaf_inv<4>, dim3(1), dim3(256), 0, s, A, lda, Li, ldl, Ui, ldu, (int)L,
                           (int)col0, status);
    else
        hipLaunchKernelGGL(k_lu_leaf_inv<8>, dim3(1), dim3(512), 0, s, A, lda, Li, ldl, Ui, ldu, (int)L,
                           (int)col0, status);
    return hipGetLastError();
}

}  // namespace spin
