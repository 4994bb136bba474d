// Leaf inversion: Gauss-Jordan elimination with partial pivoting in FP64.
//
// The paper leaves the method of the leaf inversion open and runs it on a
// single node (Alg. 1, Alg. 2 `locInverse`, Sec. 3.3); here it is Gauss-Jordan with
// partial pivoting, always in FP64 (also when the surrounding products run in
// FP32).
//
// Every tier uses implicit pivoting: rows are never moved.  Step k picks the
// unused row p with the largest |z[p][k]| (ties to the smallest row index),
// scales row p by 1/pivot and eliminates column k from every other row.  The
// storage is in place: after step k the slot of column k holds column p of
// the accumulated row transformation (it replaces the unit column that an
// augmented [A | I] would carry).  With r[k] = pivot row of step k and
// rinv[r[k]] = k, the inverse is  X[rinv[i]][r[c]] = Z[i][c].
//
// Tier 1 (L <= 128): one workgroup holds the whole block in registers.  With
//   known pivots it runs in 16-step blocks (gj_ahead); a search has it
//   cyclically distributed (thread (tr, tc) of a TR x 16 grid owns rows
//   tr + TR*a and columns tc + 16b).  A step then costs two barriers: the owners of
//   column k publish it to LDS, every wave finds the pivot redundantly (DPP
//   max, then ballots for the smallest row index), the owners of the pivot
//   row publish the scaled row, and every thread applies the rank-1 update.
// Tier 2 (L > 128): blocked Gauss-Jordan over column panels of width NB on a
//   working copy Z.  One workgroup eliminates a panel (all L rows x NB
//   columns in registers) and emits the panel's transformation U' = U - E
//   (E = unit entries at the pivot rows) and the pivot rows Q of the other
//   columns; those columns are then updated by one grouped matrix-core
//   product  Z[:, out] += U' * Q.  A final pass writes the permuted result.
//   Up to order 512 the panel's kernel runs 16-step blocks too (gj_blocked;
//   full panels of leaves of order 129 .. 256: two workgroups, leaf_duo) with
//   the same search, and an FP64 leaf is not copied first: the first panel and its product read the
//   leaf's input in place.  Above 512 a rotating-slot panel kernel works on narrower panels
//   and the input is copied into Z.
//
// Speculation: every kernel up to order 512 first tries the diagonal pivots
// (in 16-step blocks on the matrix cores, except leaf_duo), checks each choice
// exactly and falls back to its search when a check fails (gj2d_any, gj_ahead,
// gj_blocked); the result is the search's bit for bit either way.  In the blocked
// kernels a pivot outside 2^-500 .. 2^501 behind a diagonal within 2^-400 ..
// 2^401 fails its check too.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <climits>
#include <cstdlib>

#include "leaf_blocks.hpp"
#include "spin_kernels.hpp"

namespace spin {
namespace {

__device__ inline bool better(double ov, int oi, double v, int i) {
    return ov > v || (ov == v && oi < i);
}

// ---------------------------------------------------------- wave helpers ---
// Maximum over the 64 lanes of a wave (every lane receives it).  Keys are
// finite (no NaN), so max is exact and order independent.
__device__ inline double wave_max(double x) {
    x = fmax(x, dpp_f64<kDppQuadXor1>(x));
    x = fmax(x, dpp_f64<kDppQuadXor2>(x));
    x = fmax(x, dpp_f64<kDppHalfMirror>(x));
    x = fmax(x, dpp_f64<kDppMirror>(x));
    const double a = fmax(readlane_f64(x, 0), readlane_f64(x, 16));
    const double b = fmax(readlane_f64(x, 32), readlane_f64(x, 48));
    return fmax(a, b);
}

// ------------------------------------------------------------ 2-D kernel ---
// One workgroup of 16*TR threads eliminates a block of L <= TR*RR rows and
// nb <= 16*RC columns held in registers: thread (tr, tc) owns rows tr + TR*r
// and columns tc + 16*q.  A step:
//   1. the owners of column c publish it to LDS (its register slot restarts
//      as the implicit unit column);
//   2. every wave finds the pivot redundantly: key |v| of each unused row
//      (-0.5 for non-finite values, -1 for used rows), a DPP max over the
//      wave, and the smallest row index holding the maximum via ballots;
//   3. the owners of the pivot row publish it scaled by 1/pivot;
//   4. every thread applies the rank-1 update to its registers.
// WHOLE = true : the block is a whole leaf (columns = rows), read from `in`
//                and written to `out` with the pivot permutation applied.
// WHOLE = false: the block is one column panel of a blocked elimination
//                whose working copy is Z (the first panel of an FP64 leaf
//                reads the leaf's input instead); the kernel writes the panel
//                to Z, its transformation U' = U - E, the used-row flags and
//                the gathered pivot rows Q of the other columns.
struct LeafArgs {
    const void *in;
    int64_t ldi;
    void *out;
    int64_t ldo;
    int L, col0;
    int *status;
    // panel mode
    double *Z;
    int64_t ldz;
    int k0, nb;
    int *used, *rsel;
    double *Up, *Q;
    // Speculation switch of the inversion (nullable): nonzero lets the kernel
    // try the speculative elimination first; a failed attempt sets it to 0 so
    // that the later leaves of the same inversion go straight to the search.
    int *spec;
    // Whole leaves: the leaf is the inversion's only launch and resets the
    // status block itself, with speculation on (1) or off (2).
    int reset;
    // Two-workgroup panels: this panel's exchange area (multipliers and
    // inverse pivots of its 64 steps), its verdict and decision words, and
    // the number of polls after which a wait for the other workgroup gives
    // up (and the panel falls back to the search).
    double *xg;
    int *xc;
    int duo_spin;
};

// LDS of gj2d_run, in doubles (shared with the blocked tier, which runs first).
template <int TR, int RR, int RC>
struct RunLds {
    static constexpr int kL = TR * RR, kB = 16 * RC;
    static constexpr int oF = 2 * kL, oRow = oF + 2 * kL, oInt = oRow + 2 * kB;
    static constexpr int kDoubles = oInt + (kL + kB + 1) / 2;
};

template <int TR, int RR, int RC, bool WHOLE, typename TI, typename TO>
__device__ __attribute__((always_inline)) inline void gj2d_run(const LeafArgs &a, double *sm) {
    constexpr int NT = 16 * TR;
    constexpr int LMAX = TR * RR;
    constexpr int NBMAX = 16 * RC;
    constexpr int CPL = LMAX / 64;
    static_assert(CPL * 64 == LMAX, "rows must cover whole waves");
    using S = RunLds<TR, RR, RC>;
    double(*const colbuf)[LMAX] = reinterpret_cast<double(*)[LMAX]>(sm);
    // Panels: the multipliers, i.e. column c with 0 at the pivot row (the
    // pivot row is scaled in place instead), so the update needs no select.
    double(*const fbuf)[LMAX] = reinterpret_cast<double(*)[LMAX]>(sm + S::oF);
    double(*const rowbuf)[NBMAX] = reinterpret_cast<double(*)[NBMAX]>(sm + S::oRow);
    int *const pivstep = reinterpret_cast<int *>(sm + S::oInt);  // step at which a row was the pivot, or -1
    int *const prow_s = pivstep + LMAX;                          // pivot row of each step
    // Thread t holds rows tr + TR r of columns tc + 16 q.  Whole leaves put
    // the 16 threads of a row group in one wave (t = 16 tr + tc), so one wave
    // publishes the pivot row.  Panels put TR consecutive rows of one column
    // in consecutive lanes (t = TR tc + tr): their loads of the panel and
    // stores of Z and Up then cover whole column segments, which outweighs
    // spreading the pivot-row publication over all waves.
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int tr = WHOLE ? t >> 4 : t % TR, tc = WHOLE ? t & 15 : t / TR;
    const int L = a.L;
    const int k0 = WHOLE ? 0 : a.k0;
    const int nb = WHOLE ? a.L : a.nb;

    for (int i = t; i < LMAX; i += NT) pivstep[i] = -1;
    // Panel mode reads the panel and the pivot rows from `in` when it is set
    // (the first panel of an FP64 leaf, straight from the leaf's input) and
    // from Z otherwise; it always writes Z.
    const double *src = WHOLE ? nullptr : (a.in ? static_cast<const double *>(a.in) : a.Z);
    const int64_t lds = WHOLE ? 0 : (a.in ? a.ldi : a.ldz);
    double z[RR][RC];
#pragma unroll
    for (int r = 0; r < RR; ++r)
#pragma unroll
        for (int q = 0; q < RC; ++q) {
            const int row = tr + TR * r, col = tc + 16 * q;
            double v = 0.0;
            if (row < L && col < nb) {
                if (WHOLE)
                    v = (double)static_cast<const TI *>(a.in)[row + (int64_t)col * a.ldi];
                else
                    v = src[row + (int64_t)(k0 + col) * lds];
            }
            z[r][q] = v;
        }
    // Bit j: row lane + 64 j is used (or beyond L).  A per-lane integer keeps
    // the flags in a vector register; as bool arrays they become wave-wide
    // lane masks whose per-step merges cost scalar instructions, and the
    // scalar unit is shared by the CU's SIMDs.
    int usdm = 0;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
        const int row = lane + 64 * j;
        if (row >= L || (!WHOLE && k0 > 0 && a.used[row] != 0)) usdm |= 1 << j;
    }
    int bad = 0;
    // Panels gather the pivot rows of the columns outside the panel during
    // the steps: thread t < L - nb owns outside column gj, loads its entry in
    // row p at step c and stores it to Q one step later, when the load has
    // long completed.  The panel kernel never writes those columns, so the
    // values are the ones a gather after the last step would read.
    static_assert(WHOLE || LMAX <= NT, "one gathering thread per outside column");
    const bool gth = !WHOLE && nb < L && t < L - nb;
    const int gj = t < k0 ? t : t + nb;
    const double *gsrc = WHOLE ? nullptr : src + (int64_t)gj * lds;
    double *gdst = WHOLE ? nullptr : a.Q + (int64_t)gj * nb;
    double gv = 0.0;
    // All initial loads complete here (vmcnt(0), the other counters left at
    // their maximum).  Otherwise the first uses of z inside the loop carry a
    // wait for every outstanding load, which would include the gathered one.
    if constexpr (!WHOLE) __builtin_amdgcn_s_waitcnt(0xF70);
    __syncthreads();

#pragma unroll
    for (int cb = 0; cb < RC; ++cb) {
        for (int cc = 0; cc < 16; ++cc) {
            const int c = cb * 16 + cc;
            if (c >= nb) break;
            const int buf = c & 1;
            if (tc == cc) {
#pragma unroll
                for (int r = 0; r < RR; ++r) {
                    colbuf[buf][tr + TR * r] = z[r][cb];
                    if (!WHOLE) fbuf[buf][tr + TR * r] = z[r][cb];
                    z[r][cb] = 0.0;
                }
            }
            __syncthreads();
            double key[CPL];
            // Panels keep the non-finite flag as a bool, test it in thread 0's
            // wave only and take p mod TR unsigned; whole leaves measured
            // 1.8 % slower with those forms, so they keep the int forms.
            int nf = 0;
#pragma unroll
            for (int j = 0; j < CPL; ++j) {
                const double av = fabs(colbuf[buf][lane + 64 * j]);
                const bool fin = av <= DBL_MAX;
                const bool u = (usdm >> j) & 1;
                if (WHOLE)
                    nf |= (!u && !fin);
                else
                    nf = nf || (!u && !fin);
                key[j] = u ? -1.0 : (fin ? av : -0.5);
            }
            double lm = key[0];
#pragma unroll
            for (int j = 1; j < CPL; ++j) lm = fmax(lm, key[j]);
            const double best = wave_max(lm);
            int p = 0;
#pragma unroll
            for (int j = CPL - 1; j >= 0; --j) {
                const unsigned long long m = __ballot(key[j] == best);
                if (m) p = 64 * j + __builtin_ctzll(m);
            }
            p = __builtin_amdgcn_readfirstlane(p);
            if (WHOLE) {
                if ((__any(nf) || !(best > 0.0)) && bad == 0) bad = c + 1;
            } else if (wave == 0 && bad == 0 && (__any(nf) || !(best > 0.0))) {
                bad = c + 1;  // only thread 0 reports the failing step
            }
            usdm |= (p & 63) == lane ? 1 << (p >> 6) : 0;
            const double pinv = 1.0 / colbuf[buf][p];
            if (tr == (WHOLE ? p % TR : (int)((unsigned)p % TR))) {
                const int rp = WHOLE ? p / TR : (int)((unsigned)p / TR);
#pragma unroll
                for (int r = 0; r < RR; ++r) {
                    if (r == rp) {
                        if (WHOLE) {
#pragma unroll
                            for (int q = 0; q < RC; ++q) {
                                rowbuf[buf][tc + 16 * q] = z[r][q] * pinv;
                                z[r][q] = 0.0;
                            }
                            if (tc == cc) rowbuf[buf][c] = pinv;
                        } else {
                            // scaled in place; its multiplier becomes 0
#pragma unroll
                            for (int q = 0; q < RC; ++q) {
                                z[r][q] = z[r][q] * pinv;
                                rowbuf[buf][tc + 16 * q] = z[r][q];
                            }
                            if (tc == cc) {
                                rowbuf[buf][c] = pinv;
                                z[r][cb] = pinv;
                                fbuf[buf][p] = 0.0;
                            }
                        }
                    }
                }
            }
            if (t == 0) {
                pivstep[p] = c;
                prow_s[c] = p;
            }
            __syncthreads();
            if (gth) {
                if (c > 0) gdst[c - 1] = gv;
                gv = gsrc[p];
            }
            double f[RR], rv[RC];
#pragma unroll
            for (int r = 0; r < RR; ++r)
                f[r] = WHOLE ? ((tr + TR * r == p) ? -1.0 : colbuf[buf][tr + TR * r]) : fbuf[buf][tr + TR * r];
#pragma unroll
            for (int q = 0; q < RC; ++q) rv[q] = rowbuf[buf][tc + 16 * q];
#pragma unroll
            for (int r = 0; r < RR; ++r)
#pragma unroll
                for (int q = 0; q < RC; ++q) z[r][q] = fma(-f[r], rv[q], z[r][q]);
        }
    }
    __syncthreads();
    if (WHOLE) {
        // X[rinv[i]][r[c]] = Z[i][c]  with r[c] = prow_s[c], rinv[i] = pivstep[i]
        TO *out = static_cast<TO *>(a.out);
#pragma unroll
        for (int r = 0; r < RR; ++r)
#pragma unroll
            for (int q = 0; q < RC; ++q) {
                const int row = tr + TR * r, col = tc + 16 * q;
                if (row < L && col < L) {
                    const int ri = pivstep[row], rc = prow_s[col];
                    if ((unsigned)ri < (unsigned)L && (unsigned)rc < (unsigned)L)
                        out[ri + (int64_t)rc * a.ldo] = (TO)z[r][q];
                }
            }
    } else {
#pragma unroll
        for (int r = 0; r < RR; ++r)
#pragma unroll
            for (int q = 0; q < RC; ++q) {
                const int row = tr + TR * r, col = tc + 16 * q;
                if (row < L && col < nb) {
                    a.Z[row + (int64_t)(k0 + col) * a.ldz] = z[r][q];
                    a.Up[row + (int64_t)col * L] = z[r][q] - ((pivstep[row] == col) ? 1.0 : 0.0);
                }
            }
        for (int c = t; c < nb; c += NT) a.rsel[k0 + c] = prow_s[c];
        for (int row = t; row < L; row += NT) {
            if (k0 == 0)
                a.used[row] = pivstep[row] >= 0 ? 1 : 0;
            else if (pivstep[row] >= 0)
                a.used[row] = 1;
        }
        if (gth) gdst[nb - 1] = gv;
    }
    if (t == 0 && bad) atomicMin(a.status, a.col0 + k0 + bad);
}

// --------------------------------------------- blocked speculative tier ---
// The elimination of gj2d_run for blocks whose partial-pivoting choice at
// step k is row k itself, as it is at every step for strictly diagonally
// dominant blocks (their Schur complements stay dominant) and, in practice,
// for well-conditioned positive-definite ones.  Each step takes that row as
// its pivot and checks the choice exactly: the step stands when the pivot is
// finite and nonzero and no unused row holds a larger magnitude or a
// non-finite value.  As long as every earlier step stood, the unused rows are
// exactly the rows below the pivot, so a tie goes to the pivot row, which is
// what the search's smallest-index rule picks.  The outputs are written only
// when every check passed.
//
// With the pivot rows known in advance, 16 steps form one block step on the
// matrix cores.  v_mfma_f64_16x16x4f64 adds its four products to each element
// as a chain of fused multiply-adds in ascending k (checked against fma() on
// random and subnormal operands), so four of them apply 16 steps to a 16 x 16
// block with the very operations, in the very order, of gj2d_run's sixteen
// rank-1 updates, and the result is the search's bit for bit.  Block step b
// on the 16 columns / rows Kb:
//   diagonal  one wave runs the 16 steps on the 16 x 16 diagonal block, the
//             only serial chain: a reciprocal, a product and a fused
//             multiply-add per step, the pivot row and column passed between
//             lanes by DPP and lane swaps;
//   panels    one lane per row takes the 16 steps through the columns Kb
//             (its multipliers F; they are checked here), one lane per column
//             takes them through the rows Kb (the scaled pivot rows R);
//   update    every other 16 x 16 block takes four MFMAs with -F and R.
// The block lives in the accumulators of NW waves (wave w holds the row
// blocks w + NW i) and only panels pass through LDS.  While the update runs,
// the wave that holds the next diagonal block updates that one first and goes
// straight into its chain.
//
// What bounds it: FP64 vector and matrix instructions share one unit per
// SIMD, and the panels (16 x 24 instructions of a lone wave, about 3 100
// cycles), the chain (16 x 37 dependent instructions, 5 000 cycles) and the
// MFMAs follow each other there.  Placing the chain wave's own MFMAs between
// its steps gained nothing for the same reason.  Whole inversions of one leaf
// (launches included), against the earlier kernels with a barrier or a flag
// per step: order 257 325 -> 247 us, 512 758 -> 547 us; full panels of orders
// 129 .. 256 stay with leaf_duo, whose two CUs take 29 us against 34 us here
// (22 us of steps, the rest loads and stores of one CU); whole leaves have
// gj_ahead.

// Pivots whose reciprocal the chain forms without the scaling and fix-up of
// the FP64 division: for these the division leaves divisor and quotient
// unscaled, so the bits are the same.  A block whose diagonal says that it has
// others (far_entry) divides in the chain; where such a pivot comes up without
// that the block's check fails.
__device__ inline unsigned exponent_bits(double x) { return (unsigned)(__double_as_longlong(x) >> 52) & 0x7ffu; }
__device__ inline bool plain_pivot(double x) {
    return exponent_bits(x) - 523u <= 1000u;  // |x| in 2^-500 .. 2^501
}
__device__ inline bool usable_pivot(double x) { return x != 0.0 && fabs(x) <= DBL_MAX; }
__device__ inline bool pivot_fails(double x, bool div) { return !(div ? usable_pivot(x) : plain_pivot(x)); }
// A diagonal entry from which the pivot is not expected within plain_pivot's
// range, since a matrix that needs no row exchanges keeps its pivots near its
// diagonal.
__device__ inline bool far_entry(double x) { return usable_pivot(x) && exponent_bits(x) - 623u > 800u; }

// Step K of the 16 x 16 diagonal block: lane l holds row l % 16 of columns
// 4 v + l / 16.
//   - the active column (group K % 4 of D[K / 4]) passes through LDS, where
//     its values, the step's multipliers with the pivot at row K, are kept
//     for the panels; it restarts as the unit column;
//   - 1 / pivot: reciprocal estimate, two Newton steps and the division's
//     final correction, in every lane (lane (K % 4, K) holds the pivot);
//   - the pivot row (lane K of each group) is scaled in place, published, and
//     reaches the other rows by DPP inside the multiply-add; its own
//     multiplier is 0.
// A lone wave issues an instruction about every five to nine cycles, so the
// step has no branch: lanes whose store is not wanted store to a dump area.
// The step's stores go to dm + 16 K + (row) and dr + 16 K + (column).
template <bool DIV, int K>
__device__ __attribute__((always_inline)) inline void diag_step(d4_t &D, int rr, int g, double *dm, double *dr,
                                                                double *dump) {
    constexpr int V = K / 4, G = K % 4;
    const double x = D[V];
    double *const pm = (g == G ? dm : dump) + rr;
    pm[16 * K] = x;
    // the other groups read what this group wrote: LDS serves a wave's accesses
    // in order, the fences keep the compiler's order too
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double f = dm[16 * K + rr];
    __builtin_amdgcn_sched_barrier(0);  // the read goes out before the arithmetic
    double y;
    if constexpr (DIV) {
        y = 1.0 / x;
    } else {
        y = __builtin_amdgcn_rcp(x);
        y = fma(y, fma(-x, y, 1.0), y);
        y = fma(y, fma(-x, y, 1.0), y);
        y = fma(fma(-x, y, 1.0), y, y);
    }
    const double pinv = readlane_f64(y, 16 * G + K);
    const bool prow = rr == K;
    const double unit = prow ? 1.0 : 0.0;
    D[V] = g == G ? unit : x;
    const double sc = prow ? pinv : 1.0;
    double *const pr = (prow ? dr : dump) + g;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        D[v] *= sc;
        pr[16 * K + 4 * v] = D[v];
    }
    f = prow ? 0.0 : f;
    // D[v] = fma(-f, D[v] of lane K, D[v])
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %0, -%4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %1, -%4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %2, -%4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %3, -%4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
        : "+v"(D[0]), "+v"(D[1]), "+v"(D[2]), "+v"(D[3])
        : "v"(f), "n"(K));
}

template <bool DIV, int... K>
__device__ __attribute__((always_inline)) inline void diag_steps(d4_t &D, int lane, double *dm, double *dr,
                                                                 double *dump, std::integer_sequence<int, K...>) {
    lane = opaque(lane);
    (diag_step<DIV, K>(D, lane & 15, lane >> 4, dm, dr, dump), ...);
    branch_end<DIV>();
}
__device__ __attribute__((always_inline)) inline void diag_chain(bool div, d4_t &D, int lane, double *dm, double *dr,
                                                                 double *dump) {
    constexpr auto kSteps = std::make_integer_sequence<int, 16>{};
    if (div)
        diag_steps<true>(D, lane, dm, dr, dump, kSteps);
    else
        diag_steps<false>(D, lane, dm, dr, dump, kSteps);
}

// The 16 steps on one row of the block column (x: its 16 columns): F gets the
// multipliers (pitch ld).  Returns whether a checked row holds a candidate
// larger than a pivot or not finite.
template <int... K>
__device__ __attribute__((always_inline)) inline bool row_steps(double (&x)[16], const double *dr16, double pd,
                                                                double *F, int ld, std::integer_sequence<int, K...>) {
    bool bad = false;
    double r[16] = {dr16[16 * K]...};  // loaded before the stores to F, which the compiler keeps in order
    (
        [&] {
            const double f = x[K];
            F[K * ld] = f;
            bad = bad | !(fabs(f) <= fabs(row_bcast<K>(pd)));
            x[K] = 0.0;
            fmac_rows(x, r[K], f);
        }(),
        ...);
    return bad;
}

// The 16 steps on one column of the block row (y: its 16 rows): R gets the
// scaled pivot rows' entries (pitch ld).  Returns whether one is not finite,
// which every later one then is not either.
template <int... K>
__device__ __attribute__((always_inline)) inline bool col_steps(double (&y)[16], const double *dm16, double id,
                                                                double *R, int ld, std::integer_sequence<int, K...>) {
    double m[16] = {dm16[16 * K]...};
    (
        [&] {
            const double r = y[K] * row_bcast<K>(id);
            R[K * ld] = r;
            fmac_rows(y, m[K], r);
            y[K] = r + 0.0;
        }(),
        ...);
    return !(fabs(y[15]) <= DBL_MAX);
}

template <int NW, int RB, int NC>
__device__ __attribute__((always_inline)) inline bool gj_blocked(const LeafArgs &a, double *sm) {
    using S = BlkLds<NW, RB, NC>;
    constexpr int NT = 64 * NW;
    const int t = threadIdx.x, lane0 = t & 63, lane = lane0, rr = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int L = a.L, k0 = a.k0, nb = a.nb;
    if ((k0 & 15) != 0 || nb < 1 || nb > S::kCols || L > S::kRows) return false;  // the same in every thread
    const double *src = a.in ? static_cast<const double *>(a.in) : a.Z;
    const int64_t lds = a.in ? a.ldi : a.ldz;

    // lane l holds row 16 (w + NW i) + l % 16 of columns 16 c + 4 v + l / 16
    d4_t acc[RB][NC];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * (w + NW * i) + rr, col = 16 * c + 4 * v + g;
                // beyond the last step the block continues as the identity: its
                // steps leave every other value as it is
                double x = (col >= nb && row == k0 + col) ? 1.0 : 0.0;
                if (row < L && col < nb) x = src[row + (int64_t)(k0 + col) * lds];
                acc[i][c][v] = x;
            }
    // Panels of up to 256 rows load the pivot rows of the outside columns (Q)
    // here, so that the loads complete during the elimination.
    constexpr bool QPRE = RB <= 2;
    constexpr int QPT = QPRE ? (S::kRows - 64) / NW : 1;
    const int nout = L - nb;
    double qv[QPT];
    if constexpr (QPRE) {
#pragma unroll
        for (int q = 0; q < QPT; ++q) {
            const int j = w + NW * q, gj = j < k0 ? j : j + nb;
            qv[q] = (lane < nb && j < nout) ? src[(k0 + lane) + (int64_t)gj * lds] : 0.0;
        }
    }
    // the same in every wave (up to 64 columns)
    static_assert(S::kCols <= 64, "one diagonal entry per lane");
    const bool div = __any(far_entry(lane < nb ? src[(k0 + lane) * (lds + 1)] : 1.0)) != 0;
    bool viol = false;
    if (k0 > 0) {
        // the rows before the panel must be the used ones and no other
        for (int row = t; row < L; row += NT)
            if ((a.used[row] != 0) != (row < k0)) viol = true;
    }

    const int nblk = (nb + 15) >> 4, p0 = k0 >> 4;
    double *const F = sm + S::oF, *const R = sm + S::oR;
    double *const dr = sm + S::oDr, *const dm = sm + S::oDm, *const dump = sm + S::oDump;
    constexpr auto kSteps = std::make_integer_sequence<int, 16>{};
    d4_t D{0.0, 0.0, 0.0, 0.0};  // the diagonal block in the wave that runs its chain
    // block column b of every row block and row block p0 + b to panel buffer u
    auto publish = [&](const int b, const int u) {
        const int ln = opaque(lane0), rr = ln & 15, g = ln >> 4;
        double *pc = sm + S::oPc + u * 16 * S::kFLd, *pr = sm + S::oPr + u * 16 * S::kPrLd;
        const int ow = (p0 + b) % NW, oi = (p0 + b) / NW;
        static_for<NC>([&](auto c) {
            if (c == b) {
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v) pc[(4 * v + g) * S::kFLd + 16 * (w + NW * i) + rr] = acc[i][c][v];
                branch_end<c>();
            }
        });
        if (w == ow) {
            static_for<RB>([&](auto i) {
                if (i == oi) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int v = 0; v < 4; ++v) pr[rr * S::kPrLd + 16 * c + 4 * v + g] = acc[i][c][v];
                    branch_end<i>();
                }
            });
        }
    };

    publish(0, 0);
    if (w == p0 % NW) {
        static_for<RB>([&](auto i) {
            if (i == p0 / NW) {
                D = acc[i][0];
                branch_end<i>();
            }
        });
        diag_chain(div, D, lane, dm, dr, dump);
    }
#pragma unroll 1
    for (int b = 0; b < nblk; ++b) {
        const int u = S::kTwo ? b & 1 : 0;
        const int lane = opaque(lane0), rr = lane & 15, g = lane >> 4;
        double *const pc = sm + S::oPc + u * 16 * S::kFLd, *const pr = sm + S::oPr + u * 16 * S::kPrLd;
        __syncthreads();
        // ---- panels ----
        constexpr int RCH = (S::kRows + 63) / 64, CCH = (S::kCols + 63) / 64;
#pragma unroll 1
        for (int tk = w; tk < RCH + CCH; tk += NW) {
            double x[16];
            if (tk < RCH) {
                const int row = 64 * tk + lane;
                const bool chk = row >= k0 + 16 * (b + 1) && row < L;
#pragma unroll
                for (int j = 0; j < 16; ++j) x[j] = pc[j * S::kFLd + row];
                const bool bad = row_steps(x, dr + rr, dm[17 * rr], F + row, S::kFLd, kSteps);
                viol = viol | (chk & bad);
#pragma unroll
                for (int j = 0; j < 16; ++j) pc[j * S::kFLd + row] = x[j];
            } else {
                const int col = 64 * (tk - RCH) + lane;
#pragma unroll
                for (int j = 0; j < 16; ++j) x[j] = pr[j * S::kPrLd + col];
                viol = viol | col_steps(x, dm + rr, dr[17 * rr], R + col, S::kRLd, kSteps);
#pragma unroll
                for (int j = 0; j < 16; ++j) pr[j * S::kPrLd + col] = x[j];
            }
        }
        if (w == NW - 1) {
            // the checks inside the diagonal block
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = lane + 64 * q, k = e >> 4, l = e & 15;
                const double piv = dm[17 * k];
                viol = viol | pivot_fails(piv, div) | ((l > k) & !(fabs(dm[e]) <= fabs(piv))) |
                       !(fabs(dr[e]) <= DBL_MAX);
            }
        }
        __syncthreads();
        // ---- update ----
        const int p = p0 + b, ow = p % NW, oi = p / NW;  // the pivot rows' owner
        // the new values of the block column and, in their owner, of the pivot rows
        static_for<NC>([&](auto c) {
            if (c == b) {
                static_for<RB>([&](auto i) {
                    if (!(w == ow && i == oi)) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[i][c][v] = pc[(4 * v + g) * S::kFLd + 16 * (w + NW * i) + rr];
                        branch_end<NC * i + c>();
                    }
                });
            }
        });
        if (w == ow) {
            static_for<RB>([&](auto i) {
                if (i == oi) {
                    static_for<NC>([&](auto c) {
                        if (c == b) {
                            acc[i][c] = D;
                            branch_end<NC * i + c>();
                        } else {
#pragma unroll
                            for (int v = 0; v < 4; ++v) acc[i][c][v] = pr[rr * S::kPrLd + 16 * c + 4 * v + g];
                            branch_end<NC * i + c>();
                        }
                    });
                }
            });
        }
        if constexpr (!S::kTwo) __syncthreads();
        double fa[RB][4];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) fa[i][q] = -F[(4 * q + g) * S::kFLd + 16 * (w + NW * i) + rr];
        const bool more = b + 1 < nblk;
        const int nw = (p + 1) % NW, ni = (p + 1) / NW;
        if (more && w == nw) {
            __builtin_amdgcn_s_setprio(3);
            // the next diagonal block first, and its chain
            static_for<NC>([&](auto c) {
                if (c == b + 1) {
                    static_for<RB>([&](auto i) {
                        if (i == ni) {
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                    R[(4 * q + g) * S::kRLd + 16 * c + rr], fa[i][q], acc[i][c], 0, 0, 0);
                            D = acc[i][c];
                            branch_end<NC * i + c>();
                        }
                    });
                }
            });
            diag_chain(div, D, lane, dm, dr, dump);
            __builtin_amdgcn_s_setprio(0);
        }
        static_for<NC>([&](auto c) {
            if (c != b && c < nblk) {
                double fb[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) fb[q] = R[(4 * q + g) * S::kRLd + 16 * c + rr];
                static_for<RB>([&](auto i) {
                    if (!(w == ow && i == oi) && !(more && c == b + 1 && w == nw && i == ni)) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            acc[i][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[q], fa[i][q], acc[i][c], 0, 0, 0);
                        branch_end<NC * i + c>();
                    }
                });
            }
        });
        if (more) publish(b + 1, S::kTwo ? (b + 1) & 1 : 0);
    }
    if (__syncthreads_or(viol)) return false;

    const int ln = opaque(lane0), sr = ln & 15, sg = ln >> 4;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * (w + NW * i) + sr, col = 16 * c + 4 * v + sg;
                if (row < L && col < nb) {
                    const double x = acc[i][c][v];
                    a.Z[row + (int64_t)(k0 + col) * a.ldz] = x;
                    a.Up[row + (int64_t)col * L] = x - ((row == k0 + col) ? 1.0 : 0.0);
                }
            }
    for (int c = t; c < nb; c += NT) a.rsel[k0 + c] = k0 + c;
    for (int row = t; row < L; row += NT) {
        const bool piv = row >= k0 && row < k0 + nb;
        if (k0 == 0)
            a.used[row] = piv ? 1 : 0;
        else if (piv)
            a.used[row] = 1;
    }
    if constexpr (QPRE) {
#pragma unroll
        for (int q = 0; q < QPT; ++q) {
            const int j = w + NW * q, gj = j < k0 ? j : j + nb;
            if (lane < nb && j < nout) a.Q[lane + (int64_t)gj * nb] = qv[q];
        }
    } else {
#pragma unroll 8
        for (int j = w; j < nout; j += NW) {
            const int gj = j < k0 ? j : j + nb;
            if (lane < nb) a.Q[lane + (int64_t)gj * nb] = src[(k0 + lane) + (int64_t)gj * lds];
        }
    }
    return true;
}

// ------------------------------------------ blocked tier, chain ahead ---
// gj_blocked for whole leaves, with a role for each wave and the serial chain
// one block step ahead.  Block step b, between the same barriers:
//   panels  one lane per row and one per column take the steps through the
//           panels, but only as far as the multipliers F and the scaled pivot
//           rows R need, which is half the updates; the chain wave does the
//           same for the 16 rows and columns of the next diagonal block;
//   update  four MFMAs for every 16 x 16 block; meanwhile the chain wave
//           applies the block step to the next diagonal block and runs its
//           chain.
// The other half of the panels' updates is left to the matrix cores: a value
// of the block column restarts at 0 in its own step, one of the pivot rows at
// its scaled value, so the later steps are an MFMA chain from there, with 0
// for the steps before (they add a zero to a value that is not -0).  The
// operations on each element and their order stay gj_blocked's, and so the
// search's; a multiplier or scaled entry that is not finite, whose product with
// those zeros would be NaN, goes to the search.
//
// What bounds it (cycles per block step): order 128 fills the FP64 units, the
// panels 2 700 and then 80 MFMAs of 64 cycles on a SIMD, 7 800 with the loads
// before and the publication after them, the chain (2 100 + 4 600) beside
// them; order 64 waits for the chain wave, 6 700.  Each role keeps a loop of
// its own because the compiler spills where one wave's registers are live
// through another's code.  Whole inversions of one leaf, launches included,
// against gj_blocked: order 33 16.2 -> 14.4 us, 64 20.1 -> 17.5, 80 30.0 ->
// 27.3, 100 42.7 -> 37.7, 128 50 -> 43.7.
template <int N>
struct AheadLds {
    // The pitches spread rows read along a lane group's 16 lanes (kLd, and kPrLd
    // for columns too) over the banks.
    static constexpr int kLd = N + 16, kPrLd = N + 18, kMLd = 17, kMini = 16 * kMLd;
    static constexpr int oPc = 0;                        // block column b [16][kLd]
    static constexpr int oF = oPc + 16 * kLd;            // F [16][kLd]
    static constexpr int oPr = oF + 16 * kLd;            // row block b [16][kPrLd]
    static constexpr int oR = oPr + 16 * kPrLd;          // R [16][kPrLd], and from column N block column b's multiplicand
    static constexpr int oStart = oR + 16 * kPrLd;       // where row block b's values start in the update [16][kPrLd]
    static constexpr int oDr = oStart + 16 * kPrLd;      // pivot rows inside a diagonal block [2][256]
    static constexpr int oDm = oDr + 512;                // its active columns [2][256]
    static constexpr int oMini = oDm + 512;              // the next diagonal block's part of the panels, then of F
                                                         // and R [2][2][kMini]
    static constexpr int oPub = oMini + 4 * kMini;       // diagonal block before its last update [2][256]
    static constexpr int oNew = oPub + 512;              // diagonal block after its chain [2][256]
    static constexpr int oDump = oNew + 512;             // unwanted stores of the chain
    static constexpr int kDoubles = oDump + 256;
};

// A wave's part.  Waves go to the four SIMDs in turn; wave 0 is the chain's,
// and its SIMD gets the least of the rest.
struct AheadRole {
    int row, c0;  // row block and first column block held
    int task;     // 64 rows (task < N / 64) or columns of the panels, or -1
};
constexpr int ahead_waves(int N) { return N == 64 ? 6 : 12; }
constexpr int ahead_checks(int N) { return N == 64 ? 4 : 8; }  // the wave of the diagonal block's checks
__device__ inline AheadRole ahead_role(int N, int w) {
    if (N == 64) return {w == 5 ? 3 : w - 1, 0, w == 2 || w == 3 ? w - 2 : -1};
    if (w < 4) return {w - 1, 0, -1};
    if (w >= 5 && w < 8) return {w - 2, 0, -1};
    const int h = w == 4 ? 3 : w - 9;  // the last two row blocks in halves
    return {6 + (h >> 1), 4 * (h & 1), h};
}

// Four of fmac_rows' updates, j = J .. J + 3.
template <int J>
__device__ inline void fmac_quad(double &x0, double &x1, double &x2, double &x3, double r, double f) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, -%5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %4, -%5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %2, %4, -%5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %3, %4, -%5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3)
        : "v"(r), "v"(f), "n"(J), "n"(J + 1), "n"(J + 2), "n"(J + 3));
}

// Step K's updates of the entries after K: x[j] -= r[lane j] * f.
template <int K>
__device__ __attribute__((always_inline)) inline void half_step(double (&x)[16], double r, double f) {
    double t[4] = {0.0, 0.0, 0.0, 0.0};  // for entries up to K
    static_for<4>([&](auto q) {
        constexpr int J = 4 * q;
        if constexpr (J > K)
            fmac_quad<J>(x[J], x[J + 1], x[J + 2], x[J + 3], r, f);
        else if constexpr (J + 3 > K)
            fmac_quad<J>(t[0], J + 1 > K ? x[J + 1] : t[1], J + 2 > K ? x[J + 2] : t[2], x[J + 3], r, f);
    });
}

// The multipliers of one row of the block column (x).  viol: a checked row
// (kind 1) holds a candidate larger than a pivot or not finite, or another
// (kind 0) a multiplier that is not finite, which every later value then is
// not either; the block's own rows (kind 2) are not used.
template <int... K>
__device__ __attribute__((always_inline)) inline bool row_half(double (&x)[16], const double *dr16, double pd, double *F,
                                                               int ld, int kind, std::integer_sequence<int, K...>) {
    bool over = false;
    double r[16] = {dr16[16 * K]...};
    (
        [&] {
            const double f = x[K];
            F[K * ld] = f;
            over = over | !(fabs(f) <= fabs(row_bcast<K>(pd)));
            half_step<K>(x, r[K], f);
        }(),
        ...);
    return kind == 1 ? over : kind == 0 && !(fabs(x[15]) <= DBL_MAX);
}

// The scaled pivot rows' entries of one column of the block row (y), and where
// the values of that column start in the update.
template <int... K>
__device__ __attribute__((always_inline)) inline bool col_half(double (&y)[16], const double *dm16, double id, double *R,
                                                               double *start, int ld,
                                                               std::integer_sequence<int, K...>) {
    double m[16] = {dm16[16 * K]...};
    (
        [&] {
            const double r = y[K] * row_bcast<K>(id);
            R[K * ld] = r;
            start[K * ld] = r + 0.0;
            half_step<K>(y, m[K], r);
            if constexpr (K == 15) y[15] = r;
        }(),
        ...);
    return !(fabs(y[15]) <= DBL_MAX);
}

// Both for the next diagonal block: lane groups 0, 2 its rows (id = 1), groups
// 1, 3 its columns.
template <int... K>
__device__ __attribute__((always_inline)) inline void mini_half(double (&x)[16], const double (&r)[16], double id,
                                                                std::integer_sequence<int, K...>) {
    (
        [&] {
            x[K] *= row_bcast<K>(id);
            half_step<K>(x, r[K], x[K]);
        }(),
        ...);
}

// A workgroup barrier for code that the waves reach on different paths.
__device__ inline void wg_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// One wave's part of the panels of block step b; returns whether a check fails.
template <int N>
__device__ __attribute__((always_inline)) inline bool ahead_panel(double *sm, int L, int b, int task, int lane0) {
    using S = AheadLds<N>;
    constexpr auto kSteps = std::make_integer_sequence<int, 16>{};
    const int lane = opaque(lane0), rr = lane & 15;
    const double *const dr = sm + S::oDr + 256 * (b & 1), *const dm = sm + S::oDm + 256 * (b & 1);
    double x[16];
    if (task < N / 64) {
        const int row = 64 * task + lane;
        const int kind = row >= 16 * b + 16 ? (row < L ? 1 : 0) : row >= 16 * b ? 2 : 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = sm[S::oPc + j * S::kLd + row];
        return row_half(x, dr + rr, dm[17 * rr], sm + S::oF + row, S::kLd, kind, kSteps);
    }
    const int col = 64 * (task - N / 64) + lane;
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = sm[S::oPr + j * S::kPrLd + col];
    return col_half(x, dm + rr, dr[17 * rr], sm + S::oR + col, sm + S::oStart + col, S::kPrLd,
                    kSteps);
}

// A wave that holds NW blocks of row block me.row, from column block me.c0 on.
template <int N, int NW, typename TI, typename TO>
__device__ __attribute__((always_inline)) inline bool ahead_rows(const LeafArgs &a, double *sm, AheadRole me,
                                                                 int lane0) {
    using S = AheadLds<N>;
    constexpr bool kTasks = NW == 4;
    const int L = a.L, nblk = (L + 15) >> 4;
    double *const F = sm + S::oF, *const R = sm + S::oR, *const pc = sm + S::oPc, *const pr = sm + S::oPr;
    double *const pub = sm + S::oPub, *const nw = sm + S::oNew;

    d4_t acc[NW];  // lane l holds row 16 me.row + l % 16 of columns 16 (me.c0 + i) + 4 v + l / 16
    {
        // beyond the last step the block continues as the identity; loads
        // outside it go to its other entries, so that none waits in a branch
        const int row = 16 * me.row + (lane0 & 15), c = 16 * me.c0 + (lane0 >> 4);
        const TI *p = static_cast<const TI *>(a.in) + (row < L ? row : 0) + (c < L ? (int64_t)c * a.ldi : 0);
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int col = c + 16 * i + 4 * v;
                const double x = (double)*p;
                acc[i][v] = row < L && col < L ? x : (col >= L && row == col) ? 1.0 : 0.0;
                p += col + 4 < L ? 4 * a.ldi : 0;
            }
    }
    // Block column b (held in x), and its part in the next diagonal block's rows.
    auto publish_col = [&](const d4_t &x, const int b, const int rr, const int g) {
#pragma unroll
        for (int v = 0; v < 4; ++v) pc[(4 * v + g) * S::kLd + 16 * me.row + rr] = x[v];
        if (me.row == b + 1) {
            double *const mini = sm + S::oMini + 2 * S::kMini * (b & 1);
#pragma unroll
            for (int v = 0; v < 4; ++v) mini[S::kMLd * (4 * v + g) + rr] = x[v];
        }
    };
    // Row block b, the next diagonal block and its columns' part.
    auto publish_row = [&](const int b) {
        const int ln = opaque(lane0), rr = ln & 15, g = ln >> 4;
        double *const mini = sm + S::oMini + 2 * S::kMini * (b & 1);
        const int ib = b - me.c0;
        if (me.row == b) {
            double *const p = pr + rr * S::kPrLd + 16 * me.c0 + g;
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) p[16 * i + 4 * v] = acc[i][v];
        }
        if (me.row == b || me.row == b + 1) {
            static_for<NW>([&](auto i) {
                if (i == ib + 1) {
                    double *const m = me.row == b ? mini + S::kMini + S::kMLd * rr + g : pub + 256 * (~b & 1) + ln;
                    const int ld = me.row == b ? 4 : 64;
#pragma unroll
                    for (int v = 0; v < 4; ++v) m[ld * v] = acc[i][v];
                    branch_end<i>();
                }
            });
        }
    };
    if (me.c0 == 0) publish_col(acc[0], 0, lane0 & 15, lane0 >> 4);
    publish_row(0);
    if (me.row == 0 && me.c0 == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) pub[64 * v + lane0] = acc[0][v];
    }
    bool viol = false;
    wg_barrier();
    wg_barrier();
#pragma unroll 1
    for (int b = 0; b < nblk; ++b) {
        wg_barrier();
        if (kTasks && me.task >= 0) {
            __builtin_amdgcn_s_setprio(3);
            viol = viol | ahead_panel<N>(sm, L, b, me.task, lane0);
            __builtin_amdgcn_s_setprio(0);
        }
        wg_barrier();
        const int lane = opaque(lane0), rr = lane & 15, g = lane >> 4;
        const int ib = b - me.c0, end = nblk - me.c0;
        const bool own = me.row == b;
        // block i's multiplicand
        const double *const rl = R + g * S::kPrLd + rr;
        auto load = [&](const int i, double (&f)[4]) {
            const double *const r = rl + (i == ib ? N : 16 * (me.c0 + i));
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = r[4 * q * S::kPrLd];
        };
        double fa[4], fb[2][4];
        load(0, fb[0]);
        if (own) {
            __builtin_amdgcn_s_setprio(2);  // it starts later than the others
            const double *const m = sm + S::oDm + 256 * (b & 1) + rr, *const r0 = sm + S::oStart + rr * S::kPrLd + 16 * me.c0 + g;
#pragma unroll
            for (int q = 0; q < 4; ++q) fa[q] = 4 * q + g > rr ? -m[16 * (4 * q + g)] : 0.0;
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][v] = r0[16 * i + 4 * v];
            branch_end<0>();
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) fa[q] = -F[(4 * q + g) * S::kLd + 16 * me.row + rr];
            static_for<NW>([&](auto i) {
                if (i == ib) {
                    acc[i] = d4_t{0.0, 0.0, 0.0, 0.0};
                    branch_end<i>();
                }
            });
        }
        // the next block column first, so that it is published meanwhile
        const int next = ib + 1 < end ? ib + 1 : -1;
        if (next >= 0 && next < NW) {
            double f[4];
            load(next, f);
            static_for<NW>([&](auto i) {
                if (i == next) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[q], fa[q], acc[i], 0, 0, 0);
                    publish_col(acc[i], b + 1, rr, g);
                    branch_end<i>();
                }
            });
        }
        static_for<NW>([&](auto i) {
            if (i < end) {
                if constexpr (i + 1 < NW) load(i + 1, fb[(i + 1) & 1]);
                if (i != next) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(fb[i & 1][q], fa[q], acc[i], 0, 0, 0);
                    branch_end<i>();
                }
            }
        });
        if (own) {
            static_for<NW>([&](auto i) {
                if (i == ib) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[i][v] = nw[256 * (b & 1) + 64 * v + lane];
                    branch_end<i>();
                }
            });
        }
        if (b + 1 < nblk) publish_row(b + 1);
        __builtin_amdgcn_s_setprio(0);
    }
    if (__syncthreads_or(viol)) return false;

    const int ln = opaque(lane0), row = 16 * me.row + (ln & 15), c = 16 * me.c0 + (ln >> 4);
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int col = c + 16 * i + 4 * v;
            if (row < L && col < L) static_cast<TO *>(a.out)[row + (int64_t)col * a.ldo] = (TO)acc[i][v];
        }
    return true;
}

template <int N, typename TI, typename TO>
__device__ __attribute__((always_inline)) inline bool gj_ahead(const LeafArgs &a, double *sm) {
    using S = AheadLds<N>;
    const int t = threadIdx.x, lane0 = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int L = a.L;
    if (L < 1 || L > N) return false;  // the same in every thread
    constexpr auto kSteps = std::make_integer_sequence<int, 16>{};
    const int nblk = (L + 15) >> 4;

    // for the two waves that need it (an FP32 entry is never far)
    auto divide = [&] {
        if constexpr (sizeof(TI) == 4) return false;
        bool far = false;
#pragma unroll
        for (int i = lane0; i < N; i += 64)
            far = far | far_entry(i < L ? (double)static_cast<const TI *>(a.in)[i * (a.ldi + 1)] : 1.0);
        return __any(far) != 0;
    };
    // Every role has a loop of its own, with the registers that it needs; all
    // meet at the same two barriers per block step, and two before the first.
    if (w == 0) {
        const bool dv = divide();
#pragma unroll 1
        for (int b = -1; b < nblk; ++b) {
            const int lane = opaque(lane0), rr = lane & 15, g = lane >> 4;
            const int u = b & 1, n = u ^ 1;
            double *const mini = sm + S::oMini + 2 * S::kMini * u;
            wg_barrier();
            // What the wave reads from here on is not written before the next
            // block step, so its second barrier may stand anywhere.  Order 64
            // waits for this wave, which does what it can before; order 128
            // has time and leaves the SIMD to the panels (2 700 cycles, not
            // 3 700).
            if (N == 128) wg_barrier();
            if (b >= 0 && b + 1 < nblk) {
                const bool cl = g & 1;
                double *const x0 = mini + (cl ? S::kMini : 0) + rr;
                const double *const dr = sm + S::oDr + 256 * u;
                const double *const r0 = (cl ? sm + S::oDm + 256 * u : dr) + rr;
                double x[16], r[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    x[j] = x0[S::kMLd * j];
                    r[j] = r0[16 * j];
                }
                mini_half(x, r, cl ? dr[17 * rr] : 1.0, kSteps);
#pragma unroll
                for (int j = 0; j < 16; ++j) x0[S::kMLd * j] = x[j];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            if (b + 1 < nblk) {
                __builtin_amdgcn_s_setprio(3);
                const double *const pub = sm + S::oPub + 256 * n;
                double *const nw = sm + S::oNew + 256 * n;
                d4_t D;
#pragma unroll
                for (int v = 0; v < 4; ++v) D[v] = pub[64 * v + lane];
                if (b >= 0) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        D = __builtin_amdgcn_mfma_f64_16x16x4f64(mini[S::kMini + S::kMLd * (4 * q + g) + rr],
                                                                 -mini[S::kMLd * (4 * q + g) + rr], D, 0, 0, 0);
                }
                if (N == 64) wg_barrier();
                diag_chain(dv, D, lane0, sm + S::oDm + 256 * n, sm + S::oDr + 256 * n, sm + S::oDump);
#pragma unroll
                for (int v = 0; v < 4; ++v) nw[64 * v + lane] = D[v];
                __builtin_amdgcn_s_setprio(0);
            } else if (N == 64) {
                wg_barrier();
            }
        }
        return !__syncthreads_or(0);
    }
    if (w == ahead_checks(N)) {
        const bool dv = divide();
        bool viol = false;
        wg_barrier();
        wg_barrier();
#pragma unroll 1
        for (int b = 0; b < nblk; ++b) {
            const double *const dr = sm + S::oDr + 256 * (b & 1), *const dm = sm + S::oDm + 256 * (b & 1);
            wg_barrier();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = lane0 + 64 * q, k = e >> 4, l = e & 15;
                const double piv = dm[17 * k];
                const double r = dr[e];
                viol = viol | pivot_fails(piv, dv) | ((l > k) & !(fabs(dm[e]) <= fabs(piv))) |
                       !(fabs(r) <= DBL_MAX);
                // block column b's multiplicand
                sm[S::oR + k * S::kPrLd + N + l] = k >= l ? r : 0.0;
            }
            wg_barrier();
        }
        return !__syncthreads_or(viol);
    }
    const AheadRole me = ahead_role(N, w);
    if (N == 128 && w < 8 && w != 4) return ahead_rows<N, 8, TI, TO>(a, sm, me, lane0);
    return ahead_rows<N, 4, TI, TO>(a, sm, me, lane0);
}

// ------------------------------------------------- two-workgroup panel ---
// The speculative elimination of a full 64-column panel of 129 to 256 rows on
// two workgroups (two CUs), each holding 32 of its columns (eight waves of
// four columns for all rows: lane l, slot i of a wave holds row l + 64 ((i +
// k0 / 64) mod RR), so the pivot row of step c is slot 0 of lane c).
// Workgroup h owns steps 32h .. 32h + 31: the wave that holds the column runs
// the step alone (pivot row by readlane), publishes its multipliers, pivot
// and inverse pivot to LDS and raises the step's flag, and every other wave
// applies the step when it sees the flag; issue priority goes by distance to
// ownership.  The wave that owned the previous column block, which is then caught up and
// far from its next turn, stores each step's multipliers and inverse pivot
// to the panel's exchange area in device memory, and the other workgroup
// replays the step from there.
//
// The exchange area holds a signalling-NaN pattern before the panel (filled
// by leaf_duo_reset, or by the previous leaf's leaf_unpermute), so a value
// read back is either that pattern (not yet stored: read again) or the
// stored value: every 8-byte access is single-copy atomic, and no flag or
// ordering between stores is needed.  The loads and stores are device-
// coherent (agent scope), and the values of the step after next are loaded
// before the current step's update.
//
// Every wait is bounded.  Workgroup 0 posts a verdict on its own steps when
// they are done.  Workgroup 1 posts its verdict (all its checks passed, or
// not) and waits for workgroup 0's decision; workgroup 0 waits for that
// verdict, decides (commit only if both workgroups' checks passed and
// nothing timed out), and posts the decision.  Workgroup 0 is dispatched
// before workgroup 1, so a running workgroup 1 always gets a decision.
// Outputs that are not the search's input are stored before the decision
// where they cannot differ from the search's (workgroup 0's own, which it
// orders before the search; workgroup 1's once both verdicts passed); the
// rest on commit.  On abort workgroup 0 runs the search (leaf_duo).  A value
// equal to the pattern in the input only makes a wait run out, which aborts
// to the search.
constexpr unsigned long long kDuoPoison = 0x7FF4DEADBEEF0001ull;  // a signalling NaN
constexpr int kDuoSpin = 1 << 15;        // default polls of a data wait (about 64 clocks each and more)
constexpr int kDuoDecideSpin = 1 << 24;  // polls of workgroup 1's wait for the decision

__device__ inline double ld_agent(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_agent(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline int ld_agent_i(const int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_agent_i(int *p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool is_poison(double v) {
    return (unsigned long long)__double_as_longlong(v) == kDuoPoison;
}

// Doubles of one panel's exchange area at RR slots per lane: the 64 steps'
// multipliers [step][slot][lane], then the inverse pivots.
template <int RR>
constexpr int duo_panel_doubles() { return 64 * RR * 64 + 64; }
// Ints of one panel's decision area: verdict of workgroup 1, decision,
// verdict of workgroup 0 on its own steps.
constexpr int kDuoPanelInts = 3;

template <int RR>
__device__ __attribute__((always_inline)) inline bool wpanel_duo(const LeafArgs &a) {
    constexpr int NW = 8, NT = 512, CW = 4, HALF = 32;  // waves, threads, columns per wave, per workgroup
    static_assert(RR <= 4 && CW * NW == HALF, "two workgroups of 32 columns, at most 256 rows");
    __shared__ double fst[HALF][RR][64];  // this workgroup's steps' multipliers
    __shared__ double pst[2][HALF];       // their inverse pivots and pivots
    __shared__ int rdy[HALF];
    const int h = blockIdx.x;  // 0 or 1: columns and steps 32h .. 32h + 31
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int L = a.L, k0 = a.k0, nb = a.nb;
    const double *src = a.in ? static_cast<const double *>(a.in) : a.Z;
    const int64_t lds = a.in ? a.ldi : a.ldz;
    const int rot = k0 >> 6;
    if ((k0 & 63) != 0 || nb != 64 || L > 64 * RR || L <= 64 || !a.xg || !a.xc)
        return false;  // the same in both workgroups
    double *gf = a.xg;                // [64][RR][64]
    double *gp = a.xg + 64 * RR * 64;  // [64]
    int *verdict1 = a.xc, *decision = a.xc + 1, *verdict0 = a.xc + 2;
    if (t < HALF) rdy[t] = 0;
    int rowr[RR];
    int rel[RR];  // row - k0 for rows inside the leaf from k0 on, else -1
#pragma unroll
    for (int i = 0; i < RR; ++i) {
        rowr[i] = lane + 64 * ((i + rot) % RR);
        rel[i] = (i + rot < RR && rowr[i] < L) ? lane + 64 * i : -1;
    }
    double z[RR][CW];
#pragma unroll
    for (int i = 0; i < RR; ++i)
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            const int col = HALF * h + CW * w + j;
            z[i][j] = rowr[i] < L ? src[rowr[i] + (int64_t)(k0 + col) * lds] : 0.0;
        }
    // this workgroup's half of the pivot rows of the outside columns (Q)
    const int nout = L - nb, qtot = nb * nout, qhalf = (qtot + 1) / 2;
    constexpr int QPT = (4096 * (RR - 1) / 2 + NT - 1) / NT;
    double qv[QPT];
#pragma unroll
    for (int r = 0; r < QPT; ++r) {
        const int e = h * qhalf + t + NT * r, c = e % nb, j = e / nb;
        const int gj = j < k0 ? j : j + nb;
        qv[r] = (t + NT * r < qhalf && e < qtot) ? src[(k0 + c) + (int64_t)gj * lds] : 0.0;
    }
    // output stores: Q (this workgroup's half), U' with or without Z, Z
    auto store_q = [&]() {
#pragma unroll
        for (int r = 0; r < QPT; ++r) {
            const int e = h * qhalf + t + NT * r, c = e % nb, j = e / nb;
            const int gj = j < k0 ? j : j + nb;
            if (t + NT * r < qhalf && e < qtot) a.Q[c + (int64_t)gj * nb] = qv[r];
        }
    };
    auto store_up = [&](const bool with_z) {
#pragma unroll
        for (int i = 0; i < RR; ++i)
#pragma unroll
            for (int j = 0; j < CW; ++j) {
                const int row = rowr[i], col = HALF * h + CW * w + j;
                if (row < L) {
                    a.Up[row + (int64_t)col * L] = z[i][j] - ((row == k0 + col) ? 1.0 : 0.0);
                    if (with_z) a.Z[row + (int64_t)(k0 + col) * a.ldz] = z[i][j];
                }
            }
    };
    auto store_z = [&]() {
#pragma unroll
        for (int i = 0; i < RR; ++i)
#pragma unroll
            for (int j = 0; j < CW; ++j) {
                const int row = rowr[i], col = HALF * h + CW * w + j;
                if (row < L) a.Z[row + (int64_t)(k0 + col) * a.ldz] = z[i][j];
            }
    };
    // Z may be written before the decision only when the panel is read from
    // the leaf's input; otherwise Z holds the search's input.
    const bool z_early = a.in != nullptr;
    bool viol = false;
    if (h == 0 && w == 0 && k0 > 0) {
#pragma unroll
        for (int i = 0; i < RR; ++i)
            if (rowr[i] < L && ((a.used[rowr[i]] != 0) != (rowr[i] < k0))) viol = true;
    }
    __syncthreads();  // the flags are cleared

    auto own_step = [&](const int j) {
        const int c = HALF * h + CW * w + j, lc = c - HALF * h;
        const double piv = readlane_f64(z[0][j], c);
        const double pinv = 1.0 / piv;
        const bool pl = lane == c;
        double rv[CW], f[RR];
#pragma unroll
        for (int jj = 0; jj < CW; ++jj) rv[jj] = (jj == j) ? pinv : readlane_f64(z[0][jj], c) * pinv;
#pragma unroll
        for (int i = 0; i < RR; ++i) {
            f[i] = (i == 0 && pl) ? 0.0 : z[i][j];
            fst[lc][i][lane] = f[i];
        }
        if (lane == 0) {
            pst[0][lc] = pinv;
            pst[1][lc] = piv;
        }
#pragma unroll
        for (int i = 0; i < RR; ++i) z[i][j] = 0.0;  // the pivot column restarts from 0
        if (pl) {
#pragma unroll
            for (int jj = 0; jj < CW; ++jj) z[0][jj] = rv[jj];
        }
#pragma unroll
        for (int i = 0; i < RR; ++i)
#pragma unroll
            for (int jj = 0; jj < CW; ++jj) z[i][jj] = fma(-f[i], rv[jj], z[i][jj]);
        if (lane == 0) __hip_atomic_store(&rdy[lc], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // the update of step c with its multipliers and inverse pivot
    auto apply = [&](const int c, const double (&f)[RR], const double pinv) {
        const bool pl = lane == c;
        double rv[CW];
#pragma unroll
        for (int jj = 0; jj < CW; ++jj) rv[jj] = readlane_f64(z[0][jj], c) * pinv;
        if (pl) {
#pragma unroll
            for (int jj = 0; jj < CW; ++jj) z[0][jj] = rv[jj];
        }
#pragma unroll
        for (int i = 0; i < RR; ++i)
#pragma unroll
            for (int jj = 0; jj < CW; ++jj) z[i][jj] = fma(-f[i], rv[jj], z[i][jj]);
    };
    // a local step of another wave, checked by the checking wave and passed
    // to the other workgroup by the forwarding wave
    auto local_step = [&](const int c, const bool chk, const bool fwd) {
        const int lc = c - HALF * h;
        while (__hip_atomic_load(&rdy[lc], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0)
            __builtin_amdgcn_s_sleep(1);
        const double pinv = pst[0][lc];
        double f[RR];
#pragma unroll
        for (int i = 0; i < RR; ++i) f[i] = fst[lc][i][lane];
        if (fwd) {
#pragma unroll
            for (int i = 0; i < RR; ++i) st_agent(&gf[((int64_t)c * RR + i) * 64 + lane], f[i]);
            if (lane == 0) st_agent(&gp[c], pinv);
        }
        apply(c, f, pinv);
        if (chk) {
            const double piv = pst[1][lc];
            const double apiv = fabs(piv);
            bool v = !(apiv > 0.0) | !(apiv <= DBL_MAX);
#pragma unroll
            for (int i = 0; i < RR; ++i) v |= (rel[i] > c) & !(fabs(f[i]) <= apiv);
            viol |= v;
        }
    };
    // The other workgroup's 32 steps c0 .. c0 + 31, each read back from the
    // exchange area once every lane sees stored values.  The values of the
    // next DEPTH steps are in flight while a step is applied: a device-
    // coherent load takes about as long as two steps' work, and a load issued
    // further ahead is more often issued before the value is stored and must
    // be repeated.  False if a wait ran out.
    constexpr int DEPTH = 2;
    auto remote_steps = [&](const int c0) -> bool {
        double rf[DEPTH][RR], rp[DEPTH];
        auto load = [&](const int c, double (&ff)[RR], double &pp) {
#pragma unroll
            for (int i = 0; i < RR; ++i) ff[i] = ld_agent(&gf[((int64_t)c * RR + i) * 64 + lane]);
            pp = ld_agent(&gp[c]);
        };
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) load(c0 + d, rf[d], rp[d]);
#pragma unroll
        for (int k = 0; k < HALF; ++k) {
            const int c = c0 + k, d = k % DEPTH;
            auto missing = [&](const double (&ff)[RR], const double pp) {
                bool bad = is_poison(pp);
#pragma unroll
                for (int i = 0; i < RR; ++i) bad |= is_poison(ff[i]);
                return __any(bad) != 0;
            };
            // The first look is outside any loop, so the loads of the later
            // steps stay in flight; a step not yet stored is read again into
            // other registers until it is.
            if (missing(rf[d], rp[d])) {
                double tf[RR], tp;
                int spins = 0;
                do {
                    if (++spins > a.duo_spin) return false;
                    __builtin_amdgcn_s_sleep(2);
                    load(c, tf, tp);
                } while (missing(tf, tp));
#pragma unroll
                for (int i = 0; i < RR; ++i) rf[d][i] = tf[i];
                rp[d] = tp;
            }
            double f[RR];
#pragma unroll
            for (int i = 0; i < RR; ++i) f[i] = rf[d][i];
            const double pinv = rp[d];
            if (k + DEPTH < HALF) load(c + DEPTH, rf[d], rp[d]);
            apply(c, f, pinv);
        }
        return true;
    };

    bool ok = true;
    // steps 0 .. 31 (workgroup 0's), then 32 .. 63 (workgroup 1's)
    for (int half = 0; half < 2; ++half) {
        if (half != h) {
            if (ok) ok = remote_steps(HALF * half);
            continue;
        }
        for (int b = 0; b < NW; ++b) {
            // issue priority by distance to ownership
            if (w == b)
                __builtin_amdgcn_s_setprio(3);
            else if (w == b + 1)
                __builtin_amdgcn_s_setprio(2);
            else if (w == b + 2)
                __builtin_amdgcn_s_setprio(1);
            // the previous owner, just caught up, forwards the block's steps
            const bool chk = w == (b + NW / 2) % NW;
            const bool fwd = w == (b + NW - 1) % NW;
            if (w == b) {
#pragma unroll
                for (int j = 0; j < CW; ++j) own_step(j);
                __builtin_amdgcn_s_setprio(0);
            } else {
                for (int c = HALF * h + CW * b; c < HALF * h + CW * b + CW; ++c) local_step(c, chk, fwd);
            }
        }
        if (h == 0) {
            // workgroup 0's steps are all checked: post the verdict on them,
            // and store this workgroup's half of Q (the search rewrites it)
            const bool bad0 = __syncthreads_or(viol);
            if (t == 0) st_agent_i(verdict0, bad0 ? 1 : 0);
            store_q();
        }
    }
    __builtin_amdgcn_s_setprio(0);
    if (h == 0) store_up(z_early);
    const bool bad = __syncthreads_or(viol || !ok);
    // Workgroup 1 stores U' and Q (and Z when the input is separate) before
    // the decision when every step of the panel passed its check: they then
    // equal what the search would write, bit for bit, so it does not matter
    // whether they land before or after the search's own stores.
    __shared__ int early_s;

    // verdict and decision
    __shared__ int commit_s;
    if (h == 1) {
        if (t == 0) {
            st_agent_i(verdict1, bad ? 1 : 0);
            int v = -1;
            for (int spins = 0; !bad && spins < a.duo_spin; ++spins) {
                v = ld_agent_i(verdict0);
                if (v >= 0) break;
                __builtin_amdgcn_s_sleep(8);
            }
            early_s = !bad && v == 0;
        }
        __syncthreads();
        if (early_s) {
            store_q();
            store_up(z_early);
        }
    }
    if (t == 0) {
        if (h == 1) {
            int d = -1;
            for (int spins = 0; spins < kDuoDecideSpin; ++spins) {
                d = ld_agent_i(decision);
                if (d >= 0) break;
                __builtin_amdgcn_s_sleep(8);
            }
            commit_s = d == 1;
        } else {
            int v = -1;
            for (int spins = 0; !bad && spins < a.duo_spin; ++spins) {
                v = ld_agent_i(verdict1);
                if (v >= 0) break;
                __builtin_amdgcn_s_sleep(8);
            }
            const bool c = !bad && v == 0;
            st_agent_i(decision, c ? 1 : 0);
            commit_s = c;
        }
    }
    __syncthreads();
    if (!commit_s) return false;

    if (h == 1 && !early_s) {
        store_q();
        store_up(true);
    } else if (!z_early) {
        store_z();
    }
    if (h == 0) {
        for (int c = t; c < nb; c += NT) a.rsel[k0 + c] = k0 + c;
        for (int row = t; row < L; row += NT) {
            const bool piv = row >= k0 && row < k0 + nb;
            if (k0 == 0)
                a.used[row] = piv ? 1 : 0;
            else if (piv)
                a.used[row] = 1;
        }
    }
    return true;
}

// A full panel of a leaf of order 129 .. 256 on two workgroups; on abort
// (or with speculation off) workgroup 0 runs the search kernel.
__global__ void __launch_bounds__(512) leaf_duo(LeafArgs a) {
    if (a.spec && *a.spec != 0) {
        if (wpanel_duo<4>(a)) return;
        if (blockIdx.x != 0) return;
        if (threadIdx.x == 0) *a.spec = 0;
        // the stores made before the decision are complete before the search
        // rewrites the same outputs
        __threadfence();
        __syncthreads();
    } else if (blockIdx.x != 0) {
        return;
    }
    __shared__ __attribute__((aligned(16))) double sm[RunLds<32, 8, 4>::kDoubles];
    gj2d_run<32, 8, 4, false, double, double>(a, sm);
}

// Fills the exchange areas of a leaf's two-workgroup panels: every value
// with the pattern, every verdict and decision word with -1.
__global__ void __launch_bounds__(256) leaf_duo_reset(double *xg, int64_t nd, int *xc, int ni) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e < nd) xg[e] = __longlong_as_double((long long)kDuoPoison);
    if (e < ni) xc[e] = -1;
}

template <int TR, int RR, int RC, bool WHOLE>
constexpr int gj2d_waves() {
    return WHOLE ? ahead_waves(TR * RR) : TR / 4;
}

template <int TR, int RR, int RC, bool WHOLE, typename TI, typename TO>
__device__ __attribute__((always_inline)) inline void gj2d_any(const LeafArgs &a) {
    constexpr int NW = TR / 4;                 // the search's waves
    constexpr int RB = TR * RR / (16 * NW);    // 16-row blocks per wave
    static_assert(RB * 16 * NW == TR * RR && NW * 64 == 16 * TR, "row blocks cover the rows");
    static_assert(!WHOLE || (16 * RC == TR * RR && gj2d_waves<TR, RR, RC, WHOLE>() >= NW), "whole leaves are square");
    constexpr int D0 = WHOLE ? AheadLds<TR * RR>::kDoubles : BlkLds<NW, RB, RC>::kDoubles;
    constexpr int D1 = RunLds<TR, RR, RC>::kDoubles;
    __shared__ __attribute__((aligned(16))) double sm[D0 > D1 ? D0 : D1];
    bool spec;
    if (WHOLE && a.reset) {
        spec = a.reset == 1;
        if (threadIdx.x == 0) {
            for (int i = 0; i < kStatusWords; ++i) a.status[i] = (i == kStatusSpecWord && !spec) ? 0 : INT_MAX;
            a.status[kFrobCounterWord] = 0;
        }
    } else {
        spec = a.spec && *a.spec != 0;
    }
    if (spec) {
        bool ok;
        if constexpr (WHOLE)
            ok = gj_ahead<TR * RR, TI, TO>(a, sm);
        else
            ok = gj_blocked<NW, RB, RC>(a, sm);
        if (ok) return;
        if (threadIdx.x == 0) *a.spec = 0;
    }
    // the waves that only the blocked tier has
    if (WHOLE && threadIdx.x >= 16 * TR) return;
    gj2d_run<TR, RR, RC, WHOLE, TI, TO>(a, sm);
}

template <int TR, int RR, int RC, bool WHOLE, typename TI, typename TO>
__global__ void __launch_bounds__((64 * gj2d_waves<TR, RR, RC, WHOLE>())) leaf_gj2d(LeafArgs a) {
    gj2d_any<TR, RR, RC, WHOLE, TI, TO>(a);
}

// Many independent whole leaves in one grid (one workgroup each); the same
// device code as a single leaf, so every leaf's result is identical to the
// one it gets when launched alone.
template <int TR, int RR, int RC, typename TI, typename TO>
__global__ void __launch_bounds__((64 * gj2d_waves<TR, RR, RC, true>())) leaf_gj2d_batch(LeafBatch b) {
    const LeafItem &it = b.item[blockIdx.x];
    LeafArgs a{};
    a.in = it.in;
    a.ldi = it.ldi;
    a.out = it.out;
    a.ldo = it.ldo;
    a.L = (int)it.L;
    a.col0 = (int)it.col0;
    a.status = it.status;
    a.spec = it.status + kStatusSpecWord;
    gj2d_any<TR, RR, RC, true, TI, TO>(a);
}

// ---------------------------------------------------------------- tier 2 ---
struct PanelArgs {
    double *Z;
    int64_t ldz;
    int L, k0, nb, col0;
    int *used;   // L flags: row already chosen as a pivot
    int *rsel;   // L entries: pivot row of global step k
    double *Up;  // L x NB, ld L: panel transformation minus the pivot units
    int *status;
};

// The panel lives in registers with a rotating slot map: at step c, slot s of
// every thread holds panel column (s + c) mod NB, so the active column is
// always slot 0 and no register is indexed by a run-time value.
template <int NB, int RPT, int NT>
__global__ void __launch_bounds__(NT) leaf_panel(PanelArgs a) {
    constexpr int NW = NT / 64;
    __shared__ double red_v[2][NW];
    __shared__ int red_i[2][NW];
    __shared__ int red_f[2][NW];
    __shared__ double rowbuf[2][NB];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int L = a.L, k0 = a.k0, nb = a.nb;

    double z[RPT][NB];
    bool usd[RPT];
    int pst[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int row = t + NT * q;
        usd[q] = row >= L || (k0 > 0 && a.used[row] != 0);
        pst[q] = -1;
#pragma unroll
        for (int c = 0; c < NB; ++c)
            z[q][c] = (row < L && c < nb) ? a.Z[row + (int64_t)(k0 + c) * a.ldz] : 0.0;
    }
    int bad = 0;

    for (int c = 0; c < nb; ++c) {
        const int buf = c & 1;
        double best = -1.0;
        int bi = INT_MAX, nf = 0;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            if (!usd[q]) {
                // non-finite candidates keep key -0.5 so that an unused row
                // is always chosen (see tier 1)
                double av = fabs(z[q][0]);
                if (!(av <= DBL_MAX)) {
                    nf = 1;
                    av = -0.5;
                }
                if (av > best) {
                    best = av;
                    bi = t + NT * q;
                }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double ob = __shfl_xor(best, off);
            const int oi = __shfl_xor(bi, off);
            if (better(ob, oi, best, bi)) {
                best = ob;
                bi = oi;
            }
        }
        const int wnf = __any(nf);
        if (lane == 0) {
            red_v[buf][w] = best;
            red_i[buf][w] = bi;
            red_f[buf][w] = wnf;
        }
        __syncthreads();
        best = red_v[buf][0];
        bi = red_i[buf][0];
        nf = red_f[buf][0];
#pragma unroll
        for (int ww = 1; ww < NW; ++ww) {
            const double ob = red_v[buf][ww];
            const int oi = red_i[buf][ww];
            nf |= red_f[buf][ww];
            if (better(ob, oi, best, bi)) {
                best = ob;
                bi = oi;
            }
        }
        const int p = bi;
        if ((nf || !(best > 0.0)) && bad == 0) bad = c + 1;
        if (t == p % NT) {
            const int pq = p / NT;
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                if (q == pq) {
                    const double pinv = 1.0 / z[q][0];
#pragma unroll
                    for (int sl = 0; sl < NB; ++sl) {
                        rowbuf[buf][sl] = z[q][sl] * pinv;
                        z[q][sl] = 0.0;
                    }
                    rowbuf[buf][0] = pinv;
                    usd[q] = true;
                    pst[q] = c;
                }
            }
        }
        if (t == 0) a.rsel[k0 + c] = p;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const double f = (pst[q] == c) ? -1.0 : z[q][0];
            z[q][0] = 0.0;
#pragma unroll
            for (int sl = 0; sl < NB; ++sl) z[q][sl] = fma(-f, rowbuf[buf][sl], z[q][sl]);
            // rotate: slot s takes panel column (s + c + 1) mod NB
            const double z0 = z[q][0];
#pragma unroll
            for (int sl = 0; sl + 1 < NB; ++sl) z[q][sl] = z[q][sl + 1];
            z[q][NB - 1] = z0;
        }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int row = t + NT * q;
        if (row < L) {
#pragma unroll
            for (int sl = 0; sl < NB; ++sl) {
                const int c = (sl + nb) & (NB - 1);
                if (c < nb) {
                    a.Z[row + (int64_t)(k0 + c) * a.ldz] = z[q][sl];
                    a.Up[row + (int64_t)c * L] = z[q][sl] - ((pst[q] == c) ? 1.0 : 0.0);
                }
            }
            if (k0 == 0)
                a.used[row] = pst[q] >= 0 ? 1 : 0;
            else if (pst[q] >= 0)
                a.used[row] = 1;
        }
    }
    if (t == 0 && bad) atomicMin(a.status, a.col0 + k0 + bad);
}

// Q (nb x L, ld nb): Q[c][j] = Z[rsel[k0 + c]][j] for columns outside the panel.
__global__ void __launch_bounds__(256)
    leaf_gather_q(const double *__restrict__ Z, int64_t ldz, int L, int k0, int nb,
                  const int *__restrict__ rsel, double *__restrict__ Q) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)L * nb) return;
    const int c = (int)(e % nb), j = (int)(e / nb);
    if (j >= k0 && j < k0 + nb) return;
    Q[c + (int64_t)j * nb] = Z[rsel[k0 + c] + (int64_t)j * ldz];
}

template <typename TI>
__global__ void __launch_bounds__(256)
    leaf_copy_in(const TI *__restrict__ in, int64_t ldi, double *__restrict__ Z, int L) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)L * L) return;
    const int i = (int)(e % L), j = (int)(e / L);
    Z[i + (int64_t)j * L] = (double)in[i + (int64_t)j * ldi];
}

// out[rinv[i]][rsel[c]] = Z[i][c].  When xg is given, also fills the leaf's
// exchange areas for the two-workgroup panels of the next leaf (nd doubles
// with the pattern, ni decision words with -1); the leaf's panels have all
// completed when this kernel runs.
template <typename TO>
__global__ void __launch_bounds__(256)
    leaf_unpermute(const double *__restrict__ Z, int L, const int *__restrict__ rsel,
                   TO *__restrict__ out, int64_t ldo, double *__restrict__ xg, int nd,
                   int *__restrict__ xc, int ni) {
    if (xg) {
        for (int e = blockIdx.x * 256 + threadIdx.x; e < nd; e += gridDim.x * 256)
            xg[e] = __longlong_as_double((long long)kDuoPoison);
        if (blockIdx.x == 0 && (int)threadIdx.x < ni) xc[threadIdx.x] = -1;
    }
    __shared__ int rinv[kLeafMaxOrder];
    for (int k = threadIdx.x; k < L; k += 256) rinv[k] = -1;
    __syncthreads();
    for (int k = threadIdx.x; k < L; k += 256) {
        const int r = rsel[k];
        if ((unsigned)r < (unsigned)L) rinv[r] = k;
    }
    __syncthreads();
    // one column per workgroup at a time
    for (int c = blockIdx.x; c < L; c += gridDim.x) {
        const int rc = rsel[c];
        if ((unsigned)rc >= (unsigned)L) continue;
        const double *zc = Z + (int64_t)c * L;
        TO *oc = out + (int64_t)rc * ldo;
        for (int i = threadIdx.x; i < L; i += 256) {
            const int ri = rinv[i];
            if ((unsigned)ri < (unsigned)L) oc[ri] = (TO)zc[i];
        }
    }
}

// ---------------------------------------------------------------- launch ---
template <int TR, int RR, int RC, bool WHOLE, typename TI, typename TO>
hipError_t gj2d_launch(const LeafArgs &la, hipStream_t s) {
    hipLaunchKernelGGL((leaf_gj2d<TR, RR, RC, WHOLE, TI, TO>), dim3(1), dim3(64 * gj2d_waves<TR, RR, RC, WHOLE>()), 0, s, la);
    return hipGetLastError();
}

// Threads per row group of the 2-D kernel for whole leaves of order <= 128
// and for panels of leaves of order <= 256 and <= 512 (measured best on
// MI355X: 32, i.e. 512 threads, in all three; a 512-row panel takes 147 us
// with 512 threads against 169 us with 1024, a 256-row panel 93 us against
// 110 us with 256 or 1024).
constexpr int kLeaf128TR = 32;
constexpr int kPanel256TR = 32;
constexpr int kPanel512TR = 32;

template <typename TI, typename TO>
hipError_t whole_dispatch(const LeafArgs &la, hipStream_t s, const char **name) {
    if (la.L <= 64) {
        *name = "leaf_gj_regs_64";
        return gj2d_launch<16, 4, 4, true, TI, TO>(la, s);
    }
    *name = "leaf_gj_regs_128";
    return gj2d_launch<kLeaf128TR, 128 / kLeaf128TR, 8, true, TI, TO>(la, s);
}

int panel_width(int64_t L) {
    if (L <= 512) return 64;
    if (L <= 1024) return 32;
    return 16;
}

hipError_t panel_launch(const PanelArgs &pa, hipStream_t s) {
    const int L = pa.L;  // above 512
    if (L <= 1024)
        hipLaunchKernelGGL((leaf_panel<32, 1, 1024>), dim3(1), dim3(1024), 0, s, pa);
    else
        hipLaunchKernelGGL((leaf_panel<16, 2, 1024>), dim3(1), dim3(1024), 0, s, pa);
    return hipGetLastError();
}

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Leaves of order 129 .. 256 run their full panels on two workgroups
// (leaf_duo), with an exchange area per panel.  The areas sit at the start
// of every blocked leaf's scratch, so that leaves of every order find them at
// the same place and no other leaf writes them.
constexpr int kDuoPanels = 4;
constexpr int kDuoDoubles = kDuoPanels * duo_panel_doubles<4>();
constexpr int kDuoInts = kDuoPanels * kDuoPanelInts;
static_assert(kDuoInts <= 256, "the decision words are filled by one workgroup");
bool duo_leaf(int64_t L) { return L > 128 && L <= 256; }
// Polls after which a two-workgroup panel gives up waiting for the other
// workgroup: kDuoSpin, or SPIN_DUO_SPIN (a positive count; small values make
// the panels fall back to the search, for tests of that path).
int duo_spin_limit() {
    const char *e = std::getenv("SPIN_DUO_SPIN");
    const long v = e ? std::strtol(e, nullptr, 10) : 0;
    return (v > 0 && v <= kDuoSpin) ? (int)v : kDuoSpin;
}
size_t duo_bytes() { return align256(sizeof(double) * kDuoDoubles) + align256(sizeof(int) * kDuoInts); }

}  // namespace

size_t leaf_scratch_bytes(int64_t L) {
    if (L <= 128) return 0;
    const int64_t nb = panel_width(L);
    return duo_bytes() + align256(sizeof(double) * L * L) + align256(sizeof(double) * L * nb) +
           align256(sizeof(double) * L * nb) + align256(sizeof(int) * L) + align256(sizeof(int) * L);
}

bool leaf_fills_exchange(int64_t L) { return duo_leaf(L); }

int64_t leaf_launches(int64_t L, DType in_dt) {
    if (L <= 128) return 1;
    // panel and product, from order 513 on with a gather between; the exchange
    // areas' fill or the copy into Z before, the permutation after
    const int64_t panels = (L + panel_width(L) - 1) / panel_width(L);
    return panels * (L <= 512 ? 2 : 3) + (duo_leaf(L) ? 1 : 0) + (L <= 512 && in_dt == kF64 ? 0 : 1) + 1;
}

hipError_t leaf_launch(const void *in, DType in_dt, int64_t ldi, void *out, DType out_dt,
                       int64_t ldo, int64_t L64, int64_t col0, int *status, void *scratch,
                       bool exch_filled, hipStream_t s,
                       void (*trace_cb)(void *, const LaunchInfo &, int), void *trace_ctx, int reset) {
    if (reset && L64 > 128) return hipErrorInvalidValue;
    if (L64 < 1 || L64 > kLeafMaxOrder) return hipErrorInvalidValue;
    const int L = (int)L64;
    const double Ld = (double)L;
    auto cb = [&](const LaunchInfo &li, int phase) {
        if (trace_cb) trace_cb(trace_ctx, li, phase);
    };
    if (L <= 128) {
        LaunchInfo li{"leaf_gj_regs", 2.0 * Ld * Ld * Ld, 16.0 * Ld * Ld};
        cb(li, 0);
        LeafArgs la{};
        la.in = in;
        la.ldi = ldi;
        la.out = out;
        la.ldo = ldo;
        la.L = L;
        la.col0 = (int)col0;
        la.status = status;
        la.spec = status + kStatusSpecWord;
        la.reset = reset;
        hipError_t e;
        const char *name = "leaf_gj_regs";
        if (in_dt == kF64 && out_dt == kF64)
            e = whole_dispatch<double, double>(la, s, &name);
        else if (in_dt == kF32 && out_dt == kF32)
            e = whole_dispatch<float, float>(la, s, &name);
        else
            return hipErrorInvalidValue;
        li.name = name;
        cb(li, 1);
        return e;
    }
    if (!scratch) return hipErrorInvalidValue;
    const int nb = panel_width(L);
    char *p = static_cast<char *>(scratch);
    double *const xg = reinterpret_cast<double *>(p);
    p += align256(sizeof(double) * kDuoDoubles);
    int *const xc = reinterpret_cast<int *>(p);
    p += align256(sizeof(int) * kDuoInts);
    double *Z = reinterpret_cast<double *>(p);
    p += align256(sizeof(double) * L * L);
    double *Up = reinterpret_cast<double *>(p);
    p += align256(sizeof(double) * L * nb);
    double *Q = reinterpret_cast<double *>(p);
    p += align256(sizeof(double) * L * nb);
    int *rsel = reinterpret_cast<int *>(p);
    p += align256(sizeof(int) * L);
    int *used = reinterpret_cast<int *>(p);
    p += align256(sizeof(int) * L);
    const bool duo = duo_leaf(L);
    if (duo && !exch_filled) {
        LaunchInfo li{"leaf_duo_reset", 0.0, 8.0 * kDuoDoubles};
        cb(li, 0);
        hipLaunchKernelGGL(leaf_duo_reset, dim3((unsigned)((kDuoDoubles + 255) / 256)), dim3(256), 0, s,
                           xg, (int64_t)kDuoDoubles, xc, kDuoInts);
        hipError_t e = hipGetLastError();
        cb(li, 1);
        if (e != hipSuccess) return e;
    }

    const int nblk = (int)(((int64_t)L * L + 255) / 256);
    // Up to order 512 an FP64 input is read in place by the first panel and
    // its update (which writes Z); otherwise it is copied into Z first.
    const bool direct = L <= 512 && in_dt == kF64;
    if (!direct) {
        LaunchInfo li{"leaf_copy_in", 0.0, (in_dt == kF64 ? 16.0 : 12.0) * Ld * Ld};
        cb(li, 0);
        if (in_dt == kF64)
            hipLaunchKernelGGL((leaf_copy_in<double>), dim3(nblk), dim3(256), 0, s,
                               static_cast<const double *>(in), ldi, Z, L);
        else
            hipLaunchKernelGGL((leaf_copy_in<float>), dim3(nblk), dim3(256), 0, s,
                               static_cast<const float *>(in), ldi, Z, L);
        hipError_t e = hipGetLastError();
        cb(li, 1);
        if (e != hipSuccess) return e;
    }
    for (int k0 = 0; k0 < L; k0 += nb) {
        const int w = (L - k0 < nb) ? (L - k0) : nb;
        PanelArgs pa{Z, (int64_t)L, L, k0, w, (int)col0, used, rsel, Up, status};
        const bool fused = L <= 512;  // the 2-D panel kernel also gathers Q
        {
            LaunchInfo li{"leaf_gj_panel", 2.0 * Ld * w * w, 16.0 * Ld * w};
            cb(li, 0);
            hipError_t e;
            if (fused) {
                LeafArgs la{};
                la.L = L;
                la.col0 = (int)col0;
                la.status = status;
                la.spec = status + kStatusSpecWord;
                la.Z = Z;
                la.ldz = L;
                la.k0 = k0;
                la.nb = w;
                if (direct && k0 == 0) {
                    la.in = in;
                    la.ldi = ldi;
                }
                la.used = used;
                la.rsel = rsel;
                la.Up = Up;
                la.Q = Q;
                if (duo && w == 64 && k0 % 64 == 0 && k0 / 64 < kDuoPanels) {
                    la.xg = xg + (int64_t)(k0 / 64) * duo_panel_doubles<4>();
                    la.xc = xc + (k0 / 64) * kDuoPanelInts;
                    la.duo_spin = duo_spin_limit();
                    hipLaunchKernelGGL(leaf_duo, dim3(2), dim3(512), 0, s, la);
                    e = hipGetLastError();
                } else if (L <= 256)
                    e = gj2d_launch<kPanel256TR, 256 / kPanel256TR, 4, false, double, double>(la, s);
                else
                    e = gj2d_launch<kPanel512TR, 512 / kPanel512TR, 4, false, double, double>(la, s);
            } else {
                e = panel_launch(pa, s);
            }
            cb(li, 1);
            if (e != hipSuccess) return e;
        }
        if (w == L) break;
        if (!fused) {
            LaunchInfo li{"leaf_gather_q", 0.0, 16.0 * Ld * w};
            cb(li, 0);
            const int gb = (int)(((int64_t)L * w + 255) / 256);
            hipLaunchKernelGGL(leaf_gather_q, dim3(gb), dim3(256), 0, s, Z, (int64_t)L, L, k0, w,
                               rsel, Q);
            hipError_t e = hipGetLastError();
            cb(li, 1);
            if (e != hipSuccess) return e;
        }
        GemmProb pr[2];
        int np = 0;
        if (k0 > 0)
            pr[np++] = GemmProb{Up, Q, Z, Z, (int64_t)L, (int64_t)w, (int64_t)L, (int64_t)L,
                                L, k0, w, 0, 1.0, 1.0};
        if (k0 + w < L) {
            // the columns right of the first panel still live in the input
            const bool from_in = direct && k0 == 0;
            const double *c0 = from_in ? static_cast<const double *>(in) + (int64_t)(k0 + w) * ldi
                                       : Z + (int64_t)(k0 + w) * L;
            pr[np++] = GemmProb{Up, Q + (int64_t)(k0 + w) * w, c0, Z + (int64_t)(k0 + w) * L,
                                (int64_t)L, (int64_t)w, from_in ? ldi : (int64_t)L, (int64_t)L,
                                L, L - k0 - w, w, 0, 1.0, 1.0};
        }
        LaunchInfo gi{};
        cb(gi, 0);
        hipError_t e = gemm_launch(pr, np, kF64, s, &gi);
        cb(gi, 1);
        if (e != hipSuccess) return e;
    }
    {
        LaunchInfo li{"leaf_unpermute", 0.0,
                      (out_dt == kF64 ? 16.0 : 12.0) * Ld * Ld + (duo ? 8.0 * kDuoDoubles : 0.0)};
        cb(li, 0);
        const int gb = L < 1024 ? L : 1024;
        // a two-workgroup leaf leaves its exchange areas filled for the next
        double *fxg = duo ? xg : nullptr;
        if (out_dt == kF64)
            hipLaunchKernelGGL((leaf_unpermute<double>), dim3(gb), dim3(256), 0, s, Z, L, rsel,
                               static_cast<double *>(out), ldo, fxg, kDuoDoubles, xc, kDuoInts);
        else
            hipLaunchKernelGGL((leaf_unpermute<float>), dim3(gb), dim3(256), 0, s, Z, L, rsel,
                               static_cast<float *>(out), ldo, fxg, kDuoDoubles, xc, kDuoInts);
        hipError_t e = hipGetLastError();
        cb(li, 1);
        return e;
    }
}


hipError_t leaf_batch_launch(const LeafItem *items, int count, DType dt, hipStream_t s,
                             LaunchInfo *info) {
    if (count < 0 || count > kMaxLeafBatch) return hipErrorInvalidValue;
    double flops = 0, bytes = 0;
    LeafBatch small{}, big{};
    for (int i = 0; i < count; ++i) {
        if (items[i].L < 1 || items[i].L > 128) return hipErrorInvalidValue;
        const double L = (double)items[i].L;
        flops += 2.0 * L * L * L;
        bytes += 16.0 * L * L;
        if (items[i].L <= 64)
            small.item[small.count++] = items[i];
        else
            big.item[big.count++] = items[i];
    }
    hipError_t e = hipSuccess;
    if (small.count) {
        if (dt == kF64)
            hipLaunchKernelGGL((leaf_gj2d_batch<16, 4, 4, double, double>), dim3(small.count),
                               dim3(64 * ahead_waves(64)), 0, s, small);
        else
            hipLaunchKernelGGL((leaf_gj2d_batch<16, 4, 4, float, float>), dim3(small.count),
                               dim3(64 * ahead_waves(64)), 0, s, small);
        e = hipGetLastError();
    }
    if (e == hipSuccess && big.count) {
        if (dt == kF64)
            hipLaunchKernelGGL((leaf_gj2d_batch<kLeaf128TR, 128 / kLeaf128TR, 8, double, double>),
                               dim3(big.count), dim3(64 * ahead_waves(128)), 0, s, big);
        else
            hipLaunchKernelGGL((leaf_gj2d_batch<kLeaf128TR, 128 / kLeaf128TR, 8, float, float>),
                               dim3(big.count), dim3(64 * ahead_waves(128)), 0, s, big);
        e = hipGetLastError();
    }
    if (info) {
        info->name = "leaf_gj_regs_batch";
        info->flops = flops;
        info->bytes = bytes;
    }
    return e;
}

}  // namespace spin
