// Block products of the recursion on gfx950 matrix cores.
//
//   D = alpha * A * B + beta * C0 (+ I on the diagonal)        column-major views
//
// This is the paper's `multiply` (Sec. 3.3) with the `subtract` steps of
// Alg. 2 (V = IV - A22, C11 = I - VII) and the sign of `scalarMul` folded into
// the epilogue: the scheduler forms S = A22 - A21*III (alpha = -1, beta = 1),
// C12 = -III*C22 and C21 = -C22*II (alpha = -1), C11 = C11 - III*C21 in place
// (alpha = -1, beta = 1, C0 == D), and the Newton residual R = I - A*X
// (alpha = -1, add_identity).
//
// Kernel shape: a BM x BN output tile per workgroup of four or eight wave64s,
// split into WM x WN wave tiles of 16 x 16 MFMA blocks.  K advances in BK slabs
// staged global -> registers -> LDS with two LDS buffers, so the global loads of
// slab k+1 (and later ones, on the smaller tiles) are in flight while the matrix
// cores consume slab k, with one barrier per slab.
//
// Matrix-core operands are issued transposed (B^T tile as the first operand,
// A^T tile as the second), so each accumulator holds a 16 x 16 block of D^T:
// lane l owns output row m = l % 16, which makes the epilogue's stores
// contiguous down each column of the column-major result.
//   v_mfma_f64_16x16x4f64 : lane l, element v  ->  D^T row 4*v + l/16
//   v_mfma_f32_16x16x4f32 : lane l, element v  ->  D^T row 4*(l/16) + v
#include <hip/hip_runtime.h>

#include <type_traits>

#include "leaf_blocks.hpp"
#include "spin_kernels.hpp"

namespace spin {
namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

template <typename T>
struct Mma;

template <>
struct Mma<double> {
    using acc_t = d4_t;
    __device__ static inline acc_t mma(double bt, double at, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(bt, at, c, 0, 0, 0);
    }
    __device__ static inline int ncol(int lane, int v) { return 4 * v + (lane >> 4); }
};

template <>
struct Mma<float> {
    using acc_t = f4_t;
    __device__ static inline acc_t mma(float bt, float at, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(bt, at, c, 0, 0, 0);
    }
    __device__ static inline int ncol(int lane, int v) { return 4 * (lane >> 4) + v; }
};

// Up to N independent products in one grid: workgroup b belongs to the
// problem whose tile range [tile_start[q], tile_start[q+1]) contains b.
template <int N>
struct GroupArgs {
    GemmProb p[N];
    int32_t count;
    int32_t tile_start[N + 1];
    int32_t tiles_m[N];
};
static_assert(sizeof(GroupArgs<kMaxBatch>) <= 4096, "kernel arguments above 4 KiB");

// Problem of workgroup `bid` (uniform scan over the prefix sums).
template <int N>
__device__ inline int group_member(const GroupArgs<N> &g, int bid) {
    int pi = 0;
#pragma unroll
    for (int q = 1; q < N; ++q)
        if (q < g.count && bid >= g.tile_start[q]) pi = q;
    return pi;
}

// Tile (tm, tn) of the t-th workgroup of a problem with tiles_m x tiles_n
// tiles whose range starts at workgroup tstart. Workgroups are dealt to the
// eight XCDs round-robin (workgroup b runs on XCD b mod 8), and each XCD has
// its own L2: when the range and both tile counts are multiples of 8, XCD x
// gets the contiguous stretch [x T/8, (x+1) T/8) of an order made of 8 x 8
// tile blocks, so the A rows and B columns it reads stay in its own L2.
// Otherwise tiles go in plain column-major order. A lower-triangle problem
// (square tile grid) has only the T (T + 1) / 2 tiles on or below the
// diagonal, row by row: row r holds (r, 0) ... (r, r).  Every tile is
// computed exactly once, with the same arithmetic, whatever the order.
__device__ inline void tile_coords(int t, int tstart, int tiles_m, int tiles_n, bool lower, int &tm,
                                   int &tn) {
    if (lower) {
        int r = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
        while (r * (r + 1) / 2 > t) --r;
        while ((r + 1) * (r + 2) / 2 <= t) ++r;
        tm = r;
        tn = t - r * (r + 1) / 2;
        return;
    }
    if ((tstart & 7) == 0 && (tiles_m & 7) == 0 && (tiles_n & 7) == 0) {
        const int u = (t & 7) * ((tiles_m * tiles_n) >> 3) + (t >> 3);
        const int blk = u >> 6, in = u & 63;
        const int bms = tiles_m >> 3;
        tm = (blk % bms) * 8 + (in & 7);
        tn = (blk / bms) * 8 + (in >> 3);
    } else {
        tm = t % tiles_m;
        tn = t / tiles_m;
    }
}

// Tile order and k range of a product with triangular operands (tri flags):
// the tiles with the longest k range come first in the grid, so that the last
// wave of workgroups is short, and the range (whole BK slabs, kend at most K
// rounded up) leaves out the slabs in which the tile's rows of A or columns of
// B are all zero.  What is left out are products with zero: the sums are the
// same.
__device__ inline void tri_tiles(int tri, int tiles_m, int tiles_n, int &tm, int &tn) {
    if (tri & kTriALower) tm = tiles_m - 1 - tm;
    if (tri & kTriBUpper) tn = tiles_n - 1 - tn;
}
__device__ inline void tri_range(int tri, int m0, int bm, int n0, int bn, int bk, int K, int &kt0, int &kt1) {
    int lo = 0, hi = K;
    if (tri & kTriALower) hi = min(hi, m0 + bm);
    if (tri & kTriBUpper) hi = min(hi, n0 + bn);
    if (tri & kTriAUpper) lo = max(lo, m0);
    if (tri & kTriBLower) lo = max(lo, n0);
    kt0 = lo / bk;
    kt1 = max(kt0, (hi + bk - 1) / bk);
}

// Guarded path: every element loaded by itself, for products that have no
// vector of A to load (fewer rows than one, or an empty reduction).
template <int BM, int BN, int BK, int WM, int WN, typename T, int NG>
__global__ void __launch_bounds__(256) gemm_kernel(GroupArgs<NG> g) {
    constexpr int NT = 256;
    constexpr int WAVES_M = BM / WM;
    static_assert(WAVES_M * (BN / WN) == 4, "four waves per workgroup");
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int A_LD = BM + 1;  // LDS pitch of an A slab row (one k)
    constexpr int B_LD = BN + 1;  // LDS pitch of a B slab row (one k); +1 spreads banks
    constexpr int A_PT = BM * BK / NT;
    constexpr int B_PT = BN * BK / NT;
    static_assert(A_PT * NT == BM * BK && B_PT * NT == BN * BK, "tile/thread mismatch");
    using acc_t = typename Mma<T>::acc_t;

    __shared__ T As[2][BK * A_LD];
    __shared__ T Bs[2][BK * B_LD];

    const int bid = blockIdx.x;
    const int pi = group_member(g, bid);
    const GemmProb P = g.p[pi];
    const int tstart = g.tile_start[pi], tiles_m = g.tiles_m[pi];
    int tm, tn;
    tile_coords(bid - tstart, tstart, tiles_m, (P.n + BN - 1) / BN, P.lower != 0, tm, tn);

    const int tri = P.tri;
    if (tri) tri_tiles(tri, tiles_m, (P.n + BN - 1) / BN, tm, tn);
    const int M = P.m, N = P.n, K = P.k;
    const int m0 = tm * BM, n0 = tn * BN;
    const T *__restrict__ A = static_cast<const T *>(P.A);
    const T *__restrict__ B = static_cast<const T *>(P.B);
    const int64_t lda = P.lda, ldb = P.ldb;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave % WAVES_M) * WM, wn0 = (wave / WAVES_M) * WN;

    T ra[A_PT], rb[B_PT];
    auto gload = [&](int k0) {
#pragma unroll
        for (int i = 0; i < A_PT; ++i) {
            const int e = tid + NT * i, r = e % BM, c = e / BM;
            const bool ok = (m0 + r < M) && (k0 + c < K);
            ra[i] = ok ? A[(m0 + r) + (int64_t)(k0 + c) * lda] : T(0);
        }
#pragma unroll
        for (int i = 0; i < B_PT; ++i) {
            const int e = tid + NT * i, r = e % BK, c = e / BK;
            const bool ok = (k0 + r < K) && (n0 + c < N);
            rb[i] = ok ? B[(k0 + r) + (int64_t)(n0 + c) * ldb] : T(0);
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int i = 0; i < A_PT; ++i) {
            const int e = tid + NT * i, r = e % BM, c = e / BM;
            As[buf][c * A_LD + r] = ra[i];
        }
#pragma unroll
        for (int i = 0; i < B_PT; ++i) {
            const int e = tid + NT * i, r = e % BK, c = e / BK;
            Bs[buf][r * B_LD + c] = rb[i];
        }
    };

    acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

    int kt0 = 0, KT = (K + BK - 1) / BK;
    if (tri) tri_range(tri, m0, BM, n0, BN, BK, K, kt0, KT);
    if (KT > kt0) {
        gload(kt0 * BK);
        sstore(kt0 & 1);
    }
    __syncthreads();
    const int krow = lane >> 4, kcol = lane & 15;
    for (int kt = kt0; kt < KT; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < KT) gload((kt + 1) * BK);
#pragma unroll
        for (int kk = 0; kk < BK / 4; ++kk) {
            T a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = As[cur][(kk * 4 + krow) * A_LD + wm0 + i * 16 + kcol];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = Bs[cur][(kk * 4 + krow) * B_LD + wn0 + j * 16 + kcol];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = Mma<T>::mma(b[j], a[i], acc[i][j]);
        }
        if (kt + 1 < KT) sstore(cur ^ 1);
        __syncthreads();
    }

    // ---- epilogue: D = alpha * acc + beta * C0 (+ I) ------------------------
    const T *__restrict__ C0 = static_cast<const T *>(P.C0);
    T *D = static_cast<T *>(P.D);
    T *DT = static_cast<T *>(P.DT);
    const double alpha = P.alpha, beta = P.beta;
    const bool use_c = (beta != 0.0) && (C0 != nullptr);
    const bool add_i = P.add_identity != 0;
    const bool low = P.lower != 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int gm = m0 + wm0 + i * 16 + kcol;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gn = n0 + wn0 + j * 16 + Mma<T>::ncol(lane, v);
                if (gm < M && gn < N && !(low && gm < gn)) {
                    double val = alpha * (double)acc[i][j][v];
                    if (use_c) val += beta * (double)C0[gm + (int64_t)gn * P.ldc];
                    if (add_i && gm == gn) val += 1.0;
                    D[gm + (int64_t)gn * P.ldd] = (T)val;
                    if (DT != nullptr && !(low && gm == gn)) DT[gn + (int64_t)gm * P.lddt] = (T)val;
                }
            }
        }
    }
}

// Fast path.  The main loop has no control flow: the edge rows/columns of a
// tile are clamped once (what they load only reaches outputs the epilogue
// discards), each thread keeps one pointer per 16-byte global load and advances
// it by one slab per step.  RAG = false requires 16-byte aligned operands,
// leading dimensions and M that are multiples of the vector width and K a
// multiple of BK -- true for every block product of the recursion when the
// order is a multiple of 64.  RAG = true takes any operands with M at least
// the vector width: 16-byte loads at element alignment, a vector that reaches
// beyond row M - 1 loaded from row M - VW on and stored to LDS at those rows
// (its neighbours' entries, with the same values), and the last K mod BK
// columns as one more slab, loaded element by element with zeros beyond K.
// m = 1537, n = 1001, k = 777 in FP64: 113 us in the guarded kernel above,
// which loads single elements, 60 us here.
//
// The K slab is split into four contiguous chunks of KQ = BK/4 values, one per
// lane group q = lane/16, and MFMA step kk consumes k = q*KQ + kk in group q
// (any assignment of k to the four MFMA k-slots is valid as long as A and B
// agree).  B is staged k-contiguous (Bs[n][k]) so that a lane fetches its KQ
// B values with 16-byte LDS reads; A is staged m-contiguous (As[k][m]).
// NW waves per workgroup, two workgroups per CU: eight for the 128 x 128
// tile (64 x 32 each) and the 64 x 64 tile (32 x 16 each), four for the
// 32 x 32 tile.  Eight waves put four on each SIMD (two when a product
// leaves one workgroup per CU), so more of the slab loads and barriers hide
// behind other waves' matrix instructions.
//
// The 32 x 32 tile is taken where the tiles leave CUs idle, so nothing covers a
// slab's load: its loads are issued four slabs ahead from k = 256 on (FP64 256
// x 256 x 256 6.27 -> 6.11 us, 512^3 10.7 -> 10.1, 192 x 320 x 1024 17.4 ->
// 15.5, 640 x 512 x 2048 50.7 -> 46.5).  Shorter k gains nothing from loads in
// the loop that are not needed (k = 64 3.5 -> 3.7 us).  A wave's eight
// dependent 16 x 16 x 4 instructions per slab, 512 cycles, bound it then.  The
// 64 x 64 tile, often one workgroup on a CU, loads two slabs ahead from k = 128
// on in FP32, k = 512 in FP64, where it takes longer over a slab and 2688 x 336
// x 256 lost 1.3 % (FP32 1024^3 28.3 -> 25.4 us, 1024 x 960 x 2048 57.5 -> 49.9; FP64 47.4
// -> 46.8, 1280 x 1024 x 4096 278 -> 258); the 128 x 128 tile has no registers
// left for it.  The ragged forms of both tiles do the same and load the tail
// slab first, into registers of its own (FP64 1537 x 1001 x 777 63.8 -> 60.2 us,
// 333 x 200 x 1029 21.3 -> 17.4, 125^3 4.9 -> 4.7), and take only the tail's own
// steps (1777 x 1650 x 40 15.0 -> 13.0, 1537 x 1001 x 777 60.2 -> 58.7).
template <int BM, int BN, int BK, int WM, int WN, typename T, int NG, int NW, bool RAG>
__global__ void __launch_bounds__(64 * NW, NW / 2) gemm_fast(GroupArgs<NG> g) {
    constexpr int NT = 64 * NW;
    constexpr int VW = 16 / sizeof(T);
    typedef T vec_t __attribute__((ext_vector_type(VW)));
    typedef T uvec_t __attribute__((ext_vector_type(VW), aligned(sizeof(T))));
    using ld_t = std::conditional_t<RAG, uvec_t, vec_t>;  // global loads and A's LDS stores
    constexpr int WAVES_M = BM / WM;
    static_assert(WAVES_M * (BN / WN) == NW, "NW waves per workgroup");
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int KQ = BK / 4;
    static_assert(KQ % VW == 0, "lane chunk must be whole vectors");
    constexpr int A_LD = BM + VW;  // As[k][m]
    constexpr int B_LD = BK + VW;  // Bs[n][k]
    constexpr int AV = BM * BK / VW / NT;
    constexpr int BV = BN * BK / VW / NT;
    static_assert(AV * VW * NT == BM * BK && BV * VW * NT == BN * BK, "tile/thread mismatch");
    using acc_t = typename Mma<T>::acc_t;

    // a ragged tile with fewer than VW rows stores up to VW - 1 entries before
    // a slab row, into the padding of the row before it
    __shared__ __attribute__((aligned(16))) T As[2][BK * A_LD + (RAG ? VW : 0)];
    __shared__ __attribute__((aligned(16))) T Bs[2][BN * B_LD];

    const int bid = blockIdx.x;
    const int pi = group_member(g, bid);
    const GemmProb P = g.p[pi];
    const int tstart = g.tile_start[pi], tiles_m = g.tiles_m[pi];
    int tm, tn;
    tile_coords(bid - tstart, tstart, tiles_m, (P.n + BN - 1) / BN, P.lower != 0, tm, tn);
    const int tri = P.tri;
    if (tri) tri_tiles(tri, tiles_m, (P.n + BN - 1) / BN, tm, tn);
    const int M = P.m, N = P.n, K = P.k;
    const int m0 = tm * BM, n0 = tn * BN;
    const int64_t lda = P.lda, ldb = P.ldb;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave % WAVES_M) * WM, wn0 = (wave / WAVES_M) * WN;

    const T *pa[AV];
    int sa[AV];
#pragma unroll
    for (int i = 0; i < AV; ++i) {
        const int v = tid + NT * i, r = (v % (BM / VW)) * VW, c = v / (BM / VW);
        const int row = RAG ? min(m0 + r, M - VW) : m0 + r < M ? m0 + r : M - VW;
        pa[i] = static_cast<const T *>(P.A) + row + (int64_t)c * lda;
        sa[i] = RAG ? VW + c * A_LD + row - m0 : c * A_LD + r;
    }
    const T *pb[BV];
    int sb[BV];
#pragma unroll
    for (int i = 0; i < BV; ++i) {
        const int v = tid + NT * i, k = (v % (BK / VW)) * VW, n = v / (BK / VW);
        const int col = n0 + n < N ? n0 + n : N - 1;
        pb[i] = static_cast<const T *>(P.B) + k + (int64_t)col * ldb;
        sb[i] = n * B_LD + k;
    }
    const int64_t astep = (int64_t)BK * lda;

    constexpr int PF = BM == 32 ? 4 : BM == 64 ? 2 : 1;  // slabs loaded ahead
    constexpr int PFMIN = BM == 64 && sizeof(T) == 8 ? 16 : 2 * PF;  // of at least so many
    constexpr bool TAIL = RAG && PF > 1;                  // the tail slab has registers of its own
    vec_t ta[TAIL ? AV : 1], tb[TAIL ? BV : 1];
    vec_t ra[PF][AV], rb[PF][BV];
    // Rows of A beyond M and columns of B beyond N are loaded from clamped
    // (valid) addresses and not zeroed: they only reach accumulator rows and
    // columns that the epilogue discards, so the loaded values are consumed
    // by the LDS stores alone and the compute phase never waits on them.
    auto gload = [&](auto p, bool step = true) {
#pragma unroll
        for (int i = 0; i < AV; ++i) {
            ra[p][i] = *reinterpret_cast<const ld_t *>(pa[i]);
            pa[i] += step ? astep : 0;
        }
#pragma unroll
        for (int i = 0; i < BV; ++i) {
            rb[p][i] = *reinterpret_cast<const ld_t *>(pb[i]);
            pb[i] += step ? BK : 0;
        }
    };
    // the last KR = K mod BK columns of A and rows of B, zeros beyond
    const int KR = RAG ? K % BK : 0;
    auto gload_tail = [&](vec_t *xa, vec_t *xb, int slabs) {
#pragma unroll
        for (int i = 0; i < AV; ++i) {
            const int c = (tid + NT * i) / (BM / VW);
            const T *p = pa[i] + slabs * astep;
#pragma unroll
            for (int e = 0; e < VW; ++e) xa[i][e] = c < KR ? p[e] : T(0);
        }
#pragma unroll
        for (int i = 0; i < BV; ++i) {
            const int kb = ((tid + NT * i) % (BK / VW)) * VW;
            const T *p = pb[i] + slabs * BK;
#pragma unroll
            for (int e = 0; e < VW; ++e) xb[i][e] = kb + e < KR ? p[e] : T(0);
        }
    };
    constexpr std::integral_constant<int, 0> P0{};
    constexpr std::integral_constant<int, KQ> kAll{};
    auto put = [&](int buf, const vec_t *xa, const vec_t *xb) {
#pragma unroll
        for (int i = 0; i < AV; ++i) *reinterpret_cast<ld_t *>(&As[buf][sa[i]]) = xa[i];
#pragma unroll
        for (int i = 0; i < BV; ++i) *reinterpret_cast<vec_t *>(&Bs[buf][sb[i]]) = xb[i];
    };
    auto sstore = [&](int buf, auto p) { put(buf, ra[p], rb[p]); };

    acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

    const int q = lane >> 4, c16 = lane & 15;
    // B fragments are fetched one 16-byte vector (VW consecutive k) per
    // column block at a time, which bounds their registers to TN vectors.
    auto compute = [&](int buf, auto steps) {
        const T *as = &As[buf][(RAG ? VW : 0) + (q * KQ) * A_LD + wm0 + c16];
        const T *bs = &Bs[buf][(wn0 + c16) * B_LD + q * KQ];
#pragma unroll
        for (int kc = 0; kc < KQ / VW; ++kc) {
            if (kc * VW >= steps) break;
            vec_t bv[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j)
                bv[j] = *reinterpret_cast<const vec_t *>(bs + j * 16 * B_LD + kc * VW);
#pragma unroll
            for (int t = 0; t < VW; ++t) {
                const int kk = kc * VW + t;
                T a[TM];
#pragma unroll
                for (int i = 0; i < TM; ++i) a[i] = as[kk * A_LD + i * 16];
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = Mma<T>::mma(bv[j][t], a[i], acc[i][j]);
            }
        }
    };

    int KT = K / BK, kend = KT;
    if (tri) {
        int kt0;
        tri_range(tri, m0, BM, n0, BN, BK, K, kt0, kend);
        KT = max(kt0, min(KT, kend));
#pragma unroll
        for (int i = 0; i < AV; ++i) pa[i] += kt0 * astep;
#pragma unroll
        for (int i = 0; i < BV; ++i) pb[i] += kt0 * BK;
        KT -= kt0;
    }
    // a triangular k range that ends before K has no tail slab
    const bool tail = RAG && KR > 0 && (!tri || kend > K / BK);
    if constexpr (TAIL)
        if (tail) gload_tail(ta, tb, KT);
    if constexpr (RAG && !TAIL) {
        const int KS = KT + tail;
        auto next = [&](int kt) {
            if (kt < KT)
                gload(P0);
            else if (kt < KS)
                gload_tail(ra[0], rb[0], 0);
        };
        next(0);
        sstore(0, P0);
        __syncthreads();
        for (int kt = 0; kt < KS; ++kt) {
            next(kt + 1);
            compute(kt & 1, kAll);
            sstore((kt & 1) ^ 1, P0);
            __syncthreads();
        }
    } else if (KT > 0 && (PF == 1 || KT < PFMIN)) {
        gload(P0);
        sstore(0, P0);
        __syncthreads();
        for (int kt = 0; kt + 1 < KT; ++kt) {
            gload(P0);
            compute(kt & 1, kAll);
            sstore((kt & 1) ^ 1, P0);
            __syncthreads();
        }
        compute((KT - 1) & 1, kAll);
    } else if (KT > 0) {
        // Slab k lies in register set k mod PF.  Loads beyond the last slab
        // repeat it: with a condition around them the next store waits for the
        // newest loads too.
        static_for<PF>([&](auto p) { gload(p); });
        sstore(0, P0);
        __syncthreads();
        for (int k0 = 0; k0 < KT; k0 += PF) {
            static_for<PF>([&](auto p) {
                const int kt = k0 + p;
                if (kt < KT) {
                    gload(p, kt + PF + 1 < KT);
                    compute(kt & 1, kAll);
                    if (kt + 1 < KT) sstore((kt & 1) ^ 1, std::integral_constant<int, (p + 1) % PF>{});
                    __syncthreads();
                }
            });
        }
    }
    if constexpr (TAIL)
        if (tail) {
            // Column c lies where lane group c mod 4 finds it in step c / 4, so
            // that the steps beyond KR are left out.  That buffer was last read
            // two slabs ago, before a barrier.
            auto at = [](int c) { return (c & 3) * KQ + (c >> 2); };
#pragma unroll
            for (int i = 0; i < AV; ++i) {
                const int c = (tid + NT * i) / (BM / VW);
                *reinterpret_cast<ld_t *>(&As[KT & 1][sa[i] + (at(c) - c) * A_LD]) = ta[i];
            }
#pragma unroll
            for (int i = 0; i < BV; ++i) {
                const int kb = ((tid + NT * i) % (BK / VW)) * VW;
#pragma unroll
                for (int e = 0; e < VW; ++e) Bs[KT & 1][sb[i] - kb + at(kb + e)] = tb[i][e];
            }
            __syncthreads();
            compute(KT & 1, (KR + 3) / 4);
        }

    const T *__restrict__ C0 = static_cast<const T *>(P.C0);
    T *D = static_cast<T *>(P.D);
    T *DT = static_cast<T *>(P.DT);
    const double alpha = P.alpha, beta = P.beta;
    const bool use_c = (beta != 0.0) && (C0 != nullptr);
    const bool add_i = P.add_identity != 0;
    const bool low = P.lower != 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int gm = m0 + wm0 + i * 16 + c16;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gn = n0 + wn0 + j * 16 + Mma<T>::ncol(lane, v);
                if (gm < M && gn < N && !(low && gm < gn)) {
                    double val = alpha * (double)acc[i][j][v];
                    if (use_c) val += beta * (double)C0[gm + (int64_t)gn * P.ldc];
                    if (add_i && gm == gn) val += 1.0;
                    D[gm + (int64_t)gn * P.ldd] = (T)val;
                    if (DT != nullptr && !(low && gm == gn)) DT[gn + (int64_t)gm * P.lddt] = (T)val;
                }
            }
        }
    }
}

// ------------------------------------------------------------ BF16 path ---
// Products of FP32 matrices on the BF16 matrix cores with FP32 accumulation.
// v_mfma_f32_16x16x32_bf16: lane l supplies row l % 16 of an operand at
// k = 8*(l/16) .. 8*(l/16) + 7 and receives rows 4*(l/16) + v of the result
// (operands transposed as above, so the result block is D^T).  Operands are
// rounded to BF16 (round to nearest even) while they are staged into LDS,
// k-contiguous per m (A) or n (B) row so that each lane fetches its eight k
// with one 16-byte read (bf_slab).  X3 splits every operand into
// hi = bf16(x) and lo = bf16(x - hi) (x - hi is exact in FP32) and
// accumulates hi*hi + lo*hi + hi*lo, about 16 significant bits per operand
// (the lo*lo term, of relative size 2^-16, is dropped).
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));

// Element offset of 16-byte k chunk `chunk` (0 .. 3) of a slab's row.  Rows
// have a 64-byte pitch and 16 bytes more per four rows, and the chunks of a row
// an order of its quad's: the 16 lanes that a 16-byte read serves together
// ({0-3, 12-15, 20-23, 24-27} and so on) and stores to rows four apart then
// fall on different banks.  An 80-byte pitch had two lanes on each bank in
// every read: on the 128 x 128 tile 3000 x 3001 x 2000 takes 182 us instead of
// 194 as bf16x3 and 118 instead of 129 as BF16, order 2048 86 (90) and 64 (73).
__device__ inline int bf_slab(int row, int chunk) {
    const int q = row >> 2;
    return row * 32 + 8 * (q + (((chunk ^ -q) - q) & 3));
}
constexpr int bf_slab_size(int rows) { return rows * 32 + 2 * rows; }

template <int KN>
struct BfVec {
    typedef __bf16 type __attribute__((ext_vector_type(KN)));
};

template <int BM, int BN, int WM, int WN, bool X3, bool VEC, int NG, int NW = 4>
__global__ void __launch_bounds__(64 * NW, NW / 2) gemm_bf16(GroupArgs<NG> g) {
    constexpr int BK = 32;
    constexpr int NT = 64 * NW;
    constexpr int WAVES_M = BM / WM;
    static_assert(WAVES_M * (BN / WN) == NW, "NW waves per workgroup");
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int KPA = BM * BK / NT / 4;  // k per thread in the A slab (4 rows each)
    constexpr int TPC = NT / BN;           // threads per column of the B slab
    constexpr int KPB = BK / TPC;          // k per thread in the B slab
    constexpr int NP = X3 ? 2 : 1;         // hi (and lo) planes
    static_assert(KPA >= 1 && KPB % 4 == 0, "slab/thread mismatch");
    typedef typename BfVec<KPA>::type va_t;
    static_assert(BK == 32, "four 16-byte k chunks per row");

    __shared__ __attribute__((aligned(16))) __bf16 As[2][NP][bf_slab_size(BM)];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][NP][bf_slab_size(BN)];

    const int bid = blockIdx.x;
    const int pi = group_member(g, bid);
    const GemmProb P = g.p[pi];
    const int tstart = g.tile_start[pi], tiles_m = g.tiles_m[pi];
    int tm, tn;
    tile_coords(bid - tstart, tstart, tiles_m, (P.n + BN - 1) / BN, P.lower != 0, tm, tn);
    const int M = P.m, N = P.n, K = P.k;
    const int m0 = tm * BM, n0 = tn * BN;
    const float *__restrict__ A = static_cast<const float *>(P.A);
    const float *__restrict__ B = static_cast<const float *>(P.B);
    const int64_t lda = P.lda, ldb = P.ldb;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave % WAVES_M) * WM, wn0 = (wave / WAVES_M) * WN;

    // A slab: rows 4*mq .. 4*mq+3, k = kq*KPA .. kq*KPA + KPA-1
    const int mq = tid % (BM / 4), kq = tid / (BM / 4);
    const int am = m0 + 4 * mq;
    // B slab: column bn, k = bk .. bk + KPB-1
    const int bn = tid / TPC, bk = (tid % TPC) * KPB;
    const int bcol = n0 + bn;

    float ra[KPA][4], rb[KPB];
    auto gload = [&](int k0) {
#pragma unroll
        for (int j = 0; j < KPA; ++j) {
            const int k = k0 + kq * KPA + j;
            if (VEC) {
                const bool ok = am < M && k < K;
                const float4 x = *reinterpret_cast<const float4 *>(ok ? A + am + (int64_t)k * lda : A);
                ra[j][0] = ok ? x.x : 0.f;
                ra[j][1] = ok ? x.y : 0.f;
                ra[j][2] = ok ? x.z : 0.f;
                ra[j][3] = ok ? x.w : 0.f;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool ok = am + i < M && k < K;
                    const float x = *(ok ? A + am + i + (int64_t)k * lda : A);
                    ra[j][i] = ok ? x : 0.f;
                }
            }
        }
#pragma unroll
        for (int h = 0; h < KPB / 4; ++h) {
            const int k = k0 + bk + 4 * h;
            if (VEC) {
                const bool ok = bcol < N && k < K;
                const float4 x = *reinterpret_cast<const float4 *>(ok ? B + k + (int64_t)bcol * ldb : B);
                rb[4 * h + 0] = ok ? x.x : 0.f;
                rb[4 * h + 1] = ok ? x.y : 0.f;
                rb[4 * h + 2] = ok ? x.z : 0.f;
                rb[4 * h + 3] = ok ? x.w : 0.f;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool ok = bcol < N && k + i < K;
                    const float x = *(ok ? B + k + i + (int64_t)bcol * ldb : B);
                    rb[4 * h + i] = ok ? x : 0.f;
                }
            }
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            va_t hi, lo;
#pragma unroll
            for (int j = 0; j < KPA; ++j) {
                const __bf16 h = (__bf16)ra[j][i];
                hi[j] = h;
                if (X3) lo[j] = (__bf16)(ra[j][i] - (float)h);
            }
            const int k = kq * KPA, off = bf_slab(4 * mq, k >> 3) + BK * i + (k & 7);
            *reinterpret_cast<va_t *>(&As[buf][0][off]) = hi;
            if (X3) *reinterpret_cast<va_t *>(&As[buf][NP - 1][off]) = lo;
        }
        typedef __bf16 bc_t __attribute__((ext_vector_type(KPB < 8 ? KPB : 8)));
        constexpr int CW = KPB < 8 ? KPB : 8;  // elements per store
#pragma unroll
        for (int h0 = 0; h0 < KPB; h0 += CW) {
            bc_t hi, lo;
#pragma unroll
            for (int j = 0; j < CW; ++j) {
                const __bf16 h = (__bf16)rb[h0 + j];
                hi[j] = h;
                if (X3) lo[j] = (__bf16)(rb[h0 + j] - (float)h);
            }
            const int k = bk + h0;
            const int off = bf_slab(bn, k >> 3) + (k & 7);
            *reinterpret_cast<bc_t *>(&Bs[buf][0][off]) = hi;
            if (X3) *reinterpret_cast<bc_t *>(&Bs[buf][NP - 1][off]) = lo;
        }
    };

    f4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f4_t{0, 0, 0, 0};

    const int g4 = lane >> 4, c16 = lane & 15;
    const int oa = bf_slab(wm0 + c16, g4), ob = bf_slab(wn0 + c16, g4);
    constexpr int o16 = bf_slab_size(16);  // 16 rows on
    auto compute = [&](int buf) {
        bf8_t a[NP][TM], b[NP][TN];
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                a[pl][i] = *reinterpret_cast<const bf8_t *>(&As[buf][pl][oa + o16 * i]);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                b[pl][j] = *reinterpret_cast<const bf8_t *>(&Bs[buf][pl][ob + o16 * j]);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0][j], a[0][i], acc[i][j], 0, 0, 0);
                if (X3) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0][j], a[NP - 1][i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[NP - 1][j], a[0][i], acc[i][j], 0, 0, 0);
                }
            }
    };

    const int KT = (K + BK - 1) / BK;
    if (KT > 0) {
        gload(0);
        sstore(0);
        __syncthreads();
        for (int kt = 0; kt + 1 < KT; ++kt) {
            gload((kt + 1) * BK);
            compute(kt & 1);
            sstore((kt & 1) ^ 1);
            __syncthreads();
        }
        compute((KT - 1) & 1);
    }

    const float *__restrict__ C0 = static_cast<const float *>(P.C0);
    float *D = static_cast<float *>(P.D);
    float *DT = static_cast<float *>(P.DT);
    const double alpha = P.alpha, beta = P.beta;
    const bool use_c = (beta != 0.0) && (C0 != nullptr);
    const bool add_i = P.add_identity != 0;
    const bool low = P.lower != 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int gm = m0 + wm0 + i * 16 + c16;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gn = n0 + wn0 + j * 16 + 4 * g4 + v;
                if (gm < M && gn < N && !(low && gm < gn)) {
                    double val = alpha * (double)acc[i][j][v];
                    if (use_c) val += beta * (double)C0[gm + (int64_t)gn * P.ldc];
                    if (add_i && gm == gn) val += 1.0;
                    D[gm + (int64_t)gn * P.ldd] = (float)val;
                    if (DT != nullptr && !(low && gm == gn)) DT[gn + (int64_t)gm * P.lddt] = (float)val;
                }
            }
        }
    }
}

// Large products on the BF16 matrix cores: eight waves share a 256 x 256
// tile (128 x 64 per wave); 16-byte aligned rows of whole float4 vectors.  A 32-deep slab carries twice
// the flops per byte of FP32 operands loaded and per rounded operand that the
// 128 x 128 tile does.  Rounding and epilogue are gemm_bf16's.
//
// A CU holds one workgroup, so the waves cover their own latencies: the next
// slab is rounded and stored piece by piece between the matrix instructions of
// the current one, from registers loaded an iteration earlier.
//
// What bounds it: no single unit.  bf16x3 keeps the matrix cores busy for 52 %
// of the cycles and loses 9 % to LDS conflicts; with two waves on a SIMD and one
// barrier per slab, LDS reads and conversions are covered in part.  It issues 1 145
// TFLOP/s at 8192 x 8192 x 4096 (a library BF16 product of order 4096: 1 124).
// The 128 x 128 tile was bound by LDS: with an
// 80-byte pitch its reads took twice the cycles of its matrix instructions.
// bf16x3 4096^3 488 -> 357 us, 8192 x 8192 x 4096 1 897 -> 1 441 us; plain
// BF16 (the conversion of twice as many values per matrix instruction shows)
// 229 -> 209 and 996 -> 915 us against an 80-byte pitch with all conversions
// after the matrix instructions.
template <int BM, int BN, int WM, int WN, bool X3, int NG>
__global__ void __launch_bounds__(512, 1) gemm_bf16_big(GroupArgs<NG> g) {
    constexpr int BK = 32;
    constexpr int NT = 512;
    constexpr int WAVES_M = BM / WM;
    static_assert(WAVES_M * (BN / WN) == 8, "eight waves per workgroup");
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int KPA = BM * BK / NT / 4;  // k per thread in the A slab (4 rows each)
    constexpr int TPC = NT / BN;           // threads per column of the B slab
    constexpr int KPB = BK / TPC;          // k per thread in the B slab
    constexpr int NP = X3 ? 2 : 1;         // hi (and lo) planes
    static_assert(BM == 256 && KPA == 4 && KPB == 16 && TM == 8, "slab/thread mismatch");
    typedef typename BfVec<KPA>::type va_t;

    __shared__ __attribute__((aligned(16))) __bf16 As[2][NP][bf_slab_size(BM)];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][NP][bf_slab_size(BN)];

    const int bid = blockIdx.x;
    const int pi = group_member(g, bid);
    const GemmProb P = g.p[pi];
    const int tstart = g.tile_start[pi], tiles_m = g.tiles_m[pi];
    int tm, tn;
    tile_coords(bid - tstart, tstart, tiles_m, (P.n + BN - 1) / BN, false, tm, tn);
    const int M = P.m, N = P.n, K = P.k;
    const int m0 = tm * BM, n0 = tn * BN;
    const float *__restrict__ A = static_cast<const float *>(P.A);
    const float *__restrict__ B = static_cast<const float *>(P.B);
    const int64_t lda = P.lda, ldb = P.ldb;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave % WAVES_M) * WM, wn0 = (wave / WAVES_M) * WN;

    // A slab: rows 4*mq .. 4*mq+3, k = kq*KPA .. kq*KPA + KPA-1; a wave holds
    // 32 row quads of both halves of a chunk
    const int mq = (tid & 31) | ((tid >> 1) & 32), kq = ((tid >> 5) & 1) | ((tid >> 7) << 1);
    const int am = m0 + 4 * mq;
    // B slab: column bn, k = bk .. bk + KPB-1
    const int bn = tid / TPC, bk = (tid % TPC) * KPB;
    const int bcol = n0 + bn;

    float ra[KPA][4], rb[KPB];
    auto load_a = [&](int k0) {
#pragma unroll
        for (int j = 0; j < KPA; ++j) {
            const int k = k0 + kq * KPA + j;
            const bool ok = am < M && k < K;
            const float4 x = *reinterpret_cast<const float4 *>(ok ? A + am + (int64_t)k * lda : A);
            ra[j][0] = ok ? x.x : 0.f;
            ra[j][1] = ok ? x.y : 0.f;
            ra[j][2] = ok ? x.z : 0.f;
            ra[j][3] = ok ? x.w : 0.f;
        }
    };
    auto load_b = [&](int k0) {
#pragma unroll
        for (int h = 0; h < KPB / 4; ++h) {
            const int k = k0 + bk + 4 * h;
            const bool ok = bcol < N && k < K;
            const float4 x = *reinterpret_cast<const float4 *>(ok ? B + k + (int64_t)bcol * ldb : B);
            rb[4 * h + 0] = ok ? x.x : 0.f;
            rb[4 * h + 1] = ok ? x.y : 0.f;
            rb[4 * h + 2] = ok ? x.z : 0.f;
            rb[4 * h + 3] = ok ? x.w : 0.f;
        }
    };
    // row i of the thread's four, and its k chunk h
    auto store_a = [&](int buf, int i) {
        va_t hi, lo;
#pragma unroll
        for (int j = 0; j < KPA; ++j) {
            const __bf16 h = (__bf16)ra[j][i];
            hi[j] = h;
            if (X3) lo[j] = (__bf16)(ra[j][i] - (float)h);
        }
        const int off = bf_slab(4 * mq, kq >> 1) + BK * i + 4 * (kq & 1);
        *reinterpret_cast<va_t *>(&As[buf][0][off]) = hi;
        if (X3) *reinterpret_cast<va_t *>(&As[buf][NP - 1][off]) = lo;
    };
    auto store_b = [&](int buf, int h) {
        bf8_t hi, lo;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const __bf16 x = (__bf16)rb[8 * h + j];
            hi[j] = x;
            if (X3) lo[j] = (__bf16)(rb[8 * h + j] - (float)x);
        }
        const int off = bf_slab(bn, (bk >> 3) + h);
        *reinterpret_cast<bf8_t *>(&Bs[buf][0][off]) = hi;
        if (X3) *reinterpret_cast<bf8_t *>(&Bs[buf][NP - 1][off]) = lo;
    };

    f4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f4_t{0, 0, 0, 0};

    const int g4 = lane >> 4, c16 = lane & 15;
    const int oa = bf_slab(wm0 + c16, g4), ob = bf_slab(wn0 + c16, g4);
    constexpr int o16 = bf_slab_size(16);  // 16 rows on
    // Slab in buffer buf; more: the next slab goes to the other buffer and the
    // registers are loaded with the one at k2.
    auto compute = [&](int buf, auto more, int k2) {
        bf8_t b[NP][TN];
#pragma unroll
        for (int pl = 0; pl < NP; ++pl)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                b[pl][j] = *reinterpret_cast<const bf8_t *>(&Bs[buf][pl][ob + o16 * j]);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            bf8_t a[NP];
#pragma unroll
            for (int pl = 0; pl < NP; ++pl)
                a[pl] = *reinterpret_cast<const bf8_t *>(&As[buf][pl][oa + o16 * i]);
            if constexpr (more) {
                if (i == 1 || i == 2) store_b(buf ^ 1, i - 1);
                if (i == 3) load_b(k2);
                if (i >= 4) store_a(buf ^ 1, i - 4);
                if (i == TM - 1) load_a(k2);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0][j], a[0], acc[i][j], 0, 0, 0);
                if (X3) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0][j], a[NP - 1], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[NP - 1][j], a[0], acc[i][j], 0, 0, 0);
                }
            }
        }
    };

    const int KT = (K + BK - 1) / BK;
    if (KT > 0) {
        load_a(0);
        load_b(0);
#pragma unroll
        for (int i = 0; i < 4; ++i) store_a(0, i);
#pragma unroll
        for (int h = 0; h < 2; ++h) store_b(0, h);
        load_a(BK);
        load_b(BK);
        __syncthreads();
        for (int kt = 0; kt + 1 < KT; ++kt) {
            compute(kt & 1, std::true_type{}, (kt + 2) * BK);
            __syncthreads();
        }
        compute((KT - 1) & 1, std::false_type{}, 0);
    }

    const float *C0 = static_cast<const float *>(P.C0);
    float *D = static_cast<float *>(P.D);
    float *DT = static_cast<float *>(P.DT);
    const double alpha = P.alpha, beta = P.beta;
    const bool use_c = (beta != 0.0) && (C0 != nullptr);
    const bool add_i = P.add_identity != 0;
    // C0 comes two row blocks ahead of its use: with no second workgroup on the
    // CU nothing else covers the loads (C0 may be D, but an element is read and
    // written by the same lane).
    float cv[2][TN][4];
    const int gm0 = m0 + wm0 + c16, gn0 = n0 + wn0 + 4 * g4;
    const float *const cp = C0 + gm0 + (int64_t)gn0 * P.ldc;
    auto load_c = [&](int i, float (&x)[TN][4]) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const bool ok = gm0 + 16 * i < M && gn0 + 16 * j + v < N;
                x[j][v] = *(ok ? cp + 16 * i + (16 * j + v) * P.ldc : C0);
            }
    };
    if (use_c) {
        load_c(0, cv[0]);
        load_c(1, cv[1]);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int gm = m0 + wm0 + i * 16 + c16;
        float val[TN][4];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double x = alpha * (double)acc[i][j][v];
                if (use_c) x += beta * (double)cv[i & 1][j][v];
                if (add_i && gm == n0 + wn0 + j * 16 + 4 * g4 + v) x += 1.0;
                val[j][v] = (float)x;
            }
        if (use_c && i + 2 < TM) load_c(i + 2, cv[i & 1]);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gn = n0 + wn0 + j * 16 + 4 * g4 + v;
                if (gm < M && gn < N) {
                    D[gm + (int64_t)gn * P.ldd] = val[j][v];
                    if (DT != nullptr) DT[gn + (int64_t)gm * P.lddt] = val[j][v];
                }
            }
    }
}

// Tile prefix sums of up to N products for a BM x BN tiling; returns the
// number of workgroups.
template <int BM, int BN, int N>
int make_group(const GemmProb *probs, int count, GroupArgs<N> &g) {
    g = GroupArgs<N>{};
    g.count = count;
    int total = 0;
    for (int q = 0; q < N; ++q) {
        if (q < count) {
            g.p[q] = probs[q];
            const int tm = (probs[q].m + BM - 1) / BM, tn = (probs[q].n + BN - 1) / BN;
            // lower-triangle mode needs a square problem on a square tile grid
            const bool low = probs[q].lower && probs[q].m == probs[q].n && BM == BN;
            g.p[q].lower = low ? 1 : 0;
            g.tile_start[q] = total;
            g.tiles_m[q] = tm > 0 ? tm : 1;
            total += low ? tm * (tm + 1) / 2 : tm * tn;
        } else {
            g.p[q] = probs[0];
            g.tile_start[q] = 1 << 30;
            g.tiles_m[q] = 1;
        }
    }
    g.tile_start[N] = total;
    return total;
}

// One launch of up to N products that share a kernel configuration.
template <int BM, int BN, int BK, int WM, int WN, typename T, int N, int NW, bool RAG>
hipError_t launch_fast(const GemmProb *probs, int count, hipStream_t s) {
    GroupArgs<N> g;
    const int total = make_group<BM, BN, N>(probs, count, g);
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL((gemm_fast<BM, BN, BK, WM, WN, T, N, NW, RAG>), dim3(total), dim3(64 * NW), 0, s, g);
    return hipGetLastError();
}

template <typename T, int N>
hipError_t launch_edge(const GemmProb *probs, int count, hipStream_t s) {
    GroupArgs<N> g;
    const int total = make_group<32, 32, N>(probs, count, g);
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL((gemm_kernel<32, 32, 32, 16, 16, T, N>), dim3(total), dim3(256), 0, s, g);
    return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, bool X3, bool VEC, int N, int NW = 4>
hipError_t launch_bf16_group(const GemmProb *probs, int count, hipStream_t s) {
    GroupArgs<N> g;
    const int total = make_group<BM, BN, N>(probs, count, g);
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL((gemm_bf16<BM, BN, WM, WN, X3, VEC, N, NW>), dim3(total), dim3(64 * NW), 0, s, g);
    return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, bool X3, int N>
hipError_t launch_bf16_big_group(const GemmProb *probs, int count, hipStream_t s) {
    GroupArgs<N> g;
    const int total = make_group<BM, BN, N>(probs, count, g);
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL((gemm_bf16_big<BM, BN, WM, WN, X3, N>), dim3(total), dim3(512), 0, s, g);
    return hipGetLastError();
}

// K slab of the fast 128x128 kernel (FP64: 16 keeps two workgroups per CU;
// FP32: 32).  Every other fast configuration uses 32.
constexpr int kFastBK128 = 16;
constexpr int fast_bk(int tile, int es) { return (tile == 128 && es == 8) ? kFastBK128 : 32; }

// Kernel configuration of one product, a function of that product alone (its
// shape, leading dimensions and alignment), so that a product is computed
// bit for bit the same whether it is launched alone or grouped with others.
enum Path { kEdge = 0, kFast = 1, kRagged = 2 };
struct Cfg {
    int tile;   // 128, 64 or 32; 256 for the eight-wave BF16 tiles
    Path path;  // guarded, branch-free vector, vector with ragged edges
    bool operator==(const Cfg &o) const { return tile == o.tile && path == o.path; }
};

Cfg choose_cfg(const GemmProb &p, DType dt) {
    const int es = dt == kF64 ? 8 : 4;
    const int vw = 16 / es;
    // a lower-triangle problem runs only the T (T + 1) / 2 tiles on or below
    // the diagonal, so that is the count that has to fill the GPU
    const bool low = p.lower && p.m == p.n;
    auto count = [&](int64_t t) {
        const int64_t tm = (p.m + t - 1) / t, tn = (p.n + t - 1) / t;
        return low ? tm * (tm + 1) / 2 : tm * tn;
    };
    const int64_t t128 = count(128);
    const int64_t t64 = count(64);
    Cfg c;
    c.tile = (t128 >= 192) ? 128 : (t64 >= 128) ? 64 : 32;
    const bool aligned =
        ((reinterpret_cast<uintptr_t>(p.A) | reinterpret_cast<uintptr_t>(p.B)) & 15) == 0;
    if (dt == kBF16 || dt == kBF16X3) {
        // float4 loads along m (A) and along k (B)
        c.path = p.m % 4 == 0 && p.k % 4 == 0 && p.lda % 4 == 0 && p.ldb % 4 == 0 && aligned ? kFast : kEdge;
        // Eight-wave 256 x 256 tiles, one workgroup per CU, against 128 x 128
        // tiles, three per CU (without / with C0, us, 128 -> 256 tiles); not
        // for the lower-triangle mode.
        // bf16x3: where they fill at least 5/8 of their rounds over the 256
        // CUs and k covers the longer prologue: 2560 x 4096 x 512 (160 tiles)
        // 53 -> 51 / 67 -> 56; 4096^3 467 -> 340 / 478 -> 349; below the line
        // 4100 x 4092 x 516 (272) 109 -> 115, 2560 x 4096 x 128 23.7 -> 25.9.
        // With a last round up to half empty the line is k = 1024: 6144 x 6144
        // (576 tiles) k = 512 146 -> 154 / 213 -> 198, 1024 level / 332 -> 312.
        // Plain BF16: from 256 tiles on for every k (4352^3 428 -> 400, 4096 x
        // 4096 x 64 level); with fewer where the 128 x 128 tiles no longer fit
        // one round of 768 (3584 x 3584 x 512, 784 of them, 48 -> 36 / 67 -> 44;
        // but 3072 x 4096 x 768, 768 of them, 46 -> 50), and from k = 4096 on,
        // level at worst (2560 x 4096 205 -> 186 / 214 -> 190, 2048 x 5120 193
        // -> 194 / 201 -> 200; 1024 x 12288 250 -> 259 with C0, so not for
        // fewer rows).
        const int64_t big = (int64_t)((p.m + 255) / 256) * ((p.n + 255) / 256);
        const int64_t rounds = (big + 255) / 256;
        const bool filled = 8 * big >= 5 * 256 * rounds;
        const bool sparse = rounds > 1 && 4 * big <= 3 * 256 * rounds;
        const bool wide = dt == kBF16X3 ? filled && p.k >= (sparse ? 1024 : 512)
                                        : big >= 256 || (t128 > 768 && p.k >= 512) ||
                                              (filled && p.k >= 4096 && p.m >= 2048);
        if (c.path == kFast && !p.lower && wide) c.tile = 256;
        return c;
    }
    const int bk = fast_bk(c.tile, es);
    if (p.k <= 0 || p.m < vw) {
        // no vector of A to load (an empty reduction, one to three rows)
        c.path = kEdge;
        c.tile = 32;
    } else {
        c.path = p.k % bk == 0 && p.m % vw == 0 && p.lda % vw == 0 && p.ldb % vw == 0 && aligned ? kFast : kRagged;
        // A short k leaves the epilogue as most of the work, and two 128 x 128
        // workgroups on a CU cover less of it than the 64 x 64 tile's more and
        // smaller ones (the same bits), at any rate when their last round is
        // nearly empty.  FP32 with C0, 128 -> 64 tiles: 3001 x 3001 x 16 46 ->
        // 29 us, 3201 x 3201 x 130 72.6 -> 49.1; where neither holds 4095 x
        // 4095 x 130 without C0 57.4 -> 59.8.
        const int64_t rounds = (t128 + 511) / 512;
        if (c.path == kRagged && dt == kF32 && c.tile == 128 &&
            (p.k <= 96 || (p.k <= 192 && 8 * t128 < 7 * 512 * rounds)))
            c.tile = 64;
    }
    return c;
}

template <typename T, int N, bool RAG>
hipError_t launch_tile(int tile, const GemmProb *probs, int count, hipStream_t s) {
    constexpr int ES = sizeof(T);
    if (tile == 128) return launch_fast<128, 128, fast_bk(128, ES), 64, 32, T, N, 8, RAG>(probs, count, s);
    if (tile == 64) return launch_fast<64, 64, fast_bk(64, ES), 32, 16, T, N, 8, RAG>(probs, count, s);
    return launch_fast<32, 32, fast_bk(32, ES), 16, 16, T, N, 4, RAG>(probs, count, s);
}

template <typename T, int N>
hipError_t launch_cfg(Cfg c, const GemmProb *probs, int count, hipStream_t s) {
    if (c.path == kEdge) return launch_edge<T, N>(probs, count, s);
    return c.path == kFast ? launch_tile<T, N, false>(c.tile, probs, count, s)
                           : launch_tile<T, N, true>(c.tile, probs, count, s);
}

template <bool X3, int N>
hipError_t launch_cfg_bf16(Cfg c, const GemmProb *probs, int count, hipStream_t s) {
    if (c.tile == 256) return launch_bf16_big_group<256, 256, 128, 64, X3, N>(probs, count, s);
    if (c.tile == 128)
        return c.path == kFast ? launch_bf16_group<128, 128, 64, 32, X3, true, N, 8>(probs, count, s)
                      : launch_bf16_group<128, 128, 64, 64, X3, false, N>(probs, count, s);
    if (c.tile == 64)
        return c.path == kFast ? launch_bf16_group<64, 64, 32, 32, X3, true, N>(probs, count, s)
                      : launch_bf16_group<64, 64, 32, 32, X3, false, N>(probs, count, s);
    return c.path == kFast ? launch_bf16_group<32, 32, 16, 16, X3, true, N>(probs, count, s)
                  : launch_bf16_group<32, 32, 16, 16, X3, false, N>(probs, count, s);
}

const char *cfg_name(Cfg c, DType dt) {
    static const char *names[4][3][3] = {
        {{"", "gemm_f64_128x128", "gemm_f64_128x128_ragged"},
         {"", "gemm_f64_64x64", "gemm_f64_64x64_ragged"},
         {"gemm_f64_32x32_edge", "gemm_f64_32x32", "gemm_f64_32x32_ragged"}},
        {{"", "gemm_f32_128x128", "gemm_f32_128x128_ragged"},
         {"", "gemm_f32_64x64", "gemm_f32_64x64_ragged"},
         {"gemm_f32_32x32_edge", "gemm_f32_32x32", "gemm_f32_32x32_ragged"}},
        {{"gemm_bf16_128x128_edge", "gemm_bf16_128x128", ""},
         {"gemm_bf16_64x64_edge", "gemm_bf16_64x64", ""},
         {"gemm_bf16_32x32_edge", "gemm_bf16_32x32", ""}},
        {{"gemm_bf16x3_128x128_edge", "gemm_bf16x3_128x128", ""},
         {"gemm_bf16x3_64x64_edge", "gemm_bf16x3_64x64", ""},
         {"gemm_bf16x3_32x32_edge", "gemm_bf16x3_32x32", ""}}};
    if (c.tile == 256) return dt == kBF16 ? "gemm_bf16_256x256" : "gemm_bf16x3_256x256";
    const int ti = c.tile == 128 ? 0 : c.tile == 64 ? 1 : 2;
    return names[(int)dt][ti][(int)c.path];
}

}  // namespace

hipError_t gemm_launch(const GemmProb *probs, int count, DType dt, hipStream_t s, LaunchInfo *info) {
    if (count < 1 || count > kMaxBatch) return hipErrorInvalidValue;
    if (dt != kF64 && dt != kF32 && dt != kBF16 && dt != kBF16X3) return hipErrorInvalidValue;
    const int esz = (dt == kF64) ? 8 : 4;
    const double es = esz;
    // Products with an empty reduction still need their epilogue; drop only
    // products with an empty output.  Group the rest by configuration.
    GemmProb part[kMaxBatch];
    Cfg cfgs[kMaxBatch];
    bool done[kMaxBatch];
    int n_live = 0;
    double flops = 0, bytes = 0;
    // the mirror form (DT == D) relies on the lower-triangle mode, which every
    // tile shape honours for a square problem
    for (int q = 0; q < count; ++q)
        if (probs[q].DT != nullptr && probs[q].DT == probs[q].D &&
            !(probs[q].lower && probs[q].m == probs[q].n))
            return hipErrorInvalidValue;
    for (int q = 0; q < count; ++q) {
        if (probs[q].m <= 0 || probs[q].n <= 0) continue;
        part[n_live] = probs[q];
        cfgs[n_live] = choose_cfg(probs[q], dt);
        done[n_live] = false;
        ++n_live;
        const double m = probs[q].m, n = probs[q].n, k = probs[q].k;
        // a lower-triangle product computes about m (m + tile) / 2 outputs
        flops += (probs[q].lower && probs[q].m == probs[q].n) ? k * m * (m + cfgs[n_live - 1].tile)
                                                               : product_flops(probs[q].m, probs[q].n, probs[q].k, probs[q].tri);
        bytes += es * (m * k + k * n + m * n + ((probs[q].beta != 0.0) ? m * n : 0.0));
        if (probs[q].DT != nullptr) bytes += es * m * n * (probs[q].lower ? 0.5 : 1.0);
    }
    const char *name = "gemm_empty";
    hipError_t e = hipSuccess;
    for (int q = 0; q < n_live && e == hipSuccess; ++q) {
        if (done[q]) continue;
        GemmProb grp[kMaxBatch];
        int ng = 0;
        for (int r = q; r < n_live; ++r)
            if (!done[r] && cfgs[r] == cfgs[q]) {
                grp[ng++] = part[r];
                done[r] = true;
            }
        name = cfg_name(cfgs[q], dt);
        if (dt == kF64)
            e = (ng <= 2) ? launch_cfg<double, 2>(cfgs[q], grp, ng, s)
                          : launch_cfg<double, kMaxBatch>(cfgs[q], grp, ng, s);
        else if (dt == kF32)
            e = (ng <= 2) ? launch_cfg<float, 2>(cfgs[q], grp, ng, s)
                          : launch_cfg<float, kMaxBatch>(cfgs[q], grp, ng, s);
        else if (dt == kBF16)
            e = (ng <= 2) ? launch_cfg_bf16<false, 2>(cfgs[q], grp, ng, s)
                          : launch_cfg_bf16<false, kMaxBatch>(cfgs[q], grp, ng, s);
        else
            e = (ng <= 2) ? launch_cfg_bf16<true, 2>(cfgs[q], grp, ng, s)
                          : launch_cfg_bf16<true, kMaxBatch>(cfgs[q], grp, ng, s);
    }
    if (info) {
        info->name = name;
        info->flops = flops;
        info->bytes = bytes;
    }
    return e;
}

}  // namespace spin
