// FP64-accurate block products on INT8 matrix cores, for the Newton
// refinement's residual R = I - A X and update X + X R (Newton iteration as
// the stabiliser of Strassen inversion, Sec. 2.1).
//
// The emulation is the integer modular scheme of Ozaki, Uchino and Imamura
// (Ozaki scheme II, 2025) on the error-free splitting of Ozaki, Ogita, Oishi
// and Rump (2012):
//   1. split: row i of the left operand is scaled by 2^s_i and rounded to the
//      nearest integer (ties to even), column j of the right operand by 2^t_j,
//      with s_i = beta - E_i for a row maximum f 2^E_i, f in [1/2, 1), so that
//      no integer exceeds 2^beta; for each modulus m_l (pairwise coprime, at
//      most 256) the symmetric residue of every integer is stored as an int8,
//      K-contiguous per row (left) or per column (right), zero padded;
//   2. product: for each modulus, the INT8 matrix-core product of the residue
//      matrices is exact in int32 (|sum| <= k 128^2 < 2^31); it is reduced
//      into [0, m_l) and stored as one byte per element;
//   3. reconstruction: P = sum_l r_l w_l mod M (M the product of the moduli,
//      w_l its Chinese-remainder weights) in 128-bit integers is the exact
//      integer product A' B' once 2 k 2^(beta_a + beta_b) < M; P is taken
//      symmetric, rounded once to FP64 (nearest, ties to even), scaled by
//      2^-(s_i + t_j), and the epilogue (I - D, or C0 + D) rounds once more.
// A row of the left operand or a column of the right one that holds a
// non-finite value gives NaN in its row or column of the result.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <climits>
#include <cmath>
#include <cstdint>

#include "spin_kernels.hpp"

namespace spin {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned __int128 u128;

// Pairwise coprime moduli, largest first; the first n are used.
constexpr int kModuli[kOzakiMaxModuli] = {256, 255, 253, 251, 247, 241, 239, 233,
                                          229, 227, 223, 217, 211, 199, 197};

constexpr int kLimbs = 6;  // 20-bit limbs of a Chinese-remainder weight (< 2^118)

struct ModArgs {
    int count;
    int m[kOzakiMaxModuli];
    float inv[kOzakiMaxModuli];                                    // 1 / m_l
    unsigned magic[kOzakiMaxModuli];                               // floor(2^32 / m_l)
    unsigned bias[kOzakiMaxModuli];                                // least multiple of m_l >= 2^31
    unsigned pow_lo[kOzakiMaxModuli], pow_hi[kOzakiMaxModuli];     // bytes 2^(8 j) mod m_l, j = 0..3 and 4..7
    unsigned w[kOzakiMaxModuli][kLimbs];                           // weights in 20-bit limbs
    unsigned long long M_lo, M_hi;                                 // product of the moduli
    double invM;                                                   // 1 / M (approximate)
};

constexpr unsigned long long kNonFinite = 0x7ff0000000000000ull;  // |x| bits at or above: Inf / NaN
constexpr int kBadShift = INT_MIN;                                 // shift of a non-finite row

// ------------------------------------------------------------ row maxima ---
// rmax[i] = max over the row's |a| as IEEE bits (ordered like the values for
// non-negative doubles; Inf and NaN compare above every finite value).
__global__ void __launch_bounds__(256) k_rowmax(const double *__restrict__ a, int64_t lda, int m,
                                                 int k, int kchunk, unsigned long long *rmax) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    const int k0 = blockIdx.y * kchunk, k1 = min(k, k0 + kchunk);
    unsigned long long mx = 0;
    for (int q = k0; q < k1; ++q) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(a[i + (int64_t)q * lda]) &
                                     0x7fffffffffffffffull;
        mx = b > mx ? b : mx;
    }
    if (mx) atomicMax(rmax + i, mx);
}

// cmax[j] for a column-major (k x n) view: one workgroup per column.
__global__ void __launch_bounds__(256) k_colmax(const double *__restrict__ b, int64_t ldb, int k,
                                                 unsigned long long *cmax) {
    __shared__ unsigned long long red[256];
    const int j = blockIdx.x;
    unsigned long long mx = 0;
    for (int q = threadIdx.x; q < k; q += 256) {
        const unsigned long long v = (unsigned long long)__double_as_longlong(b[q + (int64_t)j * ldb]) &
                                     0x7fffffffffffffffull;
        mx = v > mx ? v : mx;
    }
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = max(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) cmax[j] = red[0];
}

__global__ void k_zero_u64(unsigned long long *p, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}

// The shift of a row or column whose largest magnitude has the bits b, max =
// f 2^E with f in [1/2, 1): beta - E; 0 for a zero maximum; kBadShift for a
// non-finite one.
__device__ inline int shift_of(unsigned long long b, int beta) {
    if (b >= kNonFinite) return kBadShift;
    if (b == 0) return 0;
    int e;
    (void)frexp(__longlong_as_double((long long)b), &e);
    return beta - e;
}

// The magnitude of the scaled, rounded integer of x under shift s (0 for a
// non-finite row) as 64 bits, and the sign of its residues.
struct Split {
    unsigned lo, hi;
    float sign;
};
__device__ inline Split split_value(double x, int s) {
    const double v = s == kBadShift ? 0.0 : rint(ldexp(x, s));  // |v| <= 2^53
    const double a = fabs(v);
    Split r;
    r.hi = (unsigned)(a * 0x1p-32);
    r.lo = (unsigned)fma((double)r.hi, -0x1p32, a);
    r.sign = v < 0.0 ? -1.0f : 1.0f;
    return r;
}

// Residues modulo m_l of four split integers, packed as signed bytes.  Any
// residue in -128 .. 127 serves, since the products are reduced again.  With
// c_j = 2^(8 j) mod m the byte sum sum_j byte_j c_j (two four-byte dot
// products) is below 2^19 and congruent to the integer; from there FP32 is
// exact but for the rounded quotient, whose error (2^-11) leaves the residue
// within m / 2 + 1/8.  The bytes are packed as r + 128.
__device__ inline unsigned pack_residues(const Split *v, int l, const ModArgs &md) {
    unsigned w = 0;
    if (l == 0) {
        // m_0 = 256: the low byte of the signed integer
#pragma unroll
        for (int u = 0; u < 4; ++u)
            w |= ((v[u].sign < 0.0f ? 0u - v[u].lo : v[u].lo) & 0xffu) << (8 * u);
        return w;
    }
    const float m = (float)md.m[l], inv = md.inv[l];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        unsigned d = __builtin_amdgcn_udot4(v[u].lo, md.pow_lo[l], 0u, false);
        d = __builtin_amdgcn_udot4(v[u].hi, md.pow_hi[l], d, false);
        const float f = (float)d;
        const float r = fmaf(-rintf(f * inv), m, f);
        w = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(r, v[u].sign, 128.0f), u, w);
    }
    return w ^ 0x80808080u;
}

// Left operand: residue planes with rows K-contiguous, plane[l][i * kp + q].
// A thread takes 16 consecutive k of one row (lanes are consecutive rows, so
// its loads coalesce) and stores 16 bytes per modulus; the four waves of a
// workgroup complete each row's 64-byte segment.  Bound by the conversion
// (about 140 instructions per element) and the stores: order 4096 with 14
// moduli 188 -> 147 us against the FP64 residues of an LDS-transposed tile.
__global__ void __launch_bounds__(256) k_split_rows(const double *__restrict__ a, int64_t lda, int m, int k,
                                                    const unsigned long long *__restrict__ mx, int beta,
                                                    int8_t *planes, int64_t mp, int kp, ModArgs md) {
    const int i = blockIdx.x * 64 + (threadIdx.x & 63), q0 = blockIdx.y * 64 + (threadIdx.x >> 6) * 16;
    const int s = i < m ? shift_of(mx[i], beta) : 0;
    Split v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int q = q0 + u;
        v[u] = split_value((i < m && q < k) ? a[i + (int64_t)q * lda] : 0.0, s);
    }
    int8_t *dst = planes + (int64_t)i * kp + q0;
#pragma unroll 2
    for (int l = 0; l < md.count; ++l) {
        v4i w;
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = (int)pack_residues(v + 4 * u, l, md);
        *reinterpret_cast<v4i *>(dst + (int64_t)l * mp * kp) = w;
    }
}

// Right operand: residue planes with columns K-contiguous, plane[l][j * kp +
// q] (the operand's own order).  Thread: four k of one column, so that loads
// (32 bytes a lane) and stores (4 bytes) of a wave are contiguous: order 4096
// with 14 moduli 302 -> 108 us against 16 k per thread with FP64 residues.
__global__ void __launch_bounds__(256) k_split_cols(const double *__restrict__ b, int64_t ldb, int k, int n,
                                                    const unsigned long long *__restrict__ mx, int beta,
                                                    int8_t *planes, int64_t np_, int kp, ModArgs md) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int chunks = kp / 4;
    if (e >= (int64_t)np_ * chunks) return;
    const int j = (int)(e / chunks), q0 = (int)(e % chunks) * 4;
    const int s = j < n ? shift_of(mx[j], beta) : 0;
    Split v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int q = q0 + u;
        v[u] = split_value((j < n && q < k) ? b[q + (int64_t)j * ldb] : 0.0, s);
    }
    int8_t *dst = planes + (int64_t)j * kp + q0;
#pragma unroll 2
    for (int l = 0; l < md.count; ++l)
        *reinterpret_cast<unsigned *>(dst + (int64_t)l * np_ * kp) = pack_residues(v, l, md);
}

// The sum s of a residue product reduced into [0, m): with u = s + bias in [0,
// 2^32), floor(u floor(2^32 / m) / 2^32) is floor(u / m) or one less.
__device__ inline unsigned reduce_sum(int s, int m, unsigned bias, unsigned magic) {
    const unsigned u = (unsigned)s + bias;
    const unsigned r = u - __umulhi(u, magic) * (unsigned)m;
    return min(r, r - (unsigned)m);
}

// ------------------------------------------------------------ INT8 GEMM ---
// For modulus l = blockIdx.z: C_l = A_l B_l over the residue planes, a 128 x
// 128 tile per workgroup (four waves of 64 x 64, 4 x 4 blocks of
// v_mfma_i32_16x16x64_i8), K in 64-byte slabs staged through LDS (two
// buffers, one barrier per slab).  Output bytes (the sums reduced into
// [0, m_l)) go to cplanes[l][i + j * mp], four consecutive rows per lane.
constexpr int kTB = 128, kSK = 64, kPitch = 80;  // LDS row pitch; two lanes share a bank in fragment reads

__global__ void __launch_bounds__(256, 2) k_gemm_i8(const int8_t *__restrict__ ap, const int8_t *__restrict__ bp,
                                                     uint8_t *__restrict__ cp, int m, int n, int64_t mp,
                                                     int64_t np_, int kp, ModArgs md) {
    __shared__ __attribute__((aligned(16))) int8_t As[2][kTB * kPitch];
    __shared__ __attribute__((aligned(16))) int8_t Bs[2][kTB * kPitch];
    const int l = blockIdx.z;
    const int i0 = blockIdx.x * kTB, j0 = blockIdx.y * kTB;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int wm = (w & 1) * 64, wn = (w >> 1) * 64;
    const int8_t *A = ap + (int64_t)l * mp * kp + (int64_t)i0 * kp;
    const int8_t *B = bp + (int64_t)l * np_ * kp + (int64_t)j0 * kp;
    // slab loads: chunk c (of 512) = row c / 4, 16-byte piece c % 4
    const int r0 = t >> 2, r1 = (t + 256) >> 2, pc = (t & 3) * 16;
    v4i ra0, ra1, rb0, rb1;
    auto load = [&](int q0) {
        ra0 = *reinterpret_cast<const v4i *>(A + (int64_t)r0 * kp + q0 + pc);
        ra1 = *reinterpret_cast<const v4i *>(A + (int64_t)r1 * kp + q0 + pc);
        rb0 = *reinterpret_cast<const v4i *>(B + (int64_t)r0 * kp + q0 + pc);
        rb1 = *reinterpret_cast<const v4i *>(B + (int64_t)r1 * kp + q0 + pc);
    };
    auto store = [&](int buf) {
        *reinterpret_cast<v4i *>(&As[buf][r0 * kPitch + pc]) = ra0;
        *reinterpret_cast<v4i *>(&As[buf][r1 * kPitch + pc]) = ra1;
        *reinterpret_cast<v4i *>(&Bs[buf][r0 * kPitch + pc]) = rb0;
        *reinterpret_cast<v4i *>(&Bs[buf][r1 * kPitch + pc]) = rb1;
    };
    v4i acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = v4i{0, 0, 0, 0};
    const int nk = kp / kSK;
    load(0);
    store(0);
    __syncthreads();
    const int fr = lane & 15, fk = (lane >> 4) * 16;
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load((kt + 1) * kSK);
        v4i fa[4], fb[4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
            fa[a] = *reinterpret_cast<const v4i *>(&As[buf][(wm + 16 * a + fr) * kPitch + fk]);
#pragma unroll
        for (int b = 0; b < 4; ++b)
            fb[b] = *reinterpret_cast<const v4i *>(&Bs[buf][(wn + 16 * b + fr) * kPitch + fk]);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[a], fb[b], acc[a][b], 0, 0, 0);
        if (kt + 1 < nk) store(buf ^ 1);
        __syncthreads();
    }
    // lane holds rows 4 (lane / 16) + v, v = 0..3, of column lane % 16 of each block
    const int mod = md.m[l];
    uint8_t *C = cp + (int64_t)l * mp * np_;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int i = i0 + wm + 16 * a + 4 * (lane >> 4);
            const int j = j0 + wn + 16 * b + (lane & 15);
            if (j >= n || i >= m) continue;
            unsigned int packed = 0;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                packed |= reduce_sum(acc[a][b][v], mod, md.bias[l], md.magic[l]) << (8 * v);
            *reinterpret_cast<unsigned int *>(C + i + (int64_t)j * mp) = packed;
        }
}

// The same product with 256 x 256 tiles: eight waves, each 128 x 64 (8 x 4
// blocks), twice the integer operations per byte of residues moved, for the
// large products of the refinement.  Residue planes padded to 256 rows.
//
// At the matrix cores' rate a 64-byte slab of a tile takes 1024 cycles; its
// fragments read 96 KB and its operands fill 32 KB of LDS, which is what LDS
// passes in that time, so nothing else may: the operands go from memory to LDS
// directly (global_load_lds), without registers, three slabs ahead in four
// buffers, with one wait for the oldest slab and one barrier per slab.  A row
// of a buffer is 64 bytes without padding; its 16-byte pieces are stored in
// the order piece ^ (-(row / 4) mod 4): each four cycles of a fragment read
// (16 bytes of 16 lanes a cycle; lanes 0-3, 12-15, 20-23, 24-27 share one, or
// 16 consecutive lanes) then touch every bank once.  With piece ^ (row / 4)
// half of the LDS cycles were bank conflicts.  Tiles go to the XCDs in groups of four tile
// rows (each XCD's L2 then sees a 4 x 8 patch of a 16 x 16 grid).  14 moduli,
// against register staging one slab ahead: order 4096 1.22 -> 0.97 ms, order
// 8192 8.0 -> 6.2 ms (2490 TOP/s, matrix cores busy 60 % at 2.0 GHz).  One
// barrier per two slabs was slower (6.8 ms at 8192), and so was issuing the
// next slab before the first matrix instructions (6.3 ms).
constexpr int kTB2 = 256, kStages = 4, kStageB = 2 * kTB2 * kSK;

// 64 lanes x 16 bytes from base + voff (per lane) to LDS byte address lds +
// 16 lane.  The LDS address goes through M0.
__device__ __attribute__((always_inline)) inline void load_to_lds(const int8_t *base, unsigned voff, unsigned lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(base), "s"(lds)
                 : "memory", "m0");
}

__global__ void __launch_bounds__(512, 1) k_gemm_i8_256(const int8_t *__restrict__ ap,
                                                         const int8_t *__restrict__ bp,
                                                         uint8_t *__restrict__ cp, int m, int n,
                                                         int64_t mp, int64_t np_, int kp, ModArgs md) {
    __shared__ __attribute__((aligned(16))) int8_t sm[kStages * kStageB];
    const int tm = (int)(mp / kTB2), tn = (int)(np_ / kTB2), T = tm * tn;
    const int l = blockIdx.x / T;
    int u = blockIdx.x % T;
    if ((T & 7) == 0) u = (u & 7) * (T >> 3) + (u >> 3);  // one stretch per XCD
    const int gsz = min(4, tm - u / (4 * tn) * 4), gr = u - u / (4 * tn) * (4 * tn);
    const int i0 = (u / (4 * tn) * 4 + gr % gsz) * kTB2, j0 = gr / gsz * kTB2;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = (w & 1) * 128, wn = (w >> 1) * 64;
    const int8_t *A = ap + (int64_t)l * mp * kp + (int64_t)i0 * kp;
    const int8_t *B = bp + (int64_t)l * np_ * kp + (int64_t)j0 * kp;
    // wave w loads rows 32 w .. 32 w + 31 of both operands, 16 rows at a time:
    // lane -> row lane / 4, stored piece lane % 4
    const int lr = 32 * w + (lane >> 2);
    const unsigned vo0 = (unsigned)lr * (unsigned)kp + (((lane & 3) ^ (-(lr >> 2) & 3)) << 4);
    const unsigned vo1 = vo0 + 16u * (unsigned)kp;  // (row + 16) / 4 has the same value mod 4
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) int8_t *)sm + 2048u * w;
    const int nk = kp / kSK;
    auto issue = [&](int kt) {
        // beyond the last slab: load it again (the buffer is not read any more)
        const int q0 = min(kt, nk - 1) * kSK;
        const unsigned d = lds0 + (unsigned)(kt & (kStages - 1)) * kStageB;
        load_to_lds(A + q0, vo0, d);
        load_to_lds(A + q0, vo1, d + 1024);
        load_to_lds(B + q0, vo0, d + kTB2 * kSK);
        load_to_lds(B + q0, vo1, d + kTB2 * kSK + 1024);
    };
    v4i acc[8][4];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = v4i{0, 0, 0, 0};
    issue(0);
    issue(1);
    issue(2);
    const int fr = lane & 15, fp = ((lane >> 4) ^ (-(fr >> 2) & 3)) << 4;
#pragma unroll 1
    for (int kt = 0; kt < nk; ++kt) {
        // this wave's part of slab kt has arrived (the two later slabs' eight
        // loads may be in flight), and its reads of slab kt - 1 are done
        asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const int8_t *as = sm + (kt & (kStages - 1)) * kStageB + (wm + fr) * kSK + fp;
        const int8_t *bs = sm + (kt & (kStages - 1)) * kStageB + kTB2 * kSK + (wn + fr) * kSK + fp;
        v4i fb[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) fb[b] = *reinterpret_cast<const v4i *>(bs + 16 * b * kSK);
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const v4i fa = *reinterpret_cast<const v4i *>(as + 16 * a * kSK);
#pragma unroll
            for (int b = 0; b < 4; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa, fb[b], acc[a][b], 0, 0, 0);
            if (a == 4) issue(kt + 3);  // behind half of the matrix instructions
        }
    }
    // The reduced bytes pass through LDS (columns of 256 bytes, 16 bytes of
    // padding) so that the stores are whole 16-byte pieces of columns.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    constexpr int kOutLd = kTB2 + 16;
    const int mod = md.m[l];
    const unsigned bias = md.bias[l], magic = md.magic[l];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int i = wm + 16 * a + 4 * (lane >> 4), j = wn + 16 * b + (lane & 15);
            unsigned packed = 0;
#pragma unroll
            for (int v = 0; v < 4; ++v) packed |= reduce_sum(acc[a][b][v], mod, bias, magic) << (8 * v);
            *reinterpret_cast<unsigned *>(sm + j * kOutLd + i) = packed;
        }
    __syncthreads();
    uint8_t *C = cp + (int64_t)l * mp * np_ + i0 + (int64_t)j0 * mp;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int x = t + 512 * e, j = x >> 4, i = (x & 15) * 16;
        *reinterpret_cast<v4i *>(C + i + (int64_t)j * mp) = *reinterpret_cast<const v4i *>(sm + j * kOutLd + i);
    }
}

// ------------------------------------------------------- reconstruction ---
__device__ inline u128 mk128(unsigned long long lo, unsigned long long hi) {
    return ((u128)hi << 64) | lo;
}

// Correct rounding (nearest, ties to even) of a < 2^127 to FP64.
__device__ inline double round_u128(u128 a) {
    const unsigned long long hi = (unsigned long long)(a >> 64), lo = (unsigned long long)a;
    if (hi == 0 && (lo >> 53) == 0) return (double)lo;
    const int msb = hi ? 127 - __builtin_clzll(hi) : 63 - __builtin_clzll(lo);
    const int sh = msb - 52;  // bits dropped, >= 1
    u128 mant = a >> sh;
    const u128 rem = a & (((u128)1 << sh) - 1), half = (u128)1 << (sh - 1);
    if (rem > half || (rem == half && (mant & 1))) mant += 1;
    return ldexp((double)(unsigned long long)mant, sh);
}

// D = epilogue(P 2^-(s_i + t_j)) with P rebuilt from its residues.
// epi 0: D = P; 1: D = I - P (m == n); 2: D = C0 + P.
// Thread: four consecutive rows of one column (one 4-byte load per modulus).
// sum_l r_l w_l is formed in 20-bit limbs of the weights (r_l w < 2^28, 15
// terms below 2^32, full-rate 24-bit multiply-adds), then taken mod 2^128;
// its quotient by M is known from the limbs in FP64 to within one, and S - q M
// lies in [-M, 2 M), which 128 bits hold, whatever S lost above them.  Bound
// by the arithmetic (about 190 instructions per element): order 4096 with 14
// moduli 316 -> 180 us against sums in 128-bit integers.
__global__ void __launch_bounds__(256) k_crt(const uint8_t *__restrict__ cp, int64_t mp, int64_t np_, int m,
                                              int n, const unsigned long long *__restrict__ amx, int beta_a,
                                              const unsigned long long *__restrict__ bmx, int beta_b,
                                              int epi, const double *__restrict__ c0, int64_t ldc,
                                              double *__restrict__ d, int64_t ldd, ModArgs md) {
    const u128 M = mk128(md.M_lo, md.M_hi), halfM = M >> 1;
    const int m4 = (m + 3) / 4;
    const int64_t total = (int64_t)m4 * n;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int i0 = (int)(e % m4) * 4, j = (int)(e / m4);
        unsigned limb[4][kLimbs];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int x = 0; x < kLimbs; ++x) limb[v][x] = 0;
        const uint8_t *src = cp + i0 + (int64_t)j * mp;
#pragma unroll 2
        for (int l = 0; l < md.count; ++l) {
            const unsigned r4 = *reinterpret_cast<const unsigned *>(src + (int64_t)l * mp * np_);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const unsigned r = (r4 >> (8 * v)) & 0xffu;
#pragma unroll
                for (int x = 0; x < kLimbs; ++x) limb[v][x] += __umul24(r, md.w[l][x]);
            }
        }
        const int tt = shift_of(bmx[j], beta_b);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + v;
            if (i >= m) break;
            u128 S = limb[v][kLimbs - 1];
            double sd = (double)limb[v][kLimbs - 1];
#pragma unroll
            for (int x = kLimbs - 2; x >= 0; --x) {
                S = (S << 20) + limb[v][x];
                sd = fma(sd, 0x1p20, (double)limb[v][x]);
            }
            S -= (u128)(unsigned)(sd * md.invM) * M;
            if ((S >> 127) != 0) S += M;  // the estimate was one too high
            if (S >= M) S -= M;           // or one too low
            const bool neg = S > halfM;
            double val = round_u128(neg ? M - S : S);
            val = neg ? -val : val;
            const int sh = shift_of(amx[i], beta_a);
            if (sh == kBadShift || tt == kBadShift)
                val = __longlong_as_double(0x7ff8000000000000ll);
            else
                val = ldexp(val, -(sh + tt));
            double out;
            if (epi == 1)
                out = (i == j ? 1.0 : 0.0) - val;
            else if (epi == 2)
                out = c0[i + (int64_t)j * ldc] + val;
            else
                out = val;
            d[i + (int64_t)j * ldd] = out;
        }
    }
}

}  // namespace

// ------------------------------------------------------------------ host ---
namespace {
u128 h_mul_mod(u128 a, u128 b, u128 M) {  // (a * b) mod M for b < 2^9
    return (a * b) % M;
}

int h_inv_mod(long long a, long long m) {  // a^-1 mod m (a, m coprime)
    long long t = 0, nt = 1, r = m, nr = ((a % m) + m) % m;
    while (nr) {
        const long long q = r / nr;
        long long tmp = t - q * nt;
        t = nt;
        nt = tmp;
        tmp = r - q * nr;
        r = nr;
        nr = tmp;
    }
    return (int)((t % m + m) % m);
}

ModArgs make_moduli(int count) {
    ModArgs md{};
    md.count = count;
    u128 M = 1;
    for (int l = 0; l < count; ++l) M *= (u128)kModuli[l];
    for (int l = 0; l < count; ++l) {
        md.m[l] = kModuli[l];
        md.inv[l] = (float)(1.0 / (double)kModuli[l]);
        md.magic[l] = (unsigned)(0x100000000ull / (unsigned long long)kModuli[l]);
        md.bias[l] = (unsigned)((0x80000000ull + kModuli[l] - 1) / kModuli[l] * kModuli[l]);
        unsigned pw = 1 % kModuli[l];
        for (int j = 0; j < 8; ++j) {
            (j < 4 ? md.pow_lo : md.pow_hi)[l] |= pw << (8 * (j & 3));
            pw = (pw << 8) % (unsigned)kModuli[l];
        }
        const u128 Ml = M / (u128)kModuli[l];
        const int ml_mod = (int)(Ml % (u128)kModuli[l]);
        const u128 wl = h_mul_mod(Ml, (u128)h_inv_mod(ml_mod, kModuli[l]), M);
        for (int x = 0; x < kLimbs; ++x) md.w[l][x] = (unsigned)(wl >> (20 * x)) & 0xfffffu;
    }
    md.M_lo = (unsigned long long)M;
    md.M_hi = (unsigned long long)(M >> 64);
    md.invM = 1.0 / ((double)md.M_hi * 18446744073709551616.0 + (double)md.M_lo);
    return md;
}

int64_t rup(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// Tile of the INT8 product: 256 x 256 when both sides hold at least four
// such tiles, else 128 x 128.
int64_t tile_for(int64_t m, int64_t n) { return (m >= 4 * kTB2 && n >= 4 * kTB2) ? kTB2 : kTB; }
}  // namespace

double ozaki_log2_modulus(int count) {
    double s = 0.0;
    for (int l = 0; l < count; ++l) s += std::log2((double)kModuli[l]);
    return s;
}

int ozaki_beta(int count, int64_t k) {
    const double lm = ozaki_log2_modulus(count);
    return (int)std::floor((lm - 1.0 - std::log2((double)(k > 0 ? k : 1))) / 2.0 - 1e-9);
}

size_t ozaki_workspace_bytes(int64_t m, int64_t n, int64_t k, int count) {
    const int64_t tile = tile_for(m, n);
    const int64_t mp = rup(m, tile), np_ = rup(n, tile), kp = rup(k > 0 ? k : 1, kSK);
    size_t b = 0;
    b += al256((size_t)count * mp * kp);   // left residues
    b += al256((size_t)count * np_ * kp);  // right residues
    b += al256((size_t)count * mp * np_);  // product residues
    b += al256(8 * (size_t)(mp + np_));    // maxima
    return b;
}

hipError_t ozaki_product(const OzakiProb &p, void *ws, hipStream_t s) {
    if (p.moduli < 2 || p.moduli > kOzakiMaxModuli || p.k > kOzakiMaxK) return hipErrorInvalidValue;
    if (p.m <= 0 || p.n <= 0) return hipSuccess;
    const int64_t m = p.m, n = p.n, k = p.k;
    const int64_t tile = tile_for(m, n);
    const int64_t mp = rup(m, tile), np_ = rup(n, tile), kp = rup(k > 0 ? k : 1, kSK);
    if (mp > INT_MAX / 2 || np_ > INT_MAX / 2 || kp > INT_MAX / 2) return hipErrorInvalidValue;
    const ModArgs md = make_moduli(p.moduli);
    char *w = static_cast<char *>(ws);
    int8_t *apl = reinterpret_cast<int8_t *>(w);
    w += al256((size_t)p.moduli * mp * kp);
    int8_t *bpl = reinterpret_cast<int8_t *>(w);
    w += al256((size_t)p.moduli * np_ * kp);
    uint8_t *cpl = reinterpret_cast<uint8_t *>(w);
    w += al256((size_t)p.moduli * mp * np_);
    unsigned long long *amax = reinterpret_cast<unsigned long long *>(w);
    unsigned long long *bmax = amax + mp;
    const int nz = (int)(mp + np_);
    hipLaunchKernelGGL(k_zero_u64, dim3((nz + 255) / 256), dim3(256), 0, s, amax, nz);
    if (k > 0) {
        const int kchunk = 64;
        const int gy = (int)std::min<int64_t>((k + kchunk - 1) / kchunk, 65535);
        hipLaunchKernelGGL(k_rowmax, dim3((unsigned)((m + 255) / 256), (unsigned)gy), dim3(256), 0, s,
                           p.A, p.lda, (int)m, (int)k, (int)((k + gy - 1) / gy), amax);
        hipLaunchKernelGGL(k_colmax, dim3((unsigned)n), dim3(256), 0, s, p.B, p.ldb, (int)k, bmax);
    }
    hipLaunchKernelGGL(k_split_rows, dim3((unsigned)(mp / 64), (unsigned)(kp / 64)), dim3(256), 0, s,
                       p.A, p.lda, (int)m, (int)k, amax, p.beta_a, apl, mp, (int)kp, md);
    const int64_t cchunks = np_ * (kp / 4);
    hipLaunchKernelGGL(k_split_cols, dim3((unsigned)((cchunks + 255) / 256)), dim3(256), 0, s, p.B,
                       p.ldb, (int)k, (int)n, bmax, p.beta_b, bpl, np_, (int)kp, md);
    if (tile == kTB2)
        hipLaunchKernelGGL(k_gemm_i8_256, dim3((unsigned)(mp / kTB2 * (np_ / kTB2) * p.moduli)), dim3(512), 0, s, apl, bpl, cpl, (int)m, (int)n, mp, np_, (int)kp, md);
    else
        hipLaunchKernelGGL(k_gemm_i8, dim3((unsigned)(mp / kTB), (unsigned)(np_ / kTB), (unsigned)p.moduli),
                           dim3(256), 0, s, apl, bpl, cpl, (int)m, (int)n, mp, np_, (int)kp, md);
    const int64_t total = (m + 3) / 4 * n;
    const int64_t blocks = std::min<int64_t>((total + 255) / 256, 16384);
    hipLaunchKernelGGL(k_crt, dim3((unsigned)blocks), dim3(256), 0, s, cpl, mp, np_, (int)m, (int)n, amax,
                       p.beta_a, bmax, p.beta_b, p.epilogue, p.C0, p.ldc, p.D, p.ldd, md);
    return hipGetLastError();
}

}  // namespace spin
