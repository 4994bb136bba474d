// Auxiliary bandwidth-bound kernels: status reset, precision conversion,
// copies, transposes and deterministic Frobenius-norm reductions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "spin_kernels.hpp"

namespace spin {
namespace {

constexpr int kNormBlocks = 256;

// Several requests' workspaces in one launch: block b resets item b.
struct ResetArgs {
    int *status[kMaxAuxBatch];
};
__global__ void k_status_reset(ResetArgs a, int spec) {
    const int i = threadIdx.x;
    int *status = a.status[blockIdx.x];
    if (i < kStatusWords) status[i] = (i == kStatusSpecWord && !spec) ? 0 : INT_MAX;
    if (i == kStatusWords) status[kFrobCounterWord] = 0;
}

__global__ void k_frob_counter_reset(int *status) { status[kFrobCounterWord] = 0; }

__global__ void k_status_copy(const int *status, int *info) {
    if (threadIdx.x == 0) info[0] = status[0] == INT_MAX ? 0 : status[0];
}

// Items of a batched launch: item q owns the blocks from start[q] on.
template <typename Item>
struct AuxArgs {
    Item item[kMaxAuxBatch];
    int32_t start[kMaxAuxBatch];
    int32_t count;
};

template <typename Item>
__device__ inline int aux_member(const AuxArgs<Item> &a) {
    int q = 0;
    while (q + 1 < a.count && (int)blockIdx.x >= a.start[q + 1]) ++q;
    return q;
}

// Conversion of (m x n) column-major views: a wave takes 1024 rows of a column
// at a time (16 elements a lane in flight).
template <typename S, typename D>
__device__ inline void convert_unit(const ConvItem &it, int64_t u, int lane) {
    const int64_t segs = (it.m + 1023) / 1024, j = u / segs, i0 = (u % segs) * 1024 + lane;
    if (j >= it.n) return;
    const S *src = static_cast<const S *>(it.src) + j * it.lds;
    D *dst = static_cast<D *>(it.dst) + j * it.ldd;
#pragma unroll
    for (int q = 0; q < 16; ++q)
        if (i0 + 64 * q < it.m) dst[i0 + 64 * q] = (D)src[i0 + 64 * q];
}
__global__ void __launch_bounds__(256) k_convert(AuxArgs<ConvItem> a) {
    const int q = aux_member(a);
    const int64_t u = (int64_t)((int)blockIdx.x - a.start[q]) * 4 + (threadIdx.x >> 6);
    if (a.item[q].to_f32)
        convert_unit<double, float>(a.item[q], u, threadIdx.x & 63);
    else
        convert_unit<float, double>(a.item[q], u, threadIdx.x & 63);
}

// dst (n x m, ldd) = src (m x n, lds)^T.  A workgroup moves one 64 x 64 tile
// through LDS: it reads down the source columns and writes down the
// destination columns, so both sides coalesce.  The row pitch of 65 doubles
// spreads the transposed LDS reads over the banks.
constexpr int kTT = 64;
__global__ void __launch_bounds__(256)
    k_transpose(const double *__restrict__ src, int64_t lds, double *__restrict__ dst, int64_t ldd,
                int64_t m, int64_t n) {
    __shared__ double tile[kTT][kTT + 1];
    const int64_t i0 = (int64_t)blockIdx.x * kTT, j0 = (int64_t)blockIdx.y * kTT;
    const int tx = threadIdx.x & (kTT - 1), ty = threadIdx.x / kTT;
    for (int jj = ty; jj < kTT; jj += 256 / kTT) {
        const int64_t i = i0 + tx, j = j0 + jj;
        if (i < m && j < n) tile[jj][tx] = src[i + j * lds];
    }
    __syncthreads();
    for (int ii = ty; ii < kTT; ii += 256 / kTT) {
        const int64_t r = j0 + tx, c = i0 + ii;  // dst row = src column
        if (r < n && c < m) dst[r + c * ldd] = tile[tx][ii];
    }
}

// Lower triangle of an order-n view mirrored onto the upper one, in place:
// d[i][j] = d[j][i] for j > i.  Workgroup t takes lower tile (r, c), r >= c
// (row by row over the T (T + 1) / 2 of them), reads it whole into LDS and
// writes its transpose into upper tile (c, r); a diagonal tile writes only its
// own strict upper part.  Each tile is read by one workgroup, and no tile
// that is written is read by another, so the update needs no ordering.
__global__ void __launch_bounds__(256) k_mirror_lower(double *__restrict__ d, int64_t ld, int64_t n) {
    __shared__ double tile[kTT][kTT + 1];
    const int t = blockIdx.x;
    int r = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while (r * (r + 1) / 2 > t) --r;
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    const int c = t - r * (r + 1) / 2;
    const int64_t i0 = (int64_t)r * kTT, j0 = (int64_t)c * kTT;  // source rows i0.., columns j0..
    const int tx = threadIdx.x & (kTT - 1), ty = threadIdx.x / kTT;
    for (int jj = ty; jj < kTT; jj += 256 / kTT) {
        const int64_t i = i0 + tx, j = j0 + jj;
        if (i < n && j < n) tile[jj][tx] = d[i + j * ld];
    }
    __syncthreads();
    for (int ii = ty; ii < kTT; ii += 256 / kTT) {
        const int64_t row = j0 + tx, col = i0 + ii;  // destination (row, col) = source (col, row)
        if (row < n && col < n && col > row) d[row + col * ld] = tile[tx][ii];
    }
}

// 2-D grid-stride zero fill of an (m x n) column-major view.
__global__ void __launch_bounds__(256) k_fill_zero(double *__restrict__ d, int64_t ld, int64_t m, int64_t n) {
    for (int64_t j = blockIdx.y; j < n; j += gridDim.y)
        for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += (int64_t)gridDim.x * 256)
            d[i + j * ld] = 0.0;
}

// Sums of squares of (m x n) views and what the refinement makes of them, in
// one launch for up to kMaxAuxBatch views.  Each wave sums whole columns (fixed
// assignment of columns to waves and fixed in-block order); the block of a view
// that finishes last, told by a counter in front of the view's partials that it
// sets back to 0, adds the partials in a fixed order, so the result does not
// depend on scheduling or on the other views.  Then
//   kFrobOnly   nothing more;
//   kFrobCheck  refinement monitor: flags divergence when |R_j|_F did not
//               decrease (out is norms + j);
//   kFrobFinal  acceptance of a refined inverse, out = norms + 3 = |X|^2 being
//               the last of the three: flags divergence unless rho = |R|_F /
//               (|A|_F |X|_F) <= kNsTol (norms[2] = |R|^2, norms[0] = |A|^2; a
//               NaN anywhere fails the test).
// Three launches for each norm before (partials, sum, check): 14 mixed requests
// of a batch spent 680 us on 70 norms, 230 us now.  What bounds a small one is
// latency: a round trip for the columns, which another XCD has just written, and
// three for the hand-over.  Right behind the kernel that wrote the view, in a
// graph, against three launches and a column at a time: order 64 5.8 -> 3.5 us,
// 192 5.9 -> 4.3, 384 6.6 -> 5.0, 768 8.5 -> 7.1, 2048 12.0 -> 11.2, 8192 156 ->
// 109; only 1024 lost, 6.7 -> 9.0.  With one column of a wave in flight 192 and 384
// took 8.3 and 9.1 us.
__device__ inline double block_sum(double s) {
    __shared__ double red[4];
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) s += __shfl_xor(s, w);
    __syncthreads();  // the previous sum has been read
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// A lane's sum over N columns, stride elements apart, from row threadIdx % 64 on:
// 16 loads are in flight whatever m is.
template <int N>
__device__ inline double frob_columns(const double *col, int64_t stride, int64_t m) {
    double s[N];
#pragma unroll
    for (int q = 0; q < N; ++q) s[q] = 0.0;
#pragma unroll(16 / N)
    for (int64_t i = threadIdx.x & 63; i < m; i += 64)
#pragma unroll
        for (int q = 0; q < N; ++q) s[q] = fma(col[i + q * stride], col[i + q * stride], s[q]);
    if constexpr (N == 4) return (s[0] + s[1]) + (s[2] + s[3]);
    if constexpr (N == 2) return s[0] + s[1];
    return s[0];
}

__global__ void __launch_bounds__(256) k_frob(AuxArgs<FrobItem> a) {
    __shared__ bool last;
    const int q = aux_member(a);
    const FrobItem &it = a.item[q];
    const int b = (int)blockIdx.x - a.start[q], nb = it.blocks;
    const int64_t m = it.m, n = it.n;
    double s = 0.0;
    // a wave takes every 4 nb-th column, up to four at a time
    const int64_t step = nb * 4, stride = step * it.ld;
    int64_t c = b * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (; c + 3 * step < n; c += 4 * step) s += frob_columns<4>(it.src + c * it.ld, stride, m);
    if (c + step < n) {
        s += frob_columns<2>(it.src + c * it.ld, stride, m);
        c += 2 * step;
    }
    if (c < n) s += frob_columns<1>(it.src + c * it.ld, stride, m);
    s = block_sum(s);
    double *const partials = it.partials;
    unsigned *const counter = reinterpret_cast<unsigned *>(partials) - 2;
    if (threadIdx.x == 0) {
        // The partial is stored device-coherently and has arrived before the
        // block is counted; nothing else is handed over, so no fence (which
        // would write back the whole L2) is needed.
        __hip_atomic_store(partials + b, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        last = (int)__hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nb - 1;
    }
    __syncthreads();
    if (!last) return;
    s = 0.0;
    for (int i = threadIdx.x; i < nb; i += 256)
        s += __hip_atomic_load(partials + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s = block_sum(s);
    if (threadIdx.x != 0) return;
    __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *it.out = s;
    if (it.then == kFrobCheck && it.j > 0 && !(s < it.out[-1])) *it.status = kStatusNsDiverged;
    if (it.then == kFrobFinal) {
        const double rho = sqrt(it.out[-1]) / (sqrt(it.out[-3]) * sqrt(s));
        if (!(rho <= kNsTol)) *it.status = kStatusNsDiverged;
    }
}

// Launches kernel k over the items, units blocks each.
template <typename Item, typename U>
hipError_t aux_launch(void (*k)(AuxArgs<Item>), const Item *items, int count, U blocks, hipStream_t s) {
    if (count < 0 || count > kMaxAuxBatch) return hipErrorInvalidValue;
    AuxArgs<Item> a{};
    int64_t total = 0;
    for (int q = 0; q < count; ++q) {
        if (items[q].m <= 0 || items[q].n <= 0) continue;
        a.item[a.count] = items[q];
        a.start[a.count++] = (int32_t)total;
        total += blocks(a.item[a.count - 1]);
        if (total > INT_MAX) return hipErrorInvalidValue;
    }
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k, dim3((unsigned)total), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t status_reset(int *const *status, int count, bool spec, hipStream_t s) {
    if (count < 1 || count > kMaxAuxBatch) return hipErrorInvalidValue;
    ResetArgs a{};
    for (int q = 0; q < count; ++q) a.status[q] = status[q];
    hipLaunchKernelGGL(k_status_reset, dim3((unsigned)count), dim3(64), 0, s, a, spec ? 1 : 0);
    return hipGetLastError();
}

hipError_t status_reset(int *status, bool spec, hipStream_t s) { return status_reset(&status, 1, spec, s); }

hipError_t status_copy(const int *status, int *info, hipStream_t s) {
    hipLaunchKernelGGL(k_status_copy, dim3(1), dim3(64), 0, s, status, info);
    return hipGetLastError();
}

hipError_t convert(const ConvItem *items, int count, hipStream_t s) {
    return aux_launch(k_convert, items, count,
                      [](const ConvItem &it) { return ((it.m + 1023) / 1024 * it.n + 3) / 4; }, s);
}

hipError_t cast_f64_to_f32(const double *src, int64_t lds, float *dst, int64_t ldd, int64_t m,
                           int64_t n, hipStream_t s) {
    const ConvItem it{src, dst, lds, ldd, m, n, 1};
    return convert(&it, 1, s);
}

hipError_t cast_f32_to_f64(const float *src, int64_t lds, double *dst, int64_t ldd, int64_t m,
                           int64_t n, hipStream_t s) {
    const ConvItem it{src, dst, lds, ldd, m, n, 0};
    return convert(&it, 1, s);
}

hipError_t fill_zero_f64(double *d, int64_t ld, int64_t m, int64_t n, hipStream_t s) {
    if (m <= 0 || n <= 0) return hipSuccess;
    const int64_t bx = (m + 255) / 256;
    dim3 grid((unsigned)(bx < 64 ? bx : 64), (unsigned)(n < 4096 ? n : 4096));
    hipLaunchKernelGGL(k_fill_zero, grid, dim3(256), 0, s, d, ld, m, n);
    return hipGetLastError();
}

hipError_t mirror_lower_f64(double *d, int64_t ld, int64_t n, hipStream_t s) {
    if (n <= 1) return hipSuccess;
    const int64_t T = (n + kTT - 1) / kTT, blocks = T * (T + 1) / 2;
    if (blocks > INT_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mirror_lower, dim3((unsigned)blocks), dim3(256), 0, s, d, ld, n);
    return hipGetLastError();
}

hipError_t transpose_f64(const double *src, int64_t lds, double *dst, int64_t ldd, int64_t m,
                         int64_t n, hipStream_t s) {
    if (m <= 0 || n <= 0) return hipSuccess;
    const int64_t gx = (m + kTT - 1) / kTT, gy = (n + kTT - 1) / kTT;
    if (gx > INT_MAX || gy > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_transpose, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, s, src, lds, dst,
                       ldd, m, n);
    return hipGetLastError();
}

// Blocks of a norm: one per 16 columns, four to a wave, or per 128 KB (64 loads a
// lane) if that is more, at most kNormBlocks, because counting a block takes about
// 20 ns, and at most one per column quartet.
int frob_partials_count(int64_t m, int64_t n) {
    const int64_t b = std::max<int64_t>((n + 15) / 16, (m * n + 16383) / 16384);
    return (int)std::max<int64_t>(std::min<int64_t>({b, (n + 3) / 4, kNormBlocks}), 1);
}

hipError_t frob_counter_reset(int *status, hipStream_t s) {
    hipLaunchKernelGGL(k_frob_counter_reset, dim3(1), dim3(1), 0, s, status);
    return hipGetLastError();
}

hipError_t frob(const FrobItem *items, int count, hipStream_t s) {
    return aux_launch(k_frob, items, count,
                      [](FrobItem &it) {
                          it.blocks = frob_partials_count(it.m, it.n);
                          return (int64_t)it.blocks;
                      },
                      s);
}

hipError_t frob2(const double *src, int64_t ld, int64_t m, int64_t n, double *partials,
                 double *out, hipStream_t s) {
    const FrobItem it{src, ld, m, n, partials, out, nullptr, kFrobOnly, 0, 0};
    return frob(&it, 1, s);
}

}  // namespace spin
