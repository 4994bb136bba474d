// Device helpers of the 16-step block eliminations (leaf.hip, lu.hip).  Not
// installed.
//
// A 16 x 16 block lives in the accumulator layout of v_mfma_f64_16x16x4f64
// with the operands swapped: lane l holds row l % 16 of columns 4 v + l / 16,
// so a wave's loads and stores cover 16 consecutive rows of four columns.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

namespace spin {
namespace {

// DPP control words (GFX9 encoding).
constexpr int kDppQuadXor1 = 0xB1;   // quad_perm [1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;   // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;
constexpr int kDppMirror = 0x140;

// Every control used here reads a lane of the same row, so all lanes are
// written and the move needs no initial value.
template <int CTRL>
__device__ inline double dpp_f64(double x) {
    const int lo =
        __builtin_amdgcn_mov_dpp((int)(__double_as_longlong(x) & 0xffffffff), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(__double_as_longlong(x) >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ inline double readlane_f64(double x, int lane) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

typedef double d4_t __attribute__((ext_vector_type(4)));
template <int NW, int RB, int NC>
struct BlkLds {
    static constexpr int kRows = 16 * NW * RB, kCols = 16 * NC;
    // two panel buffers where 160 KB hold them: the panels of the next block
    // step are then written while the current ones are still read
    static constexpr bool kTwo = NW * RB <= 16;
    static constexpr int kBufs = kTwo ? 2 : 1;
    // pitches that spread the 16 x 4 element accesses of a wave over the banks
    static constexpr int kFLd = kRows + 16, kPrLd = kCols + 4, kRLd = kCols + 16;
    static constexpr int oPc = 0;                        // column panel [16][kFLd], per buffer
    static constexpr int oF = oPc + kBufs * 16 * kFLd;   // F [16][kFLd]
    static constexpr int oPr = oF + 16 * kFLd;           // row panel [16][kPrLd], per buffer
    static constexpr int oR = oPr + kBufs * 16 * kPrLd;  // R [16][kRLd]
    static constexpr int oDr = oR + 16 * kRLd;           // pivot rows inside the diagonal block
    static constexpr int oDm = oDr + 256;                // its active columns
    static constexpr int oDump = oDm + 256;              // unwanted stores of the chain
    static constexpr int kDoubles = oDump + 16 * 15 + 16;
};

// The same value, unknown to the compiler: what is computed from it (lane
// masks, addresses) is computed anew and not held in registers across loops.
__device__ inline int opaque(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Ends a branch taken for one of several register blocks.  Without it the
// compiler merges the branches' common ends into one with a run-time index,
// which puts the indexed registers into scratch memory.
template <int I>
__device__ __attribute__((always_inline)) inline void branch_end() {
    asm volatile("; block %0" ::"n"(I));
}

// f(0), ..., f(N - 1) with constant arguments.
template <typename F, int... I>
__device__ __attribute__((always_inline)) inline void static_for_seq(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __attribute__((always_inline)) inline void static_for(F f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// x[j] = fma(-f, r of lane j, x[j]) for all 16 j, the lane within each group
// of 16 (DPP row_newbcast).  The wait states before the first DPP read cover
// a vector write of r just before it.
__device__ inline void fmac_rows(double (&x)[16], double r, double f) {
#define SPIN_FMAC(J) "v_fmac_f64_dpp %" #J ", %16, -%17 row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"
    asm("s_nop 1\n\t" SPIN_FMAC(0) SPIN_FMAC(1) SPIN_FMAC(2) SPIN_FMAC(3) SPIN_FMAC(4) SPIN_FMAC(5) SPIN_FMAC(6)
            SPIN_FMAC(7) SPIN_FMAC(8) SPIN_FMAC(9) SPIN_FMAC(10) SPIN_FMAC(11) SPIN_FMAC(12) SPIN_FMAC(13)
                SPIN_FMAC(14) SPIN_FMAC(15)
        : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]),
          "+v"(x[8]), "+v"(x[9]), "+v"(x[10]), "+v"(x[11]), "+v"(x[12]), "+v"(x[13]), "+v"(x[14]), "+v"(x[15])
        : "v"(r), "v"(f));
#undef SPIN_FMAC
}

// The value of lane K of each lane's own group of 16.
template <int K>
__device__ inline double row_bcast(double x) {
    return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + K, 0xf, 0xf, true);
}

}  // namespace
}  // namespace spin
