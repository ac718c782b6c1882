// Three 32x32 factors on rows of 32^3 floats in one launch, on the matrix cores (fp32): X read and Y written once.
//
// A row is X[a][p1][p2].  For one value of `a`, the last two factors are a product of small matrices, F1^T X_a F0, whose
// intermediate stays in the accumulators: they are the B operand of the second product as they are (mfma_pair_kernel.hpp
// says why).  Each of the sixteen wavefronts does that for two values of `a`, with X read straight into operand
// registers.  The first factor needs all values of `a`, so the row passes through LDS (128 KB) once, and
// each wavefront takes 64 columns of it into registers.  A second barrier then frees LDS: while the first factor is
// multiplied and stored by some wavefronts, others are already at the next row, whose loads are issued as
// soon as the operand registers are free.
//
// 1024 rows take 61 us back to back in a graph and 66 as separate calls (77 and 78 before, with the row in LDS between all
// three products and two more barriers), 4000 rows 238 (299).  A row costs its compute unit 15 us, of which the products are 10.2 at the matrix cores' full rate; with memory
// at 4.3 TB/s beside them the chip's power allows them no more than about 110 TFLOP/s, 12 us.  One row alone takes
// 14 us, four wavefronts on a SIMD in turn.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "mfma_kernel.hpp"    // MfmaF32x16, MfmaF32x32

namespace km {

struct Row32Shape {
    static constexpr int P = 32, NW = 16, NT = NW * 64, ROW = P * P * P;
    static constexpr int APW = P / NW;                 // values of the first digit per wavefront
    static constexpr int LDS_BYTES = (ROW + 3 * P * P) * 4;
};

template <bool KEEP>
__global__ __launch_bounds__(Row32Shape::NT, 4)
void mfma_row32_multiply(const float* __restrict__ Xg, float* __restrict__ Yg, const float* __restrict__ F0,
                         const float* __restrict__ F1, const float* __restrict__ F2,       // in order of application
                         int64_t num_rows, int64_t rows_per_wg, int order)
{
    typedef Row32Shape Sh;
    typedef Vec16<float>::type V;
    constexpr int P = Sh::P, NW = Sh::NW, ROW = Sh::ROW, APW = Sh::APW;
    extern __shared__ __attribute__((aligned(16))) unsigned char row32_lds[];
    float* const z = reinterpret_cast<float*>(row32_lds);
    float* const f0 = z + ROW;
    float* const f1 = f0 + P * P;
    float* const f2 = f1 + P * P;
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);

    {
        const int p = tid / P, q = tid % P;            // NT == P * P
        // 32x32x2 B operand, contraction index 8j + 4h + t; A operand in the order of the accumulators, 8j + 4h + t too
        f0[((p / 8) * 64 + p / 4 % 2 * 32 + q) * 4 + p % 4] = F0[tid];
        f1[((p / 8) * 64 + p / 4 % 2 * 32 + q) * 4 + p % 4] = F1[tid];
        // 16x16x4 A operand, block of 16 columns, contraction index 16j + 4t + g
        f2[(((q / 16) * 2 + p / 16) * 64 + p % 4 * 16 + q % 16) * 4 + p % 16 / 4] = F2[tid];
    }
    int64_t row = (int64_t)blockIdx.x * rows_per_wg, step = 1, end = row + rows_per_wg;
    if (order == 2) {
        row = blockIdx.x;
        step = gridDim.x;
        end = num_rows;
    } else if (order == 3) {
        const int64_t per = num_rows / 8, xcd = blockIdx.x % 8;
        row = xcd * per + blockIdx.x / 8;
        step = gridDim.x / 8;
        end = (xcd + 1) * per;
    }
    if (end > num_rows) end = num_rows;

    const int col = lane % 32, h = lane / 32, i = lane % 16, g = lane / 16;
    const uint32_t in_off = (uint32_t)(col * P + 4 * h) * 4u;
    V x[APW][P / 8];
    auto fetch = [&](int64_t r, int a) __attribute__((always_inline)) {
        const char* src = reinterpret_cast<const char*>(Xg + r * ROW + (wave + a * NW) * P * P);
#pragma unroll
        for (int j = 0; j < P / 8; ++j) x[a][j] = *reinterpret_cast<const V*>(src + (in_off + 32u * j));
    };
    if (row < end)
#pragma unroll
        for (int a = 0; a < APW; ++a) fetch(row, a);
    const int turn = (wave / 2) % 2 * 32;              // this wavefront's window of the intermediate has its halves swapped
    __syncthreads();
#pragma unroll
    for (int a = 0; a < APW; ++a)
#pragma unroll
        for (int j = 0; j < P / 8; ++j) asm volatile("" : "+v"(x[a][j]));       // (waited for here: in the loop the compiler would wait for the stores behind them too)
    for (; row < end; row += step) {
        int at = lane * 4;
        asm volatile("" : "+v"(at));                   // (the factors would be held in registers over the rows)
#pragma unroll
        for (int a = 0; a < APW; ++a) {
            MfmaF32x32::Acc d0, d1;
#pragma unroll
            for (int v = 0; v < 16; ++v) d0[v] = d1[v] = 0.f;
#pragma unroll
            for (int j = 0; j < P / 8; ++j) {
                const V f = *reinterpret_cast<const V*>(f0 + at + j * 256);
#pragma unroll
                for (int t = 0; t < 4; ++t) d0 = MfmaF32x32::mma(x[a][j][t], f[t], d0);
            }
            if (row + step < end) fetch(row + step, a);
#pragma unroll
            for (int j = 0; j < P / 8; ++j) {
                const V f = *reinterpret_cast<const V*>(f1 + at + j * 256);
#pragma unroll
                for (int t = 0; t < 4; ++t) d1 = MfmaF32x32::mma(f[t], d0[4 * j + t], d1);
            }
            // Register v is row q1 = 8 (v/4) + 4 h + v%4.  Where h is set, rows 2k and 2k + 1 change places, so that the two
            // halves of the wavefront write to different banks.
            float* const to = z + (wave + a * NW) * P * P + 4 * h * P + col;
            float* const even = to + h * P;
            float* const odd = to - h * P;
#pragma unroll
            for (int v = 0; v < 16; ++v) (v % 2 ? odd : even)[(8 * (v / 4) + v % 4) * P] = d1[v];
        }
        __syncthreads();
        // first digit: this wavefront's 64 columns of the intermediate
        V zz[P / 4];
        const float* const from = z + g * P * P + 64 * wave + 4 * i;
#pragma unroll
        for (int t = 0; t < P / 4; ++t) zz[t] = *reinterpret_cast<const V*>(from + 4 * t * P * P);
        __syncthreads();                               // read by everybody: the next row may follow while this one is multiplied
        float* const y = Yg + row * ROW + 4 * g * P * P + 64 * wave + ((4 * i) ^ turn);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            MfmaF32x16::Acc acc[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[e][v] = 0.f;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const V f = *reinterpret_cast<const V*>(f2 + at + (m * 2 + j) * 256);
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] = MfmaF32x16::mma(f[t], zz[4 * j + t][e], acc[e]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                V w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = acc[e][v];
                out_store<KEEP>(w, reinterpret_cast<V*>(y + (16 * m + v) * P * P));
            }
        }
    }
}

}  // namespace km
