// All factors of a row of 4^7 floats in one launch: 4x4 ones, two 2x2 ones in the place of each as it comes.  X is read and Y
// written once.
//
// A row is seven digits of two bits, and their factors are applied last digit first, as in Algorithm 1.  As it loads the row a thread
// has the last digit in its 16-byte vectors, and its quad of lanes the one before, whose factor it applies by reading the
// other three lanes' registers.  Then it holds two digits (sixteen values) at a time, and at the end the first one for
// whole vectors of the last; three exchanges through LDS change what it holds.  Digits stay where they are in the row, so
// a thread writes its results over what it has read; the exchange between digits 5 and 4 and digits 3 and 2 stays
// within a wavefront, and a thread ends with the vectors it began with, so two barriers a row are all.  Every load and store of
// global memory is 1 KB in a piece.  LDS strides are padded against bank conflicts.  The other factors are
// wave-uniform: scalar loads, as in fused_kernel.hpp.
//
// Bound by memory: 1024 rows take 22.3 us (6.0 TB/s; 37.7 before), 20000 rows 451 us (5.8 TB/s; 569 before); 1024 rows of 2^14 22.3 us
// (35 before).  The kernel that ran these rows (fused_multi_kernel.hpp with four super-stages) gave a row to 256
// threads that load, multiply and store it in turn, all workgroups in step; here the next row is on its way into
// registers meanwhile (16 more of the 64 that two workgroups of 1024 threads leave a thread).  (Digit 6 through LDS too, five
// stages: 23.1 us.  The first two digits in one stage, results stored 4 bytes a lane: 24.2.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_kernel.hpp"   // Vec16, as_constant
#include "plan.hpp"           // ROW4_*

namespace km {

struct Row4Shape {
    static constexpr int NT = ROW4_THREADS, ROW = ROW4_ELEMS, N = ROW4_DIGITS;
    static constexpr int D3 = 64 + 4, D2 = 4 * D3, BLOCK = 4 * D2 + 16;  // LDS strides of digits 3, 2 and (1, 6); 16 and 4 of 4 and 5
    static_assert(16 * BLOCK * 4 == ROW4_LDS_BYTES && 16 * NT == ROW, "the planner's numbers");
};
// What is applied to each digit of the row, in the order of the Kronecker product: a 4x4 factor (g null), or two 2x2
// ones, f before g.
struct Row4Factors {
    const float* f[Row4Shape::N];
    const float* g[Row4Shape::N];
};

// d[.] <- what is applied to four values of a digit, for every e
template <int E>
__device__ __forceinline__ void row4_apply(const Row4Factors& fa, int digit, float (&d)[4][E])
{
    const float *f = fa.f[digit - 1], *g = fa.g[digit - 1];
    asm volatile("" : "+s"(f), "+s"(g));               // (all factors would be held in scalar registers over the rows, and spill)
    const auto cf = as_constant(f);
    if (g) {
        const auto cg = as_constant(g);
#pragma unroll
        for (int e = 0; e < E; ++e) {
#pragma unroll
            for (int i = 0; i < 4; i += 2) {           // the later factor: the digit's low bit
                const float y0 = __builtin_fmaf(d[i + 1][e], cg[2], d[i][e] * cg[0]), y1 = __builtin_fmaf(d[i + 1][e], cg[3], d[i][e] * cg[1]);
                d[i][e] = y0;
                d[i + 1][e] = y1;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float y0 = __builtin_fmaf(d[i + 2][e], cf[2], d[i][e] * cf[0]), y1 = __builtin_fmaf(d[i + 2][e], cf[3], d[i][e] * cf[1]);
                d[i][e] = y0;
                d[i + 2][e] = y1;
            }
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        float y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            y[q] = d[0][e] * cf[q];
#pragma unroll
            for (int p = 1; p < 4; ++p) y[q] = __builtin_fmaf(d[p][e], cf[4 * p + q], y[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q][e] = y[q];
    }
}
// The same for a digit that is the place of a lane in its quad: c is what row4_lane_factors gives the lane.
__device__ __forceinline__ void row4_lane_factors(const Row4Factors& fa, int digit, int lane, float (&c)[4])
{
    const float *f = fa.f[digit - 1], *g = fa.g[digit - 1];
#pragma unroll
    for (int p = 0; p < 4; ++p) c[p] = !g ? f[4 * p + lane % 4] : p < 2 ? g[2 * p + lane % 2] : f[2 * (p - 2) + lane / 2 % 2];
}
__device__ __forceinline__ void row4_apply_lane(bool pair, const float (&c)[4], const float (&v)[4], float (&y)[4])
{
    // (The compiler takes a move for each operand from another lane of a fused multiply-add.  s_nop: a register may be read so
    // two instructions after it was written, at the earliest; the instructions below keep that distance among themselves.)
    if (pair) {
        float w[4];
        asm("s_nop 1\n\t"
            "v_mul_f32_dpp %4, %8, %12 quad_perm:[0,0,2,2] row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %5, %9, %12 quad_perm:[0,0,2,2] row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %6, %10, %12 quad_perm:[0,0,2,2] row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %7, %11, %12 quad_perm:[0,0,2,2] row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %4, %8, %13 quad_perm:[1,1,3,3] row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %5, %9, %13 quad_perm:[1,1,3,3] row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %6, %10, %13 quad_perm:[1,1,3,3] row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %7, %11, %13 quad_perm:[1,1,3,3] row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %0, %4, %14 quad_perm:[0,1,0,1] row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %1, %5, %14 quad_perm:[0,1,0,1] row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %2, %6, %14 quad_perm:[0,1,0,1] row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %3, %7, %14 quad_perm:[0,1,0,1] row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %0, %4, %15 quad_perm:[2,3,2,3] row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %1, %5, %15 quad_perm:[2,3,2,3] row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %2, %6, %15 quad_perm:[2,3,2,3] row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %3, %7, %15 quad_perm:[2,3,2,3] row_mask:0xf bank_mask:0xf\n\t"
            : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3]), "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
            : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]));
        return;
    }
    asm("s_nop 1\n\t"
        "v_mul_f32_dpp %0, %4, %8 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
        "v_mul_f32_dpp %1, %5, %8 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
        "v_mul_f32_dpp %2, %6, %8 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
        "v_mul_f32_dpp %3, %7, %8 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %4, %9 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %5, %9 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %6, %9 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %7, %9 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %4, %10 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %5, %10 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %6, %10 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %7, %10 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %4, %11 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %5, %11 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %6, %11 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %7, %11 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]));
}
__device__ __forceinline__ void row4_transpose(const float (&a)[4][4], float (&b)[4][4])
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j][i] = a[i][j];
}

__global__ __launch_bounds__(Row4Shape::NT, 8)
void fused_row4_multiply(const float* __restrict__ Xg, float* __restrict__ Yg, Row4Factors fa, int64_t num_rows)
{
    typedef Row4Shape Sh;
    typedef Vec16<float>::type V;
    constexpr int ROW = Sh::ROW, D3 = Sh::D3, D2 = Sh::D2, BLOCK = Sh::BLOCK;
    extern __shared__ __attribute__((aligned(16))) unsigned char row4_lds[];
    float* const lds = reinterpret_cast<float*>(row4_lds);
    const int tid = threadIdx.x, l = tid % 64;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);

    V x[4];
    auto fetch = [&](int64_t r) __attribute__((always_inline)) {
        const float* src = Xg + r * ROW + w * 256 + 4 * l;
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = stream_load(reinterpret_cast<const V*>(src + k * 4096));
    };
    if (blockIdx.x >= num_rows) return;
    fetch(blockIdx.x);
    float c6[4];
    row4_lane_factors(fa, 6, l, c6);
    const bool pair6 = fa.g[5] != nullptr;
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(x[k]), "+v"(c6[k]));      // (waited for here: in the loop the compiler would wait for the stores behind them too)
    // this thread's vectors of digit 7 in LDS, k the first digit
    float* const own = lds + (l % 4) * BLOCK + (w / 4) * D2 + (w % 4) * D3 + (l / 16) * 16 + (l / 4 % 4) * 4;
    for (int64_t row = blockIdx.x; row < num_rows; row += gridDim.x) {
        float a[4][4], b[4][4];
        // digits 7, in a vector, and 6, in a quad of lanes; vector k is digit 1
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e][k] = x[k][e];
        if (row + gridDim.x < num_rows) fetch(row + gridDim.x);
        row4_apply(fa, 7, a);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float v[4] = {a[0][k], a[1][k], a[2][k], a[3][k]};
            float q[4];
            row4_apply_lane(pair6, c6, v, q);
            *reinterpret_cast<V*>(own + k * 4 * BLOCK) = V{q[0], q[1], q[2], q[3]};
        }
        __syncthreads();
        // digits 5 and 4 of this wavefront's block of 1024 (a value of digits 1 and 6), lanes along digits 2, 3 and 7
        {
            float* at = lds + w * BLOCK + (l / 16) * D2 + (l / 4 % 4) * D3 + l % 4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) a[j][i] = at[i * 16 + j * 4];
            row4_apply(fa, 5, a);
            row4_transpose(a, b);
            row4_apply(fa, 4, b);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) at[i * 16 + j * 4] = b[i][j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");           // (within the wavefront: no barrier)
        __builtin_amdgcn_wave_barrier();
        // digits 3 and 2 of the same block, lanes along digits 4, 5 and 7
        {
            float* at = lds + w * BLOCK + l;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) a[j][i] = at[i * D2 + j * D3];
            row4_apply(fa, 3, a);
            row4_transpose(a, b);
            row4_apply(fa, 2, b);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) at[i * D2 + j * D3] = b[i][j];
        }
        __syncthreads();
        // digit 1, on the vectors that this thread wrote at first (so no barrier before it writes those of the next row)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const V v = *reinterpret_cast<const V*>(own + k * 4 * BLOCK);
#pragma unroll
            for (int e = 0; e < 4; ++e) a[k][e] = v[e];
        }
        row4_apply(fa, 1, a);
        float* const y = Yg + row * ROW + w * 256 + 4 * l;
#pragma unroll
        for (int k = 0; k < 4; ++k) stream_store(V{a[k][0], a[k][1], a[k][2], a[k][3]}, reinterpret_cast<V*>(y + k * 4096));
    }
}

}  // namespace km
