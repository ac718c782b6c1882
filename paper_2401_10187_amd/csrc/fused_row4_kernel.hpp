// All factors of a row of 4^7 floats in one launch: 4x4 ones, two 2x2 ones in the place of each as it comes.  X is read and Y
// written once.
//
// A row is seven digits of two bits.  A thread holds one or two digits (sixteen values) at a time and applies their
// factors in registers, the last digit first, as Algorithm 1 does; four exchanges through LDS give it the next ones.  Digits
// stay where they are in the row, so a thread writes its results over what it has read and an exchange takes one barrier;
// those between digits 6 and 5 and digits 4 and 3, and between the first two digits, stay within a wavefront and take none.
// The last digit is a 16-byte vector and the first two are applied to whole vectors of it, so every load and store of global memory is
// 256 bytes or more in a piece.  LDS strides are padded against bank conflicts.  Factors are wave-uniform: scalar loads,
// as in fused_kernel.hpp.
//
// Bound by memory: 1024 rows take 23 us (5.8 TB/s; 37.7 before), 20000 rows 449 us (5.8 TB/s; 569 before); 1024 rows of 2^14 23 us
// (35 before).  The kernel that ran these rows (fused_multi_kernel.hpp with four super-stages) gave a row to 256
// threads that load, multiply and store it in turn, all workgroups in step; here the next row is on its way into
// registers meanwhile (16 more of the 64 that two workgroups of 1024 threads leave a thread).  (The first two digits in
// one stage, sixteen values, results stored 4 bytes a lane: one exchange less, 24.2 us.  Digits in the order 7, 1, 4, 3, 6, 5, 2, three
// exchanges: 21.9 us, but intermediates overflow that do not in Algorithm 1's order.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_kernel.hpp"   // Vec16, as_constant
#include "plan.hpp"           // ROW4_*

namespace km {

struct Row4Shape {
    static constexpr int NT = ROW4_THREADS, ROW = ROW4_ELEMS, N = ROW4_DIGITS;
    static constexpr int D4 = 64 + 4, D3 = 4 * D4, BLOCK = 4 * D3;       // LDS strides of digits 4, 3 and (1, 2)
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
    constexpr int ROW = Sh::ROW, D4 = Sh::D4, D3 = Sh::D3, BLOCK = Sh::BLOCK;
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
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(x[k]));      // (waited for here: in the loop the compiler would wait for the stores behind them too)
    for (int64_t row = blockIdx.x; row < num_rows; row += gridDim.x) {
        float a[4][4], b[4][4];
        // digit 7, in a vector; vector k is digit 1
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e][k] = x[k][e];
        if (row + gridDim.x < num_rows) fetch(row + gridDim.x);
        row4_apply(fa, 7, a);
        {
            float* to = lds + (w / 4) * BLOCK + (w % 4) * D3 + (l / 16) * D4 + (l % 16) * 4;
#pragma unroll
            for (int k = 0; k < 4; ++k) *reinterpret_cast<V*>(to + k * 4 * BLOCK) = V{a[0][k], a[1][k], a[2][k], a[3][k]};
        }
        __syncthreads();
        // digits 6 and 5: this wavefront's block of 1024, lanes along digits 3, 4 and 7
        {
            float* at = lds + w * BLOCK + (l / 16) * D3 + (l / 4 % 4) * D4 + l % 4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) a[j][i] = at[i * 16 + j * 4];
            row4_apply(fa, 6, a);
            row4_transpose(a, b);
            row4_apply(fa, 5, b);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) at[i * 16 + j * 4] = b[i][j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");           // (within the wavefront: no barrier)
        __builtin_amdgcn_wave_barrier();
        // digits 4 and 3 of the same block, lanes along digits 5 to 7
        {
            float* at = lds + w * BLOCK + l;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) a[j][i] = at[i * D3 + j * D4];
            row4_apply(fa, 4, a);
            row4_transpose(a, b);
            row4_apply(fa, 3, b);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) at[i * D3 + j * D4] = b[i][j];
        }
        __syncthreads();
        // digit 2, whole vectors of digit 7, wavefronts along digits 3 and 4, lanes along digits 1, 5 and 6
        float* const to = lds + (w / 4) * D3 + (w % 4) * D4 + (l % 16) * 4;
        {
            float* at = to + (l / 16) * 4 * BLOCK;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const V v = *reinterpret_cast<const V*>(at + k * BLOCK);
#pragma unroll
                for (int e = 0; e < 4; ++e) a[k][e] = v[e];
            }
            row4_apply(fa, 2, a);
#pragma unroll
            for (int k = 0; k < 4; ++k) *reinterpret_cast<V*>(at + k * BLOCK) = V{a[k][0], a[k][1], a[k][2], a[k][3]};
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // digit 1, lanes along digits 2, 5 and 6
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const V v = *reinterpret_cast<const V*>(to + ((l / 16) + 4 * k) * BLOCK);
#pragma unroll
            for (int e = 0; e < 4; ++e) a[k][e] = v[e];
        }
        __syncthreads();                               // read by everybody: the next row may be written
        row4_apply(fa, 1, a);
        float* const y = Yg + row * ROW + (l / 16) * 1024 + w * 64 + (l % 16) * 4;
#pragma unroll
        for (int k = 0; k < 4; ++k) stream_store(V{a[k][0], a[k][1], a[k][2], a[k][3]}, reinterpret_cast<V*>(y + k * 4096));
    }
}

}  // namespace km
