// Sliced multiplies on the matrix cores whose digits stay where they are (fp32).
//
// Algorithm 1 moves the digit that a factor produces to the front of the row, so after all factors the digits are in
// order again.  Only the first and the last layout are given, though: if every launch of a plan leaves its digits in
// place, the result is the same row and the traffic of each launch is better.  A launch on the last two digits then
// reads and writes contiguous matrices, and one on any digit before them multiplies a P x R block of a row from the left
// by the factor's transpose, whose rows of R elements are read and written in runs of 256 bytes.  Two kernels:
//
//   mfma_chain_multiply     the last two factors, F1 (x) F0 with both P x P: Y_i = F1^T X_i F0 for the
//                           contiguous P x P matrices X_i of X.  The accumulators of the first product (row
//                           register, column lane) are the B operand of the second one as they are, so the
//                           intermediate never leaves the registers of the wavefront that has the matrix.
//   mfma_digit_multiply     one factor on a digit with R elements behind it: Y_m = F^T X_m for P x R blocks X_m.
//                           Columns run along the lanes of the B operand, four of them per lane in
//                           consecutive column blocks, so X goes from memory into operand registers, and the
//                           accumulators to memory, in 16-byte accesses without passing LDS.
//
// Both keep the factors in LDS in operand order (one conflict-free 16-byte read feeds four steps) and have no barrier
// after loading them: every wavefront walks over its own matrices or runs of columns with the loads of the next
// ones ahead.  Whole calls, launches that rotate -> these: 1024 x 64x64^3 1.157 -> 0.987 ms (0.60 for two factors at 114
// TFLOP/s, 0.38 for the first at 5.7 TB/s; three launches of 0.387 before), 16 x 64x64^4 1.59 -> 1.37, 1024 x 48x48^3
// 0.513 -> 0.359, 256 x (96x96, 48x48^2) 0.308 -> 0.223.  The first kernel is bound by the matrix cores within the chip's power (a loop
// of nothing but these products reaches 135 TFLOP/s on ordinary numbers, 150 on zeros), the second by memory.
// Four wavefronts to a compute unit are the best for the second: each touches P rows, R elements apart, and more of them at
// a time cost the memory more than they hide (64x64: 0.379 ms with one workgroup per compute unit, 0.416 with two, 0.425
// with three; 16x16 on 2 GB 0.182 and 0.205; 128 columns per wavefront 0.391).
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include <stdint.h>
#include "mfma_kernel.hpp"    // MfmaF32x16
#include "plan.hpp"           // CHAIN_*, DIGIT_*

namespace km {

template <int P>
struct ChainShape {
    static constexpr int NB = P / 16;                  // blocks of 16 rows or columns
    static constexpr int LDS_BYTES = 2 * P * P * 4;
};

template <int P, bool KEEP>
__global__ __launch_bounds__(CHAIN_THREADS, 2)
void mfma_chain_multiply(const float* __restrict__ Xg, float* __restrict__ Yg, const float* __restrict__ F0,
                         const float* __restrict__ F1, int64_t count)      // factors in order of application
{
    typedef MfmaF32x16 OP;
    typedef Vec16<float>::type V;
    constexpr int NB = ChainShape<P>::NB, NW = CHAIN_THREADS / 64;
    typedef float W __attribute__((ext_vector_type(NB), aligned(NB % 2 == 0 ? 4 * NB : 4)));    // a lane's columns of an output row
    const int tid = threadIdx.x, lane = tid % 64, i = lane % 16, g = lane / 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);

    // f0, B operand of the first product: block n holds columns NB * lane + n, so that a lane's results are neighbours in
    // memory.  f1, A operand of the second one: its contraction indices in the order of the first one's accumulators.
    extern __shared__ __attribute__((aligned(16))) unsigned char chain_lds[];
    float* const f0 = reinterpret_cast<float*>(chain_lds);
    float* const f1 = f0 + P * P;
    for (int e = tid; e < P * P; e += CHAIN_THREADS) {
        const int p = e / P, q = e % P, r = p % 16;
        f0[(((p / 16) * NB + q % NB) * 64 + r / 4 * 16 + q / NB) * 4 + p % 4] = F0[e];
        f1[(((q / 16) * NB + p / 16) * 64 + r / 4 * 16 + q % 16) * 4 + r % 4] = F1[e];
    }
    __syncthreads();

    const int64_t step = (int64_t)gridDim.x * NW, first = (int64_t)blockIdx.x * NW + wave;
    if (first >= count) return;
    const uint32_t in_off = (uint32_t)(i * P + 4 * g) * 4u, out_off = (uint32_t)(4 * g * P + NB * i) * 4u;
    V x[NB][NB];                                       // rows 16b + i, elements 16j + 4g of the matrix: A operand
    auto fetch = [&](const char* src, int j) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            x[b][j] = *reinterpret_cast<const V*>(src + (in_off + (uint32_t)((16 * b * P + 16 * j) * 4)));
    };
    {
        const char* src = reinterpret_cast<const char*>(Xg + first * (P * P));
#pragma unroll
        for (int j = 0; j < NB; ++j) fetch(src, j);
    }
    for (int64_t m = first; m < count; m += step) {
        // a chunk of the next matrix takes the place of this one's as soon as that is used (after the last matrix it is
        // read once more, for nothing: a condition would make the compiler wait for the loads)
        const char* src = reinterpret_cast<const char*>(Xg + (m + step < count ? m + step : m) * (P * P));
        int at = lane * 4;
        asm volatile("" : "+v"(at));                   // (the factors would be held in registers over the matrices, and spill)
        const V* fa = reinterpret_cast<const V*>(f0 + at);
        const V* fb = reinterpret_cast<const V*>(f1 + at);
        OP::Acc d0[NB][NB];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) d0[b][n][v] = 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            V f[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n) f[n] = fa[(j * NB + n) * 64];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int n = 0; n < NB; ++n) d0[b][n] = OP::mma(x[b][j][t], f[n][t], d0[b][n]);
            fetch(src, j);
        }
        char* dst = reinterpret_cast<char*>(Yg + m * (P * P));
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            OP::Acc d1[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) d1[n][v] = 0.f;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const V f = fb[(q * NB + b) * 64];
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int n = 0; n < NB; ++n) d1[n] = OP::mma(f[v], d0[b][n][v], d1[n]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                W w;
#pragma unroll
                for (int n = 0; n < NB; ++n) w[n] = d1[n][v];
                W* const y = reinterpret_cast<W*>(dst + (out_off + (uint32_t)((16 * q + v) * P * 4)));
                if constexpr (KEEP) *y = w;              // (out_store would take W for its naturally aligned like)
                else __builtin_nontemporal_store(w, y);
            }
        }
    }
}

// Columns are counted through the rows and the digits before this one.  A wavefront takes runs of 64 columns; R is a multiple
// of 64, so a run belongs to one block.  The four runs of a workgroup lie side by side, and so do those of the workgroups
// that the chip holds at once, which go on a whole grid further each time; two such stretches of 256 columns are a
// tile.  (Two runs of a wavefront side by side, or two stretches of a workgroup, leave holes in what is read and
// written at a time: 1024 x 64x64^3 0.07 ms slower.)  `go`: blocks and columns from one run of a wavefront to its next.
struct DigitStep {
    int64_t blocks, cols;
};
template <int MB, bool KEEP>
__global__ __launch_bounds__(DIGIT_THREADS, 2)
void mfma_digit_multiply(const float* __restrict__ Xg, float* __restrict__ Yg, const float* __restrict__ Fg, int P, int Q,
                         int64_t R, int64_t num_runs, DigitStep go)
{
    typedef MfmaF32x16 OP;
    typedef Vec16<float>::type V;
    constexpr int AHEAD = MB <= 5 ? 2 : 1;             // chunks of 16 rows in flight (64x64: one 0.41 ms, two 0.38)
    extern __shared__ __attribute__((aligned(16))) unsigned char digit_lds[];
    float* const lds = reinterpret_cast<float*>(digit_lds);
    const int tid = threadIdx.x, lane = tid % 64, i = lane % 16, g = lane / 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int chunks = P / 16;

    for (int e = tid; e < P * 16 * MB; e += DIGIT_THREADS) {       // the factor in operand order: Q == 16 * MB
        const int p = e / (16 * MB), q = e % (16 * MB);
        lds[(((p / 16) * MB + q / 16) * 64 + p % 16 / 4 * 16 + q % 16) * 4 + p % 4] = Fg[e];
    }
    __syncthreads();

    // a run: its number, and where its columns are in X and Y
    struct Place { int64_t n, block, c; };
    auto uniform = [](int64_t v) __attribute__((always_inline)) {
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
        return (int64_t)(((uint64_t)hi << 32) | lo);
    };
    constexpr int NW = DIGIT_THREADS / 64;
    const int64_t stride = (int64_t)gridDim.x * NW;
    auto step = [&](Place& w) __attribute__((always_inline)) {
        w.n += stride;
        w.block += go.blocks;
        w.c += go.cols;
        if (w.c >= R) { w.c -= R; w.block += 1; }
    };
    Place xw;
    xw.n = (int64_t)blockIdx.x * NW + wave;
    if (xw.n >= num_runs) return;
    xw.block = uniform(xw.n * 64 / R);
    xw.c = uniform(xw.n * 64 % R);
    Place yw = xw;

    const uint32_t in_off = (uint32_t)(4 * g * R + 4 * i) * 4u;
    V x[AHEAD + 1][4];                                 // row 16j + 4g + t, columns 4i ... of the run
    int ahead = 0;
    auto fetch = [&](V (&d)[4]) __attribute__((always_inline)) {
        if (ahead == chunks) {
            ahead = 0;
            // (after the last run its own first chunks are read again, for nothing)
            if (xw.n + stride < num_runs) step(xw);
        }
        int64_t row = R * 4;
        asm volatile("" : "+s"(row));                  // (multiples of it would be held in scalar registers, and spill)
        const char* base = reinterpret_cast<const char*>(Xg + xw.block * P * R + xw.c) + (int64_t)(16 * ahead) * row;
#pragma unroll
        for (int t = 0; t < 4; ++t) d[t] = stream_load(reinterpret_cast<const V*>(base + t * row + in_off));
        ++ahead;
    };
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) fetch(x[d]);

    OP::Acc acc[MB][4];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[m][e][v] = 0.f;
    };
    clear();
    int j = 0;
    auto chunk = [&](auto slot) __attribute__((always_inline)) {
        constexpr int S = decltype(slot)::value;
        fetch(x[(S + AHEAD) % (AHEAD + 1)]);
        __builtin_amdgcn_sched_barrier(0);             // (the compiler would move the loads behind the products)
        const V* fa = reinterpret_cast<const V*>(lds) + (j * MB) * 64 + lane;
        V f[MB];
#pragma unroll
        for (int m = 0; m < MB; ++m) f[m] = fa[m * 64];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[m][e] = OP::mma(f[m][t], x[S][t][e], acc[m][e]);
        if (++j == chunks) {
            j = 0;
            if (yw.n < num_runs) {
                int64_t row = R * 4;
                asm volatile("" : "+s"(row));
                char* base = reinterpret_cast<char*>(Yg + yw.block * Q * R + yw.c);
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        V w;
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[e] = acc[m][e][v];
                        out_store<KEEP>(w, reinterpret_cast<V*>(base + (16 * m + v) * row + in_off));
                    }
            }
            clear();
            step(yw);
        }
    };
    // (one exit for a round of the ring: an exit after each chunk makes the compiler wait for the loads ahead.  What is
    // computed past the last run is stored nowhere.)
    while (yw.n < num_runs) {
        chunk(std::integral_constant<int, 0>());
        chunk(std::integral_constant<int, 1>());
        if constexpr (AHEAD == 2) chunk(std::integral_constant<int, 2>());
    }
}

}  // namespace km
