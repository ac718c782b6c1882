// Rows of P^(3G) floats in one launch and of P^(4G) floats in two, square factors of an odd size P (fp32; P = 5 with G = 2 and
// P = 3 with G = 3).
//
// A tile is a cube: three groups of G digits, E = P^G values each (5^6 = 25^3, 3^9 = 27^3 elements), contiguous where it is
// read.  A thread holds the E values of one group in registers, applies the group's factors to them and changes to the group before it
// through LDS; the last group comes first, as in Algorithm 1.  Digits stay where they are, so a thread writes its values over
// those it has read, and an exchange takes one barrier.  A row of 3G digits is one tile.  A row of 4G digits takes two launches of two
// groups each.  The first one leaves the row in an order that makes the second one's tiles contiguous too, and writes it in runs of
// E^2 elements; the second one's results are runs of E elements (100 and 108 bytes), which cost it a quarter of its rate.  (The two middle groups
// first, then the two outer ones, reads and writes all runs of E^2, 1000 x 5x5^8 1.26 ms, but intermediates overflow that do
// not in Algorithm 1's order.  Three groups and one, 1.32.)
// Lanes run along the two groups behind the one in registers, 4 bytes a lane (rows of odd length start on no boundary); the LDS
// stride of the first group is congruent to E modulo the 64 banks, so an access meets a bank twice only at the ends of
// runs.  The next tile's loads are issued before the current one is multiplied.
//
// Bound by memory.  1000 x 5x5^8 1.61 -> 1.34 ms (two launches of 0.60 and 0.74; a plain copy of X takes 0.58), 40 rows
// 75 -> 56 us; 1000 x 3x3^12 1.99 -> 1.83; 1024 x 5x5^6 42 -> 31 us, 4096 rows 142 -> 121; 1024 x 3x3^9 46 -> 34.  (What ran these rows,
// fused_multi_kernel.hpp, loads, multiplies and stores a tile in turn and stores element-sized pieces of 100 and 108 bytes.)
// Loads are ordinary ones: at the ends of a wavefront's 256 bytes its neighbour reads the same lines.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_kernel.hpp"   // ipow, as_constant
#include "plan.hpp"           // cube_stride

namespace km {

// A tile is three groups of G digits of size P: E = P^G values each.
template <int P_, int G_>
struct CubeShape {
    static constexpr int P = P_, G = G_, E = (int)ipow(P, G), EE = E * E;
    static constexpr int NT = (EE + 63) / 64 * 64;
    static constexpr int S1 = cube_stride(E);          // LDS stride of the first group
    static constexpr int LDS_BYTES = E * S1 * 4;
    static constexpr int WAVES = 2 * (NT / 64) / 4;    // two workgroups per compute unit, per SIMD
};
// The factors of each group in the order of the Kronecker product.
struct CubeFactors {
    const float* f[3][3];
};

// The G factors of a group, last one first, on its E values.
template <int P, int G>
__device__ __forceinline__ void cube_apply(const float* const (&f)[3], float (&d)[(int)ipow(P, G)])
{
    constexpr int E = (int)ipow(P, G);
#pragma unroll
    for (int k = G - 1; k >= 0; --k) {
        const float* fk = f[k];
        asm volatile("" : "+s"(fk));                   // (all factors would be held in scalar registers over the tiles)
        const auto c = as_constant(fk);
        const int below = (int)ipow(P, G - 1 - k);     // values of the digits behind this one
#pragma unroll
        for (int s = 0; s < E / P; ++s) {
            const int at = s / below * below * P + s % below;
            float y[P];
#pragma unroll
            for (int q = 0; q < P; ++q) {
                y[q] = d[at] * c[q];
#pragma unroll
                for (int p = 1; p < P; ++p) y[q] = __builtin_fmaf(d[at + p * below], c[p * P + q], y[q]);
            }
#pragma unroll
            for (int q = 0; q < P; ++q) d[at + q * below] = y[q];
        }
    }
}

// PART 0: rows of three groups, all factors.  Rows of four groups g1 ... g4: PART 1 applies the last two to tiles (row, g1) of
// X and leaves the row in the order g3, g1, g2, g4, which makes tiles (row, g3) contiguous too; PART 2 applies the first two to those.
template <int P, int G, int PART>
__global__ __launch_bounds__((CubeShape<P, G>::NT), (CubeShape<P, G>::WAVES))
void fused_cube_multiply(const float* __restrict__ Xg, float* __restrict__ Yg, CubeFactors fa, int64_t tiles)
{
    typedef CubeShape<P, G> Sh;
    constexpr int E = Sh::E, EE = Sh::EE, S1 = Sh::S1;
    constexpr int64_t EEE = (int64_t)E * EE;
    extern __shared__ __attribute__((aligned(16))) unsigned char cube_lds[];
    float* const lds = reinterpret_cast<float*>(cube_lds);
    const int u = (int)threadIdx.x < EE ? (int)threadIdx.x : EE - 1;     // (what is left of the last wavefront does the last one's work again: no access hangs on a condition)
    const int ua = u / E, ub = u % E;
    const uint32_t in4 = (uint32_t)u * 4u, out4 = PART == 2 ? (uint32_t)(ua * EE + ub) * 4u : in4;

    // each XCD (workgroup b runs on XCD b % 8) walks its own part of the tiles; grids that do not split by 8: one tile each
    int64_t first = blockIdx.x, step = gridDim.x, end = tiles;
    if (gridDim.x % 8 == 0) {
        const int64_t part = (tiles + 7) / 8, xcd = blockIdx.x % 8;
        first = xcd * part + blockIdx.x / 8;
        step = gridDim.x / 8;
        if ((xcd + 1) * part < tiles) end = (xcd + 1) * part;
    }

    float x[E];
    auto fetch = [&](int64_t t) __attribute__((always_inline)) {
        const char* src = reinterpret_cast<const char*>(Xg + t * EEE);
        int64_t go = EE * 4;
        asm volatile("" : "+s"(go));                   // (multiples of it would be held in scalar registers, and spill)
#pragma unroll
        for (int k = 0; k < E; ++k) {
            x[k] = *reinterpret_cast<const float*>(src + in4);
            src += go;
        }
    };
    if (first >= end) return;
    fetch(first);
    // (waited for here: in the loop the compiler would have to allow for a first round without stores behind the loads,
    // and wait for the last tile's stores with every tile)
#pragma unroll
    for (int k = 0; k < E; ++k) asm volatile("" : "+v"(x[k]));
    for (int64_t t = first; t < end; t += step) {
        float d[E];
#pragma unroll
        for (int k = 0; k < E; ++k) lds[k * S1 + u] = x[k];
        __syncthreads();
        if (t + step < end) fetch(t + step);
        if constexpr (PART != 2) {                     // the tile's third group
            float* at = lds + ua * S1 + ub * E;
#pragma unroll
            for (int k = 0; k < E; ++k) d[k] = at[k];
            cube_apply<P, G>(fa.f[2], d);
#pragma unroll
            for (int k = 0; k < E; ++k) at[k] = d[k];
            __syncthreads();
        }
        {                                              // the second
            float* at = lds + ua * S1 + ub;
#pragma unroll
            for (int k = 0; k < E; ++k) d[k] = at[k * E];
            if constexpr (PART != 1) {
                cube_apply<P, G>(fa.f[1], d);
#pragma unroll
                for (int k = 0; k < E; ++k) at[k * E] = d[k];
                __syncthreads();
#pragma unroll
                for (int k = 0; k < E; ++k) d[k] = lds[k * S1 + u];
            }
        }
        __syncthreads();                               // read by everybody: the next tile may be written
        cube_apply<P, G>(fa.f[PART == 1 ? 1 : 0], d);
        {
            char* dst = reinterpret_cast<char*>(Yg + (PART == 0 ? t * EEE : t / E * (EEE * E) + t % E * (PART == 1 ? EE : E)));
            int64_t go = (PART == 0 ? EE : EEE) * 4;
            asm volatile("" : "+s"(go));
#pragma unroll
            for (int k = 0; k < E; ++k) {
                *reinterpret_cast<float*>(dst + out4) = d[k];
                dst += go;
            }
        }
    }
}

}  // namespace km
