// One sliced-multiply iteration for small factors of any shape: the form of the generic kernel (generic_kernel.hpp) for factors
// whose 128 slices fit LDS whole.
//
// A unit of work is the same 128 consecutive slices times 32 factor columns.  The slices are one contiguous run of X,
// numbered through all rows, and are copied to LDS rows of an odd stride, so that the lanes of a wavefront, one
// slice each, read from different banks.  Two wavefronts take the first half of the unit's columns, two the other; a thread keeps
// NC columns of its slice in registers and walks over the slice once, the factor's elements coming as scalars.  NC is what the
// columns need (1 to 16), so nothing is multiplied on padding; where NC does not divide them, the last columns are
// computed by two wavefronts, alike.  The other form always multiplies 32 columns by chunks of 16: 57 times the work
// for a 3x3 factor.
// Bound by memory and, on small launches, by the latency of one pass.  Calls with such a launch, us, the other form -> this one:
// 1000000 x (2x3) 25.5 -> 11.5, 300000 x (5x40) 71 -> 29, 100000 x (3x100) 63 -> 20, 100000 x (33x5) fp64 16.9 -> 9.5, 100000 x (20x7)
// 8.0 -> 5.8; 115 x (25x125, 11x3, 3x7, 18x121) 207 -> 142, 295 x (3x3, 7x3, 20x40, 4x16) 50.6 -> 39.5, 2 x (35x5, 10x2, 7x67) 15.7 -> 12.4;
// 22 of 160 drawn problems have one: 1.18 times as fast on average, none slower.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_kernel.hpp"   // Vec16, as_constant
#include "generic_kernel.hpp" // GEN_*

namespace km {

// columns per thread: a power of two that covers half a unit's columns
KM_HOST_DEVICE constexpr int gen_small_columns(int Q) { return Q <= 2 ? 1 : Q <= 4 ? 2 : Q <= 8 ? 4 : Q <= 16 ? 8 : 16; }

// The NC columns of one slice, whose elements x gives.
template <typename T, int NC, class Elem>
__device__ __forceinline__ void small_multiply(T (&acc)[NC], const T* __restrict__ Fg, int P, int Q, Elem x)
{
    const auto f = as_constant(Fg);
#pragma unroll
    for (int j = 0; j < NC; ++j) acc[j] = T(0);
    int p = 0;
    for (; p + 4 <= P; p += 4) {
        T v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = x(p + i);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NC; ++j) acc[j] += v[i] * f[(p + i) * Q + j];
    }
    for (; p < P; ++p) {
        const T v = x(p);
#pragma unroll
        for (int j = 0; j < NC; ++j) acc[j] += v * f[p * Q + j];
    }
}

// FEW: P is at most GEN_FEW, and a thread reads its slice by itself: what 64 lanes read one after the other is one run, and no
// barrier is needed.
template <typename T, int NC, bool FEW>
__global__ __launch_bounds__(GEN_THREADS)
void sliced_multiply_small(const T* __restrict__ Xg, const T* __restrict__ Fg, T* __restrict__ Yg, int64_t S, int P, int Q,
                           int64_t num_slices, int64_t num_units, unsigned p_magic)
{
    typedef typename Vec16<T>::type V;
    constexpr int VN = Vec16<T>::N, AHEAD = 8;         // vectors in flight per thread
    static_assert(GEN_THREADS == 2 * GEN_TS && GEN_TS == GEN_SLICES, "two groups of columns per slice");
    extern __shared__ __attribute__((aligned(16))) unsigned char small_lds[];
    T* const lds = reinterpret_cast<T*>(small_lds);
    const int tid = threadIdx.x, rs = gen_small_stride(P);
    const int half = __builtin_amdgcn_readfirstlane(tid / GEN_TS), s = tid % GEN_TS;
    const int q_groups = (Q + GEN_TQ - 1) / GEN_TQ;
    const bool narrow = num_slices < (int64_t)1 << 31; // 32-bit divisions will do

    for (int64_t unit = blockIdx.x; unit < num_units; unit += gridDim.x) {
        int64_t tile = unit;
        int group = 0;
        if (q_groups > 1) unit_of(unit, num_units / q_groups, q_groups, tile, group);
        const int64_t g0 = tile * GEN_TS;
        const T* src = Xg + g0 * P;                    // (128 P elements from the start: on a 16-byte boundary)
        const int64_t rest = num_slices - g0;
        const int q_last = Q - NC, q_first = group * GEN_TQ + half * NC;
        const int q0 = q_first < q_last ? q_first : q_last;
        T acc[NC];
        if constexpr (FEW) {
            const T* xs = src + (s < rest ? s : 0) * P;
            T x[GEN_FEW];
            if (P % VN == 0) {                         // whole vectors, on their boundaries
#pragma unroll
                for (int p = 0; p < GEN_FEW; p += VN)
                    if (p < P) {
                        const V v = *reinterpret_cast<const V*>(xs + p);
#pragma unroll
                        for (int k = 0; k < VN; ++k) x[p + k] = v[k];
                    }
            } else {
#pragma unroll
                for (int p = 0; p < GEN_FEW; ++p)
                    if (p < P) x[p] = xs[p];
            }
            const auto f = as_constant(Fg + q0);
#pragma unroll
            for (int j = 0; j < NC; ++j) acc[j] = T(0);
#pragma unroll
            for (int p = 0; p < GEN_FEW; ++p)
                if (p < P)
#pragma unroll
                    for (int j = 0; j < NC; ++j) acc[j] += x[p] * f[p * Q + j];
        } else {
            const int n = (rest < GEN_TS ? (int)rest : GEN_TS) * P;
            for (int e0 = tid * VN; e0 < n; e0 += AHEAD * GEN_THREADS * VN) {
                V v[AHEAD];
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) {
                    const int e = e0 + i * GEN_THREADS * VN;
                    if (e + VN <= n) v[i] = *reinterpret_cast<const V*>(src + e);
                    else if (e < n)                    // the end of X inside a vector
#pragma unroll
                        for (int k = 0; k < VN; ++k) v[i][k] = e + k < n ? src[e + k] : T(0);
                }
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) {
                    const int e = e0 + i * GEN_THREADS * VN;
                    if (e < n) {
                        const int row = (int)__umulhi((unsigned)e, p_magic);
                        int left = P - (e - row * P);  // elements left in the slice (P > GEN_FEW: a vector is in two at most)
                        T* to = lds + e + row * (rs - P);
#pragma unroll
                        for (int k = 0; k < VN; ++k)
                            if (e + k < n) to[k + (k >= left ? rs - P : 0)] = v[i][k];
                    }
                }
            }
            __syncthreads();
            const T* xs = lds + s * rs;
            small_multiply<T, NC>(acc, Fg + q0, P, Q, [&](int p) { return xs[p]; });
        }
        if (s < rest) {
            int64_t row = narrow ? (int64_t)((uint32_t)g0 / (uint32_t)S) : g0 / S;
            int64_t c = g0 - row * S + s;              // slice in the row, or in one of the next
            if (c >= S) {
                const int64_t more = S >= GEN_TS ? 1 : (int64_t)((uint32_t)c / (uint32_t)S);
                row += more;
                c -= more * S;
            }
            T* y = Yg + row * (S * Q) + c + q0 * S;
            if (NC >= VN && S == 1) {                  // rows of one slice: a thread's columns lie side by side
                typedef T Loose __attribute__((ext_vector_type(VN), aligned(sizeof(T))));
#pragma unroll
                for (int j = 0; j + VN <= NC; j += VN) {
                    Loose w;
#pragma unroll
                    for (int k = 0; k < VN; ++k) w[k] = acc[j + k];
                    *reinterpret_cast<Loose*>(y + j) = w;
                }
            } else
#pragma unroll
                for (int j = 0; j < NC; ++j) y[j * S] = acc[j];
        }
        if constexpr (!FEW) __syncthreads();           // read by everybody: the next unit may be copied
    }
}

}  // namespace km
