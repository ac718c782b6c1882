// One sliced-multiply iteration on the matrix cores, fp32, one slice per lane: the form of the run-time-shape MFMA family
// (mfma_any_kernel.hpp) for factors of up to 128 rows and columns on many slices.
//
// The contraction of a slice with the factor (Algorithm 1's inner loop),
//     D[q][s] = sum_p F[p][q] * X[s*P + p],
// on the 4x4x1 MFMA: sixteen blocks of four columns times four slices at a time, one contraction index each.  With the
// factor as the A operand and one block of it broadcast to all sixteen (cbsz 4, abid the block), the sixteen blocks are
// 64 slices, one per lane, times four columns: P needs no padding at all, Q only to a multiple of 4, where the 16x16x4
// instruction computes 16 columns for what is left of them (112 for 100, 80 for 65).  Its rate is the larger one's: 144 TFLOP/s
// on ordinary numbers, 135 of 16x16x4, both at the clock that power allows.
//
// A wavefront takes tiles of 64 consecutive slices, numbered through all rows, one contiguous run of X, and needs no
// other wavefront: its slices go through registers into LDS of its own, U vectors of each at a time (a chunk; LANE_U says
// which), while the next chunk, of this tile or the next one, is on its way into registers.  A lane then reads its own
// slice vector by vector and multiplies all columns of it, 4G accumulators; the factor lies in LDS as [vector of P][column], so that
// its operands are one read per 64 columns and four indices.  Slices that are no whole vectors are read in unaligned
// ones; the last vector of a slice is always P - 4 .. P - 1, and what it shares with the one before is not multiplied again,
// so nothing is read past a slice and nothing but the slice's own elements ever meets the factor.  The last chunk may likewise
// start inside the one before.
// Results: lanes are renumbered, slice 4 * (lane % 16) + lane / 16, so that exchanging lane groups of 16 and 32 (four swaps
// for four registers) leaves a lane with four consecutive slices of one column: 16-byte stores, and a quarter as many (a
// wavefront has at most 63 memory operations outstanding; 100 stores of 4 bytes after each tile held it up for 13000
// of 48000 cycles).  Tiles that leave a row, and the last one, store element by element.
//
// Bound by memory for P, Q up to 50 and by the power that matrix cores and memory draw together above.  Whole calls, the
// other forms -> this one, us: 256 x 65x65^3 689 -> 481 (88 TFLOP/s), 256 x 72x72^3 853 -> 576, 2048 x 36x36^3 496 -> 449 (5.1 TB/s),
// 1024 x 24x24^4 2014 -> 1888; against the generic kernel's small form 6 x 10x5^7 244 -> 144.  lane_wins in plan.hpp says where it is
// taken: for 100x100 the form with the factor in registers stays, 152 us a launch in a chain and 157 here.
// What follows was measured by launches repeated on one X, part of which the last-level cache then holds, and compares
// variants of this kernel only.  Chunk lengths as template parameters: with one length for all classes and the run-time length
// beside it 100x100 took 172 us instead of 142 and 24x24 141 instead of 120.  Non-persistent workgroups, the dispatcher evens
// the chip out: 24x24 in one round of resident workgroups 129, one tile per wavefront 120; with factors of more than 32 columns,
// whose way into LDS costs more, two tiles per wavefront (100x100: one 152, two 142, three 157; 50x50: 229 and 225).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "plan.hpp"           // lane_units, lane_waves

namespace km {

typedef float lane_vec __attribute__((ext_vector_type(4)));
typedef float lane_vec_any __attribute__((ext_vector_type(4), aligned(4)));     // at any element

// One contraction index: G groups of four columns, group n from block n % 16 of operand register n / 16.
template <int G>
__device__ __forceinline__ void lane_products(lane_vec (&acc)[G], const lane_vec* f, float x, int t)
{
#define KM_LANE(n) if constexpr (n < G) acc[n] = __builtin_amdgcn_mfma_f32_4x4x1f32(f[n / 16][t], x, acc[n], 4, n % 16, 0);
    KM_LANE(0) KM_LANE(1) KM_LANE(2) KM_LANE(3) KM_LANE(4) KM_LANE(5) KM_LANE(6) KM_LANE(7)
    KM_LANE(8) KM_LANE(9) KM_LANE(10) KM_LANE(11) KM_LANE(12) KM_LANE(13) KM_LANE(14) KM_LANE(15)
    KM_LANE(16) KM_LANE(17) KM_LANE(18) KM_LANE(19) KM_LANE(20) KM_LANE(21) KM_LANE(22) KM_LANE(23)
    KM_LANE(24) KM_LANE(25) KM_LANE(26) KM_LANE(27) KM_LANE(28) KM_LANE(29) KM_LANE(30) KM_LANE(31)
#undef KM_LANE
}

// Four registers x four groups of 16 lanes, transposed.
__device__ __forceinline__ lane_vec lane_transpose(lane_vec d)
{
    auto swap = [](float& a, float& b, bool far) {
        const auto w = far ? __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false)
                           : __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(w[0]);
        b = __uint_as_float(w[1]);
    };
    float d0 = d[0], d1 = d[1], d2 = d[2], d3 = d[3];
    swap(d0, d2, true);
    swap(d1, d3, true);
    swap(d0, d1, false);
    swap(d2, d3, false);
    return lane_vec{d0, d1, d2, d3};
}

// S_magic: lane_row_magic(S); s_magic: 2^32 / S rounded up where a tile holds several rows (1 < S < 64), else 0.
template <int G, int U>
__global__ __launch_bounds__(LANE_THREADS, lane_waves(G, U))
void mfma_lane_sliced_multiply(const float* __restrict__ Xg, const float* __restrict__ Fg, float* __restrict__ Yg, int64_t S, int P,
                               int Q, int chunks, uint64_t S_magic, unsigned s_magic, int64_t num_slices, int64_t num_tiles, int keep)
{
    constexpr int NR = (G + 15) / 16, NW = LANE_THREADS / 64, US = U | 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char lane_lds[];
    const int tid = threadIdx.x, lane = tid % 64, mine = lane % 16 * 4 + lane / 16;      // this lane's slice of a tile
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int units = (P + 3) / 4, left = P % 4, whole = left ? units - 1 : units;
    lane_vec* const fl = reinterpret_cast<lane_vec*>(lane_lds);
    lane_vec* const xl = fl + units * 4 * G + wave * 64 * US;

    // this workgroup's groups of NW tiles: the XCD (workgroup b runs on XCD b % 8) owns a contiguous part of them
    const int64_t groups = (num_tiles + NW - 1) / NW, base = groups / 8, rem = groups % 8, xcd = blockIdx.x % 8;
    const int64_t g_end = (xcd + 1) * base + (xcd + 1 < rem ? xcd + 1 : rem), g_step = gridDim.x / 8;
    int64_t group = xcd * base + (xcd < rem ? xcd : rem) + blockIdx.x / 8;
    if (group >= g_end) return;

    lane_vec next[U];
    auto fetch = [&](int64_t t, int c) {
        if (t >= num_tiles) return;
        const float* src = Xg + t * (64 * (int64_t)P);
        const int last = t + 1 < num_tiles ? 63 : (int)(num_slices - t * 64) - 1;        // (slices past the last one: that one again)
        const int u0 = c * U < units - U ? c * U : units - U;
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int e = i * 64 + lane, row = e / U, p = 4 * (e % U + u0);
            next[i] = *reinterpret_cast<const lane_vec_any*>(src + ((row < last ? row : last) * P + (p < P - 4 ? p : P - 4)));
        }
    };
    auto place = [&]() {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int e = i * 64 + lane;
            xl[e + e / U * (US - U)] = next[i];
        }
    };

    fetch(group * NW + wave, 0);
    // the factor: vector u of column q holds rows 4u .. 4u + 3 (the last one P - 4 .. P - 1)
    constexpr int FB = G > 16 ? 5 : G > 8 ? 3 : 1;       // loads in flight before the first is stored
    for (int i0 = tid; i0 < units * 4 * G; i0 += LANE_THREADS * FB) {
        lane_vec v[FB];
#pragma unroll
        for (int k = 0; k < FB; ++k) {
            const int i = i0 + LANE_THREADS * k, u = i / (4 * G), q = i % (4 * G), p = u * 4 < P - 4 ? u * 4 : P - 4;
            if (i < units * 4 * G)
#pragma unroll
                for (int t = 0; t < 4; ++t) v[k][t] = Fg[(p + t) * Q + (q < Q ? q : Q - 1)];     // (columns past Q are dropped)
        }
#pragma unroll
        for (int k = 0; k < FB; ++k)
            if (i0 + LANE_THREADS * k < units * 4 * G) fl[i0 + LANE_THREADS * k] = v[k];
    }
    __syncthreads();
    int column[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) column[r] = 64 * r + lane < 4 * G ? 64 * r + lane : 4 * G - 1;

    place();
    int64_t ng = group;                                  // what is fetched next: chunk nc of this wavefront's tile in group ng
    int nc = 1;
    if (nc == chunks) { nc = 0; ng += g_step; }
    if (ng < g_end) fetch(ng * NW + wave, nc);
    for (; group < g_end; group += g_step) {
        const int64_t tile = group * NW + wave;
        lane_vec acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = lane_vec{0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < chunks; ++c) {
            const int u0 = c * U < units - U ? c * U : units - U, stop = c + 1 < chunks ? u0 + U : whole;
            const lane_vec* xr = xl + mine * US - u0;
            // (the wavefront's LDS operations run in order; this keeps the compiler from moving reads ahead of place())
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            lane_vec x0, x1, f0[NR], f1[NR];
            auto take = [&](int u, lane_vec& x, lane_vec* f) {
                const int v = u < u0 + U ? u : u0 + U - 1;
                x = xr[v];
#pragma unroll
                for (int r = 0; r < NR; ++r) f[r] = fl[v * 4 * G + column[r]];
            };
            // two sets of operands in turn, one on its way while the other is multiplied
            int u = c * U;
            take(u, x0, f0);
            while (u < stop) {
                take(u + 1, x1, f1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 4; ++t) lane_products<G>(acc, f0, x0[t], t);
                if (++u >= stop) {
                    x0 = x1;
#pragma unroll
                    for (int r = 0; r < NR; ++r) f0[r] = f1[r];
                    break;
                }
                take(u + 1, x0, f0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 4; ++t) lane_products<G>(acc, f1, x1[t], t);
                ++u;
            }
            if (c + 1 == chunks && left) {               // the last vector: its last P % 4 elements
                if (left > 2) lane_products<G>(acc, f0, x0[1], 1);
                if (left > 1) lane_products<G>(acc, f0, x0[2], 2);
                lane_products<G>(acc, f0, x0[3], 3);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (ng < g_end) {
                if (ng * NW + wave < num_tiles) place();
                if (++nc == chunks) { nc = 0; ng += g_step; }
                if (ng < g_end) fetch(ng * NW + wave, nc);
            }
        }
        if (tile >= num_tiles) continue;

        // permuted store: (slice s of row r, column q) -> Y[r*(S*Q) + q*S + s]
        const int64_t g0 = tile * 64, r0 = S == 1 ? g0 : (int64_t)__umul64hi((uint64_t)g0, S_magic), s0 = g0 - r0 * S;
        if (s0 + 64 <= S && g0 + 64 <= num_slices) {
            const int column0 = lane / 16;
            float* y = Yg + r0 * (S * Q) + s0 + lane % 16 * 4 + column0 * S;
            // (the empty asm keeps the compiler from merging the two forms, with ordinary stores, and from exchanging lanes for
            // all groups ahead of the branch, which takes as many registers again)
            if (keep) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    asm volatile("; ordinary" : "+v"(acc[g]));
                    const lane_vec d = lane_transpose(acc[g]);
                    if (g + 1 < G || 4 * g + column0 < Q) *reinterpret_cast<lane_vec_any*>(y) = d;
                    y += 4 * S;
                }
            } else {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    asm volatile("; non-temporal" : "+v"(acc[g]));
                    const lane_vec d = lane_transpose(acc[g]);
                    if (g + 1 < G || 4 * g + column0 < Q) __builtin_nontemporal_store(d, reinterpret_cast<lane_vec_any*>(y));
                    y += 4 * S;
                }
            }
            continue;
        }
        int64_t s = s0 + mine, r = r0;
        if (s >= S) {                                    // the tile goes on in the next row, or over several short ones
            const int n = s_magic ? (int)__umulhi((unsigned)s, s_magic) : S == 1 ? (int)s : 1;
            r += n;
            s -= n * S;
        }
        if (g0 + mine < num_slices) {
            float* y = Yg + r * (S * Q) + s;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (g + 1 < G || v == 0 || 4 * g + v < Q) { *y = acc[g][v]; y += S; }
        }
    }
}

}  // namespace km
