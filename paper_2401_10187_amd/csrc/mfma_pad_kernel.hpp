// One sliced-multiply iteration on the matrix cores for a factor of run-time shape (P, Q up to 128) that
// stays in registers: the form of the run-time-shape MFMA family (mfma_any_kernel.hpp) that most factors of
// this size take; larger ones, tall ones and those that chunked_form_wins in plan.hpp names are walked through
// LDS in chunks by the other.
//
// The contraction of a slice with the factor (Algorithm 1's inner loop) is the dense product
//     D[q][s] = sum_p F[p][q] * X[s*P + p]
// on the 16x16x4 MFMA of the element type: the factor is the A operand, slices are the B operand, one
// contraction index per lane group and step.  A workgroup has SG groups of QB wavefronts; wavefront wq of a
// group holds factor columns 16*wq .. 16*wq + 15, all P rows of them, in up to 32 registers (fp64 64) from start to
// end, and multiplies the group's BPW blocks of 16 slices out of LDS.  A tile is 16*BPW*SG consecutive
// slices, numbered through all rows, so one contiguous run of X: nothing is assumed of the row length, the
// last tile may be ragged.  Workgroups are resident and walk over their share of the tiles; the next
// tile is on its way into registers while the current one is multiplied, and moves to the other LDS buffer
// before the results are stored, so waiting for it never means waiting for this tile's stores.
//
// Bound by the matrix cores for large factors and by memory for small ones.  Whole calls, the chunked form ->
// this one, ms: 64 x 100x100^3 0.785 -> 0.451 (85 TFLOP/s, 56 % of what a large fp32 product reaches), 64 x
// 99x99^3 0.866 -> 0.450, 64 x 127x127^3 1.61 -> 1.02, 1024 x 50x50^3 0.947 -> 0.730, 512 x
// 60x60^3 0.661 -> 0.591; fp64 32 x 100x100^3 0.730 -> 0.459, 64 x 84x84^3 0.639 -> 0.501, 1024 x 33x33^3 0.544 -> 0.398, 1024 x
// 30x30^3 0.323 -> 0.214.  (fp32 steps that lane_wins in plan.hpp names are launched with a slice per lane instead.)  What
// the chunked form spends and this one does not: a second pass over LDS for the factor with every unit, two
// barriers per chunk with no load in flight behind them, and products on P padded to 16.
// Registers decide how many workgroups share a compute unit, so the kernel is compiled for four lengths of
// the contraction (one class for all took 0.70 ms for 20x20^4 and 2.7 for 1024 x 24x24^4, now 0.48 and 2.0).
//
// Step 0 holds what P leaves over a multiple of 4 (1 to 4 indices; both operands are zeroed past it, since
// what lies behind a slice may be NaN), the steps of chunk 0 what they leave over a multiple of 4 steps: all
// other chunks are four whole steps, and no product is spent on padding P further.  Columns past Q are
// computed on zeros and dropped.
// LDS rows (one slice each) have a stride of 4 times an odd number of floats, or 2 times an odd number of
// doubles, so that the 64 operand reads of a step (16 slices x 4 consecutive p) start in different banks (counters:
// 40-46 % of the LDS-active cycles are conflicts all the same, of an LDS that is active 18-32 % of the time).  What
// keeps 100x100^3 at 58 % busy matrix cores is 112 columns for 100 and seven wavefronts on four SIMDs.  Slices
// that are not whole 16-byte vectors keep the stride P, so that the tile is copied in vectors all the same (it
// starts on a 16-byte boundary): most such strides meet a bank twice, those next to a multiple of 64 four
// times, which costs less than dealing the elements to padded rows one by one (512 x 62x62^3 0.84 ms that
// way, 256 x 65x65^3 0.63).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "mfma_kernel.hpp"    // MfmaF32x16, MfmaF64x16, join_blocks
#include "plan.hpp"           // pad_shape

namespace km {

template <typename T> struct PadOp;
template <> struct PadOp<float> { typedef MfmaF32x16 OP; };
template <> struct PadOp<double> { typedef MfmaF64x16 OP; };

// Is `i` at most `last`?  (The empty asm keeps the answers from being held in scalar registers over the tiles.)
__device__ __forceinline__ bool pad_has(int i, int last)
{
    asm volatile("" : "+s"(last));
    return i <= last;
}

constexpr int PAD_STREAM = 2;              // non-temporal, as stream_load
__device__ __forceinline__ void pad_load(float& v, __amdgpu_buffer_rsrc_t rsrc, int at) { v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, at, 0, 0)); }
__device__ __forceinline__ void pad_load(double& v, __amdgpu_buffer_rsrc_t rsrc, int at) { v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsrc, at, 0, 0)); }

// WHOLE: slices are whole 16-byte vectors.  Both operands are then read by buffer loads whose resource ends where
// the operand does: what is past it comes as zero, no lane branches, and all loads of a tile go out together.  The
// first tile is asked for before the factor (in the other order its way to memory came after the factor's: 2 x
// 48x96^2 10.0 -> 9.2 us, 2064 x 64x32^2 29.4 -> 21.2, 60 x 60x60^3 82 -> 75, 32 x 100x100^3 fp64 490 -> 459).
// Slices that are not whole vectors keep the branches: without them, large problems were slower (1024 x 50x50^3
// 0.730 -> 0.810 ms, 1024 x 33x33^3 fp64 0.398 -> 0.455).  (Of the 11 % the fetch
// without branches costs most, the order and the factor's loads 2 %; on 33x33 these are the 12 %.)
// drain: wait for the next tile before the results of this one are stored, which keeps reads and writes apart in
// time; other workgroups of the compute unit use it meanwhile (us without -> with: 1000 x 44x44^3 454 -> 430, 512 x
// 60x60^3 602 -> 591, fp64 2000 x 30x30^3 556 -> 534, 1000 x 36x36^3 426 -> 418).  The long fp64 classes run one
// workgroup per compute unit or two, where hardly anybody does: 32 x 100x100^3 457 -> 509.
// (The test for the end of X inside a vector in every form of the kernel made 1024 x 24x24^4 2.66 instead of 2.01 ms.)
template <typename T, int QB, int KC, bool KEEP, bool WHOLE>
__global__ __launch_bounds__(64 * QB * pad_groups(QB), pad_waves(sizeof(T), QB, KC))
void mfma_pad_sliced_multiply(const T* __restrict__ Xg, const T* __restrict__ Fg, T* __restrict__ Yg,
                              int64_t S, int P, int Q, int rs, unsigned p_magic, unsigned s_magic,
                              int64_t num_slices, int64_t num_tiles)
{
    typedef typename PadOp<T>::OP OP;
    typedef typename Vec16<T>::type V;
    constexpr int VN = Vec16<T>::N, SG = pad_groups(QB), NT = 64 * QB * SG, BPW = pad_blocks(sizeof(T), QB, KC);
    constexpr int TS = 16 * BPW * SG, RV = pad_vectors(sizeof(T), QB, KC);
    constexpr bool drain = WHOLE && (sizeof(T) == 4 || KC <= 4);
    extern __shared__ __attribute__((aligned(16))) unsigned char pad_lds[];
    T* const lds = reinterpret_cast<T*>(pad_lds);
    const int tid = threadIdx.x, lane = tid % 64, j = lane % 16, g = lane / 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int wq = wave % QB, ws = wave / QB;
    const int steps = (P + 3) / 4, left = (P - 1) % 4 + 1;          // indices of step 0
    const int head = (steps - 1) % 4 + 1, last = (steps - 1) / 4;   // steps of chunk 0; the last chunk

    // this workgroup's tiles: the XCD (workgroup b runs on XCD b % 8) owns a contiguous part of them
    const int64_t base = num_tiles / 8, rem = num_tiles % 8, xcd = blockIdx.x % 8;
    const int64_t t_end = (xcd + 1) * base + (xcd + 1 < rem ? xcd + 1 : rem), t_step = gridDim.x / 8;
    int64_t tile = xcd * base + (xcd < rem ? xcd : rem) + blockIdx.x / 8;

    V pf[RV];
    const int tile_elems = TS * P;
    const int rounds = (tile_elems - wave * 64 * VN + NT * VN - 1) / (NT * VN);      // vectors of this wavefront's threads
    auto fetch = [&](int64_t t) {
        const T* src = Xg + t * tile_elems;
        const int64_t rest = (num_slices - t * TS) * P;
        const int valid = rest < tile_elems ? (int)rest : tile_elems;
        if constexpr (WHOLE) {
            auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), 0, valid * (int)sizeof(T), 0x00020000);
#pragma unroll
            for (int i = 0; i < RV; ++i)
                if (i == 0 || i < rounds)
                    pf[i] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (tid + i * NT) * 16, 0, PAD_STREAM));
        } else {
#pragma unroll
            for (int i = 0; i < RV; ++i) {
                const int e0 = (tid + i * NT) * VN;
                if (e0 + VN <= valid) pf[i] = stream_load(reinterpret_cast<const V*>(src + e0));
                else if (e0 < valid)                     // the end of X inside a vector
#pragma unroll
                    for (int k = 0; k < VN; ++k) pf[i][k] = e0 + k < valid ? src[e0 + k] : T(0);
            }
        }
    };
    if (tile >= t_end) return;
    if constexpr (WHOLE) fetch(tile);                    // (on its way while the factor is asked for)
    // chunk c >= 1 starts at index first + 16 * (c - 1)
    const int first = left + 4 * (head - 1);
    T a[KC][4];
    {
        const int q = wq * 16 + j;
        [[maybe_unused]] auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(Fg), 0, P * Q * (int)sizeof(T), 0x00020000);
#pragma unroll
        for (int c = 0; c < KC; ++c)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int p = (c > 0 ? first + 16 * (c - 1) + 4 * t : t > 0 ? left + 4 * (t - 1) : 0) + g;
                const bool in = q < Q && (c > 0 ? c <= last : t > 0 ? t < head : g < left);
                if constexpr (WHOLE) pad_load(a[c][t], rsrc, in ? (p * Q + q) * (int)sizeof(T) : 0x7ffffff0);    // (past the end: zero)
                else a[c][t] = in ? Fg[p * Q + q] : T(0);
            }
    }

    // vector i of a thread: element e0 of the tile, and where it goes in LDS
    int at[RV];
#pragma unroll
    for (int i = 0; i < RV; ++i) {
        const int e0 = (tid + i * NT) * VN, row = (int)__umulhi((unsigned)e0, p_magic);
        at[i] = e0 + row * (rs - P);
    }
    auto place = [&](T* buf) {
#pragma unroll
        for (int i = 0; i < RV; ++i) {
            const int e0 = (tid + i * NT) * VN;
            if (e0 < tile_elems) *reinterpret_cast<V*>(buf + at[i]) = pf[i];
        }
    };
    if constexpr (!WHOLE) fetch(tile);
    place(lds);
    if (tile + t_step < t_end) fetch(tile + t_step);
    __syncthreads();
    int cur = 0;
    for (; tile < t_end; tile += t_step) {
        const T* b = lds + cur * TS * rs + (ws * 16 * BPW + j) * rs + g;
        typename OP::Acc acc[BPW];
#pragma unroll
        for (int k = 0; k < BPW; ++k)
#pragma unroll
            for (int v = 0; v < OP::NACC; ++v) acc[k][v] = T(0);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (t == 0 || pad_has(t + 1, head)) {
                T bv[BPW];
#pragma unroll
                for (int k = 0; k < BPW; ++k) {
                    bv[k] = b[16 * k * rs + (t > 0 ? left + 4 * (t - 1) : 0)];
                    if (t == 0) bv[k] = g < left ? bv[k] : T(0);
                }
#pragma unroll
                for (int k = 0; k < BPW; ++k) acc[k] = OP::mma(a[0][t], bv[k], acc[k]);
            }
#pragma unroll
        for (int c = 1; c < KC; ++c)
            if (pad_has(c, last)) {
                T bv[4][BPW];
                const T* bc = b + first + 16 * (c - 1);
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int k = 0; k < BPW; ++k) bv[t][k] = bc[16 * k * rs + 4 * t];
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int k = 0; k < BPW; ++k) acc[k] = OP::mma(a[c][t], bv[t][k], acc[k]);
            }
        if (tile + t_step < t_end) {
            place(lds + (cur ^ 1) * TS * rs);
            if (tile + 2 * t_step < t_end) fetch(tile + 2 * t_step);
            if constexpr (drain) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }

        // permuted store: (slice s of row r, column q) -> Y[r*(S*Q) + q*S + s]
        const int64_t g0 = tile * TS, r0 = g0 / S, s0 = g0 - r0 * S;
        constexpr int PER = OP::JOIN_BLOCKS ? 2 : 1;     // blocks stored together
#pragma unroll
        for (int k = 0; k < BPW; k += PER) {
            const int mine = (ws * BPW + k) * 16 + (OP::JOIN_BLOCKS ? lane % 32 : j);      // slice of the tile
            int64_t s = s0 + mine, r = r0;
            if (s >= S) {                                // the tile goes on in the next row, or over several short ones
                const int n = s_magic ? (int)__umulhi((unsigned)s, s_magic) : S == 1 ? (int)s : 1;
                r += n;
                s -= n * S;
            }
            const bool live = g0 + mine < num_slices;
            T* Yc = Yg + r * (S * Q) + s;
#pragma unroll
            for (int v = 0; v < OP::NACC; ++v) {
                if constexpr (OP::JOIN_BLOCKS) {
                    join_blocks(acc[k], acc[k + 1], v);
                    const int q = wq * 16 + 8 * (lane / 32) + v;
                    if (live && q < Q) out_store<KEEP>(acc[k][v], &Yc[(int64_t)q * S]);
                    if (live && q + 4 < Q) out_store<KEEP>(acc[k + 1][v], &Yc[(int64_t)(q + 4) * S]);
                } else {
                    const int q = wq * 16 + OP::row_lane(lane) + OP::row_reg(v);
                    if (live && q < Q) out_store<KEEP>(acc[k][v], &Yc[(int64_t)q * S]);
                }
            }
        }
        __syncthreads();      // the other buffer is complete; this one has been read by everybody
        cur ^= 1;
    }
}

}  // namespace km
