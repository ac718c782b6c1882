// Every factor of a Kron-Matmul applied to a short row inside one launch, on the matrix cores, for problems
// of few rows, which are bound by latency: by how long one workgroup takes from its start to its end.
//
// As in row_kernel.hpp the whole row is the tile, one workgroup per row: it loads the row of X, applies factor N, N-1,
// ..., 1 by the rule of Algorithm 1 (slice s times column q goes to q*(K/P) + s) between two LDS buffers
// and writes the row of Y; factor shapes are run-time values.  A step is the dense product
// D[q][s] = sum_p F[p][q] * X[s*P + p] on the 16x16x4 MFMA of the element type: the factor is the A operand
// (rows q), slices are the B operand (columns s), one contraction index per lane group and MFMA (p = 4t + g).
// A unit is one 16x16 block of the result, units of one factor column block following each other; a wavefront
// takes a run of them, so that it seldom changes its columns of the factor.
//
// What keeps the chain of latencies short: the A operand of a unit is read straight from global memory
// into registers, and the loads of the next step's first unit are issued among this step's products, so a
// factor costs neither a pass through LDS nor a memory latency of its own; the first step's are in flight
// together with the row's.  Where rows are few the B operands of a unit are all read before its first product, and the
// last step's results go straight to Y instead of through LDS, a barrier and a read.  What remains of a step, some 2000 cycles for a unit
// whose products take 500, is instructions one after the other: the host works out all that depends on the shapes alone, a
// step's numbers are one cache line of the arguments.  No loop holds a division.  Contraction indices past P are zeroed in both
// operands (what lies behind a slice may be NaN); rows q and columns s past the ends are computed on clamped
// addresses and dropped.
// Bound by latency: 10 x (52x50, 65x20), two steps, takes 5.0 us from launch to launch on a stream where an empty launch
// takes 1.6 (5.8 before the three things above: 11 x 50x50^2 7.3 -> 6.4, 2 x 80x80^2 10.4 -> 9.3, 280 x (5x4, 4x17)
// 4.8 -> 4.1; 13.6 on the FMA kernel, whose factors go through LDS and whose 130 busy threads add up 117
// products one after the other; fp64 20.1 -> 6.7 against two launches); 200 x 50x50^2 20.0 -> 6.7 (9.3 in two launches
// of the factor-in-register kernel), 33 x 80x80^2 20.2 -> 9.7, 300 x (32x32, 64x3) 19.9 -> 4.7, 5 x (111x82, 7x9)
// 14.9 -> 5.2.  Sixteen wavefronts when units are many or rows few, four (four rows to a compute unit) otherwise; a
// first version with the factors in LDS took 8.7 us on the first of these, 1.2 of it staging them, and a loop over
// rows around all of it 0.4 us more on every problem, though it ran once.
// Slices of a multiple of 8 elements are padded by 4 in LDS, which spreads the 64 operand reads of an MFMA
// (16 slices x 4 consecutive p) over the banks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "mfma_kernel.hpp"                 // MfmaF32x16, MfmaF64x16, Vec16, stream_load, stream_store
#include "plan.hpp"                        // rowm_slice_stride, RowmShape

namespace km {

template <typename T> struct RowmOp;
template <> struct RowmOp<float> { typedef MfmaF32x16 OP; };
template <> struct RowmOp<double> { typedef MfmaF64x16 OP; };

// One factor's step, in order of application (last factor of the product first), with what the host can work out of it.
struct alignas(64) RowmStep {
    const void* f;
    int P, Q, S;                           // S: slices of the row the step reads
    int units, share;                      // 16x16 blocks of its result; those of a wavefront
    unsigned blocks_magic;                 // unit / slice blocks = (unit * blocks_magic) >> 32
    int blocks;                            // slice blocks
    int first, last, last_round;           // contraction indices of chunk 0, 1 to 16; the last chunk; the last round
    int stride;                            // of the slices in LDS
    unsigned out_magic;                    // c / P of the next step if its slices are padded (0: they are not): (c * out_magic) >> 32
};
struct RowmArgs {
    RowmStep step[ROWM_MAXF];
    unsigned in_magic;                     // out_magic for the row of X
    int n;
    int buf_elems;                         // elements of one row buffer; the second one follows it
};

// factor column block of a unit
__device__ __forceinline__ int rowm_column_block(const RowmStep& st, int unit)
{
    return st.blocks == 1 ? unit : (int)__umulhi((unsigned)unit, st.blocks_magic);
}

// position in LDS of element c of a row that is read in slices of P elements
__device__ __forceinline__ int rowm_at(int c, unsigned magic) { return magic ? c + 4 * (int)__umulhi((unsigned)c, magic) : c; }

// Is there a chunk c (of chunks 0 to `last`)?  The empty asm keeps the answers from being held in
// scalar registers over a loop: asking costs one instruction.
__device__ __forceinline__ bool rowm_chunk(int c, int last)
{
    asm volatile("" : "+s"(last));
    return c <= last;
}

// Contraction indices are taken in chunks of 16, the first one holding what P leaves over (1 to 16 of them).
// The operand registers hold ROWM_CHUNKS chunks; a longer contraction takes as many rounds of them.
//
// Where a wavefront finds the A operand of a unit: element t of lane group g in chunk c is row
// p = first + 16(c - 1) + 4t + g (4t + g in chunk 0) of factor column q, `step` bytes apart for each t.
struct RowmOperand {
    __amdgpu_buffer_rsrc_t rsrc;
    int at, next, step, last;              // byte offsets in the round's first chunk and in the second one; the last chunk (-1: no unit)
};
template <typename T>
__device__ __forceinline__ RowmOperand rowm_operand(const RowmStep& st, int unit, int round, int j, int g)
{
    const int q = rowm_column_block(st, unit) * 16 + j, row = st.Q * (int)sizeof(T);
    RowmOperand o;
    // (elements past the factor's last row, which chunk 0 may ask for, are past the end of the resource and read as zero)
    o.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(st.f), 0, st.P * row, 0x00020000);
    o.at = g * row + (q < st.Q ? q : st.Q - 1) * (int)sizeof(T);
    o.step = 4 * row;
    o.next = o.at + (st.first + round * ROWM_CHUNKS * 16) * row;
    if (round > 0) o.at = o.next - 16 * row;
    const int last = st.last - round * ROWM_CHUNKS;
    o.last = last < ROWM_CHUNKS ? last : ROWM_CHUNKS - 1;
    return o;
}
__device__ __forceinline__ void rowm_load(float& v, const RowmOperand& o, int at)
{
    v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(o.rsrc, at, 0, 0));
}
__device__ __forceinline__ void rowm_load(double& v, const RowmOperand& o, int at)
{
    v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(o.rsrc, at, 0, 0));
}
// chunk c of the operand (chunks are asked for in order)
template <typename T>
__device__ __forceinline__ void rowm_load_chunk(T (&a)[4], RowmOperand& o, int c)
{
    if (c == 1) o.at = o.next;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        rowm_load(a[t], o, o.at);
        o.at += o.step;
    }
}

template <typename T, int NW>
__global__ __launch_bounds__(NW * 64, NW / 4)
void row_mfma_sliced_multiply(const T* __restrict__ Xg, T* __restrict__ Yg, int k_in, int k_out, const RowmArgs ra)
{
    typedef typename RowmOp<T>::OP OP;
    typedef typename Vec16<T>::type V;
    constexpr int VN = Vec16<T>::N, NT = NW * 64, KC = ROWM_CHUNKS;
    extern __shared__ __attribute__((aligned(16))) unsigned char rowm_lds[];
    T* const lds = reinterpret_cast<T*>(rowm_lds);
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);

    const int64_t row = blockIdx.x;
    const int j = lane % 16, g = lane / 16;
    T a[KC][4];                                      // A operand of the wavefront's next unit
    if (wave * ra.step[0].share < ra.step[0].units) {
        RowmOperand o = rowm_operand<T>(ra.step[0], wave * ra.step[0].share, 0, j, g);
#pragma unroll
        for (int c = 0; c < KC; ++c)
            if (rowm_chunk(c, o.last)) rowm_load_chunk(a[c], o, c);
    }
    {
        const T* src = Xg + row * k_in;
        const unsigned magic = ra.in_magic;
        if (k_in % VN == 0) {                        // (a padded slice is a multiple of 8 elements: a vector stays inside it)
            for (int c0 = tid * VN; c0 < k_in; c0 += 4 * NT * VN) {
                V v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c0 + i * NT * VN < k_in) v[i] = stream_load(reinterpret_cast<const V*>(src + c0 + i * NT * VN));
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c0 + i * NT * VN < k_in) *reinterpret_cast<V*>(lds + rowm_at(c0 + i * NT * VN, magic)) = v[i];
            }
        } else {
            for (int c0 = tid; c0 < k_in; c0 += 4 * NT) {
                T v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c0 + i * NT < k_in) v[i] = src[c0 + i * NT];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c0 + i * NT < k_in) lds[rowm_at(c0 + i * NT, magic)] = v[i];
            }
        }
    }
    __syncthreads();

    T* buf = lds;
    T* out = lds + ra.buf_elems;
    // The last step's results go straight to Y with sixteen wavefronts or a short row, else through LDS in whole vectors (922 x
    // 50x50^2 fp64 24.7 us straight, 23.9 through LDS; 280 x (5x4, 4x17) 4.3 and 4.6; sixteen wavefronts with both ways compiled in
    // 2 % slower throughout).
    const bool straight = NW == 16 || k_out * (int)sizeof(T) <= 8192;
    for (int i = 0; i < ra.n; ++i) {
        const RowmStep st = ra.step[i];
        const bool more = i + 1 < ra.n;
        const RowmStep& nx = ra.step[more ? i + 1 : i];
        const int begin = wave * st.share, share = begin + st.share, end = share < st.units ? share : st.units;
        for (int unit = begin; unit < end; ++unit) {
            const int qb = rowm_column_block(st, unit);
            const int s = (unit - qb * st.blocks) * 16 + j;
            const T* b = buf + (s < st.S ? s : st.S - 1) * st.stride + g;
            typename OP::Acc acc;
#pragma unroll
            for (int v = 0; v < OP::NACC; ++v) acc[v] = T(0);
            for (int round = 0; round <= st.last_round; ++round) {
                // Rows that have their compute unit to themselves: the round's B operands are all asked for before the first product,
                // one LDS latency (four rows to a unit hide it from each other, and it would cost them registers).
                constexpr bool AHEAD = NW == 16;
                const T* from = b + (st.first + 16 * (round * KC - 1));      // chunk c: 16c elements on
                const int here = st.last - round * KC;
                T bv[KC][4];
                if (round == 0) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) bv[0][t] = b[4 * t + g < st.first ? 4 * t : 0];
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t) bv[0][t] = from[4 * t];
                }
#pragma unroll
                for (int c = 1; c < KC; ++c)
                    if (AHEAD && rowm_chunk(c, here))
#pragma unroll
                        for (int t = 0; t < 4; ++t) bv[c][t] = from[16 * c + 4 * t];
                if (round == 0) {
                    // (the empty asm keeps the reads out of branches of their own)
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        asm volatile("" : "+v"(bv[0][t]));
                        if (4 * t + g >= st.first) { bv[0][t] = T(0); a[0][t] = T(0); }
                    }
                }
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (t == 0 || round > 0 || rowm_chunk(4 * t + 1, st.first)) acc = OP::mma(a[0][t], bv[0][t], acc);
                // What comes next (this unit's next round, the next unit of this step, the first one of the next
                // step) takes the operand registers as the products free them.
                RowmOperand o;
                o.last = -1;
                if (round < st.last_round) {
                    o = rowm_operand<T>(st, unit, round + 1, j, g);
                } else if (unit + 1 < end) {         // (the same columns of the factor: it has the operand already)
                    if (st.last_round > 0 || rowm_column_block(st, unit + 1) != qb) o = rowm_operand<T>(st, unit + 1, 0, j, g);
                } else if (more && wave * nx.share < nx.units) {
                    o = rowm_operand<T>(nx, wave * nx.share, 0, j, g);
                }
                if (rowm_chunk(0, o.last)) rowm_load_chunk(a[0], o, 0);
#pragma unroll
                for (int c = 1; c < KC; ++c) {
                    if (rowm_chunk(c, here)) {
                        if (!AHEAD)
#pragma unroll
                            for (int t = 0; t < 4; ++t) bv[c][t] = from[16 * c + 4 * t];
#pragma unroll
                        for (int t = 0; t < 4; ++t) acc = OP::mma(a[c][t], bv[c][t], acc);
                    }
                    if (rowm_chunk(c, o.last)) rowm_load_chunk(a[c], o, c);
                }
            }
            if (more || !straight) {
#pragma unroll
                for (int v = 0; v < OP::NACC; ++v) {
                    const int q = qb * 16 + OP::row_lane(lane) + OP::row_reg(v);
                    if (q < st.Q && s < st.S) out[rowm_at(q * st.S + s, st.out_magic)] = acc[v];
                }
            } else {
                T* y = Yg + row * k_out + s;
#pragma unroll
                for (int v = 0; v < OP::NACC; ++v) {
                    const int q = qb * 16 + OP::row_lane(lane) + OP::row_reg(v);
                    if (q < st.Q && s < st.S) y[q * st.S] = acc[v];
                }
            }
        }
        if (!more && straight) return;
        if (more && begin >= end && wave * nx.share < nx.units) {        // idle in this step
            RowmOperand o = rowm_operand<T>(nx, wave * nx.share, 0, j, g);
#pragma unroll
            for (int c = 0; c < KC; ++c)
                if (rowm_chunk(c, o.last)) rowm_load_chunk(a[c], o, c);
        }
        __syncthreads();
        T* other = buf; buf = out; out = other;
    }

    T* dst = Yg + row * k_out;
    if (k_out % VN == 0) {
        for (int c = tid * VN; c < k_out; c += NT * VN) stream_store(*reinterpret_cast<const V*>(buf + c), reinterpret_cast<V*>(dst + c));
    } else {
        for (int c = tid; c < k_out; c += NT) dst[c] = buf[c];
    }
}

}  // namespace km
