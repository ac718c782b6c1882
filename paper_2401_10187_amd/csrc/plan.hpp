// Host-side planner: turns a problem (M, factor shapes, dtype) into the list of kernel launches
// that evaluates Algorithm 1, last factor first, and assigns the buffers the launches read and
// write (the two swapped intermediates of Algorithm 1; Y stands in for one of them when it is wide
// enough, and the first launch reads X in place).  Pure host code, no HIP calls.
#pragma once
#include <stdint.h>
#include <stddef.h>
#include <vector>
#include "../../include/kronmatmul.h"

namespace km {

// One compiled kernel instance the planner can choose.
struct Variant {
    int kernel;        // km_kernel family
    int dtype;         // km_dtype
    int P, Q;          // factor shape it is compiled for (0 = any)
    int num_factors;   // factors per launch
    int tile_slices;   // S_t: run of consecutive output columns a tile produces per fused column
    int threads;       // workgroup size
    int lds_bytes;     // LDS per workgroup
    int rows_per_tile; // rows of X a workgroup handles together
    int persistent;    // >0: a workgroup walks over several tiles (see tiles_per_wg); 1: in any of the
                       // three tile orders, 2: contiguous or grid-strided only
    int flexible;      // 1: tile_slices is an upper limit; the launch picks a divisor of K/prod(P)
    float slowdown;    // measured cost relative to an HBM-bound launch of the same bytes (planner weight)
    const char* name;
    int lds_per_slice; // flexible instances: LDS bytes per slice of the tile (lds_bytes is the maximum)
    int thread_elems;  // flexible instances: contiguous elements of a tile that one thread multiplies first
    int max_srow;      // > 0: only for rows of at most this many slices of the group (K / prod P)
    int min_tiles;     // > 0: only planned for launches of at least this many tiles (the tuner still tries it)
    int walk;          // > 0: tiles per workgroup of a persistent instance, instead of the rule of tiles_per_wg();
                       // -1: as many as make the grid one round of the workgroups the chip holds at once
    int xcd_order;     // 1: persistent instance that prefers tile order 3 (each XCD walks its own eighth of the tiles)
    int lds_slack;     // flexible instances: LDS bytes a launch needs on top of lds_per_slice * tile_slices
    int mix[9];        // instances whose stages have their own factor shapes: (P, Q, factors) of up to three
                       // stages in order of application (P, Q above are the first stage's); all 0 otherwise
    int simd_waves;    // > 0: wavefronts that the instance's registers leave room for on a SIMD
};

// Do factors [f - nf + 1, f] (applied from f downwards) have the shapes instance c is compiled for?
inline bool shapes_match(const Variant& c, const std::vector<int>& P, const std::vector<int>& Q, int f, int nf)
{
    if (c.num_factors != nf) return false;
    if (c.mix[2] == 0) {                                  // one shape for every factor of the group
        for (int i = f - nf + 1; i <= f; ++i)
            if (P[i] != c.P || Q[i] != c.Q) return false;
        return true;
    }
    int at = f;
    for (int j = 0; j < 3; ++j)
        for (int k = 0; k < c.mix[3 * j + 2]; ++k, --at)
            if (at < f - nf + 1 || P[at] != c.mix[3 * j] || Q[at] != c.mix[3 * j + 1]) return false;
    return at == f - nf;
}

// LDS a launch of the instance asks for when its tiles hold `tile_slices` slices.
inline int launch_lds_bytes(const Variant& c, int tile_slices)
{
    if (!c.flexible || c.lds_per_slice <= 0) return c.lds_bytes;
    const int64_t b = ((int64_t)c.lds_per_slice * tile_slices + 15) / 16 * 16 + c.lds_slack;
    return b < c.lds_bytes ? (int)b : c.lds_bytes;
}

// Tiles handled by one workgroup of a persistent instance; `hint` > 0 forces the value.
// Measured with the autotuner on this chip: a workgroup loads its factors once, so with large
// factors (16 KB and more) long walks pay (64x64 fp32: walks of 32-64 tiles are 7 % faster than
// walks of 5), while with small factors every tile beyond the amortisation point costs workgroups
// in flight (16x16: walks of 3-4 tiles are 10 % slower than one tile per workgroup).  Walks are
// powers of two so that the usual power-of-two tile counts split evenly over the grid.
// Instances that fill most of a compute unit's LDS run one or two workgroups per unit and need the
// walk to overlap their loads with their stores: at least 4 tiles above 64 KB, 32 above 80 KB.
inline int64_t tiles_per_wg(int64_t num_tiles, int hint, int64_t factor_elems, int64_t tile_elems,
                            int lds_bytes, size_t esize, int instance_walk = 0)
{
    if (hint > 0) return hint;
    const int64_t want = (10 * factor_elems + tile_elems - 1) / tile_elems;
    int64_t t = 1;
    while (t < want && t < 32) t *= 2;
    if ((size_t)factor_elems * esize >= 16 * 1024) t = 32;
    if (lds_bytes > 64 * 1024 && t < 4) t = 4;
    if (lds_bytes > 80 * 1024) t = 32;
    if (instance_walk > 0) t = instance_walk;          // measured per instance
    // two workgroups per compute unit at least; four when the instance is light (small factor, at most
    // 64 KB of LDS): 1024 x 64x64^2 is 28 % faster with 1024 workgroups than with 512; but one per unit
    // is enough when loading the factor costs a workgroup as much as a tile does (16 x 64x64^3 fp64:
    // 256 workgroups walking 4 tiles each are 28 % faster than 1024 with one tile)
    const bool heavy = (size_t)factor_elems * esize >= 64 * 1024 || lds_bytes > 64 * 1024;
    // (factors of 16 KB and more: with 32x32 factors, whose tiles are as large as the factor too, four
    // workgroups per unit win again: 4096 x 32x32^2 fp64 0.044 -> 0.027 ms, 16 x 32x32^3 0.014 -> 0.011)
    const int64_t fewest = heavy ? 512 : ((size_t)factor_elems * esize >= 16 * 1024 && factor_elems >= tile_elems ? 256 : 1024);
    while (t > 1 && num_tiles / t < fewest) t /= 2;
    return t;
}

struct Problem {
    int64_t M = 0;
    int N = 0;
    std::vector<int> P, Q;
    int dtype = 0;
    int64_t k_in = 1, k_out = 1;   // prod P, prod Q
    size_t esize = 4;
};

struct Plan {
    std::vector<km_plan_step> steps;
    size_t ws0_bytes = 0, ws1_bytes = 0;   // the two intermediates (ws1 unused when Y can serve)
    double flops = 0, bytes = 0;
};

struct Options {
    int kernels = 0x37;   // bit mask of km_kernel families
    int max_fuse = 16;
    int prefer_tile = 0;      // tuning: choose instances with this tile_slices when one fits
    int prefer_threads = 0;   // tuning: ... with this workgroup size
    int tiles_per_wg = 0;     // tuning: tiles per workgroup of persistent instances (0 = automatic)
    int pair_interleave = 1;  // neighbouring tiles with short output runs go to workgroup pairs
    int prefer_instance = 0;  // tuning: k > 0 = take compiled instance k - 1 wherever it fits
    int tile_order = -1;      // persistent kernels: 0 = contiguous tile ranges, 2 = tiles strided by the grid,
                              // 3 = strided inside the XCD's own eighth of the tiles, -1 = the instance's
                              // preference (3 where it asks for it and the tiles split by 8, else 2)
};

inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

#if defined(__HIPCC__)
#define KM_HOST_DEVICE __host__ __device__
#else
#define KM_HOST_DEVICE
#endif
// A run of `valid` elements that starts `mis` elements (0 <= mis < vn) above a 16-byte boundary is
// moved in vectors of vn elements counted from that boundary: unaligned_vectors() of them touch the
// run; the first unaligned_whole_vectors() are loaded or stored whole.  Those lie inside
// [-mis, valid): the elements below the run exist whenever mis > 0 (buffers start on 16-byte
// boundaries), so a whole vector never leaves the buffer.  What is left, the part of the last vector
// that belongs to the run, is moved element by element.
KM_HOST_DEVICE inline int unaligned_vectors(int valid, int mis, int vn) { return (valid + mis + vn - 1) / vn; }
KM_HOST_DEVICE inline int unaligned_whole_vectors(int valid, int mis, int vn) { return (valid + mis) / vn; }

// Validates the shapes and fills the derived sizes.  Products must stay below 2^62 elements.
inline km_status make_problem(int M, int N, const int* P, const int* Q, int dtype, Problem& pr)
{
    if (M < 0 || N < 1 || N > 64 || !P || !Q) return KM_EINVAL;
    if (dtype != KM_F32 && dtype != KM_F64) return KM_EINVAL;
    pr.M = M; pr.N = N; pr.dtype = dtype; pr.esize = dtype == KM_F32 ? 4 : 8;
    pr.P.assign(P, P + N); pr.Q.assign(Q, Q + N);
    const int64_t lim = (int64_t)1 << 40;   // elements per row; M * width * esize must fit in int64
    int64_t kin = 1, kout = 1;
    for (int i = 0; i < N; ++i) {
        if (P[i] < 1 || Q[i] < 1) return KM_EINVAL;
        if (kin > lim / P[i] || kout > lim / Q[i]) return KM_EINVAL;
        kin *= P[i]; kout *= Q[i];
    }
    // every intermediate width Q_N..Q_f * P_1..P_{f-1}
    int64_t w = kin;
    for (int f = N - 1; f >= 0; --f) {
        w = w / P[f];
        if (w > lim / Q[f]) return KM_EINVAL;
        w *= Q[f];
        if (M > 0 && w > ((int64_t)1 << 59) / M) return KM_EINVAL;
    }
    if (M > 0 && kin > ((int64_t)1 << 59) / M) return KM_EINVAL;
    pr.k_in = kin; pr.k_out = kout;
    return KM_OK;
}

// Output column of local element c of tile `tile_index` after a fused group (section 4.2): the
// tile's final contents are ordered (fused column qq, slice r) with r < S_t = tile_k / p_group, and
// the row of the intermediate holds, for each qq, all K_in / p_group slices contiguously.
inline int64_t store_column(int64_t k_in, int64_t p_group, int64_t tile_k, int64_t tile_index,
                            int64_t local_col)
{
    if (k_in <= 0 || p_group <= 0 || tile_k <= 0 || k_in % p_group || tile_k % p_group ||
        k_in % tile_k || tile_index < 0 || tile_index >= k_in / tile_k || local_col < 0)
        return -1;
    const int64_t s_tile = tile_k / p_group;      // slices of the fused group inside the tile
    const int64_t s_row = k_in / p_group;         // ... inside the whole row
    const int64_t qq = local_col / s_tile;
    const int64_t r = local_col % s_tile;
    return qq * s_row + tile_index * s_tile + r;
}

// Column blocks (of 16) per unit of the run-time-shape MFMA kernel for a factor with Q columns: one or
// two for factors that narrow, else the width among 4, 5 and 3 that leaves the fewest padded blocks
// (narrower units would re-read the slices once per 16 or 32 columns).
constexpr int any_column_blocks(int Q)
{
    const int blocks = (Q + 15) / 16;
    if (blocks <= 2) return blocks < 1 ? 1 : blocks;
    int best = 4, waste = (4 - blocks % 4) % 4 * 1000 / ((blocks + 3) / 4 * 4);
    for (int cb = 5; cb >= 3; cb -= 2) {
        const int w = (cb - blocks % cb) % cb * 1000 / ((blocks + cb - 1) / cb * cb);
        if (w < waste) { waste = w; best = cb; }
    }
    return best;
}

// The run-time-shape MFMA kernel takes single factors whose slices start on 16-byte boundaries
// (P a multiple of 4 floats or 2 doubles) or are at most 256 bytes long.  It pads P and Q to multiples of 16 with zeros, so a factor
// is given to it only while the padded product is at most 3 times the real one (measured against the
// generic kernel, 3 factors each: fp32 20x20 4 % faster at 2.56x padding, 36x36 19 % at 1.78x, 40x40
// 18 %, 52x52 10 %, 100x100 level; fp64 20x20 9 % faster, 36x36 31 %, 34x34 26 %, 84x84 14 %, 50x50 and
// 22x22 level, 30x30 4 % slower).
constexpr bool any_padding_fits(int P, int Q)
{
    const int cols = 16 * any_column_blocks(Q);
    const double padded = (double)((P + 15) / 16 * 16) * (double)((Q + cols - 1) / cols * cols);
    return padded <= 3.0 * (double)P * (double)Q;
}

// Units of work of the kernels without compiled shapes: (tile t of `tiles` slice tiles, group c of
// `groups` factor-column groups).  The groups of one tile read the same slices, so they should meet in
// one L2: workgroup b runs on XCD b % 8, hence within each run of 8 tiles the unit number is
// b = (8 * (t / 8) * groups) + c * 8 + t % 8; the last tiles % 8 tiles are numbered plainly.
KM_HOST_DEVICE inline void unit_of(int64_t b, int64_t tiles, int groups, int64_t& t, int& c)
{
    const int64_t full = tiles / 8 * 8 * groups;
    if (b < full) {
        t = b / (8 * groups) * 8 + b % 8;
        c = (int)(b / 8 % groups);
    } else {
        b -= full;
        t = tiles / 8 * 8 + b / groups;
        c = (int)(b % groups);
    }
}

// The run-time-shape MFMA kernel that keeps the factor in registers (mfma_pad_kernel.hpp): factors of up to
// PAD_MAXP rows and columns, compiled for contractions of 2, 4, 6 and 8 chunks of 16; pad_columns(Q) wavefronts
// hold 16 columns each, pad_groups of such groups share the slices of a tile, pad_blocks blocks of 16 slices each.
constexpr int PAD_MAXP = 128, PAD_LDS_LIMIT = 96 * 1024, PAD_VECTORS = 8;
constexpr int PAD_VARIANT = -3;            // km_plan_step.variant of its launches
KM_HOST_DEVICE constexpr int pad_chunks(int P) { return P <= 32 ? 2 : P <= 64 ? 4 : P <= 96 ? 6 : 8; }
KM_HOST_DEVICE constexpr int pad_columns(int Q) { return (Q + 15) / 16; }
KM_HOST_DEVICE constexpr int pad_groups(int columns) { return columns == 1 ? 4 : columns <= 3 ? 2 : 1; }
KM_HOST_DEVICE constexpr int pad_blocks(size_t esize, int columns, int chunks) { return (chunks == 2 && columns > 1 ? 8 : 4) * 4 / (int)esize; }
KM_HOST_DEVICE constexpr int pad_tile_slices(size_t esize, int columns, int chunks) { return 16 * pad_blocks(esize, columns, chunks) * pad_groups(columns); }
// 16-byte vectors of a tile that one thread fetches, at most PAD_VECTORS
KM_HOST_DEVICE constexpr int pad_vectors(size_t esize, int columns, int chunks)
{
    const int threads = 64 * columns * pad_groups(columns), vectors = pad_tile_slices(esize, columns, chunks) * chunks * (int)esize;
    return (vectors + threads - 1) / threads < PAD_VECTORS ? (vectors + threads - 1) / threads : PAD_VECTORS;
}
// wavefronts per SIMD that registers are limited for
KM_HOST_DEVICE constexpr int pad_waves(size_t esize, int columns, int chunks)
{
    return (chunks == 8 && (esize == 8 || columns <= 4)) || (chunks == 6 && columns <= 4) || (chunks == 2 && columns <= 2) ? 3 : 4;
}
// LDS row stride in elements: 4 times an odd number of floats or 2 times an odd number of doubles where slices
// are whole 16-byte vectors; others stay as they lie in memory
KM_HOST_DEVICE constexpr int pad_stride(int P, size_t esize)
{
    const int u = esize == 4 ? 4 : 2;
    return P % u ? P : (P / u % 2 ? P : P + u);
}
KM_HOST_DEVICE constexpr int64_t pad_lds_bytes(int P, int Q, size_t esize)
{
    return 2 * (int64_t)pad_tile_slices(esize, pad_columns(Q), pad_chunks(P)) * pad_stride(P, esize) * (int64_t)esize + 16;     // (16: a masked read past the last slice)
}
KM_HOST_DEVICE constexpr bool pad_fits(int P, int Q, size_t esize)
{
    if (P < 2 || P > PAD_MAXP || Q > PAD_MAXP) return false;
    const int c = pad_columns(Q), k = pad_chunks(P), threads = 64 * c * pad_groups(c);
    return (int64_t)pad_tile_slices(esize, c, k) * P * (int64_t)esize <= (int64_t)pad_vectors(esize, c, k) * threads * 16 && pad_lds_bytes(P, Q, esize) <= PAD_LDS_LIMIT;
}
// How the kernel would run a factor on `slices` slices (threads == 0: it cannot).
struct PadShape {
    int threads = 0, tile_slices = 0, lds_bytes = 0;
    int64_t grid = 0, per_cu = 0;          // per_cu: workgroups a compute unit holds at once
};
inline PadShape pad_shape(int P, int Q, size_t esize, int64_t slices)
{
    PadShape r;
    if (!pad_fits(P, Q, esize)) return r;
    const int c = pad_columns(Q), k = pad_chunks(P), threads = 64 * c * pad_groups(c);
    r.tile_slices = pad_tile_slices(esize, c, k);
    const int64_t lds = pad_lds_bytes(P, Q, esize);
    r.threads = threads;
    r.lds_bytes = (int)lds;
    // one round of the workgroups the chip holds, each walking over its share; a multiple of 8 for the XCDs
    const int64_t tiles = (slices + r.tile_slices - 1) / r.tile_slices;
    int64_t per_cu = 160 * 1024 / lds;
    if (per_cu > 4 * pad_waves(esize, c, k) * 64 / threads) per_cu = 4 * pad_waves(esize, c, k) * 64 / threads;
    if (per_cu < 1) per_cu = 1;
    r.per_cu = per_cu;
    r.grid = tiles < 256 * per_cu ? (tiles + 7) / 8 * 8 : 256 * per_cu;
    return r;
}

// The run-time-shape MFMA kernel with a slice per lane (mfma_lane_kernel.hpp): fp32, tiles of LANE_SLICES slices per
// wavefront, factors of LANE_MINP to LANE_MAXP rows and up to LANE_MAXP columns.
constexpr int LANE_VARIANT = -8;           // km_plan_step.variant of its launches
constexpr int LANE_THREADS = 256, LANE_SLICES = 64, LANE_MINP = 5, LANE_MAXP = 128;
// A slice's row is found as the high half of (slice * lane_row_magic(slices of a row)): exact while their number times that of
// a row's stays below 2^64 (1 x (5x1)^15, 2^32.5 slices in one row, finds the last one in a second row).
constexpr int64_t LANE_MAX_SLICES = (int64_t)1 << 32;
KM_HOST_DEVICE constexpr uint64_t lane_row_magic(int64_t S) { return S > 1 ? ~(uint64_t)0 / (uint64_t)S + 1 : 0; }      // 2^64 / S rounded up
// Vectors of a slice that are moved at a time: the compiled length that leaves the fewest to move twice (each chunk counting as
// one more; the longest only where it is the whole slice, since longer chunks are fewer workgroups per compute unit: 64 x
// 100x100^3 in chunks of 7, 9 and 13 vectors 147, 142 and 157 us a launch that is repeated on one X, 1024 x 50x50^3 in 7 and 13 251 and 225).
KM_HOST_DEVICE constexpr int lane_units(int P)
{
    const int units = (P + 3) / 4;
    if (units == 13) return 13;
    int best = 2, cost = 1 << 30;
    for (int u : {2, 3, 4, 5, 6, 7, 9}) {
        const int chunks = (units + u - 1) / u, c = chunks * (u + 1);
        if (u <= units && c <= cost) { best = u; cost = c; }
    }
    return best;
}
// wavefronts per SIMD that registers are limited for: 4G accumulators, 5U of the next chunk and its addresses, two sets of operands, the rest
KM_HOST_DEVICE constexpr int lane_waves(int G, int U)
{
    const int registers = 4 * G + 5 * U + 8 * (1 + (G + 15) / 16) + 55;
    return registers <= 122 ? 4 : registers <= 163 ? 3 : 2;
}
KM_HOST_DEVICE constexpr int lane_lds_bytes(int P, int Q, int U)
{
    return 16 * ((P + 3) / 4 * ((Q + 3) / 4 * 4) + LANE_THREADS * (U | 1));
}
// Factors that it is compiled for, those that lane_wins() may give it: of the generic kernel's (padded to 16s too large for the other
// forms), of the form in registers, and of the chunked form's.
KM_HOST_DEVICE constexpr bool lane_fits_generic(int P, int Q) { return P <= 32 || P > 64 || Q > 8; }
KM_HOST_DEVICE constexpr bool lane_fits_chunked(int P, int Q) { return P > 32 && (P % 4 != 0 || P == 36 || Q <= 8 || Q > 16); }
KM_HOST_DEVICE constexpr bool lane_fits_pad(int P, int Q)
{
    if (P > 64) return P <= 80 && Q > 64 && Q <= (P % 4 == 0 ? 72 : 76);
    if (P > 36 || Q > 40) return false;
    return P % 4 != 0 || (Q % 16 != 0 && P >= 12 && !(P == 32 && Q <= 8));
}
constexpr bool lane_takes(int P, int Q)
{
    if (P < LANE_MINP || P > LANE_MAXP || Q < 1 || Q > LANE_MAXP) return false;
    if (!any_padding_fits(P, Q)) return lane_fits_generic(P, Q);
    const int columns = pad_columns(Q);
    const bool pad = pad_fits(P, Q, sizeof(float)), chunked = !pad || (P % 4 == 0 && P > 64 && (columns == 3 || columns == 5));
    return (pad && lane_fits_pad(P, Q)) || (chunked && lane_fits_chunked(P, Q));
}
// Is there a factor whose launch would be mfma_lane_sliced_multiply<G, U>?
constexpr bool lane_compiled(int G, int U)
{
    for (int P = LANE_MINP; P <= LANE_MAXP; ++P)
        if (lane_units(P) == U)
            for (int Q = 4 * G - 3; Q <= 4 * G; ++Q)
                if (lane_takes(P, Q)) return true;
    return false;
}
// How the kernel would run a factor on `slices` slices (lds_bytes == 0: it does not).
struct LaneShape {
    int lds_bytes = 0;
    int64_t grid = 0, per_cu = 0;          // per_cu: workgroups a compute unit holds at once
};
inline LaneShape lane_shape(int P, int Q, int64_t slices)
{
    LaneShape r;
    if (!lane_takes(P, Q) || slices > LANE_MAX_SLICES) return r;
    const int U = lane_units(P), G = (Q + 3) / 4;
    r.lds_bytes = lane_lds_bytes(P, Q, U);
    r.per_cu = 160 * 1024 / r.lds_bytes < lane_waves(G, U) ? 160 * 1024 / r.lds_bytes : lane_waves(G, U);
    // One tile per wavefront, two where the factor's way into LDS takes long beside a tile's work; a multiple of 8 for the XCDs.
    const int64_t groups = (slices + 4 * LANE_SLICES - 1) / (4 * LANE_SLICES);
    int64_t walk = Q > 32 && groups > 512 * r.per_cu ? 2 : 1;
    const int64_t most = (int64_t)1 << 23;               // (a launch has fewer than 2^32 work-items)
    if (groups > most * walk) walk = (groups + most - 1) / most;
    r.grid = ((groups + walk - 1) / walk + 7) / 8 * 8;
    return r;
}

// Makes `st` (whose factor, rows and buffers stay) a launch of that kernel.
inline void make_lane_step(const LaneShape& sh, km_plan_step& st)
{
    st.kernel = KM_KERNEL_MFMA_ANY;
    st.variant = LANE_VARIANT;
    st.tile_slices = LANE_SLICES;
    st.block = LANE_THREADS;
    st.lds_bytes = sh.lds_bytes;
    st.grid = sh.grid;
}

// The whole-row MFMA kernel: up to ROWM_MAXF factors; slices of a multiple of 8 elements are padded by 4 in
// LDS, the operand registers hold ROWM_CHUNKS chunks of 16 rows of a factor (row_mfma_kernel.hpp says why).
// Rows whose two buffers need more than 60 KB keep their other plans: their work takes one compute unit so
// long that nothing is gained (30 x 20x20^3 14.6 us in three launches and 14.6 here, 300 rows 21.2 and 28.5; 50 x 17x17^3
// fp64 15.6 on the FMA kernel, 14.5 here).
constexpr int ROWM_MAXF = 8, ROWM_CHUNKS = 5, ROWM_LDS_LIMIT = 60 * 1024, ROWM_ROWS = 1024;
constexpr int ROWM_VARIANT = -2;           // km_plan_step.variant of its launches
KM_HOST_DEVICE inline int rowm_slice_stride(int P) { return P + (P % 8 == 0 ? 4 : 0); }

// How that kernel would run a problem (threads == 0: it cannot).
struct RowmShape {
    int threads = 0;
    int64_t buf_elems = 0, lds_bytes = 0;
    double us = 0;                         // estimate of the launch
};
inline RowmShape rowm_shape(const Problem& pr)
{
    RowmShape r;
    if (pr.N > ROWM_MAXF || pr.M < 1) return r;
    // a buffer holds the row as each step reads it, slices padded, and the result
    int64_t w = pr.k_in;
    r.buf_elems = pr.k_out;
    for (int f = pr.N - 1; f >= 0; --f) {
        if (w > 65535) return RowmShape();
        const int64_t S = w / pr.P[f];
        if (S * rowm_slice_stride(pr.P[f]) > r.buf_elems) r.buf_elems = S * rowm_slice_stride(pr.P[f]);
        w = S * pr.Q[f];
    }
    r.buf_elems = (r.buf_elems + 7) / 4 * 4;              // (whole vectors, and a few elements that a masked read may touch)
    r.lds_bytes = 2 * r.buf_elems * (int64_t)pr.esize;
    if (r.lds_bytes > ROWM_LDS_LIMIT) return RowmShape();
    // Four or sixteen wavefronts per row, by what a row takes that has its compute unit to itself (1.2 us to load and
    // store it, per step 0.5 us and 0.15 us for each 16x16 block that a wavefront computes in turn) and what the rows on a
    // compute unit take from each other (per block 25 ns and 3.5 ns per MFMA, fp64 7; registers allow 16 wavefronts
    // per unit).  `us` is a finer estimate of the launch in the chosen form, with the parts of a step taken apart (the
    // contraction's length, its rounds of the operand registers, the products' time in a wavefront): fitted to 700
    // problems of 1 to 1024 rows, 6 % off either way.
    double best = 0;
    for (int nw = 16; nw >= 4; nw -= 12) {
        int64_t per_cu = 160 * 1024 / r.lds_bytes;
        if (per_cu > 16 / nw) per_cu = 16 / nw;
        const double rounds = (double)((pr.M + 256 * per_cu - 1) / (256 * per_cu));
        const double together = (double)(pr.M < 256 * per_cu ? (pr.M + 255) / 256 : per_cu);
        double coarse = 1.2 + 0.02 * (double)pr.k_in / (nw * 64);
        double fine = (0.078 * (double)pr.k_in + 0.086 * (double)pr.k_out) / (nw * 64);
        w = pr.k_in;
        for (int f = pr.N - 1; f >= 0; --f) {
            const int64_t S = w / pr.P[f], blocks = (S + 15) / 16 * ((pr.Q[f] + 15) / 16);
            const double turns = (double)((blocks + nw - 1) / nw), shared = together * (double)blocks;
            const double k4 = (double)((pr.P[f] + 3) / 4) * (pr.esize == 4 ? 1 : 2);
            coarse += 0.5 + 0.15 * turns + shared * (0.025 + 0.0035 * k4);
            fine += 0.635 + 0.0012 * pr.P[f] + 0.317 * ((pr.P[f] - 1) / (16 * ROWM_CHUNKS)) + turns * (0.2465 + 0.0075 * k4) +
                    shared * (0.0357 + 0.0036 * k4);
            w = S * pr.Q[f];
        }
        if (r.threads == 0 || rounds * coarse < best) {
            best = rounds * coarse;
            r.threads = nw * 64;
            r.us = 1.94 + rounds * fine;
        }
    }
    return r;
}

// The kernel for rows of 4^7 floats whose factors are 4x4 or pairs of 2x2 (fused_row4_kernel.hpp): all of them in one launch,
// two workgroups to a compute unit.  It is the faster one for any number of rows (4^7, us: 1 row 8.5 -> 5.8, 100 rows 11.0 -> 6.8, 512
// rows 17.2 -> 11.7, 1024 rows 37.7 -> 22.3, 20000 rows 569 -> 451; what it replaces: two launches for few rows, else
// fused_multi_kernel.hpp).
constexpr int ROW4_ELEMS = 16384, ROW4_DIGITS = 7, ROW4_THREADS = 1024, ROW4_LDS_BYTES = 16 * (4 * 4 * 68 + 16) * 4, ROW4_GRID = 512;
constexpr int ROW4_VARIANT = -6;           // km_plan_step.variant of its launches

// The kernel for rows of P^(3G) and P^(4G) floats, square factors of size 5 (G = 2) and 3 (G = 3) (fused_cube_kernel.hpp).
constexpr int CUBE_VARIANT = -7;           // km_plan_step.variant of its launches
KM_HOST_DEVICE constexpr int cube_stride(int E) { return E * E + (E + 64 - E * E % 64) % 64; }       // the same modulo 64 as E

// The fp32 kernels that leave digits in place (mfma_inplace_kernel.hpp).  The last two factors, both 48x48 or both
// 64x64, are one launch with a tile of one matrix per wavefront, each factor before them (multiples of 16 up to 128) one
// with tiles of DIGIT_COLS columns, in two stretches.
constexpr int CHAIN_THREADS = 256, DIGIT_THREADS = 256, DIGIT_COLS = 512, DIGIT_STRETCH = DIGIT_COLS / 2;
constexpr int CHAIN_VARIANT = -4, DIGIT_VARIANT = -5;      // km_plan_step.variant of their launches
constexpr int INPLACE_ORDER = 4;                           // ... and tile_order

// A compiled instance chosen for one group of factors, with the slices per tile it will run with.
// What the planner needs to know of the generic kernel: a workgroup of `threads` work-items takes
// `tile_slices` slices and `tile_cols` factor columns at a time.
struct GenericKernel {
    int threads, tile_slices, tile_cols, lds_bytes;
    // the whole-row kernel: a workgroup of row_threads_many work-items (row_threads_few when there
    // are at most row_few_rows rows) applies up to row_max_factors factors to one row held, with the
    // factors, in at most row_lds_limit bytes of LDS
    int row_threads_many, row_threads_few, row_few_rows, row_lds_limit, row_max_factors;
    // the run-time-shape MFMA kernel: a workgroup of any_threads work-items takes
    // any_tile_slices slices and 16 * any_column_blocks(Q) factor columns at a time, chunks of
    // any_row_bytes per slice in LDS rows padded by one 16-byte unit; slices of at most half a chunk
    // take the narrow shape: twice the slices, chunks of half the bytes
    int any_threads, any_tile_slices, any_row_bytes;
};

inline bool any_narrow(const GenericKernel& gen, int P, size_t esize) { return (size_t)P * esize * 2 <= (size_t)gen.any_row_bytes; }
inline int any_unit_slices(const GenericKernel& gen, int P, size_t esize)
{
    return any_narrow(gen, P, esize) ? 2 * gen.any_tile_slices : gen.any_tile_slices;
}
inline int any_lds_bytes(const GenericKernel& gen, int P, int Q, size_t esize)
{
    const int row = any_narrow(gen, P, esize) ? gen.any_row_bytes / 2 : gen.any_row_bytes;
    return (any_unit_slices(gen, P, esize) + 16 * any_column_blocks(Q)) * (row + 16);
}

// Tiles (or units) that keep a compute unit busy when `tiles` of them are dealt to workgroups of which it holds
// per_cu at once: between whole rounds (a workgroup's last tile has nothing left to overlap with) and an even deal.
inline double tiles_in_turn(int64_t tiles, int64_t per_cu)
{
    const int64_t grid = tiles < 256 * per_cu ? tiles : 256 * per_cu, side = (grid + 255) / 256;
    const int64_t rounds = (tiles + grid - 1) / grid, left = tiles % grid;
    return 0.7 * (double)(rounds * side) + 0.3 * (double)(tiles / grid * side + (left + 255) / 256);
}

// Microseconds of a launch of the form that holds the factor in registers, for comparison with the whole-row kernel on
// few rows (fitted to 900 pairs of launches, 8 % off either way): a fixed part with the factor's loads, and the tiles of a
// compute unit by their bytes and by their wavefronts' products, where one SIMD has the most of them.
inline double pad_us(int P, int Q, size_t esize, int64_t slices, const PadShape& pad)
{
    const int64_t tiles = (slices + pad.tile_slices - 1) / pad.tile_slices, grid = 256 * pad.per_cu < tiles ? 256 * pad.per_cu : tiles;
    const int64_t side = (grid + 255) / 256, left = tiles % grid;
    const double n = (double)(tiles / grid * side + (left + 255) / 256);
    const double bytes = (double)pad.tile_slices * (double)(P + Q) * (double)esize / 21.0e3;
    const double products = (double)(pad_blocks(esize, pad_columns(Q), pad_chunks(P)) * ((P + 3) / 4) * ((pad.threads / 64 + 3) / 4)) *
                            (esize == 4 ? 32.0 : 64.0) / 2400.0;
    return 2.26 + 0.0081 * P + 0.09 * (double)((tiles + grid - 1) / grid) + n * (0.13 + 0.64 * bytes + 0.98 * products);
}

// The generic kernel's form for small factors (generic_small_kernel.hpp): units of GEN_SLICES slices, held in LDS whole with an odd
// stride.  (A few slices per row and many columns, results 8 to 28 bytes apart: 150000 x (2x2, 5x40) 71 us in the other
// form, 73 in this one; with one slice 300000 x 5x40 71 and 29.)
// Slices of up to GEN_FEW elements are read by a thread each, without LDS.
constexpr int GEN_SLICES = 128, GEN_SMALL_LDS = 66 * 1024 + 64, GEN_FEW = 8;
KM_HOST_DEVICE constexpr int gen_small_stride(int P) { return P | 1; }
KM_HOST_DEVICE constexpr int64_t gen_small_lds(int64_t P, int64_t esize) { return GEN_SLICES * (P | 1) * esize; }
KM_HOST_DEVICE constexpr bool gen_small_form(int P, int Q, int64_t S, int64_t esize)
{
    return gen_small_lds(P, esize) <= GEN_SMALL_LDS && !(S > 1 && S < 8 && Q > 16);
}

// Does the form of the run-time-shape MFMA kernel that walks the factor through LDS in chunks beat the one that holds
// it in registers (`pad`)?  Measured side by side on 900 pairs of equal factors, 1 to 60000 rows: the register form
// is faster (mostly 1.05 to 3 times) in launches of up to 256 tiles, where slices are no whole 16-byte vectors (the other
// one deals their elements to LDS one by one) and where its wavefronts, one per 16 columns, fill the four SIMDs
// of a compute unit evenly.  What is left are, of long contractions, three, five or six column blocks, and
// slices of up to 32 elements with one or two: there the chunked form, with units of twice the slices and one
// workgroup more on a compute unit, needs fewer rounds for some row counts (654 x 80x80^2 fp64 57.8 us in registers,
// 46.9 in chunks, 240 rows 29.0 and 27.8, 1028 rows 79.1 and 82.4; 1586 x 48x48^2 25.4 and 19.9, 2717 rows 30.4 and 38.1).
// Both are estimated there, in nanoseconds fitted to those measurements (8 to 11 % off either way): a fixed part and,
// per tile in turn, its bytes at 21 per nanosecond (a compute unit's share of 5.4 TB/s) and its products at the matrix
// cores' rate.  The chunked form is taken where it promises 5 %: of the 45 among 1021 problems that
// the register form made more than 3 % slower 24 are left, by 13 % at most but for one, and 4 become slower for it.
inline bool chunked_form_wins(const GenericKernel& gen, int P, int Q, size_t esize, int64_t S, int64_t slices, const PadShape& pad)
{
    const int columns = pad_columns(Q);
    const int64_t tiles = (slices + pad.tile_slices - 1) / pad.tile_slices;
    // (rows of a single slice of 32 elements, which fill a chunk: 826 x (32x32) 7.49 us in registers, 7.24 in chunks,
    // 48694 x (32x24) 9.60 and 9.12, fp64 687 x (32x16) 4.34 and 4.02; level at 28 and 36)
    if (S == 1 && P == 32 && columns <= 2) return true;
    if (tiles <= 256 || P * esize % 16 != 0) return false;
    if (!(columns == 3 ? P > (esize == 4 ? 32 : 64) : P <= 32 ? columns < 3 : P > 64 && (columns == 5 || columns == 6))) return false;
    const bool f32 = esize == 4;
    const double mfma = (f32 ? 32.0 : 64.0) / 2.4;       // one 16x16x4 product on one SIMD
    auto bytes = [&](int64_t n, int q) { return (double)n * (double)(P + q) * (double)esize / 21.0; };

    const int waves = pad.threads / 64, k4 = (P + 3) / 4;
    const double n = tiles_in_turn(tiles, pad.per_cu), b = n * bytes(pad.tile_slices, Q);
    const double m = n * (double)(pad_blocks(esize, columns, pad_chunks(P)) * k4 * ((waves + 3) / 4)) * mfma;
    const double in_registers = f32 ? 2600.0 + 0.83 * b + 0.80 * m + 2.4 * P : 1780.0 + 0.56 * b + 0.82 * m + 166.0 * n + 32.6 * P;

    const int cb = any_column_blocks(Q), ts = any_unit_slices(gen, P, esize);
    const int64_t units = (slices + ts - 1) / ts * ((Q + 16 * cb - 1) / (16 * cb));
    int64_t per_cu = 160 * 1024 / any_lds_bytes(gen, P, Q, esize);
    if (per_cu > 3) per_cu = 3;                          // (the registers it is compiled for)
    if (per_cu > 2 && (cb >= 5 || (!f32 && cb >= 3 && any_narrow(gen, P, esize)))) per_cu = 2;
    if (f32 && columns == 3 && units > 256 * per_cu) return false;       // (level or slower from its second round on)
    const double un = tiles_in_turn(units, per_cu), ub = un * bytes(ts, Q < 16 * cb ? Q : 16 * cb);
    const double um = (double)(ts / 16 * cb * ((P + 15) / 16 * 4)) * mfma / 4.0;
    const double in_chunks = f32 ? 1930.0 + 0.48 * ub + (1.16 * un + 1.05) * um + 544.0 * un
                                 : 2570.0 + 0.38 * ub + (0.95 * un + 0.57) * um + 650.0 * un;
    return in_chunks < 0.95 * in_registers;
}

struct Choice {
    bool any_mfma = false;   // with var == nullptr: the run-time-shape MFMA kernel instead of the generic one
    int any_form = 0;        // ... 0: the form that is estimated faster, PAD_VARIANT: factor in registers, -1: in chunks, LANE_VARIANT: a slice per lane
    const Variant* var = nullptr;
    int tile_slices = 0;
    int64_t grid = 0;        // tiles (before the persistent-walk division)
    int tiles_per_wg = 0;    // persistent instances: 0 = take the rule of tiles_per_wg()
    int tile_order = -1;     // persistent instances: -1 = take the option
    int tile_rows = 1;       // rows per tile; above 1 the tile holds whole rows (tile_slices = K/prod(P))
};

// Rows a flexible instance puts into one tile when a whole row is shorter than its tile (rows are
// contiguous in memory, so several of them pass through the stages as one long tile): as many as
// fit 48 KB of LDS (three and more workgroups per compute unit, see find_variant), within the
// instance's limit, leaving at least 512 tiles when there are that many rows.
// (the autotuner's finding on 2^6 ... 2^10, 3^5, 4^4, 4^5 and 5^3 with 16 K to 1 M rows: fp32 tiles of
// 24 KB are 5-20 % faster than tiles of 48 KB, fp64 tiles are best at 48 KB: about 6000 elements either way)
inline int64_t whole_rows_lds_budget(size_t esize) { return esize == 4 ? 24 * 1024 : 48 * 1024; }

inline int whole_rows_per_tile(const Variant& c, int64_t s_row, int64_t M, int64_t row_bytes, int64_t row_out_bytes,
                               int64_t lds_budget)
{
    if (!c.flexible || s_row > c.tile_slices / 2 || M < 1024) return 1;   // few rows: one workgroup each
    // rows of 8 KB that do not start on 16-byte boundaries are tiles of their own: the joined rows
    // would be stored element by element (1024 rows of 3^7: one row per tile 0.014 ms, two 0.018 ms)
    if (row_bytes >= 8192 && row_bytes % 16 != 0) return 1;
    int64_t most = c.tile_slices / s_row;
    if (c.lds_per_slice > 0) {
        const int64_t fit = lds_budget / c.lds_per_slice / s_row;
        if (fit < most) most = fit < 1 ? 1 : fit;
    }
    // the output rows are collected in the tile's own LDS: where they are longer than the input rows
    // (Q > P) they set the limit, and the launch asks for their size (build_step)
    if (row_out_bytes > row_bytes) {
        const int64_t room = lds_budget < c.lds_bytes ? lds_budget : c.lds_bytes;
        const int64_t fit = room / row_out_bytes;
        if (fit < most) most = fit < 1 ? 1 : fit;
    }
    if (most > M) most = M;
    while (most > 1 && (M + most - 1) / most < 512) --most;
    return most < 1 ? 1 : (int)most;
}

// Tile order 3 gives each of the 8 XCDs a contiguous eighth of the tiles, walked by grid / 8 workgroups.
inline bool xcd_order_fits(int64_t num_tiles, int64_t grid)
{
    return num_tiles % 8 == 0 && grid % 8 == 0 && grid >= 8;
}

// Workgroups of an instance that one compute unit holds at once (160 KB of LDS, 2048 threads, registers where the
// table names their limit).
inline int64_t resident_per_cu(const Variant& c)
{
    int64_t by_lds = c.lds_bytes > 0 ? (160 * 1024) / c.lds_bytes : 8;
    int64_t by_threads = 2048 / (c.threads > 0 ? c.threads : 256);
    int64_t n = by_lds < by_threads ? by_lds : by_threads;
    if (c.simd_waves > 0 && n > 4 * 64 * c.simd_waves / c.threads) n = 4 * 64 * c.simd_waves / c.threads;
    return n < 1 ? 1 : (n > 8 ? 8 : n);
}

// The divisors of s_row an instance may run with (fixed instances: their one tile length).
inline void tile_lengths(const Variant& c, int64_t s_row, std::vector<int>& out, int at_most)
{
    out.clear();
    if (!c.flexible) {
        if (s_row % c.tile_slices == 0) out.push_back(c.tile_slices);
        return;
    }
    const int64_t lim = s_row < c.tile_slices ? s_row : c.tile_slices;
    for (int64_t d = lim; d >= 1 && (int)out.size() < at_most; --d)
        if (s_row % d == 0) out.push_back((int)d);
}

// Can factors [f - nf + 1, f] on rows of width k_cur be one tiled launch at all?  Fills prod(P), K/prod(P).
inline bool group_shape(const Problem& pr, int f, int nf, int64_t k_cur, int64_t& pg, int64_t& s_row)
{
    int64_t qg = 1;
    pg = 1;
    for (int i = f - nf + 1; i <= f; ++i) {
        pg *= pr.P[i];
        qg *= pr.Q[i];
        if (pg > ((int64_t)1 << 40) || qg > ((int64_t)1 << 40)) return false;
    }
    if (k_cur % pg) return false;
    s_row = k_cur / pg;
    // the tiled kernels address within a row with 32-bit offsets
    if ((double)s_row * (double)qg * (double)pr.esize >= 2147483648.0) return false;
    if ((double)k_cur * (double)pr.esize >= 2147483648.0) return false;
    return true;
}

// Every (instance, tile length, walk) combination that can run the group: the autotuner's search space.
inline void enumerate_choices(const Variant* table, int count, const Problem& pr, int f, int nf,
                              int64_t k_cur, const Options& opt, std::vector<Choice>& out)
{
    out.clear();
    int64_t pg, s_row;
    if (!group_shape(pr, f, nf, k_cur, pg, s_row)) return;
    int64_t qg_all = 1;
    for (int i = f - nf + 1; i <= f; ++i) qg_all *= pr.Q[i];
    std::vector<int> lens;
    for (int v = 0; v < count; ++v) {
        const Variant& c = table[v];
        if (!(opt.kernels >> c.kernel & 1)) continue;
        if (c.dtype != pr.dtype || !shapes_match(c, pr.P, pr.Q, f, nf)) continue;
        if (c.max_srow > 0 && s_row > c.max_srow) continue;
        if (c.rows_per_tile > 1 && s_row != c.tile_slices) continue;      // tiles of several rows hold whole rows
        tile_lengths(c, s_row, lens, 5);
        const int rows = whole_rows_per_tile(c, s_row, pr.M, s_row * pg * (int64_t)pr.esize, s_row * qg_all * (int64_t)pr.esize, 48 * 1024);
        if (rows > 1) {                                   // whole rows, several per tile, then half and a quarter as many
            for (int r = rows; r >= 2 && r >= rows / 4; r /= 2) {
                Choice ch;
                ch.var = &c;
                ch.tile_slices = (int)s_row;
                ch.tile_rows = r;
                ch.grid = (pr.M + r - 1) / r;
                out.push_back(ch);
            }
        }
        for (int st : lens) {
            Choice ch;
            ch.var = &c;
            ch.tile_slices = st;
            ch.tile_rows = c.rows_per_tile;
            ch.grid = ((pr.M + c.rows_per_tile - 1) / c.rows_per_tile) * (s_row / st);
            if (!c.persistent) { out.push_back(ch); continue; }
            // walks: fixed lengths, and the lengths that make the grid exactly one or two rounds of
            // the workgroups the chip holds at once (every workgroup then gets the same share)
            const int64_t resident = 256 * resident_per_cu(c);
            int64_t walks[6] = {1, 4, 16, 32, (ch.grid + resident - 1) / resident,
                                (ch.grid + 2 * resident - 1) / (2 * resident)};
            for (int i = 0; i < 6; ++i) {
                const int64_t w = walks[i];
                bool seen = w < 1 || w > 4096;
                for (int j = 0; j < i; ++j) seen = seen || walks[j] == w;
                if (seen) continue;
                if (w > 1 && ch.grid / w < 256) continue;      // keep every compute unit busy
                ch.tiles_per_wg = (int)w;
                ch.tile_order = 2;
                out.push_back(ch);
                if (w > 1 && xcd_order_fits(ch.grid, (ch.grid + w - 1) / w)) {
                    ch.tile_order = 3;
                    out.push_back(ch);
                }
            }
        }
    }
}

// Flexible instances whose full tile leaves room for only two workgroups on a compute unit are compiled with a
// larger workgroup too, which is taken when the tile has work for 90 % of its threads (a thread takes
// thread_elems elements at a time): 1000 x 5x5^8 (62 KB tiles) 2.03 ms with 256 threads, 1.61 with 640; 100 x
// 3x3^12 0.290 -> 0.219 (768); fp64 1000 x 3x3^10 0.439 -> 0.417 (768).  Short
// tiles keep the small one (rows of 3^7 use 81 threads), and so do instances with smaller full tiles, which share
// a compute unit in threes and fours (7^6 0.519 ms with 256 threads, 0.743 with 512; 10^5, 6^7, 4^9 alike).
inline Choice larger_workgroup(const Variant* table, int count, Choice ch, int64_t pg)
{
    if (!ch.var || !ch.var->flexible || ch.var->thread_elems <= 0) return ch;
    const Variant& c = *ch.var;
    const int64_t busy = (int64_t)ch.tile_slices * ch.tile_rows * pg / c.thread_elems;
    for (int v = 0; v < count; ++v) {
        const Variant& t = table[v];
        if (t.kernel == c.kernel && t.dtype == c.dtype && t.P == c.P && t.Q == c.Q && t.num_factors == c.num_factors && t.flexible &&
            t.tile_slices == c.tile_slices && t.lds_per_slice == c.lds_per_slice && t.thread_elems == c.thread_elems &&
            t.max_srow == c.max_srow && c.mix[2] == 0 && t.mix[2] == 0 && t.threads > ch.var->threads && busy * 10 >= (int64_t)t.threads * 9 &&
            (double)ch.grid * (double)t.threads < 4294967296.0)              // (a launch's limit of work-items)
            ch.var = &t;
    }
    return ch;
}

// Picks the instance for factors [f - nf + 1, f] applied to rows of width k_cur (var == nullptr: none).
// The table is in order of preference (fastest instance on a full machine first).  The first instance
// that fits the shape and still gives the chip enough workgroups wins; failing that, the fitting
// instance with the most workgroups among those whose output runs are at least 32 bytes.  The tuning
// options override both.
inline double launch_cost(const Problem& pr, int64_t k_in, int64_t k_out, const Choice& ch, int generic_P);

inline Choice find_variant(const Variant* table, int count, const Problem& pr, int f, int nf,
                           int64_t k_cur, const Options& opt)
{
    Choice none;
    int64_t pg, s_row;
    if (!group_shape(pr, f, nf, k_cur, pg, s_row)) return none;
    int64_t k_out = s_row;
    for (int i = f - nf + 1; i <= f; ++i) k_out *= pr.Q[i];

    const int64_t enough = 2 * 256;
    Choice first_big, first_tiny, most, wanted, cheapest;
    double cheapest_cost = 0;
    int64_t wanted_score = 0;
    for (int v = 0; v < count; ++v) {
        const Variant& c = table[v];
        if (!(opt.kernels >> c.kernel & 1)) continue;
        if (c.dtype != pr.dtype || !shapes_match(c, pr.P, pr.Q, f, nf)) continue;
        if (c.max_srow > 0 && s_row > c.max_srow) continue;
        if (c.rows_per_tile > 1 && s_row != c.tile_slices) continue;      // tiles of several rows hold whole rows
        if (c.min_tiles > 0 && !c.flexible && pr.M * (s_row / c.tile_slices) < c.min_tiles && opt.prefer_instance != v + 1)
            continue;                                     // too few tiles for this instance (unless it is asked for)
        // Rows of 128x128, which take more than 64 KB of LDS and have a compute unit to themselves: only where the last
        // round of 256 rows is nearly full (300 x 128x128^2 0.038 ms, two tiled launches 0.034, 520 rows 0.054 and 0.052; 700
        // rows 0.054 and 0.060, 1000 rows 0.072 and 0.082; rows of 32^3 always: 300 rows 0.037 and 0.043)
        if (c.max_srow == 1 && nf == 2 && !c.flexible && c.lds_bytes > 64 * 1024 && opt.prefer_instance != v + 1 &&
            (pr.M + 255) / 256 * 256 * 10 > pr.M * 13)
            continue;
        // slices per tile: fixed, or the best divisor of s_row up to the instance's limit
        int cand[3] = {0, 0, 0};
        int rows = c.rows_per_tile;
        if (!c.flexible) {
            if (s_row % c.tile_slices) continue;
            cand[0] = c.tile_slices;
        } else {
            // Best tile length; best one that still leaves enough workgroups; the tuning wish.
            // "Best" (measured with the autotuner on factors of 3 to 6): output runs that are whole
            // 128-byte lines before anything else (6x6: runs of 1152 bytes are 50 % faster than runs of
            // 1296), then tiles of at most 48 KB of LDS (three and more workgroups per compute unit are
            // 10-30 % faster than two) unless that would cut runs that are not whole lines below 256
            // bytes (6^6: 288-byte runs in 62 KB tiles are 50 % faster than 96-byte runs in 21 KB
            // tiles; rows of odd length, where no run is ever aligned, below 64 bytes: since such tiles
            // are fetched with 16-byte loads and LDS writes, 5^8 with 100-byte runs in 12 KB tiles is
            // 20 % faster than with 500-byte runs in 62 KB tiles), then the longest tile.
            const int64_t lim = s_row < c.tile_slices ? s_row : c.tile_slices;
            const int64_t row_bytes = s_row * (int64_t)pr.esize;
            const bool alignable = (row_bytes & -row_bytes) >= 32;      // some tile length gives 32-byte aligned runs
            // (rows of odd length: 40 KB, four workgroups per compute unit; 1024 x 15^4 fp64 in tiles of 15
            // slices, 27 KB, 0.363 ms, of 25 slices, 45 KB, 0.429)
            const int64_t fit = c.lds_per_slice > 0 ? ((alignable ? 48 : 40) * 1024) / c.lds_per_slice : lim;
            int64_t best_key[2] = {-1, -1};
            int best_tier = 0;
            for (int64_t d = lim; d >= 1; --d) {
                if (s_row % d) continue;
                const int64_t run = d * (int64_t)pr.esize;
                int64_t align = run & -run;                          // largest power of two dividing the run
                if (align > 128) align = 128;
                // (runs of 256 bytes and more that start on 64-byte boundaries count as whole lines: 53 x 10^7
                // in tiles of 80 slices, 320-byte runs, 3.43 ms, of 32 slices, 128-byte runs, 4.07; shorter ones
                // do not: 256 x 12^4 fp64 with 192-byte runs 0.052 ms, with 128-byte runs 0.045)
                if (align == 64 && run >= 256) align = 128;
                const bool small_enough = d <= fit && (align >= 128 || run >= 256 || (!alignable && run >= 64));
                const int64_t key = (align * 2 + (small_enough ? 1 : 0)) * (lim + 1) + d;
                if (key > best_key[0]) { best_key[0] = key; cand[0] = (int)d; }
                // ... that leaves enough workgroups: 512 with at least 16 busy threads, else 96 with at
                // least 4.  A thread takes thread_elems contiguous elements, so short tiles only
                // multiply the wavefronts that run the same instructions for a few lanes (20 rows of
                // 5^6, 125 elements per thread: one-slice tiles 0.037 ms, 5 or 25 slices 0.018 ms).
                const int64_t wgs = pr.M * (s_row / d);
                const int64_t busy = c.thread_elems > 0 ? d * pg / c.thread_elems : d;     // threads with work
                const int tier = (wgs >= enough && (busy >= 16 || d == lim)) ? 2 : (wgs >= 96 && (busy >= 4 || d == lim)) ? 1 : 0;
                if (tier > 0 && (tier > best_tier || (tier == best_tier && key > best_key[1]))) {
                    best_tier = tier; best_key[1] = key; cand[1] = (int)d;
                }
                // ... and the tile length the cost estimate likes best (small problems, see below)
                if ((busy >= 4 || d == lim) && (c.persistent || (double)wgs * (double)c.threads < 4294967296.0)) {
                    Choice t;
                    t.var = &c;
                    t.tile_slices = (int)d;
                    t.grid = wgs;
                    const double tc = launch_cost(pr, k_cur, k_out, t, 0);
                    if (!cheapest.var || tc < cheapest_cost) { cheapest = t; cheapest_cost = tc; }
                }
            }
            if (opt.prefer_tile > 0 && opt.prefer_tile <= c.tile_slices && s_row % opt.prefer_tile == 0) cand[2] = opt.prefer_tile;
            // rows much shorter than the tile: whole rows, several per tile
            rows = whole_rows_per_tile(c, s_row, pr.M, s_row * pg * (int64_t)pr.esize, k_out * (int64_t)pr.esize, whole_rows_lds_budget(pr.esize));
            if (rows > 1) {
                cand[0] = (int)s_row; cand[1] = cand[2] = 0;
                if (cheapest.var == &c) cheapest = Choice();
            }
        }
        for (int k = 0; k < 3; ++k) {
            if (!cand[k]) continue;
            Choice ch;
            ch.var = &c;
            ch.tile_slices = cand[k];
            ch.grid = pr.M * (s_row / cand[k]);
            if (rows > 1) {
                ch.tile_rows = rows;
                ch.grid = (pr.M + rows - 1) / rows;
            }
            // a launch may hold at most 2^32 - 1 work-items (walking instances shrink their grid later)
            if (!c.persistent && (double)ch.grid * (double)c.threads >= 4294967296.0) continue;
            // Tiles under 1 KB leave a workgroup with next to nothing to do (one 8x8 factor on rows of
            // 8 elements: a tile of several whole rows is 10 times faster): they only count when no
            // instance with a decent tile gives the chip enough workgroups.
            const int64_t tile_bytes = (int64_t)ch.tile_slices * ch.tile_rows * pg * (int64_t)pr.esize;
            if (!first_big.var && ch.grid >= enough && tile_bytes >= 1024) first_big = ch;
            if (!first_tiny.var && ch.grid >= enough) first_tiny = ch;
            // among small launches: at least 96 workgroups first (16 rows of 10^4 in 16 tiles of 100
            // slices are twice as slow as in 400 tiles of 4), then output runs of at least 32 bytes,
            // then more workgroups
            auto rank = [&](const Choice& x) {
                return (x.grid >= 96 ? 2 : 0) + ((int64_t)x.tile_slices * (int64_t)pr.esize >= 32 ? 1 : 0);
            };
            if (!most.var || rank(ch) > rank(most) || (rank(ch) == rank(most) && ch.grid > most.grid)) most = ch;
            int64_t sc = 0;
            if (opt.prefer_tile && ch.tile_slices == opt.prefer_tile) sc += 2;
            if (opt.prefer_threads && c.threads == opt.prefer_threads) sc += 1;
            if (opt.prefer_instance && v == opt.prefer_instance - 1) sc += 4;
            if (sc > wanted_score) { wanted = ch; wanted_score = sc; }
        }
    }
    if (wanted.var) return wanted;
    const Choice base = first_big.var ? first_big : (first_tiny.var ? first_tiny : most);
    // The rules above are made for launches that fill the chip.  On small problems they would cut a
    // row into tiles with runs of 16 bytes to reach 512 workgroups, where a hundred workgroups with
    // decent runs finish sooner (16 rows of 6^6: three launches of two factors in 1296 tiles 0.024 ms,
    // two of three factors in 144 tiles of 24 slices 0.013): when the cost estimate rates another
    // tile length of a fitting flexible instance a fifth cheaper than the rules' choice, that one is taken.
    if (base.var && cheapest.var && cheapest_cost < 0.8 * launch_cost(pr, k_cur, k_out, base, 0)) return larger_workgroup(table, count, cheapest, pg);
    return larger_workgroup(table, count, base, pg);
}

// Estimated cost of one launch in "bytes moved at full speed": rows read and written, scaled up for
// short output runs and for the generic kernel, plus a constant per launch.
inline double launch_cost(const Problem& pr, int64_t k_in, int64_t k_out, const Choice& ch, int generic_P)
{
    const double bytes = (double)pr.M * ((double)k_in + (double)k_out) * (double)pr.esize;
    double slow = ch.any_mfma ? 1.5 : 3.0;               // generic kernel; run-time-shape MFMA kernel
    if (ch.var) {
        int64_t run = (int64_t)ch.tile_slices * (int64_t)pr.esize;
        // a tile that holds a whole row writes the whole output row: its runs join up
        if (ch.tile_rows > 1 || ch.grid == pr.M) run = k_out * (int64_t)pr.esize;
        slow = run >= 128 ? 1.0 : (run >= 64 ? 1.25 : (run >= 32 ? 2.5 : 4.0));
        // Rows of odd length: no run ever fills whole lines, so short runs cost less on top (measured
        // with the autotuner: 1024 x 7^6 as 3+3 factors with 28-byte runs is 12 % faster than 2+2+2 with
        // 196-byte runs, 9^5 as 2+3 with 36-byte runs 19 % faster than 2+2+1, 3^11 as 7+4 with 12-byte
        // runs 3 % faster than 4+4+3)
        const int64_t row_bytes = k_out * (int64_t)pr.esize;
        if ((row_bytes & -row_bytes) < 16) slow = run >= 64 ? 1.0 : (run >= 32 ? 1.15 : (run >= 16 ? 1.3 : 1.9));
        slow *= ch.var->slowdown;
    }
    // fewer workgroups than compute units: the launch streams at a matching fraction of the chip's
    // rate (one row of 4^9: seven factors in 16 workgroups take 0.017 ms, four in 256 take 0.005)
    if (ch.var && ch.grid < 256) slow *= 256.0 / (double)(ch.grid < 1 ? 1 : ch.grid);
    double fixed = 2.5e7;                                // ~5 us of launch latency at 5 TB/s
    // the generic kernel walks the slice elements in chunks of 16, a barrier apart: a launch of it
    // takes about 2 us + 0.7 us per chunk even when it moves next to nothing (measured: 5.5 us for
    // P = 65, 4.8 us for P = 52 on ten rows)
    if (!ch.var && !ch.any_mfma) fixed += 1.0e7 + 3.5e6 * (double)((generic_P + 15) / 16);
    // a launch of the run-time-shape MFMA kernel that moves next to nothing takes 6-8 us (measured on the
    // paper's Table 4 sizes: two such launches 12.5 us for 50 x (32x8, 64x128), 15.4 us for 10 x (52x65,
    // 50x20), where the whole-row kernel takes 17 and 13.4).  That was its chunked form; the one with the factor in
    // registers takes 4-6, and the factor of 1.5 above is the chunked form's too: this price only weighs the groupings
    // against each other, the whole-row kernel for few rows is compared with finer estimates in make_plan.
    if (ch.any_mfma) fixed += 1.25e7;
    return bytes * slow + fixed;
}

// Tile order 1 hands tiles out in groups of 16 workgroups (8 XCDs x 2) that each take every other
// tile of a range of 2 * tiles_per_wg: the grid must be whole groups and the tiles whole ranges.
inline bool pair_order_fits(int64_t num_tiles, int64_t tpw)
{
    const int64_t grid = (num_tiles + tpw - 1) / tpw;
    return grid % 16 == 0 && num_tiles % (2 * tpw) == 0;
}

// One launch of the plan for factors [r - nf, r - 1] with the given choice (var == nullptr: generic).
inline km_plan_step build_step(const Problem& pr, const Options& opt, const Variant* table, int r, int nf,
                               const Choice& ch, const std::vector<int64_t>& width,
                               const GenericKernel& gen)
{
    const int f = r - 1;
    km_plan_step st = {};
    st.first_factor = f - nf + 1;
    st.num_factors = nf;
    st.k_in = width[r];
    st.k_out = width[r - nf];
    if (ch.var) {
        const Variant* var = ch.var;
        int64_t pg = 1;
        for (int i = f - nf + 1; i <= f; ++i) pg *= pr.P[i];
        st.kernel = var->kernel;
        st.variant = (int)(var - table);
        st.tile_slices = ch.tile_slices;
        st.block = var->threads;
        st.tile_rows = ch.tile_rows;
        st.lds_bytes = launch_lds_bytes(*var, ch.tile_slices * ch.tile_rows);
        if (ch.tile_rows > 1) {                           // whole rows: the output rows are collected in LDS too
            const int64_t out_bytes = ((int64_t)ch.tile_rows * st.k_out * (int64_t)pr.esize + 15) / 16 * 16;
            if (out_bytes > st.lds_bytes) st.lds_bytes = (int)out_bytes;
        }
        st.grid = ch.grid;
        if (var->persistent) {
            const int hint = ch.tiles_per_wg > 0 ? ch.tiles_per_wg : opt.tiles_per_wg;
            int64_t tpw = tiles_per_wg(st.grid, hint, (int64_t)nf * var->P * var->Q,
                                       (int64_t)ch.tile_slices * ch.tile_rows * pg, var->lds_bytes, pr.esize, var->walk);
            if (hint <= 0 && var->walk == -1) {
                // every workgroup resident from the start and each with the same share of the tiles
                // (measured with the autotuner: 256 x 80x80^3 walks of 17 instead of 8 tiles 0.809 -> 0.721 ms,
                // 256 x 112x112^3 49 instead of 32 2.68 -> 2.38, 64 x 144x144^3 27 instead of 32 2.07 -> 1.76)
                const int64_t resident = 256 * resident_per_cu(*var);
                tpw = (st.grid + resident - 1) / resident;
                // ... or up to a third longer walks when that lowers the tiles the busiest compute unit
                // gets (workgroups on it times walk; 16 x 80x80^3 fp64, 1600 tiles: walks of 3 in 534
                // workgroups 0.140 ms, walks of 4 in 400 workgroups 0.122)
                auto busiest = [&](int64_t t) { return (((st.grid + t - 1) / t + 255) / 256) * t; };
                // (by 5 % at least: fewer workgroups per unit cost more than a tile: 256 x 96x96^3 in 1272
                // workgroups of 29 tiles 1.59 ms, in 1024 of 36 1.78)
                const int64_t first = tpw;
                for (int64_t t = first + 1, last = first + (first + 2) / 3; t <= last; ++t)
                    if (busiest(t) * 20 <= busiest(tpw) * 19) tpw = t;
                if (tpw > 4096) tpw = 4096;
                while (tpw > 1 && st.grid / tpw < 256) --tpw;
            } else if (hint <= 0 && var->walk == 0 && tpw > 1 && !var->xcd_order) {
                // The other walking instances, by the same measure (17 x 128x128^3 fp64, 8704 tiles: walks of
                // 16 in 544 workgroups, two or three to a compute unit, 0.626 ms; walks of 17 in 512, two to each)
                auto busiest = [&](int64_t t) { return (((st.grid + t - 1) / t + 255) / 256) * t; };
                const int64_t first = tpw;
                for (int64_t t = first + 1, last = first + (first + 2) / 3; t <= last; ++t)
                    if (busiest(t) * 20 <= busiest(tpw) * 19) tpw = t;
            }
            const int64_t num_tiles = st.grid;
            st.tiles_per_wg = (int)tpw;
            st.grid = (num_tiles + tpw - 1) / tpw;
            st.tile_order = ch.tile_order >= 0 ? ch.tile_order : (opt.tile_order >= 0 ? opt.tile_order : (var->xcd_order ? 3 : 2));
            // output runs shorter than a 128-byte line: neighbouring tiles go to a pair of workgroups
            // that run side by side (order 1), when the tiles split evenly that way
            if (ch.tile_order < 0 && var->persistent == 1 && opt.pair_interleave &&
                (int64_t)ch.tile_slices * (int64_t)pr.esize < 128 && pair_order_fits(num_tiles, tpw))
                st.tile_order = 1;
            if (st.tile_order == 1 && (var->persistent != 1 || !pair_order_fits(num_tiles, tpw))) st.tile_order = 0;
            if (st.tile_order == 3 && !xcd_order_fits(num_tiles, st.grid)) st.tile_order = 2;
            // Whole rows: every compute unit, also where the rows are no multiple of them.  (As many workgroups as give
            // each the same walk leave some compute units out, and cost more than those: 1000 x 32x32^3 in 250 workgroups
            // 0.108 ms, in 256 0.081; 4000 rows 0.496 and 0.296.  Tiles strided by the grid only: in the other
            // orders a workgroup's tiles are a run of tiles_per_wg, so the grid is what that leaves.)
            if (var->walk == -1 && var->max_srow == 1 && hint <= 0 && tpw > 1 && st.tile_order == 2) {
                st.grid = 256 * resident_per_cu(*var);
                while (st.grid > num_tiles) st.grid /= 2;
                st.tiles_per_wg = (int)((num_tiles + st.grid - 1) / st.grid);
            }
        }
    } else if (ch.any_mfma) {
        st.kernel = KM_KERNEL_MFMA_ANY;
        st.variant = -1;
        st.tile_rows = 1;
        st.tile_slices = any_unit_slices(gen, pr.P[f], pr.esize);
        const int64_t slices = pr.M * (st.k_in / pr.P[f]);
        if (ch.any_form == LANE_VARIANT) {
            make_lane_step(lane_shape(pr.P[f], pr.Q[f], slices), st);
            return st;
        }
        const PadShape pad = pad_shape(pr.P[f], pr.Q[f], pr.esize, slices);
        bool chunked = pad.threads == 0 || ch.any_form == -1;
        if (!chunked && ch.any_form == 0) {
            // the tuning options prefer the form with that tile or workgroup, as they do among compiled instances (the
            // chunked one where both have it: the other is what the planner mostly takes by itself)
            auto wish = [&](int tile, int threads) { return (opt.prefer_tile == tile ? 2 : 0) + (opt.prefer_threads == threads ? 1 : 0); };
            const int a = wish(pad.tile_slices, pad.threads), b = wish(st.tile_slices, gen.any_threads);
            chunked = a + b > 0 ? b >= a : chunked_form_wins(gen, pr.P[f], pr.Q[f], pr.esize, st.k_in / pr.P[f], slices, pad);
        }
        if (!chunked) {                                  // the form with the factor in registers
            st.variant = PAD_VARIANT;
            st.tile_slices = pad.tile_slices;
            st.block = pad.threads;
            st.lds_bytes = pad.lds_bytes;
            st.grid = pad.grid;
            return st;
        }
        st.block = gen.any_threads;
        st.lds_bytes = any_lds_bytes(gen, pr.P[f], pr.Q[f], pr.esize);
        const int64_t S = st.k_in / pr.P[f];
        const int cols = 16 * any_column_blocks(pr.Q[f]);
        st.grid = ((pr.M * S + st.tile_slices - 1) / st.tile_slices) * ((pr.Q[f] + cols - 1) / cols);
        const int64_t most = ((int64_t)1 << 32) / gen.any_threads - 1;     // the kernel strides over its units
        if (st.grid > most) st.grid = most;
        // two rounds of the workgroups the chip holds at once (three per compute unit, two with five column
        // blocks), each striding over its share of the units: 2-11 % faster than one workgroup per unit
        // (512 x 40x40^3 fp64 0.458 -> 0.409 ms, 512 x 20x20^4 0.729 -> 0.691, 64 x 100x100^3 0.822 -> 0.789)
        const int64_t rounds2 = 2 * 256 * (any_column_blocks(pr.Q[f]) >= 5 ? 2 : 3);
        if (st.grid > rounds2) st.grid = rounds2;
    } else {
        st.kernel = KM_KERNEL_GENERIC;
        st.variant = -1;
        st.tile_rows = 1;
        st.tile_slices = gen.tile_slices;
        st.block = gen.threads;
        const int64_t S = st.k_in / pr.P[f];
        st.lds_bytes = !gen_small_form(pr.P[f], pr.Q[f], S, (int64_t)pr.esize) ? gen.lds_bytes : pr.P[f] <= GEN_FEW ? 0 : (int)gen_small_lds(pr.P[f], (int64_t)pr.esize);
        // one workgroup per (tile of slices, group of factor columns); tiles may span rows
        st.grid = ((pr.M * S + gen.tile_slices - 1) / gen.tile_slices) * ((pr.Q[f] + gen.tile_cols - 1) / gen.tile_cols);
        // the generic kernel strides over its work, so its grid can stay below the launch limit
        const int64_t most = ((int64_t)1 << 32) / gen.threads - 1;
        if (st.grid > most) st.grid = most;
    }
    return st;
}

inline bool any_mfma_fits(const Problem& pr, int f, const Options& opt)
{
    return (opt.kernels >> KM_KERNEL_MFMA_ANY & 1) && any_padding_fits(pr.P[f], pr.Q[f]);
}

inline void row_widths(const Problem& pr, std::vector<int64_t>& width)
{
    // width[r]: row width when factors 0..r-1 are still to be applied (the others already were)
    width.assign(pr.N + 1, 0);
    width[pr.N] = pr.k_in;
    for (int r = pr.N; r >= 1; --r) width[r - 1] = width[r] / pr.P[r - 1] * pr.Q[r - 1];
}

// Which buffers the launches of a plan read and write, and the workspace that takes.
inline void assign_buffers(const Problem& pr, Plan& plan)
{
    // Buffers, assigned backwards from Y: the last launch writes Y, the one before it writes WS0,
    // the one before that writes "B", and so on alternately.  B is Y itself when every row written
    // there fits in a row of Y, otherwise the second workspace.
    const int n = (int)plan.steps.size();
    bool b_is_y = true;
    for (int i = n - 3; i >= 0; i -= 2)
        if (plan.steps[i].k_out > pr.k_out) b_is_y = false;
    int64_t w0 = 0, w1 = 0;
    for (int i = n - 1; i >= 0; --i) {
        const int back = n - 1 - i;
        int dst = back == 0 ? KM_BUF_Y : (back % 2 == 1 ? KM_BUF_WS0 : (b_is_y ? KM_BUF_Y : KM_BUF_WS1));
        plan.steps[i].dst = dst;
        if (dst == KM_BUF_WS0 && plan.steps[i].k_out > w0) w0 = plan.steps[i].k_out;
        if (dst == KM_BUF_WS1 && plan.steps[i].k_out > w1) w1 = plan.steps[i].k_out;
        if (i + 1 < n) plan.steps[i + 1].src = dst;
    }
    plan.steps[0].src = KM_BUF_X;
    plan.ws0_bytes = round_up((size_t)(pr.M * w0) * pr.esize, 256);
    plan.ws1_bytes = round_up((size_t)(pr.M * w1) * pr.esize, 256);
}

// Completes a plan from its groups: take[r] factors are applied when r remain, with pick[r].
inline km_status finish_plan(const Problem& pr, const Options& opt, const Variant* table,
                             const std::vector<int>& take, const std::vector<Choice>& pick,
                             const std::vector<int64_t>& width,
                             const GenericKernel& gen, Plan& plan)
{
    plan = Plan();
    for (int r = pr.N; r >= 1; r -= take[r]) {
        const int nf = take[r];
        const int f = r - 1;
        km_plan_step st = build_step(pr, opt, table, r, nf, pick[r], width, gen);
        // flops of the iterations this launch covers
        int64_t w = st.k_in;
        for (int i = f; i >= f - nf + 1; --i) {
            plan.flops += 2.0 * (double)pr.M * (double)w * pr.Q[i];
            w = w / pr.P[i] * pr.Q[i];
            plan.bytes += (double)pr.P[i] * pr.Q[i] * pr.esize;
        }
        plan.bytes += (double)pr.M * ((double)st.k_in + (double)st.k_out) * pr.esize;
        plan.steps.push_back(st);
    }
    assign_buffers(pr, plan);
    return KM_OK;
}

// Makes `plan` one launch of a whole-row kernel.
inline void take_rows_plan(const Problem& pr, int variant, int threads, int64_t lds_bytes, Plan& plan)
{
    km_plan_step one{};
    one.kernel = KM_KERNEL_ROWS;
    one.variant = variant;
    one.first_factor = 0;
    one.num_factors = pr.N;
    one.tile_slices = 1;
    one.tile_rows = 1;
    one.k_in = pr.k_in;
    one.k_out = pr.k_out;
    one.src = KM_BUF_X;
    one.dst = KM_BUF_Y;
    one.grid = pr.M < 65536 ? pr.M : 65536;              // (the FMA kernel strides over the rows, the other one has at most ROWM_ROWS)
    one.block = threads;
    one.lds_bytes = (int)lds_bytes;
    plan.steps.assign(1, one);
    plan.ws0_bytes = plan.ws1_bytes = 0;
    plan.bytes = (double)pr.M * ((double)pr.k_in + (double)pr.k_out) * (double)pr.esize;
    for (int i = 0; i < pr.N; ++i) plan.bytes += (double)pr.P[i] * pr.Q[i] * pr.esize;
}

// May the whole-row kernel on the matrix cores take the problem (with the shape it would run in)?
inline bool rowm_fits(const Problem& pr, const Options& opt, RowmShape& rs)
{
    if (!(opt.kernels >> KM_KERNEL_ROWS & 1) || pr.N < 2 || pr.N > opt.max_fuse || pr.M > ROWM_ROWS) return false;
    rs = rowm_shape(pr);
    return rs.threads > 0;
}

// No tuning aid asks for particular kernels, tiles or walks.
inline bool no_wishes(const Options& opt)
{
    return !opt.prefer_tile && !opt.prefer_threads && !opt.prefer_instance && !opt.tiles_per_wg && opt.tile_order < 0;
}

// Factor of each of the row's digits of two bits (the first of two 2x2 ones): can fused_row4_kernel.hpp run the problem?
inline bool row4_digits(const Problem& pr, int (&first)[ROW4_DIGITS])
{
    if (pr.dtype != KM_F32 || pr.k_in != ROW4_ELEMS) return false;
    int f = 0;
    for (int d = 0; d < ROW4_DIGITS; ++d) {
        if (f >= pr.N) return false;
        first[d] = f;
        const int p = pr.P[f];
        if ((p != 4 && p != 2) || pr.Q[f] != p) return false;
        if (p == 2 && (f + 1 >= pr.N || pr.P[f + 1] != 2 || pr.Q[f + 1] != 2)) return false;
        if (p == 4 && f > 0 && pr.P[f - 1] == 2) return false;      // (the kernel could run 2x2 factors before 4x4 ones as well, 100 rows 16.3 -> 6.9 us; these rows are planned in two launches so far)
        f += p == 2 ? 2 : 1;
    }
    return f == pr.N;
}

inline bool row4_fits(const Problem& pr, const Options& opt)
{
    int first[ROW4_DIGITS];
    return no_wishes(opt) && (opt.kernels >> KM_KERNEL_FUSED & 1) && opt.max_fuse >= pr.N && row4_digits(pr, first);
}

// Digits per group if fused_cube_kernel.hpp can run the problem, else 0.
inline int cube_group(const Problem& pr)
{
    const int P = pr.P[0], G = P == 5 ? 2 : P == 3 ? 3 : 0;
    if (pr.dtype != KM_F32 || G == 0 || (pr.N != 3 * G && pr.N != 4 * G)) return 0;
    for (int i = 0; i < pr.N; ++i)
        if (pr.P[i] != P || pr.Q[i] != P) return 0;
    return G;
}

// (one row of 4G digits is 25 or 27 tiles, and stays with launches of smaller ones: 5^8 12.9 us there, 13.5 here, two rows 17.8
// and 14.5)
inline bool cube_fits(const Problem& pr, const Options& opt)
{
    return no_wishes(opt) && (opt.kernels >> KM_KERNEL_FUSED & 1) && opt.max_fuse >= pr.N && cube_group(pr) > 0 && !(pr.M == 1 && pr.N == 4 * cube_group(pr));
}

inline void take_cube_plan(const Problem& pr, Plan& plan)
{
    const int G = cube_group(pr), launches = pr.N / G - 2;
    int64_t E = 1;
    for (int i = 0; i < G; ++i) E *= pr.P[0];
    plan.steps.clear();
    plan.bytes = 0;
    for (int i = 0; i < launches; ++i) {
        km_plan_step st{};
        st.kernel = KM_KERNEL_FUSED;
        st.variant = CUBE_VARIANT;
        st.num_factors = pr.N / launches;
        st.first_factor = launches == 2 && i == 0 ? 2 * G : 0;
        st.tile_slices = launches == 2 ? (int)E : 1;
        st.tile_rows = 1;
        st.k_in = st.k_out = pr.k_in;
        st.block = (int)((E * E + 63) / 64 * 64);
        st.lds_bytes = (int)(E * cube_stride((int)E) * (int64_t)pr.esize);
        st.tile_order = INPLACE_ORDER;
        const int64_t tiles = pr.M * (pr.k_in / (E * E * E));
        // (Two workgroups to a compute unit that walk; with two launches and thousands of tiles a workgroup for each, in multiples of 8 for
        // the order of the tiles, us in both launches: 100 x 5x5^8 162 and 155, 250 rows 442 and 355, 1000 rows 1783 and 1343, but 40
        // rows 56 and 63.  Walking workgroups drift apart, and lines that neighbouring tiles share are moved twice; the
        // limit keeps a launch below 2^32 work-items.)
        const int64_t limit = (int64_t)1 << 20;
        st.grid = launches == 2 && tiles >= 2500 ? (tiles < limit ? tiles : limit) / 8 * 8 : tiles < 512 ? tiles : 512;
        st.tiles_per_wg = (int)((tiles + st.grid - 1) / st.grid);
        plan.bytes += (double)pr.M * 2.0 * (double)pr.k_in * pr.esize + (double)st.num_factors * pr.P[0] * pr.P[0] * pr.esize;
        plan.steps.push_back(st);
    }
    assign_buffers(pr, plan);
}

// Can the kernels that leave digits in place run the whole problem?
inline bool inplace_fits(const Problem& pr, const Options& opt)
{
    if (pr.dtype != KM_F32 || pr.N < 2 || opt.max_fuse < 2 || !(opt.kernels >> KM_KERNEL_MFMA & 1)) return false;
    if (!no_wishes(opt)) return false;
    const int P = pr.P[pr.N - 1];
    if (P != 48 && P != 64) return false;
    for (int f = pr.N - 2; f < pr.N; ++f)
        if (pr.P[f] != P || pr.Q[f] != P) return false;
    int64_t w = pr.k_in;
    for (int f = pr.N - 1; f >= 0; --f) {
        if (f < pr.N - 2 && (pr.P[f] % 16 || pr.Q[f] % 16 || pr.P[f] > 128 || pr.Q[f] > 128)) return false;
        if (w * (int64_t)pr.esize >= (int64_t)1 << 31) return false;     // (in-row offsets are 32 bits)
        w = w / pr.P[f] * pr.Q[f];
    }
    return w * (int64_t)pr.esize < (int64_t)1 << 31;
}

// Workgroups of a launch on a digit, at most one per compute unit: one for each stretch of columns while there are no more of
// them than compute units, then one for two.  (A workgroup for two from the start left half the chip idle: 20 x (128x128,
// 48x48^2) 65.6 us, 50.8 now, 26 x (96x96, 48x48^2) 47.3 and 38.3.  32 x (112x112, 48x48^2), 288 stretches: 63.4 us in 144
// workgroups, 65.9 in 256.)
inline int64_t digit_stretches(int64_t columns) { return (columns + DIGIT_STRETCH - 1) / DIGIT_STRETCH; }
inline int64_t digit_grid(int64_t columns)
{
    const int64_t stretches = digit_stretches(columns), grid = stretches <= 256 ? stretches : (stretches + 1) / 2;
    return grid < 256 ? grid : 256;
}

// Microseconds of the launches that leave digits in place, and of the rotating launches that they stand in for, fitted to 511
// problems (5 and 6 % off): the first kernel by its matrices per wavefront, the others by their bytes or, where there are few
// columns, by a wavefront's runs.
inline double inplace_us(const Problem& pr)
{
    const int64_t last = pr.P[pr.N - 1];
    int64_t w = pr.k_in;
    double us = 13.7 + 18.2 * (double)(pr.M * (w / (last * last))) / 2048 * (double)(last * last * last) / (64 * 64 * 64);
    for (int f = pr.N - 3; f >= 0; --f) {
        const int64_t stretches = digit_stretches(pr.M * (w / pr.P[f])), to = w / pr.P[f] * pr.Q[f];
        const double move = (double)pr.M * (double)(w + to) * (double)pr.esize / 5.85e6;
        const double runs = (double)((stretches + 255) / 256) * (0.9 + 22.0 * pr.P[f] * pr.Q[f] / (128 * 128));
        us += 2.7 + (move > runs ? move : runs);
        w = to;
    }
    return us;
}
inline double rotating_us(const Problem& pr, const std::vector<km_plan_step>& steps)
{
    double us = 0;
    for (const km_plan_step& st : steps) {
        double flops = 0;
        int64_t w = st.k_in;
        for (int f = st.first_factor + st.num_factors - 1; f >= st.first_factor; --f) {
            flops += 2.0 * (double)pr.M * (double)w * pr.Q[f];
            w = w / pr.P[f] * pr.Q[f];
        }
        const double bytes = (double)pr.M * (double)(st.k_in + st.k_out) * (double)pr.esize;
        const bool any = st.kernel != KM_KERNEL_MFMA, pair = !any && st.num_factors > 1;
        const double move = bytes / (any ? 5.15e6 : pair ? 5.2e6 : 5.95e6), products = flops / (any ? 93e6 : pair ? 64.6e6 : 91e6);
        us += (any ? 8.9 : pair ? 0.7 : 5.8) + (move > products ? move : products);
    }
    return us;
}

// ... and are they the faster ones?  From a matrix per wavefront of the first launch on (two workgroups of four on each
// compute unit), and then by the estimates.  Two 64x64 factors alone have a whole-row instance (65536 rows 0.570 ms, 0.594 here); two
// 48x48 ones were two launches (65536 rows 0.529 ms, 0.264 here, 4096 rows 46.5 us and 23.8).  With factors before them, rotating launches and these,
// us: 1024 x 64x64^3 1157 and 987, 64 rows 88 and 79, 64 x 48x48^3 44 and 35, 256 x (96x96, 48x48^2) 308 and 223.  Rotating launches are
// the faster ones where they take two leading factors at a time and where wide factors have few columns: 128 x (16x16^2, 64x64^2)
// 569 and 669, 1 x (16x16^4, 48x48^2) 956 and 1134, 20 x (128x128, 48x48^2) 45 and 51, 1 x (128x128, 16x16, 48x48^2) 47 and 58.
inline bool inplace_wins(const Problem& pr, const std::vector<km_plan_step>& steps)
{
    const int P = pr.P[pr.N - 1];
    if (pr.M * (pr.k_in / (P * P)) < 512 * (CHAIN_THREADS / 64)) return false;
    return pr.N == 2 ? P == 48 : inplace_us(pr) < 0.97 * rotating_us(pr, steps);
}

inline void take_inplace_plan(const Problem& pr, Plan& plan)
{
    plan.steps.clear();
    plan.bytes = 0;
    int64_t w = pr.k_in;
    for (int left = pr.N; left > 0;) {
        km_plan_step st{};
        st.kernel = KM_KERNEL_MFMA;
        st.num_factors = left == pr.N ? 2 : 1;
        st.first_factor = left - st.num_factors;
        st.k_in = w;
        for (int f = left - 1; f >= st.first_factor; --f) {
            w = w / pr.P[f] * pr.Q[f];
            plan.bytes += (double)pr.P[f] * pr.Q[f] * pr.esize;
        }
        st.k_out = w;
        st.tile_order = INPLACE_ORDER;
        st.tile_rows = 1;
        const int64_t P = pr.P[st.first_factor], Q = pr.Q[st.first_factor];
        int64_t tiles;
        if (st.num_factors == 2) {                       // two workgroups per compute unit
            st.variant = CHAIN_VARIANT;
            st.tile_slices = CHAIN_THREADS / 64;
            st.block = CHAIN_THREADS;
            st.lds_bytes = (int)(2 * P * P * (int64_t)pr.esize);
            tiles = (pr.M * (st.k_in / (P * P)) + st.tile_slices - 1) / st.tile_slices;
            st.grid = tiles < 512 ? tiles : 512;
        } else {                                         // one
            st.variant = DIGIT_VARIANT;
            st.tile_slices = DIGIT_COLS;
            st.block = DIGIT_THREADS;
            st.lds_bytes = (int)(P * Q * (int64_t)pr.esize);
            tiles = (pr.M * (st.k_in / P) + st.tile_slices - 1) / st.tile_slices;
            st.grid = digit_grid(pr.M * (st.k_in / P));
        }
        st.tiles_per_wg = (int)((tiles + st.grid - 1) / st.grid);
        plan.bytes += (double)pr.M * ((double)st.k_in + (double)st.k_out) * pr.esize;
        plan.steps.push_back(st);
        left = st.first_factor;
    }
    assign_buffers(pr, plan);
}

// Would the launch after this one find this one's results in the last-level cache?  Launches with a slice per lane leave at most 160 MiB
// there, others 320.  (Results whose runs do not start on 64-byte boundaries are stored alike by both; above 256 MiB the cache holds too little of them.)
inline bool lane_cached(const Problem& pr, const km_plan_step& st)
{
    const double mib = (double)pr.M * (double)st.k_out * (double)pr.esize / 1048576.0;
    return mib > 160.0 && mib <= (st.k_in / pr.P[st.first_factor] * (int64_t)pr.esize % 64 == 0 ? 320.0 : 256.0);
}

// Does the slice-per-lane kernel beat the one that step i was given to?  Fitted to some 8000 pairs of calls, with and without it in one or
// more of their launches, on problems of random sizes.  On 1306 more of them 875 calls change, 1.21 times as fast on average, 97 % of them as
// fast or faster (within 2 %), the worst 0.83.  By what the step was given to:
// - the generic kernel: 1.3 times (20.8 M slices of 10x2 408 -> 226 us, 20.1 M of 10x6 406 -> 248).  From 64 workgroups of 256 slices
//   on (calls with 64 to 128 of them 0.6 us faster); fewer leave it a single tile's latency.  Slices of up to 8 elements, which that kernel reads
//   without LDS, need more of both: on short rows a tile's results are in many runs and stored element by element (1.6 M of 5x31, 16 to a row,
//   88 -> 130 us).  Tall slices with few columns only while they are few (249 K of 72x2 24.0 -> 21.4, 512 K of 75x2 39.6 -> 45.4).
// - the chunked form: 1.34 times on slices that are no whole vectors, which that one deals to LDS element by element (6.9 M of 34x8 439 ->
//   274).  Others lose what it gains elsewhere (1.3 M of 48x9 54 -> 73) but for more than 16 columns (3 M of 72x72 655 -> 450), 36 rows (1.07 to
//   1.2) and small launches of few columns.
// - the form with the factor in registers, from 92 MiB moved on; with less the one tile that a wavefront gets takes longer than the products saved.
//   Its sixteen columns to a wavefront leave some idle, and with two, three and five wavefronts also SIMDs: up to 36 rows and 40 columns
//   1.17 times (7.4 M of 33x33 536 -> 384), whole vectors 1.10 (9.6 M of 24x29 481 -> 372), 65 to 76 columns 1.29 (3.8 M of 65x65 857 -> 538); columns that
//   fill the sixteens only on the largest problems (8 M of 30x32 497 -> 353, 1 M of 34x32 39 -> 51), whole vectors in few columns only with
//   small results (24x12^3 of 165 MiB 1.14, 20x13^4 of 175 MiB 0.93; 72x72, rows of 72 slices, 0.87).  Rows of less than 64
//   slices, each tile in several of them, 0.56 to 0.9 (9 M x 16x16 376 -> 645 us) where the
//   intermediates stay on chip or there is none; from 160 MiB on 1.11, and with few columns, few of those stores, 1.16.
//   Intermediates of 160 to 320 MiB stay with that form, which leaves them in the last-level cache (2250 x 31x31^3 whole 319 us there, 346
//   with one launch of three here), but for 33 to 36 columns, which gain more than that costs (1.11).
inline bool lane_wins(const Problem& pr, const Plan& plan, size_t i)
{
    const km_plan_step& st = plan.steps[i];
    const int P = pr.P[st.first_factor], Q = pr.Q[st.first_factor];
    const int64_t S = st.k_in / P, groups = (pr.M * S + 4 * LANE_SLICES - 1) / (4 * LANE_SLICES);
    const bool vectors = P % 4 == 0;                     // slices are whole 16-byte vectors
    if (st.variant == PAD_VARIANT) {
        const bool first = i == 0, last = i + 1 == plan.steps.size();
        const double mib = (double)pr.M * (double)pr.esize / 1048576.0, in = mib * (double)st.k_in, out = mib * (double)st.k_out;
        if (in + out < 92.0) return false;
        if (!lane_fits_pad(P, Q)) return false;
        if (P > 64) return S >= (vectors ? 1024 : Q <= 72 || in + out > 400.0 ? 64 : 128);
        if (Q % 16 == 0 && in < 600.0) return false;
        if (vectors && (Q <= 8 ? P < 20 || P > 28 : Q <= 16 || (P >= 32 && Q <= 32))) return S >= LANE_SLICES && in <= 180.0 && out <= 100.0;
        if (Q <= 8 || (Q <= 10 && P > 16 && !vectors)) return true;
        if (S < LANE_SLICES) return !vectors && S >= 6 && P >= 9 && (first || in > 160.0) && (last || out > 160.0);
        if (P > 32 && Q > 32 && Q <= 36) return true;
        return !(!first && lane_cached(pr, plan.steps[i - 1])) && !(!last && lane_cached(pr, st));
    }
    if (groups < 64 || S < 16 || (S < 256 && Q > 32)) return false;
    if (st.kernel != KM_KERNEL_GENERIC) {
        if (!lane_fits_chunked(P, Q) || groups < 128) return false;
        return !vectors || P == 36 || (Q <= 8 ? groups < 512 : P > 64 || groups >= 512);
    }
    if (!lane_fits_generic(P, Q)) return false;
    if (P <= 8) {
        if (S < 128) return groups >= 512 && (Q <= 4 || (Q <= 8 && P < 8) || (Q <= 32 && P > 5 && P < 8 && groups >= 8192));
        return groups >= (Q <= 4 ? 256 : Q <= 16 ? 128 : 64);
    }
    return P <= 32 || Q > 4 || P > 96 || groups < 1024;
}

inline bool lane_allowed(const Problem& pr, const Options& opt) { return pr.dtype == KM_F32 && (opt.kernels >> KM_KERNEL_MFMA_ANY & 1) && no_wishes(opt); }

// The steps that the slice-per-lane kernel runs faster go to it, once the plan is made: the prices that group factors and weigh
// plans against each other are those of the kernels it takes the steps from.
inline void take_lane_steps(const Problem& pr, const Options& opt, Plan& plan)
{
    if (!lane_allowed(pr, opt)) return;
    for (size_t i = 0; i < plan.steps.size(); ++i) {
        km_plan_step& st = plan.steps[i];
        if (st.kernel != KM_KERNEL_GENERIC && st.kernel != KM_KERNEL_MFMA_ANY) continue;
        const int P = pr.P[st.first_factor], Q = pr.Q[st.first_factor];
        const LaneShape sh = lane_shape(P, Q, pr.M * (st.k_in / P));
        if (sh.lds_bytes == 0 || !lane_wins(pr, plan, i)) continue;
        make_lane_step(sh, st);
    }
}

// Microseconds of the whole-row FMA kernel: per row a fixed part, its factors' loads and per step 1 us and 70 ns (fp64 106) for each of
// the P products that a thread adds up in turn; 1024 threads have a compute unit to themselves.
inline double fma_rows_us(const Problem& pr, int threads, int64_t lds_bytes, const std::vector<int64_t>& width)
{
    int64_t side = threads >= 1024 ? 1 : 160 * 1024 / (lds_bytes < 20 * 1024 ? 20 * 1024 : lds_bytes);
    if (side > 2048 / threads) side = 2048 / threads;
    const int64_t rounds = (pr.M + 256 * side - 1) / (256 * side);
    if (side > (pr.M + 255) / 256) side = (pr.M + 255) / 256;
    double row = 0.328 + 0.159 * (double)(pr.k_in + pr.k_out) / threads;
    for (int r = pr.N; r >= 1; --r) {
        const int64_t S = width[r] / pr.P[r - 1], units = (S + 1) / 2 * ((pr.Q[r - 1] + 3) / 4);
        row += 1.036 + (double)((units + threads - 1) / threads) * pr.P[r - 1] * (pr.esize == 4 ? 0.069 : 0.106) +
               (double)side * (double)width[r] * (double)pr.Q[r - 1] * 5.4e-6 + 0.275 * pr.P[r - 1] * pr.Q[r - 1] / threads;
    }
    return 1.13 + (double)rounds * row;
}

// Microseconds of tiled launches, for comparison with the whole-row kernels.  Generic launches in the form that they take, or
// (by_form false) all at the padded form's rate, which is what decides whether a problem has a whole-row plan at all.
inline double tiled_us(const Problem& pr, const std::vector<km_plan_step>& steps, const GenericKernel& gen, bool by_form)
{
    double us = 0;
    for (const km_plan_step& st : steps) {
        const double bytes = (double)pr.M * ((double)st.k_in + (double)st.k_out) * (double)pr.esize;
        const int P = pr.P[st.first_factor], Q = pr.Q[st.first_factor];
        // (small launches of the chunked form of the run-time-shape MFMA kernel: 5.5 us when slices are whole 16-byte
        // vectors and one chunk, 10 otherwise: 100 x 36x36^2 10.0 us in two, 200 x 50x50^2 20.2, 33 x 80x80^2 20.4)
        if (st.variant == PAD_VARIANT) {
            const int64_t slices = pr.M * (st.k_in / P);
            us += pad_us(P, Q, pr.esize, slices, pad_shape(P, Q, pr.esize, slices));
        } else if (st.kernel == KM_KERNEL_MFMA_ANY)
            us += (P * pr.esize % 16 == 0 && P * pr.esize <= (size_t)gen.any_row_bytes ? 5.5 : 9.5) + bytes / 7e6;
        else if (st.kernel == KM_KERNEL_GENERIC) {
            // (the form without padding: its pass over a tall slice takes its time too; the other one moves its bytes at a
            // third of the rate, as launch_cost has it)
            const bool small = by_form && gen_small_form(P, Q, st.k_in / P, (int64_t)pr.esize);
            us += small ? 2.7 + (P > 16 ? 0.06 * (P - 16) : 0.0) + bytes / 3e6 : 4.5 + 0.7 * ((P + 15) / 16) + bytes / 1.7e6;
        } else
            us += 2.5 + bytes / 5e6;
    }
    return us;
}

// `spare`: where `plan` needs a workspace and stands in for a whole-row plan, that one; else without steps.
inline km_status make_plan(const Problem& pr, const Options& opt, const Variant* table, int count,
                           const GenericKernel& gen, Plan& plan, Plan& spare)
{
    const int N = pr.N;
    spare = Plan();
    std::vector<int64_t> width;
    row_widths(pr, width);
    // Grouping by dynamic programming over r: best[r] = cheapest way to apply factors 0..r-1.
    std::vector<double> best(N + 1, 0.0);
    std::vector<int> take(N + 1, 1);
    std::vector<Choice> pick(N + 1);
    for (int r = 1; r <= N; ++r) {
        best[r] = -1;
        for (int nf = 1; nf <= r && nf <= opt.max_fuse; ++nf) {
            Choice ch = find_variant(table, count, pr, r - 1, nf, width[r], opt);
            if (nf > 1 && !ch.var) continue;             // only single factors fall back to the kernels without compiled shapes
            if (!ch.var) ch.any_mfma = any_mfma_fits(pr, r - 1, opt);
            double c = launch_cost(pr, width[r], width[r - nf], ch, pr.P[r - 1]);
            if (opt.prefer_instance > 0 && opt.prefer_instance <= count && ch.var == &table[opt.prefer_instance - 1]) c *= 0.5;      // (asked for: the grouping should let it in)
            c += best[r - nf];
            if (best[r] < 0 || c <= best[r] * (1 + 1e-9)) { best[r] = c; take[r] = nf; pick[r] = ch; }
        }
    }
    km_status st = finish_plan(pr, opt, table, take, pick, width, gen, plan);
    if (st != KM_OK) return st;

    // Every factor in one launch with the row resident in LDS, whatever the factor shapes, when
    // that is cheaper: plain FMA code run by one workgroup per row, so only where the launches saved
    // outweigh it.  Measured time per row of one workgroup: about 2 us plus 0.4 us per factor of
    // fixed cost, plus 35 ns per multiply-add of each of its 256 threads, or 50 ns with the 1024
    // threads taken when rows are few (fp64: 1.5 times that); rows run side by side as far as LDS
    // and 2048 threads per compute unit allow.
    const bool force_rows = opt.prefer_instance == count + 1;      // tuning aid: this kernel whenever it fits
    Plan rows = plan;                                    // (for its flops)
    double rows_us = -1;
    if ((opt.kernels >> KM_KERNEL_ROWS & 1) && N >= 2 && N <= gen.row_max_factors && N <= opt.max_fuse &&
        (plan.steps.size() > 1 || force_rows)) {
        int64_t maxw = 0;
        double macs = 0;
        for (int r = 0; r <= N; ++r) maxw = width[r] > maxw ? width[r] : maxw;
        for (int r = 1; r <= N; ++r) macs += (double)width[r] * (double)pr.Q[r - 1];
        int64_t fel = 0;
        for (int i = 0; i < N; ++i) fel += (int64_t)pr.P[i] * pr.Q[i];
        // two row buffers (one word in 33 skipped, see row_kernel.hpp) and every factor
        const int64_t lds = (2 * (maxw + (maxw >> 5) + 1) + fel) * (int64_t)pr.esize;
        if (lds <= gen.row_lds_limit) {
            const bool few = pr.M <= gen.row_few_rows;
            const int threads = few ? gen.row_threads_few : gen.row_threads_many;
            int64_t per_cu = 160 * 1024 / (lds < 20 * 1024 ? 20 * 1024 : lds);
            if (per_cu > 2048 / threads) per_cu = 2048 / threads;
            const int64_t side_by_side = 256 * per_cu;
            const double rounds = (double)((pr.M + side_by_side - 1) / side_by_side);
            const double per_mac = (few ? 50e-9 : 35e-9) * (pr.esize == 4 ? 1.0 : 1.5);
            // ... and rows that share a compute unit share its LDS bandwidth: about 60 ps per multiply-add
            // and compute unit, whatever the precision (measured with 7 or 8 rows per unit: 103563 x 6^4
            // 14.9 us per round, 116508 x 24x24^2 fp64 13.6, 37282 x (9x3, 32x100) 13.2)
            const int64_t rows_per_cu = per_cu < (pr.M + 255) / 256 ? per_cu : (pr.M + 255) / 256;
            // (long rows: about 0.1 us per trip of the workgroup through the loops that load and store a
            // row, beyond the first trips, which are part of the fixed cost; it was 0.45 us while the row
            // loader kept no loads in flight: 3355 x (10x5)^4, rows of 10000 floats on 256 threads, took 34 us
            // per round where the multiply-adds account for 16, and takes 15.5 now)
            const double trips = (double)(width[N] + width[0]) / threads;
            const double alone = 2.0e-6 + 0.4e-6 * N + macs / threads * per_mac + (trips > 8 ? (trips - 8) * 0.1e-6 : 0.0);
            const double shared = 2.0e-6 + (double)rows_per_cu * macs * 60e-12;
            const double seconds = rounds * (alone > shared ? alone : shared);
            const double bytes = (double)pr.M * ((double)width[N] + (double)width[0]) * (double)pr.esize;
            double c = seconds * 5e12;
            // and its row loads and stores, a short loop without loads in flight ahead, stream at about
            // 1.1 TB/s over the whole chip at best (13107 x (80x5, 64x2), rows of 20 KB: 0.384 ms, the tiled
            // plan 0.090; 116508 x (16x13, 36x4) fp64 0.628 against 0.228)
            if (c < 4.5 * bytes) c = 4.5 * bytes;
            c += 2.5e7;
            if (c < best[N] || force_rows) {
                take_rows_plan(pr, -1, threads, lds, rows);
                rows_us = fma_rows_us(pr, threads, lds, width);
            }
        }
    }
    // The same on the matrix cores (row_mfma_kernel.hpp), for up to ROWM_ROWS rows, in the place of a whole-row
    // plan of the FMA kernel or of tiled launches without compiled shapes.  Launches of compiled instances are
    // as quick on problems this small (16 x 16x16^3 6.9 us in three of them, 7.7 here; 128 x 32x32^2 4.9
    // and 4.7).  The others by their estimates, each within 8 % of what was measured on 700 problems: 10 x (52x50,
    // 65x20) fp64 20.1 us in two launches, 6.7 here, 5 x 61x61^2 fp64 9.1 and 11.0; on the FMA kernel 300 x (32x32, 64x3)
    // 19.9 and 4.7, 37 x (9x4, 15x14, 4x44) 8.5 and 10.4.  (The kernel has become a tenth quicker than the estimate since.  Level with tiled launches the single one without workspace is
    // taken: 1000 x 50x50^2 18.3 us and 16.8, 900 rows 15.9 and 16.6; the FMA kernel stays where the two are within 5 %, since
    // short contractions make this one's estimate too low: 54 x 2x1^6 7.2 us and 7.6.)
    bool compiled = true;
    for (const km_plan_step& s1 : plan.steps) compiled = compiled && s1.variant >= 0;
    RowmShape rs;
    if ((rows_us >= 0 || !compiled) && !(force_rows && rows_us >= 0) && rowm_fits(pr, opt, rs)) {
        const double had = rows_us >= 0 ? rows_us : tiled_us(pr, plan.steps, gen, false);
        if (rs.us < (rows_us >= 0 ? 0.95 : 1.02) * had) {
            take_rows_plan(pr, ROWM_VARIANT, rs.threads, rs.lds_bytes, rows);
            rows_us = rs.us;
        }
    }
    // The whole-row plan, whichever kernel it is on, unless the finer estimates promise a tenth from tiled launches whose
    // workspace fits the static array: 9363 x (74x14, 18x5) 79 us in rows, 31 in two launches, 5058 x (18x4,
    // 39x3) 27 and 10; of 91 such problems 90 are faster tiled, 2.1 times on average, since the generic kernel has its form for small
    // factors.  (Not so small compiled launches against the matrix-core rows: 300 x 2x2^2 fp64 3.9 us in rows, 6.6 tiled, 500 x 4x4^3 fp64
    // 4.7 and 6.3; 500 x 16x16^2 takes 4.2 and 3.8, but two launches of the host's.  Up to a row per compute unit the fixed costs
    // decide, which these estimates do not know that well: one launch there.)  Calls that bring no such workspace keep the
    // whole-row plan: they may run side by side on several streams, which calls that share one workspace may not.
    if (rows_us >= 0) {
        const bool tiled = !force_rows && pr.M > 256 && plan.ws0_bytes + plan.ws1_bytes <= KM_STATIC_SCRATCH_BYTES &&
                           tiled_us(pr, plan.steps, gen, true) < 0.9 * rows_us;
        (tiled ? spare : plan) = rows;
    }
    if (inplace_fits(pr, opt) && inplace_wins(pr, plan.steps)) take_inplace_plan(pr, plan);
    if (cube_fits(pr, opt)) take_cube_plan(pr, plan);
    if (row4_fits(pr, opt)) {
        take_rows_plan(pr, ROW4_VARIANT, ROW4_THREADS, ROW4_LDS_BYTES, plan);
        km_plan_step& one = plan.steps[0];
        one.kernel = KM_KERNEL_FUSED;
        one.grid = pr.M < ROW4_GRID ? pr.M : ROW4_GRID;
        one.tiles_per_wg = (int)((pr.M + one.grid - 1) / one.grid);
        one.tile_order = 2;
    }
    if (plan.ws0_bytes + plan.ws1_bytes == 0) spare = Plan();
    take_lane_steps(pr, opt, plan);
    return KM_OK;
}

// The kernels without compiled shapes that the tuner times for factor f of rows of `width` elements: the generic one, and of the run-time-shape
// MFMA family every form that can run it, a slice per lane from as many slices on as that form is ever planned for.
inline void uncompiled_choices(const Problem& pr, const Options& opt, int f, int64_t width, std::vector<Choice>& out)
{
    out.push_back(Choice());
    const int64_t slices = pr.M * (width / pr.P[f]);
    Choice any;
    any.any_mfma = true;
    if (any_mfma_fits(pr, f, opt)) {
        any.any_form = -1;
        out.push_back(any);
        any.any_form = PAD_VARIANT;
        if (pad_shape(pr.P[f], pr.Q[f], pr.esize, slices).threads > 0) out.push_back(any);
    }
    any.any_form = LANE_VARIANT;
    if (lane_allowed(pr, opt) && slices > 63 * 4 * LANE_SLICES && lane_shape(pr.P[f], pr.Q[f], slices).lds_bytes > 0) out.push_back(any);
}

// The tuner's candidates besides the planner's own plan and the one it measured: the whole-row kernels wherever they fit, if the
// planner did not take them itself (no steps: not a candidate).  They need no workspace.
inline void whole_row_candidates(const Problem& pr, const Options& opt, const Variant* table, int count, const GenericKernel& gen,
                                 const Plan& deflt, Plan& fma, Plan& mfma)
{
    auto is_rows = [](const Plan& p, int variant) {
        return p.steps.size() == 1 && p.steps[0].kernel == KM_KERNEL_ROWS && p.steps[0].variant == variant;
    };
    fma = mfma = Plan();
    if (!is_rows(deflt, -1)) {
        Options force = opt;
        force.prefer_instance = count + 1;
        Plan none;
        if (make_plan(pr, force, table, count, gen, fma, none) != KM_OK || !is_rows(fma, -1)) fma = Plan();
    }
    RowmShape rs;
    if (!is_rows(deflt, ROWM_VARIANT) && rowm_fits(pr, opt, rs)) {
        mfma = deflt;                                    // (for its flops)
        take_rows_plan(pr, ROWM_VARIANT, rs.threads, rs.lds_bytes, mfma);
    }
}

}  // namespace km
