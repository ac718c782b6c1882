// Compiled instances: LDS-staged MFMA kernels, fp32.
#include "launch_mfma.hpp"
#include "mfma_row32_kernel.hpp"
#include "instances.hpp"

namespace km {

// whole rows of 32^3 have a kernel of their own
template <>
struct MfmaLauncher<MfmaF32x32, 32, 32, 3, 1, 16, 1> {
template <bool KEEP>
static hipError_t run(const LaunchArgs& a)
{
    typedef MfmaShape<MfmaF32x32, 32, 32, 3, 1, 16, 1> Sh;
    static_assert(Row32Shape::LDS_BYTES <= Sh::LDS_BYTES && Row32Shape::NT == Sh::NT, "what the instance table says");
    const km_plan_step& st = *a.st;
    auto kern = mfma_row32_multiply<KEEP>;
    static unsigned char lds_ok[64];
    hipError_t e = allow_lds((const void*)kern, Row32Shape::LDS_BYTES, lds_ok);
    if (e != hipSuccess || a.prepare_only) return e;
    const int64_t rows = a.pr->M, per = st.tiles_per_wg;
    if (st.k_in != Row32Shape::ROW || st.k_out != Row32Shape::ROW) return hipErrorInvalidValue;
    if (per < 1 || (st.tile_order == 2 ? st.grid > rows || st.grid * per < rows : (rows + per - 1) / per != st.grid)) return hipErrorInvalidValue;
    if (st.tile_order != 0 && st.tile_order != 2 && st.tile_order != 3) return hipErrorInvalidValue;
    if (st.tile_order == 3 && !xcd_order_fits(rows, st.grid)) return hipErrorInvalidValue;
    const int f = st.first_factor;
    hipLaunchKernelGGL(kern, dim3((unsigned)st.grid), dim3(Row32Shape::NT), Row32Shape::LDS_BYTES, a.stream, (const float*)a.src, (float*)a.dst,
                       (const float*)a.factors[f + 2], (const float*)a.factors[f + 1], (const float*)a.factors[f], rows, per, st.tile_order);
    return hipGetLastError();
}
};

#define KM_Y_KM_F32(OP, P, Q, NF, ST, NW, QS) template hipError_t launch_mfma<OP, P, Q, NF, ST, NW, QS>(const LaunchArgs&);
#define KM_Y_KM_F64(...)
#define KM_Y(OP, DT, P, Q, NF, ST, NW, QS) KM_Y_##DT(OP, P, Q, NF, ST, NW, QS)
#define KM_NONE(...)
KM_INSTANCES(KM_NONE, KM_Y, KM_NONE, KM_NONE, KM_NONE, KM_NONE, KM_NONE)
}  // namespace km
