// Launcher of the run-time-shape MFMA kernel with a slice per lane (declared in launch.hpp).
#pragma once
#include "launch.hpp"
#include "mfma_lane_kernel.hpp"

namespace km {

template <int G, int U>
static hipError_t launch_lane_shape(const LaunchArgs& a)
{
    const km_plan_step& st = *a.st;
    const int f = st.first_factor, P = a.pr->P[f], Q = a.pr->Q[f];
    auto kern = mfma_lane_sliced_multiply<G, U>;
    static unsigned char lds_ok[64];
    hipError_t e = allow_lds((const void*)kern, lane_lds_bytes(LANE_MAXP, 4 * G, U), lds_ok);
    if (e != hipSuccess || a.prepare_only) return e;
    const int64_t S = st.k_in / P, slices = a.pr->M * S;
    const LaneShape sh = lane_shape(P, Q, slices);
    if (sh.lds_bytes == 0 || st.block != LANE_THREADS || st.grid != sh.grid || st.lds_bytes != sh.lds_bytes || st.tile_slices != LANE_SLICES) return hipErrorInvalidValue;
    // (output runs that do not start on 64-byte boundaries: ordinary stores, as in launch_any.hpp)
    const bool keep = a.keep_output || S * (int64_t)sizeof(float) % 64 != 0;
    hipLaunchKernelGGL(kern, dim3((unsigned)st.grid), dim3((unsigned)st.block), (size_t)st.lds_bytes, a.stream, (const float*)a.src,
                       (const float*)a.factors[f], (float*)a.dst, S, P, Q, ((P + 3) / 4 + U - 1) / U, lane_row_magic(S),
                       S >= LANE_SLICES || S == 1 ? 0u : (unsigned)(((1ull << 32) + (unsigned long long)S - 1) / (unsigned long long)S),
                       slices, (slices + LANE_SLICES - 1) / LANE_SLICES, keep ? 1 : 0);
    return hipGetLastError();
}

template <int U>
hipError_t launch_mfma_lane(const LaunchArgs& a)
{
    const km_plan_step& st = *a.st;
    const int P = a.pr->P[st.first_factor], Q = a.pr->Q[st.first_factor];
    if (a.pr->dtype != KM_F32 || st.num_factors != 1 || st.k_in % P || lane_units(P) != U) return hipErrorInvalidValue;
    switch ((Q + 3) / 4) {
#define KM_LANE(n) case n: if constexpr (lane_compiled(n, U)) return launch_lane_shape<n, U>(a); break;
        KM_LANE(1) KM_LANE(2) KM_LANE(3) KM_LANE(4) KM_LANE(5) KM_LANE(6) KM_LANE(7) KM_LANE(8)
        KM_LANE(9) KM_LANE(10) KM_LANE(11) KM_LANE(12) KM_LANE(13) KM_LANE(14) KM_LANE(15) KM_LANE(16)
        KM_LANE(17) KM_LANE(18) KM_LANE(19) KM_LANE(20) KM_LANE(21) KM_LANE(22) KM_LANE(23) KM_LANE(24)
        KM_LANE(25) KM_LANE(26) KM_LANE(27) KM_LANE(28) KM_LANE(29) KM_LANE(30) KM_LANE(31) KM_LANE(32)
#undef KM_LANE
    }
    return hipErrorInvalidValue;
}

}  // namespace km
