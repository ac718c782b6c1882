// Rows of P^(3G) and P^(4G) floats: the kernel's instances, with their launcher.
#include "launch.hpp"
#include "fused_cube_kernel.hpp"

namespace km {

template <int P, int G>
static hipError_t launch_cube_shape(const LaunchArgs& a)
{
    typedef CubeShape<P, G> Sh;
    const km_plan_step& st = *a.st;
    const Problem& pr = *a.pr;
    static unsigned char lds_ok[64];
    hipError_t e = allow_lds((const void*)fused_cube_multiply<P, G>, Sh::LDS_BYTES, lds_ok);
    if (e != hipSuccess || a.prepare_only) return e;
    const int64_t cube = (int64_t)Sh::E * Sh::EE;
    const int64_t tiles = pr.M * (pr.k_in / cube);
    const bool row = pr.N == 3 * G, ends = !row && st.first_factor == 0;
    if (st.num_factors != (row ? 3 : 2) * G || (!row && !ends && st.first_factor != G) || (row && st.first_factor != 0)) return hipErrorInvalidValue;
    if (st.block != Sh::NT || st.lds_bytes != Sh::LDS_BYTES || st.grid < 1 || st.grid > tiles || (st.grid % 8 && st.grid != tiles)) return hipErrorInvalidValue;
    CubeFactors fa{};
    auto group = [&](int at, int first) { for (int k = 0; k < G; ++k) fa.f[at][k] = (const float*)a.factors[first + k]; };
    if (row) {
        for (int k = 0; k < 3; ++k) group(k, k * G);
    } else if (ends) {
        group(0, 0);
        group(2, 3 * G);
    } else {
        group(0, G);
        group(1, 2 * G);
    }
    hipLaunchKernelGGL((fused_cube_multiply<P, G>), dim3((unsigned)st.grid), dim3(Sh::NT), Sh::LDS_BYTES, a.stream, (const float*)a.src,
                       (float*)a.dst, fa, tiles, ends ? (int64_t)Sh::E : (int64_t)1, ends ? pr.k_in : cube, ends ? cube : (int64_t)Sh::EE);
    return hipGetLastError();
}

hipError_t launch_cube(const LaunchArgs& a)
{
    switch (cube_group(*a.pr)) {
        case 2: return launch_cube_shape<5, 2>(a);
        case 3: return launch_cube_shape<3, 3>(a);
    }
    return hipErrorInvalidValue;
}

}  // namespace km
