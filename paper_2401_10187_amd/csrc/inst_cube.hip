// Rows of P^(3G) and P^(4G) floats: the kernel's instances, with their launcher.
#include "launch.hpp"
#include "fused_cube_kernel.hpp"

namespace km {

template <int P, int G, int PART>
static hipError_t launch_cube_part(const LaunchArgs& a)
{
    typedef CubeShape<P, G> Sh;
    const km_plan_step& st = *a.st;
    const Problem& pr = *a.pr;
    auto kern = fused_cube_multiply<P, G, PART>;
    static unsigned char lds_ok[64];
    hipError_t e = allow_lds((const void*)kern, Sh::LDS_BYTES, lds_ok);
    if (e != hipSuccess || a.prepare_only) return e;
    const int64_t tiles = pr.M * (pr.k_in / ((int64_t)Sh::E * Sh::EE));
    if (st.num_factors != (PART == 0 ? 3 : 2) * G || st.first_factor != (PART == 1 ? 2 * G : 0) || pr.N != (PART == 0 ? 3 : 4) * G) return hipErrorInvalidValue;
    if (st.block != Sh::NT || st.lds_bytes != Sh::LDS_BYTES || st.grid < 1 || st.grid > tiles || (st.grid % 8 && st.grid != tiles)) return hipErrorInvalidValue;
    CubeFactors fa{};
    for (int i = 0; i < st.num_factors; ++i) fa.f[i / G + (PART == 1 ? 1 : 0)][i % G] = (const float*)a.factors[st.first_factor + i];
    hipLaunchKernelGGL(kern, dim3((unsigned)st.grid), dim3(Sh::NT), Sh::LDS_BYTES, a.stream, (const float*)a.src, (float*)a.dst, fa, tiles);
    return hipGetLastError();
}

template <int P, int G>
static hipError_t launch_cube_shape(const LaunchArgs& a)
{
    if (a.pr->N == 3 * G) return launch_cube_part<P, G, 0>(a);
    return a.st->first_factor ? launch_cube_part<P, G, 1>(a) : launch_cube_part<P, G, 2>(a);
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
