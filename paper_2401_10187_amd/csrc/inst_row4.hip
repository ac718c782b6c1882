// The kernel for rows of 4^7 floats, with its launcher.
#include "launch.hpp"
#include "fused_row4_kernel.hpp"

namespace km {

hipError_t launch_row4(const LaunchArgs& a)
{
    const km_plan_step& st = *a.st;
    const Problem& pr = *a.pr;
    static unsigned char lds_ok[64];
    hipError_t e = allow_lds((const void*)fused_row4_multiply, ROW4_LDS_BYTES, lds_ok);
    if (e != hipSuccess || a.prepare_only) return e;
    int first[ROW4_DIGITS];
    if (!row4_digits(pr, first) || st.first_factor != 0 || st.num_factors != pr.N || st.grid < 1 || st.grid > pr.M) return hipErrorInvalidValue;
    if (st.block != ROW4_THREADS || st.lds_bytes != ROW4_LDS_BYTES) return hipErrorInvalidValue;
    Row4Factors fa;
    for (int d = 0; d < ROW4_DIGITS; ++d) {
        fa.f[d] = (const float*)a.factors[first[d]];
        fa.g[d] = pr.P[first[d]] == 2 ? (const float*)a.factors[first[d] + 1] : nullptr;
    }
    hipLaunchKernelGGL(fused_row4_multiply, dim3((unsigned)st.grid), dim3(ROW4_THREADS), ROW4_LDS_BYTES, a.stream, (const float*)a.src,
                       (float*)a.dst, fa, pr.M);
    return hipGetLastError();
}

}  // namespace km
