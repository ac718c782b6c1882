// The MFMA kernels that leave digits in place (fp32), with their launchers.
#include "launch.hpp"
#include "mfma_inplace_kernel.hpp"

namespace km {

template <int P, bool KEEP>
static hipError_t launch_chain_shape(const LaunchArgs& a)
{
    const km_plan_step& st = *a.st;
    auto kern = mfma_chain_multiply<P, KEEP>;
    static unsigned char lds_ok[64];
    hipError_t e = allow_lds((const void*)kern, ChainShape<P>::LDS_BYTES, lds_ok);
    if (e != hipSuccess || a.prepare_only) return e;
    const float* f0 = (const float*)a.factors[st.first_factor + 1];    // applied first
    const float* f1 = (const float*)a.factors[st.first_factor];
    const int64_t count = a.pr->M * (st.k_in / (P * P));
    if (st.k_in % (P * P) || st.k_out != st.k_in || st.block != CHAIN_THREADS || st.lds_bytes != ChainShape<P>::LDS_BYTES || st.grid < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)st.grid), dim3(CHAIN_THREADS), ChainShape<P>::LDS_BYTES, a.stream, (const float*)a.src,
                       (float*)a.dst, f0, f1, count);
    return hipGetLastError();
}

template <int P>
struct ChainLauncher {
    template <bool KEEP> static hipError_t run(const LaunchArgs& a) { return launch_chain_shape<P, KEEP>(a); }
};

hipError_t launch_chain(const LaunchArgs& a)
{
    const Problem& pr = *a.pr;
    const int f = a.st->first_factor, P = pr.P[f];
    if (pr.dtype != KM_F32 || a.st->num_factors != 2 || f + 2 != pr.N) return hipErrorInvalidValue;
    if (pr.Q[f] != P || pr.P[f + 1] != P || pr.Q[f + 1] != P) return hipErrorInvalidValue;
    if (P == 48) return launch_either<ChainLauncher<48>>(a);
    if (P == 64) return launch_either<ChainLauncher<64>>(a);
    return hipErrorInvalidValue;
}

template <int MB>
struct DigitLauncher {
template <bool KEEP>
static hipError_t run(const LaunchArgs& a)
{
    const km_plan_step& st = *a.st;
    const Problem& pr = *a.pr;
    const int f = st.first_factor, P = pr.P[f], Q = pr.Q[f];
    auto kern = mfma_digit_multiply<MB, KEEP>;
    static unsigned char lds_ok[64];
    hipError_t e = allow_lds((const void*)kern, 128 * 16 * MB * (int)sizeof(float), lds_ok);
    if (e != hipSuccess || a.prepare_only) return e;
    int64_t R = 1;                                       // elements behind the digit: all of them contracted already
    for (int k = f + 1; k < pr.N; ++k) R *= pr.Q[k];
    if (P % 16 || P > 128 || Q != 16 * MB || R % 64 || st.k_in % (P * R) || st.k_out != st.k_in / P * Q) return hipErrorInvalidValue;
    if (st.grid < 1 || st.block != DIGIT_THREADS || st.lds_bytes != P * Q * (int)sizeof(float)) return hipErrorInvalidValue;
    const int64_t runs = pr.M * (st.k_in / P) / 64, on = st.grid * (DIGIT_THREADS / 64) * 64;
    hipLaunchKernelGGL(kern, dim3((unsigned)st.grid), dim3(DIGIT_THREADS), (size_t)st.lds_bytes, a.stream, (const float*)a.src,
                       (float*)a.dst, (const float*)a.factors[f], P, Q, R, runs, DigitStep{on / R, on % R});
    return hipGetLastError();
}
};

hipError_t launch_digit(const LaunchArgs& a)
{
    if (a.pr->dtype != KM_F32 || a.st->num_factors != 1) return hipErrorInvalidValue;
    switch (a.pr->Q[a.st->first_factor] / 16) {
        case 1: return launch_either<DigitLauncher<1>>(a);
        case 2: return launch_either<DigitLauncher<2>>(a);
        case 3: return launch_either<DigitLauncher<3>>(a);
        case 4: return launch_either<DigitLauncher<4>>(a);
        case 5: return launch_either<DigitLauncher<5>>(a);
        case 6: return launch_either<DigitLauncher<6>>(a);
        case 7: return launch_either<DigitLauncher<7>>(a);
        case 8: return launch_either<DigitLauncher<8>>(a);
    }
    return hipErrorInvalidValue;
}

}  // namespace km
