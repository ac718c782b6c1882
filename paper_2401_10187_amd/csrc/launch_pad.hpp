// Launcher of the run-time-shape MFMA kernel with the factor in registers (declared in launch.hpp).
#pragma once
#include "launch.hpp"
#include "mfma_pad_kernel.hpp"

namespace km {

template <typename T, int QB, int KC, bool KEEP, bool WHOLE>
static hipError_t launch_pad_shape(const LaunchArgs& a)
{
    const km_plan_step& st = *a.st;
    const int f = st.first_factor, P = a.pr->P[f], Q = a.pr->Q[f];
    auto kern = mfma_pad_sliced_multiply<T, QB, KC, KEEP, WHOLE>;
    static unsigned char lds_ok[64];
    hipError_t e = allow_lds((const void*)kern, PAD_LDS_LIMIT, lds_ok);
    if (e != hipSuccess || a.prepare_only) return e;
    const int64_t S = st.k_in / P, slices = a.pr->M * S;
    const PadShape sh = pad_shape(P, Q, sizeof(T), slices);
    if (sh.threads == 0 || st.block != sh.threads || st.grid != sh.grid || st.lds_bytes != sh.lds_bytes || st.tile_slices != sh.tile_slices) return hipErrorInvalidValue;
    auto magic = [](int64_t d) { return (unsigned)(((1ull << 32) + (unsigned long long)d - 1) / (unsigned long long)d); };
    // (element numbers of a tile stay below 2^16, slice numbers below S + the tile's.  A row at least as long as a
    // tile is left at most once.)
    hipLaunchKernelGGL(kern, dim3((unsigned)st.grid), dim3((unsigned)st.block), (size_t)st.lds_bytes, a.stream,
                       (const T*)a.src, (const T*)a.factors[f], (T*)a.dst, S, P, Q, pad_stride(P, sizeof(T)), magic(P),
                       S >= sh.tile_slices || S == 1 ? 0u : magic(S), slices, (slices + sh.tile_slices - 1) / sh.tile_slices);
    return hipGetLastError();
}

template <typename T, int KC, int QB>
static hipError_t launch_pad_qb(const LaunchArgs& a)
{
    const int P = a.pr->P[a.st->first_factor];
    // (output runs that do not start on 64-byte boundaries: ordinary stores, as in launch_any.hpp)
    const bool keep = a.keep_output || (a.st->k_in / P) * (int64_t)sizeof(T) % 64 != 0;
    const bool whole = P % (16 / (int)sizeof(T)) == 0;
    hipError_t e = hipSuccess;
    for (int k = 0; k < 2 && e == hipSuccess; ++k) {
        if (!a.prepare_only && (k == 1) != keep) continue;               // preparing takes both store forms
        e = whole ? (k ? launch_pad_shape<T, QB, KC, true, true>(a) : launch_pad_shape<T, QB, KC, false, true>(a))
                  : (k ? launch_pad_shape<T, QB, KC, true, false>(a) : launch_pad_shape<T, QB, KC, false, false>(a));
    }
    return e;
}

template <typename T, int KC>
hipError_t launch_mfma_pad(const LaunchArgs& a)
{
    const km_plan_step& st = *a.st;
    const int P = a.pr->P[st.first_factor], Q = a.pr->Q[st.first_factor];
    if (st.num_factors != 1 || st.k_in % P || pad_chunks(P) != KC) return hipErrorInvalidValue;
    switch (pad_columns(Q)) {
        case 1: return launch_pad_qb<T, KC, 1>(a);
        case 2: return launch_pad_qb<T, KC, 2>(a);
        case 3: return launch_pad_qb<T, KC, 3>(a);
        case 4: return launch_pad_qb<T, KC, 4>(a);
        case 5: return launch_pad_qb<T, KC, 5>(a);
        case 6: return launch_pad_qb<T, KC, 6>(a);
        case 7: return launch_pad_qb<T, KC, 7>(a);
        case 8: return launch_pad_qb<T, KC, 8>(a);
    }
    return hipErrorInvalidValue;
}

}  // namespace km
