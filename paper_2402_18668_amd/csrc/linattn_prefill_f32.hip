// The fp32 prefill (linattn_prefill_f32.h) for d' = 8, 16, 24, and its host side; d' = 32 is built in a file of its own (it
// takes as long to compile as these together).
#include "linattn_prefill_f32.h"

namespace based {

namespace pf32 {
extern template hipError_t launch_dp<32>(const void *, const void *, const void *, void *, float *, int, void *, int, int,
                                         int, int, DecayArg, hipStream_t);
}

size_t prefill_f32_workspace_bytes(int U, int N, int dp, int dv)
{
    const int G = pf32::segments(U, N, dp, dv);
    return G > 1 ? (size_t)U * (dv / pf32::COLS) * G * pf32::entry_floats(dp) * sizeof(float) : 0;
}

hipError_t launch_prefill_f32(const void *q, const void *k, const void *v, void *y, float *state, int has_init,
                              void *workspace, const float *gamma, const void *gate, int H, int U, int N, int dp, int dv,
                              int dtype, hipStream_t s)
{
    if (prefill_f32x3_supported(dp, dtype, N))
        return launch_prefill_f32x3(q, k, v, y, state, has_init, workspace, gamma, gate, H, U, N, dv, s);
    const pf32::DecayArg dec{gamma, gate, H};
    switch (dp) {
    case 8: return pf32::launch_dp<8>(q, k, v, y, state, has_init, workspace, U, N, dv, dtype, dec, s);
    case 16: return pf32::launch_dp<16>(q, k, v, y, state, has_init, workspace, U, N, dv, dtype, dec, s);
    case 24: return pf32::launch_dp<24>(q, k, v, y, state, has_init, workspace, U, N, dv, dtype, dec, s);
    case 32: return pf32::launch_dp<32>(q, k, v, y, state, has_init, workspace, U, N, dv, dtype, dec, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace based
