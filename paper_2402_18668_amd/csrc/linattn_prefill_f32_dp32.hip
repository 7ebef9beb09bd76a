// The fp32 prefill (linattn_prefill_f32.h) for d' = 32.
#include "linattn_prefill_f32.h"

namespace based {

namespace pf32 {
template hipError_t launch_dp<32>(const void *, const void *, const void *, void *, float *, int, void *, int, int, int, int,
                                  DecayArg, hipStream_t);
}

}  // namespace based
