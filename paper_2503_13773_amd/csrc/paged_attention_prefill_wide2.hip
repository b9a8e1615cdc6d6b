#include "pa_prefill_wide.h"

namespace kvc {

template hipError_t launch_prefill_wide<2>(const void *, const void *, const void *, const int32_t *, const int32_t *, const int32_t *,
                                           void *, const PrefillParams &, hipStream_t);

}  // namespace kvc
