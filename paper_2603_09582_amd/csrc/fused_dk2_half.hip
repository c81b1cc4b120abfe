// Instantiation of the fused kernel for ceil(d / 32) = 2 where d ends in the first half of the last 32
// channels.
#include "fused_impl.h"

namespace binattn {
template int launch_fused_dk<2, FORM_HALF>(const FusedParams &, int, hipStream_t);
template int launch_onehead_dk<2, FORM_HALF>(const FusedParams &, int, hipStream_t);
}
