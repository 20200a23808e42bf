// Blocked convolution on fp16 MFMA with two-term operands (conv_h2.h): the
// kernels over a converted filter, for every other pair of input and output blocks.
#include "conv_h2.h"

namespace neo {
namespace conv_detail {

template hipError_t dispatch_h2<true, true>(const ConvConfig&, int, bool, const H2Args&, hipStream_t);

}  // namespace conv_detail
}  // namespace neo
