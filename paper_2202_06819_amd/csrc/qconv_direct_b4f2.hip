// Direct convolution kernels (qconv_direct.h) for 4-bit operands and filter
// images of 2-fragment channel blocks, in a translation unit of their own.
#include "qconv_direct.h"

namespace qconv {

DirectInstance g_direct_b4f2[] = {QCONV_DIRECT_SET(4, 2) QCONV_DIRECT_SET16(2)};
int g_direct_b4f2_count = (int)(sizeof(g_direct_b4f2) / sizeof(g_direct_b4f2[0]));

}  // namespace qconv
