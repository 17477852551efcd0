// Direct convolution kernels (qconv_direct.h) for 4-bit operands and filter
// images of 4-fragment channel blocks, in a translation unit of their own.
#include "qconv_direct.h"

namespace qconv {

DirectInstance g_direct_b4f4[] = {QCONV_DIRECT_SET(4, 4) QCONV_DIRECT_SET16(4)};
int g_direct_b4f4_count = (int)(sizeof(g_direct_b4f4) / sizeof(g_direct_b4f4[0]));

}  // namespace qconv
