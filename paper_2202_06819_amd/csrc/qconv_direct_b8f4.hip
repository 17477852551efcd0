// Direct convolution kernels (qconv_direct.h) for 8-bit operands and filter
// images of 4-fragment channel blocks, in a translation unit of their own.
#include "qconv_direct.h"

namespace qconv {

DirectInstance g_direct_b8f4[] = {QCONV_DIRECT_SET(8, 4)};
int g_direct_b8f4_count = (int)(sizeof(g_direct_b8f4) / sizeof(g_direct_b8f4[0]));

}  // namespace qconv
