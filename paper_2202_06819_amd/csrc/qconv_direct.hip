// Registry of the direct convolution kernels (qconv_direct.h); the instances
// are compiled in qconv_direct_b*.hip.
#include "qconv_internal.h"

namespace qconv {

extern DirectInstance g_direct_b4f2[], g_direct_b4f4[], g_direct_b8f2[], g_direct_b8f4[];
extern int g_direct_b4f2_count, g_direct_b4f4_count, g_direct_b8f2_count, g_direct_b8f4_count;

const DirectInstance *direct_instance(int bits, int fkb, int np, int fp, int ext, int la, int multi, int lin, int resident, int two_steps) {
    const DirectInstance *t = bits == 4 ? (fkb == 2 ? g_direct_b4f2 : g_direct_b4f4) : (fkb == 2 ? g_direct_b8f2 : g_direct_b8f4);
    const int n = bits == 4 ? (fkb == 2 ? g_direct_b4f2_count : g_direct_b4f4_count)
                            : (fkb == 2 ? g_direct_b8f2_count : g_direct_b8f4_count);
    for (int i = 0; i < n; ++i)
        if (t[i].bits == bits && t[i].fkb == fkb && t[i].np == np && t[i].fp == fp && t[i].ext == ext && t[i].la == la &&
            t[i].multi == multi && t[i].lin == lin && t[i].resident == resident &&
            t[i].two_steps == two_steps)
            return &t[i];
    return nullptr;
}

}  // namespace qconv
