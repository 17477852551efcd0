// Relayout-and-pack for gfx950: int8 N x C x H x W  ->  channel-packed
// N x H x W x C (Sec. 1: eight 4-bit values per 32-bit word along the channel
// axis; Sec. 3.3: channels innermost so consumers read it coalesced).
//
// The operation is a transpose of each image's C x (H*W) plane.  A workgroup
// owns a tile of PK_C channels x 64 pixels, with two threads per channel.  It
// reads the tile row by row (each channel's pixels are contiguous in NCHW: 32
// bytes per lane, two lanes per 64-byte row segment), saturates every value into
// the target range and parks it in LDS; it then reads 8 channels x 4 pixels per
// lane as dwords, transposes the bytes in registers, packs nibbles and writes
// each pixel's words.  The LDS row pitch is 17 dwords: the dwords a wave of a
// 64-channel tile reads at once (8 channel groups 136 dwords apart, 8 pixel
// quads) lie in 64 banks, those of a 128-channel tile (16 groups, 4 quads) in 32,
// two to a bank.
//
// The kernel is HBM-bound: every input byte is read once and every output byte
// written once.  PK_C is 64, except where 128 pays: the channels fill whole pairs of
// 64-channel tiles, so that no more rows are staged, and 2048 workgroups or more
// are left.  A pixel's packed words are then written in 64-byte runs (4-bit)
// instead of 32-byte ones: 41x256x108x108 32.8 against 37.6 us, 41x128x108x108
// 17.1 against 18.2, 64x2048x28x28 27.2 against 27.4.  With a half-empty tile it
// costs more than it gives (41x160x108x108 27.0 against 23.9, 41x192x108x108 28.4
// against 26.6), and on small tensors the larger workgroups take up to 0.2 us
// longer (16x192x1x1 2.9 against 2.8, 16x96x56x56 4.1 against 3.9).
//
// Rows of 11 pixels or more are read with 16-byte loads, unaligned where the row is:
// 41x256x108x109 33 us, with byte loads 199.  Shorter ones (filters, 1x1 images)
// are read byte by byte, which moves less: 1024x2048x1x1 24.0 against 29.2 us,
// 1024x256x3x3 6.2 against 6.5; at 12 pixels it is 6.8 against 6.3.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qconv_internal.h"

namespace qconv {

constexpr int PK_P = 64;          // pixels per tile (64-byte segments of each channel row)
constexpr int PK_PITCH = 68;      // LDS row pitch in bytes
constexpr int PK_SHORT = 11;      // rows below so many pixels are read by bytes

// Same renumbering as the convolution kernels: block b runs on XCD b % 8;
// give every XCD a contiguous range so neighbouring pixel tiles (which share
// cache lines at row ends) meet in one L2.
__device__ __forceinline__ int pack_xcd_block(int b, int g) {
    const int x = b % 8, i = b / 8, q = g / 8, r = g % 8;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + i;
}

__device__ __forceinline__ uint32_t byte_of(uint32_t v, int j) { return (v >> (8 * j)) & 0xFFu; }

// 4x4 byte transpose: byte k of result j is byte j of t[k].
__device__ __forceinline__ uint32_t gather_byte(const uint32_t (&t)[4], int j) {
    return byte_of(t[0], j) | (byte_of(t[1], j) << 8) | (byte_of(t[2], j) << 16) | (byte_of(t[3], j) << 24);
}

// (ptiles, ctiles, nb: the divisors of the block and image decompositions)
// PK_C: channels per tile, 2 PK_C threads (phase 2: PK_C / 8 channel groups x 16
// pixel quads).  This launch's workgroups are those from `first` on of `blocks`.
template <int BITS, bool SIGNED, int PK_C>
__global__ void __launch_bounds__(2 * PK_C)
    pack_nchw(const int8_t *__restrict__ src, const int8_t *end, uint8_t *__restrict__ dst, int c, int hw,
              FastDiv ptiles, FastDiv ctiles, FastDiv nb, int first, int blocks) {
    constexpr int LO = SIGNED ? -(1 << (BITS - 1)) : 0;
    constexpr int HI = SIGNED ? (1 << (BITS - 1)) - 1 : (1 << BITS) - 1;
    __shared__ __attribute__((aligned(16))) uint8_t tile[PK_C * PK_PITCH];
    const int tid = threadIdx.x;
    int bid = pack_xcd_block(first + (int)blockIdx.x, blocks);
    const int rest = (int)fdiv((uint32_t)bid, ptiles);
    const int pt = bid - rest * (int)ptiles.d;
    const int img = (int)fdiv((uint32_t)rest, ctiles);
    const int ct = rest - img * (int)ctiles.d;
    const int c0 = ct * PK_C;
    const int p0 = pt * PK_P;
    const int8_t *plane = src + (size_t)img * c * hw;
    // destination pixel of (img, pix): nb images interleaved per pixel
    // (nb = 1: plain N x H x W x C)
    const int ig = (int)fdiv((uint32_t)img, nb);
    const size_t obase = (size_t)ig * hw * nb.d + (img - ig * (int)nb.d);
    auto out_pixel = [&](int px) { return obase + (size_t)px * nb.d; };

    // ---- phase 1: PK_C channel rows x 64 pixels; a lane reads 32 consecutive
    // pixels of one row, saturates them and parks them in LDS
    {
        const int row = tid >> 1;
        const int seg = (tid & 1) * 32;
        const int ch = c0 + row;
        uint32_t v[8];
        const int8_t *rp = plane + (size_t)ch * hw + p0 + seg;
        if (ch < c && hw >= PK_SHORT && p0 + seg < hw && rp + 32 <= end) {
            // (rows of any length: the loads are unaligned where the row is, and
            // those past a row's end read the next row, whose pixels are not stored)
            uint4 a, b;
            __builtin_memcpy(&a, rp, 16);
            __builtin_memcpy(&b, rp + 16, 16);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
            v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        } else {
            // short rows, and the tensor's last bytes
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint32_t w = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int px = p0 + seg + 4 * e + k;
                    if (ch < c && px < hw) w |= (uint32_t)(uint8_t)rp[4 * e + k] << (8 * k);
                }
                v[e] = w;
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            uint32_t w = v[e];
            if constexpr (BITS == 4) {
                // byte-parallel range test (for signed values on v + 8, added per
                // byte without carries); only words with a byte out of range
                // take the per-byte clamp
                const uint32_t t = SIGNED ? (((w & 0x7F7F7F7Fu) + 0x08080808u) ^ (w & 0x80808080u)) : w;
                if ((t & 0xF0F0F0F0u) != 0u) {
                    uint32_t o = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int x = (int)(int8_t)byte_of(w, k);
                        o |= ((uint32_t)(x < LO ? LO : (x > HI ? HI : x)) & 0xFFu) << (8 * k);
                    }
                    w = o;
                }
            }
            *reinterpret_cast<uint32_t *>(tile + row * PK_PITCH + seg + 4 * e) = w;
        }
    }
    __syncthreads();

    // ---- phase 2: a lane takes 8 channels (group g) x 4 pixels (quad q):
    // 8 dword reads, an in-register transpose, and one output word (4-bit) or
    // two (8-bit) per pixel
    const int g = tid % (PK_C / 8);
    const int q = tid / (PK_C / 8);
    const int cg = c0 + 8 * g;
    if (cg >= c) return;
    uint32_t d[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) d[i] = *reinterpret_cast<const uint32_t *>(tile + (8 * g + i) * PK_PITCH + 4 * q);
    if constexpr (BITS == 4) {
        // byte j of t[k]: channel 8g+2k in the low nibble, 8g+2k+1 in the high one, of pixel j
        uint32_t t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = (d[2 * k] & 0x0F0F0F0Fu) | ((d[2 * k + 1] << 4) & 0xF0F0F0F0u);
        uint32_t *out = reinterpret_cast<uint32_t *>(dst);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int pix = p0 + 4 * q + j;
            if (pix < hw) out[out_pixel(pix) * (c / 8) + cg / 8] = gather_byte(t, j);
        }
    } else {
        const uint32_t lo4[4] = {d[0], d[1], d[2], d[3]};
        const uint32_t hi4[4] = {d[4], d[5], d[6], d[7]};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int pix = p0 + 4 * q + j;
            if (pix >= hw) continue;
            uint32_t *out = reinterpret_cast<uint32_t *>(dst + out_pixel(pix) * c + cg);   // c % 4 == 0
            out[0] = gather_byte(lo4, j);
            if (cg + 4 < c) out[1] = gather_byte(hi4, j);
        }
    }
}

hipError_t launch_pack(const int8_t *src, void *dst, int32_t n, int32_t c, int32_t h, int32_t w, int32_t bits,
                       int32_t is_signed, int32_t nb, hipStream_t stream) {
    const int hw = h * w;
    const int ptiles = (hw + PK_P - 1) / PK_P;
    const int c64 = (c + 63) / 64;
    const bool wide = c64 % 2 == 0 && (long long)n * ptiles * (c64 / 2) >= 2048;   // (see the top)
    const int pkc = wide ? 128 : 64;
    const int ctiles = (c + pkc - 1) / pkc;
    const long long blocks = (long long)n * ptiles * ctiles;
    uint8_t *d = static_cast<uint8_t *>(dst);
    const int8_t *end = src + (size_t)n * c * hw;
    const dim3 block(2 * pkc);
    const FastDiv dp = make_fastdiv((uint32_t)ptiles), dc = make_fastdiv((uint32_t)ctiles),
                  dn = make_fastdiv((uint32_t)(nb > 0 ? nb : 1));
    auto go = [&](auto kernel) {
        launch_slices(blocks, 2 * pkc, [&](long long first, unsigned count) {
            hipLaunchKernelGGL(kernel, dim3(count), block, 0, stream, src, end, d, c, hw, dp, dc, dn, (int)first,
                               (int)blocks);
        });
    };
    if (pkc == 128) {
        if (bits == 4 && is_signed)
            go(pack_nchw<4, true, 128>);
        else if (bits == 4)
            go(pack_nchw<4, false, 128>);
        else
            go(pack_nchw<8, true, 128>);
    } else {
        if (bits == 4 && is_signed)
            go(pack_nchw<4, true, 64>);
        else if (bits == 4)
            go(pack_nchw<4, false, 64>);
        else
            go(pack_nchw<8, true, 64>);
    }
    return hipGetLastError();
}

}  // namespace qconv
