// Patch unrolling for convolutions with very few input channels (the 3-channel
// 7x7 stride-2 stem of a ResNet): filter taps are folded into the channel
// axis, so the layer runs on the channel-packed kernels at a useful MMA depth.
//
//   dst[n][u][q][(b*taps_w + s)*C + c] =
//       src[n][c][u*stride_h + b - pad_h][q*stride_w + s - pad_w]
//
// for b < taps_h, s < taps_w (0 outside the input, and 0 for channels from
// taps_h*taps_w*C to c_out).  Folding every filter row turns the layer into a
// 1x1 convolution; folding groups of stride_h rows turns a strided R-row
// filter into a ceil(R/stride_h)-row one at stride 1.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qconv_internal.h"

namespace qconv {

namespace {

// One workgroup per output row (image, u).  The taps_h source rows of all C
// channels that the row reads are staged in LDS with their zero padding, and
// a table gives each output channel's LDS offset (-1 for a zero channel);
// the threads then assemble 16-byte output vectors from it, consecutive
// threads writing consecutive vectors of the row.  (Workgroups that loop over
// several rows were slower: every row's loads, barrier and stores form one
// latency chain, and one resident workgroup per row overlaps them best.)
__global__ void __launch_bounds__(256) unroll_patches(const int8_t *__restrict__ src, int8_t *__restrict__ dst,
                                                      UnrollArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    int32_t *table = reinterpret_cast<int32_t *>(smem);
    uint8_t *rows = smem + 4 * a.c_out;
    const int real = a.taps_h * a.taps_w * a.c;
    for (int ch = threadIdx.x; ch < a.c_out; ch += 256) {
        int off = -1;
        if (ch < real) {
            const int tap = ch / a.c, ci = ch - tap * a.c;
            const int b = tap / a.taps_w, s = tap - b * a.taps_w;
            off = (ci * a.taps_h + b) * a.lw + s;
        }
        table[ch] = off;
    }
    const int nrb = a.c * a.taps_h;
    const int vpp = a.c_out / 16;
    const unsigned row = (unsigned)a.first + blockIdx.x;
    const int u = (int)(row % (unsigned)a.out_h);
    const int img = (int)(row / (unsigned)a.out_h);
    // staged row rb = ci * taps_h + b holds source row u*stride_h + b - pad_h
    // of channel ci; each thread takes one column of up to 8 rows at a time,
    // so that their loads are in flight together
    for (int x = threadIdx.x; x < a.lw; x += 256) {
        const int col = x - a.pad_w;
        const bool col_ok = col >= 0 && col < a.w;
        for (int rb0 = 0; rb0 < nrb; rb0 += 8) {
            uint8_t vals[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int rb = rb0 + e;
                const int ci = rb / a.taps_h, b = rb - ci * a.taps_h;
                const int y = u * a.stride_h + b - a.pad_h;
                vals[e] = 0;
                if (rb < nrb && col_ok && y >= 0 && y < a.h)
                    vals[e] = (uint8_t)src[(((int64_t)img * a.c + ci) * a.h + y) * a.w + col];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (rb0 + e < nrb) rows[(rb0 + e) * a.lw + x] = vals[e];
        }
    }
    __syncthreads();
    int8_t *out = dst + ((int64_t)img * a.out_h + u) * a.wout * a.c_out;
    for (int v = threadIdx.x; v < a.wout * vpp; v += 256) {
        const int q = v / vpp, j = v - q * vpp;
        const int base = q * a.stride_w;
        const int4 *t4 = reinterpret_cast<const int4 *>(table + 16 * j);
        uint32_t words[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int4 o = t4[g];
            const int oo[4] = {o.x, o.y, o.z, o.w};
            uint32_t word = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (oo[e] >= 0) word |= (uint32_t)rows[oo[e] + base] << (8 * e);
            words[g] = word;
        }
        *reinterpret_cast<uint4 *>(out + (int64_t)v * 16) = uint4{words[0], words[1], words[2], words[3]};
    }
}

// The same for runs of at least 16 bytes (taps_w * C: the bytes of one output
// pixel that come from one source row, contiguous if the staged rows hold their
// columns' channels side by side).  An output vector is then a 16-byte window of
// one staged row, or its first bytes one window and the rest another, and a
// window is five aligned words shifted together: 10 LDS reads and about 30
// instructions a vector against 20 and 90 when its bytes are gathered one by
// one.  A thread's vectors all have the same place in their pixel, so where the
// windows start is worked out once, and the rows are counted on: with run-time
// divisions both kernels spent longer on those.  N=16 224x224x3 folded into 115
// rows of 64 channels: 9.4 us against 11.4 by single bytes; what is left is one
// round of loads, a barrier and one round of stores a workgroup.
__global__ void __launch_bounds__(256) unroll_runs(const int8_t *__restrict__ src, int8_t *__restrict__ dst,
                                                   UnrollArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int c = a.c;
    const int run = a.taps_w * c;
    const int row_bytes = (a.lw * c + 3) & ~3;
    const uint32_t row = (uint32_t)a.first + blockIdx.x;
    const int img = (int)fdiv(row, a.div_out_h);
    const int u = (int)row - img * a.out_h;
    const int nrb = c * a.taps_h;
    uint8_t *rows = smem + 16;   // (a window may start up to 15 bytes before its row)
    const int8_t *image = src + (int64_t)img * c * a.h * a.w;
    const int y0 = u * a.stride_h - a.pad_h;
    for (int x = threadIdx.x; x < a.lw; x += 256) {
        const int col = x - a.pad_w;
        const bool col_ok = col >= 0 && col < a.w;
        // (row, channel) pairs, counted on rather than divided out
        int b = 0, ci = 0;
        for (int rb0 = 0; rb0 < nrb; rb0 += 8) {
            uint8_t vals[8];
            int lb = b, lc = ci;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int y = y0 + lb;
                vals[e] = 0;
                if (rb0 + e < nrb && col_ok && y >= 0 && y < a.h)
                    vals[e] = (uint8_t)image[((int64_t)lc * a.h + y) * a.w + col];
                if (++lc == c) {
                    lc = 0;
                    ++lb;
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (rb0 + e < nrb) rows[b * row_bytes + x * c + ci] = vals[e];
                if (++ci == c) {
                    ci = 0;
                    ++b;
                }
            }
        }
    }
    // this thread's place in a pixel: vector j, its first window's start, the
    // second's (moved back by the bytes the first gives), and masks of the bytes
    // each gives
    const int vpp = a.c_out / 16;
    const int per = a.pixels_per_round;   // 256 / vpp (vpp divides 256)
    const int q0 = (int)fdiv(threadIdx.x, a.div_vpp), j = (int)threadIdx.x - q0 * vpp;
    const int b0 = (int)fdiv((uint32_t)(16 * j), a.div_run), o = 16 * j - b0 * run, first = min(16, run - o);
    const int real = a.taps_h * run;
    int start[2];
    uint32_t give[2][4];
    start[0] = b0 < a.taps_h ? b0 * row_bytes + o : 0;
    start[1] = first < 16 && b0 + 1 < a.taps_h ? (b0 + 1) * row_bytes - first : 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        give[0][w] = give[1][w] = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 4 * w + e;
            if (16 * j + k < real) give[k < first ? 0 : 1][w] |= 0xFFu << (8 * e);
        }
    }
    __syncthreads();
    int8_t *out = dst + ((int64_t)img * a.out_h + u) * a.wout * a.c_out;
    const int step = a.stride_w * c;
    for (int q = q0; q < a.wout; q += per) {
        uint32_t word[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const int at = 16 + start[n] + q * step;
            const uint32_t *p = reinterpret_cast<const uint32_t *>(smem + (at & ~3));
            uint32_t v[5];
#pragma unroll
            for (int i = 0; i < 5; ++i) v[i] = p[i];
#pragma unroll
            for (int w = 0; w < 4; ++w)
                word[w] |= __builtin_amdgcn_alignbyte(v[w + 1], v[w], (uint32_t)at & 3u) & give[n][w];
        }
        *reinterpret_cast<uint4 *>(out + ((int64_t)q * vpp + j) * 16) = uint4{word[0], word[1], word[2], word[3]};
    }
}

// Runs long enough for unroll_runs, whose threads keep one vector of a pixel,
// and its staged rows (with the bytes its windows may read around them) in LDS.
int64_t unroll_runs_lds(const UnrollArgs &a) {
    return 16 + (int64_t)a.taps_h * ((a.lw * (int64_t)a.c + 3) & ~int64_t(3)) + 20;
}
bool use_unroll_runs(const UnrollArgs &a) {
    return a.taps_w * a.c >= 16 && 256 % (a.c_out / 16) == 0 && unroll_runs_lds(a) <= 64 * 1024;
}

}  // namespace

int64_t unroll_lds_bytes(const UnrollArgs &a) { return 4ll * a.c_out + (int64_t)a.c * a.taps_h * a.lw; }

hipError_t launch_unroll(const int8_t *src, int8_t *dst, const UnrollArgs &a, hipStream_t stream) {
    const int64_t blocks = (int64_t)a.n * a.out_h;
    if (blocks == 0 || a.wout == 0) return hipSuccess;
    const bool runs = use_unroll_runs(a);
    UnrollArgs r = a;
    if (runs) {
        r.div_out_h = make_fastdiv((uint32_t)a.out_h);
        r.div_vpp = make_fastdiv((uint32_t)(a.c_out / 16));
        r.div_run = make_fastdiv((uint32_t)(a.taps_w * a.c));
        r.pixels_per_round = 256 / (a.c_out / 16);
    }
    const size_t lds = (size_t)(runs ? unroll_runs_lds(a) : unroll_lds_bytes(a));
    launch_slices(blocks, 256, [&](long long first, unsigned count) {
        r.first = (int32_t)first;
        if (runs)
            hipLaunchKernelGGL(unroll_runs, dim3(count), dim3(256), lds, stream, src, dst, r);
        else
            hipLaunchKernelGGL(unroll_patches, dim3(count), dim3(256), lds, stream, src, dst, r);
    });
    return hipGetLastError();
}

}  // namespace qconv
