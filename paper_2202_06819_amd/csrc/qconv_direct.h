// Convolution straight from global memory: no input band in LDS.
//
// The wide kernels stage a tile's input band in LDS, widen it there and meet
// at a barrier for every stage.  Here a wave owns an output tile (16 FP pixels
// x 32 NP channels) by itself: per step (one filter tap x 64 channels) every
// lane loads the 16 channels of its pixel that its MFMA operand needs -- 8
// packed bytes for 4 bits, 16 for 8 -- from global memory, where the other taps
// of a window hit the CU's L1, and widens them in registers.  Padding is an
// out-of-range buffer offset.  The filters come from the prepared image of
// whichever wide tile the caller chose.
//   DEPTH (WRES = false): filters are read from the image step by step; `wd`
//     waves of a workgroup share one output tile, each over a range of the
//     steps, and meet once to add their sums through LDS.  For layers with few
//     output tiles: a wide workgroup walks its channel chunks one after the
//     other with a memory latency in each, here all of a wave's loads (LA
//     steps) are in flight at once.
//   RESIDENT (WRES = true): the channel tile's whole filter block is copied to
//     LDS once, and a workgroup's waves walk pixel tiles on their own, with no
//     barrier: one wave's loads and epilogue run under the others' MFMAs.  For
//     1x1 layers, whose stages in the wide kernels are mostly waits.
#pragma once

#include "qconv_kernels.h"

namespace qconv {

// ---- the requantiser in f32.  t = floor((A*mult + 2^(shift-1)) / 2^shift) of an
// accumulator acc = A * 2^acc_shift is floor(x) with x = acc*m + 0.5 and m =
// mult * 2^(-shift-acc_shift).  With rounding toward minus infinity one fma
// gives x rounded down, whose floor is floor(x): integers are representable
// below 2^24, and past that the clamp decides alone.  It needs acc and mult
// within 2^24 (both then exact in f32).  v_cvt_pk_u8_f32 floors (in that
// rounding mode), saturates to [0, 255] and packs in one instruction; a scale
// 2^s and an offset put the ends of the clamp range on those of the byte.  That
// is 3 instructions a value (a conversion, an fma, a packing conversion)
// against v_mad_i64_i32 (two issue slots), v_med3 and a shift-or.
struct DirectEpilogue {   // what the epilogue helpers read, of one job
    int32_t mode, acc_shift, shift, lo, hi, res_signed, k, m;
    const uint8_t *res;
    uint8_t *yptr;
};

// f32 results of this wave round toward minus infinity from here on.  The
// requantiser's have to be its only ones: no division by a run-time value, which
// the compiler works out through f32 reciprocals and conversions.
__device__ __forceinline__ void round_down_f32() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 2" : : : "memory");
#endif
}

// |v| <= room (room < 2^31), for every v: the sum is formed in unsigned, where it
// may wrap.
__host__ __device__ constexpr bool within(int32_t v, uint32_t room) { return (uint32_t)v + room <= 2u * room; }
static_assert(within(1 << 24, 1u << 24) && within(-(1 << 24), 1u << 24) && !within((1 << 24) + 1, 1u << 24) &&
              !within(-(1 << 24) - 1, 1u << 24) && !within(INT32_MAX, 1u << 24) && !within(INT32_MIN, 1u << 24) &&
              within(0, 0u) && !within(1, 0u) && !within(-1, 0u));

// Byte N of w = floor(x) saturated to [0, 255] (N = 0 starts a word).
template <int N>
__device__ __forceinline__ uint32_t pack_u8(float x, uint32_t w) {
    uint32_t r;
    if constexpr (N == 0)
        asm("v_cvt_pk_u8_f32 %0, %1, 0, 0" : "=v"(r) : "v"(x));
    else
        asm("v_cvt_pk_u8_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "n"(N), "v"(w));
    return r;
}

// Byte N of w as a float.
template <int N>
__device__ __forceinline__ float byte_f32(uint32_t w) {
    return (float)((w >> (8 * N)) & 0xFFu);
}

// The f32 form over FP fragments of a run of 4*FK channels.  4 bits: bytes hold
// 16 times the value, so a byte's saturation is the clamp and its high nibble
// the result; even and odd channels gather in two words.  8 bits: bytes hold
// the value plus 128, or twice the value for a clamp of [0, 127].  A residual
// joins in the fma's addend.
template <int BITS, int FP, int FK, bool RES>
__device__ __forceinline__ void epilogue_f32(const DirectEpilogue &a, const FloatEpilogue &fe, v4i (&acc)[FP][FK],
                                             int mbase, int cb, int l16, const float (&mul)[4 * FK],
                                             const uint32_t (&rw)[FP][4 * FK * BITS / 32]) {
    constexpr int CPW = 32 / BITS;
    constexpr int NWD = 4 * FK / CPW;
    const float c0 = fe.addend;
#pragma unroll
    for (int tn = 0; tn < FP; ++tn) {
        uint32_t words[NWD];
        auto value = [&](int e, float add) { return __builtin_fmaf((float)acc[tn][e / 4][e % 4], mul[e], add); };
#pragma unroll
        for (int wd = 0; wd < NWD; ++wd) {
            if constexpr (BITS == 4) {
                float av[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) av[i] = c0;
                if constexpr (RES) {
                    // 16 r + 8 (16 (r + 8) + 8 for signed values), in bytes
                    const uint32_t even = ((rw[tn][wd] << 4) & 0xF0F0F0F0u) ^ fe.res_xor;
                    const uint32_t odd = (rw[tn][wd] & 0xF0F0F0F0u) ^ fe.res_xor;
                    av[0] = byte_f32<0>(even); av[2] = byte_f32<1>(even); av[4] = byte_f32<2>(even); av[6] = byte_f32<3>(even);
                    av[1] = byte_f32<0>(odd); av[3] = byte_f32<1>(odd); av[5] = byte_f32<2>(odd); av[7] = byte_f32<3>(odd);
                }
                uint32_t ev = pack_u8<0>(value(8 * wd + 0, av[0]), 0u), od = pack_u8<0>(value(8 * wd + 1, av[1]), 0u);
                ev = pack_u8<1>(value(8 * wd + 2, av[2]), ev);
                od = pack_u8<1>(value(8 * wd + 3, av[3]), od);
                ev = pack_u8<2>(value(8 * wd + 4, av[4]), ev);
                od = pack_u8<2>(value(8 * wd + 5, av[5]), od);
                ev = pack_u8<3>(value(8 * wd + 6, av[6]), ev);
                od = pack_u8<3>(value(8 * wd + 7, av[7]), od);
                words[wd] = (((ev >> 4) & 0x0F0F0F0Fu) | (od & 0xF0F0F0F0u)) ^ fe.out_xor;
            } else {
                float av[4] = {c0, c0, c0, c0};
                if constexpr (RES) {
                    const uint32_t r = rw[tn][wd] ^ fe.res_xor;
                    av[0] = __builtin_fmaf(byte_f32<0>(r), fe.res_scale, c0);
                    av[1] = __builtin_fmaf(byte_f32<1>(r), fe.res_scale, c0);
                    av[2] = __builtin_fmaf(byte_f32<2>(r), fe.res_scale, c0);
                    av[3] = __builtin_fmaf(byte_f32<3>(r), fe.res_scale, c0);
                }
                uint32_t w = pack_u8<0>(value(4 * wd + 0, av[0]), 0u);
                w = pack_u8<1>(value(4 * wd + 1, av[1]), w);
                w = pack_u8<2>(value(4 * wd + 2, av[2]), w);
                w = pack_u8<3>(value(4 * wd + 3, av[3]), w);
                words[wd] = ((w >> fe.out_shift) & fe.out_mask) ^ fe.out_xor;
            }
        }
        const int m = mbase + tn * 16 + l16;
        if (m < a.m) store_run<BITS, FK>(a, m, cb, words);
    }
}

// FKB: fragments per channel block of the image (the tile's frag_k).  LA: steps
// in flight; MULTI: a wave has more than LA steps (at least two rounds of LA).
// LIN: a 1x1 filter at stride 1 without padding.  B16 (4 bits): steps come in
// pairs, 128 channels, and a lane loads the 16 bytes of both at once, 32
// consecutive channels (its granules are 2 gq and 2 gq + 1); for channels in whole
// 128s.  The loads, not the arithmetic, bound these kernels: 1x1 256->64 at 56x56
// N=64 takes 9.2 us with them and 12.1 with 8-byte loads, 2048->512 at 7x7 9.6 and
// 12.6.  3x3 filters keep one step a load: with two, 28x28 128->128 N=64 went from
// 14.3 to 14.7 us and 14x14 256->256 from 21.2 to 18.0, where the wide kernels
// take 13.3 and 11.9.
// Spilled registers: multipliers, biases, start sums, two rounds of loads and the
// residual's words are live together in 256 VGPRs (two waves a SIMD).  Of the 184
// instances eight spill, all resident 1x1 from images of 4-fragment blocks with
// NP 2: with the bias and residual epilogue FP 4 by 13-21 registers (4 bits) and
// 39-63 (8 bits) and FP 2 of LA 4 in one round by 6 (4 bits); without it FP 2 of
// LA 4 in several rounds by 3 (8 bits).  direct_margin asks more of the first.
template <int BITS, int FKB, int NP, int FP, bool EXT, int LA, bool MULTI, bool LIN, bool WRES, bool B16 = false>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) conv_direct(DirectArgs a) {
    constexpr int NF = 2 * NP;                       // MFMA rows of 16 channels per wave
    constexpr bool WHOLE = FKB == 4 && NP == 2;      // the wave's channels are one image block
    constexpr int FE = WHOLE ? 4 : 2;                // fragments of a run of consecutive channels per lane
    constexpr int NBK = NF / FE;
    constexpr int CB = 64 * BITS / 8;                // bytes of a step's channels of one pixel
    constexpr int AS = WRES && LA % 2 == 0 ? 2 : LA; // filter fragment sets
    static_assert(!B16 || (BITS == 4 && LIN && WRES && LA % 2 == 0), "two steps a load: 4-bit resident 1x1");
    constexpr int US = B16 ? 2 : 1;                  // steps of a load
    constexpr int LB = LA / US;                      // loads in flight of a fragment
    using Raw = std::conditional_t<BITS == 4 && !B16, u32x2, u32x4>;

    round_down_f32();
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15;
    const int gq = lane >> 4;

    // ---- this wave's tile: pixel tile mt, channel tile kb, part wd_i of the depth
    const int ji = !WRES && (int)blockIdx.x >= a.job_groups ? 1 : 0;
    const DirectJob &jb = a.job[ji];
    const int lb = ji ? xcd_block((int)blockIdx.x - a.job_groups, (int)gridDim.x - a.job_groups)
                      : xcd_block((int)blockIdx.x, a.job_groups);
    int mt, kb, wd_i = 0;
    if constexpr (WRES) {
        const int wg = (int)fdiv((uint32_t)lb, a.div_kb);
        kb = lb - wg * a.kblocks;
        mt = wg * a.wt + wave;
    } else {
        const int wt_i = (int)fdiv((uint32_t)wave, a.div_wd);
        wd_i = wave - wt_i * a.wd;
        const int tile = lb * a.wt + wt_i;
        if (tile >= a.tiles) return;   // (several tiles a workgroup: no barrier)
        if (a.pixel_fast) {
            kb = (int)fdiv((uint32_t)tile, a.div_mt);
            mt = tile - kb * a.mtiles;
        } else {
            mt = (int)fdiv((uint32_t)tile, a.div_kb);
            kb = tile - mt * a.kblocks;
        }
    }

    const __amdgpu_buffer_rsrc_t rx = make_brsrc(jb.x, jb.xrange);
    const __amdgpu_buffer_rsrc_t rw = make_brsrc(a.w, a.wbytes);

    // image offsets of the wave's channel pairs (32 channels; past the last
    // pair the last one is read again and never stored)
    int wpair[NP];
    int chan[NBK];   // the lane's first channel of each run
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int pair0 = kb * NP + p;
        const int pair = min(pair0, a.pairs - 1);
        const int blk = FKB == 4 ? pair >> 1 : pair;
        const int kt = (int)fdiv((uint32_t)blk, a.div_wk);
        wpair[p] = jb.ws0 + kt * a.kt_stride + (blk - kt * a.wk) * (FKB * 256) + (FKB == 4 ? (pair & 1) * 512 : 0);
        if (!WHOLE || p == 0) {
            const int blk0 = FKB == 4 ? pair0 >> 1 : pair0;
            chan[WHOLE ? 0 : p] = blk0 * FKB * 16 + gq * 4 * FKB + (FKB == 4 && !WHOLE ? (pair0 & 1) * 8 : 0);
        }
    }
    const int lane_w = gq * (B16 ? 2 : 1) * a.psw + l16 * 16;

    // ---- this wave's steps: [step0, step0 + steps)
    const int step0 = WRES ? 0 : wd_i * jb.steps_per_wave;
    const int steps = WRES ? jb.steps : max(0, min(jb.steps_per_wave, jb.steps - step0));
    const int rounds = (steps + LA - 1) / LA;

    // the step (B16: pair of steps) whose operands are loaded next: its tap, and its offsets in the
    // input and in the image.  (The increments are held in scalar registers:
    // taken from the argument block, the selects below become loads.)
    auto held = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int taps = held(jb.taps), fs = held(jb.s), xpix = held(a.xpix), xs_row = held(jb.xs_row),
              xs_chunk = held(jb.xs_chunk), ws_tap = held(a.tk16), ws_chunk = held(jb.ws_chunk);
    int s_i = 0, tap = 0, left, xs, ws;
    auto first_step = [&] {
        left = steps / US;
        if constexpr (LIN) {
            xs = step0 * CB;
            ws = step0 * ws_chunk;
        } else {
            const int j = (int)fdiv((uint32_t)step0, jb.div_taps);
            tap = step0 - j * taps;
            const int r_i = (int)fdiv((uint32_t)tap, jb.div_s);
            s_i = tap - r_i * fs;
            xs = (r_i * a.w_in + s_i) * xpix + j * CB;
            ws = j * 4 * a.psw + tap * ws_tap;
        }
        if (left <= 0) {   // a wave without steps reads zeros
            tap = 31;
            ws = 0;
        }
    };
    auto next_step = [&] {
        --left;
        if constexpr (LIN) {
            xs += CB * US;
            ws += left > 0 ? ws_chunk : 0;
        } else {
            // (scalar selects by mask: as conditionals they end up in vector
            // registers, and a scalar offset there costs a loop per load)
            const int row = -(int)(s_i + 1 == fs), chunk = -(int)(tap + 1 == taps), more = -(int)(left > 0);
            s_i = held((s_i + 1) & ~row);
            xs = held(xs + ((xs_chunk & chunk) | (((xs_row & row) | (xpix & ~row)) & ~chunk)));
            ws = held(ws + (((ws_chunk & chunk) | (ws_tap & ~chunk)) & more));
            tap = held((((tap + 1) & ~chunk) & more) | (31 & ~more));   // 31: a step past the last reads zeros
        }
    };

    // ---- the pixels: byte offset of the window's first tap, and a mask of
    // the taps outside the image (bit 31 always set).  (Lanes whose channels
    // lie past a pixel of fewer than 64 read its first ones: their filters are
    // zero, and no load passes the tensor's end.)
    const int lane_c = B16 ? gq * 16 : gq * (CB / 4) < a.xpix ? gq * (CB / 4) : 0;
    uint32_t voff[FP], bad[FP];
    auto set_pixels = [&](int mtile) {
        const int m0 = mtile * (FP * 16) + l16;
        if constexpr (LIN) {
#pragma unroll
            for (int tn = 0; tn < FP; ++tn)
                voff[tn] = (uint32_t)(min(m0 + tn * 16, a.m - 1) * xpix + lane_c);
            return;
        }
        int pp = 0, qq = 0, img = 0;
        // rows of at least 16 pixels: the next fragment is one step on, not a
        // division (not in the last tile, whose pixels past the output repeat
        // the last one)
        const bool walk = a.q >= 16 && (mtile + 1) * (FP * 16) <= a.m;
#pragma unroll
        for (int tn = 0; tn < FP; ++tn) {
            if (tn == 0 || !walk) {
                const int m = min(m0 + tn * 16, a.m - 1);
                img = (int)fdiv((uint32_t)m, a.div_pq);
                const int rem = m - img * a.pq;
                pp = (int)fdiv((uint32_t)rem, a.div_q);
                qq = rem - pp * a.q;
            } else {
                qq += 16;
                const bool over = qq >= a.q;
                qq -= over ? a.q : 0;
                pp += over ? 1 : 0;
                const bool next = pp >= a.p;
                pp = next ? 0 : pp;
                img += next ? 1 : 0;
            }
            const int h0 = pp * a.sh, w0 = qq * a.sw;   // in the padded image
            voff[tn] = (uint32_t)(((img * a.h_in + h0) * a.w_in + w0) * xpix + lane_c);
            uint32_t b = 0x80000000u;
            if (jb.padded) {
                const int slo = min(max(jb.pw - w0, 0), fs), shi = min(fs, a.w_in + jb.pw - w0);
                const uint32_t full = (1u << fs) - 1u;
                const uint32_t cols = full & ~(((1u << max(shi, 0)) - 1u) & ~((1u << slo) - 1u));
                for (int r_i = 0; r_i < jb.r; ++r_i) {
                    const bool in = (uint32_t)(h0 + r_i - jb.ph) < (uint32_t)a.h_in;
                    b |= (in ? cols : full) << (r_i * fs);
                }
            }
            bad[tn] = b;
        }
    };

    v4i A[AS][NF];
    Raw B[LB][FP];
    auto load_b = [&](int u) {
        // (bounds checks see the lane's offset, not the scalar one: 1x1 steps,
        // whose last chunk may pass the tensor's end, add theirs to the lane's;
        // other filters run here only with whole chunks)
        const uint32_t step = LIN ? (left > 0 ? (uint32_t)xs : 0x80000000u) : 31u - (uint32_t)tap;
#pragma unroll
        for (int tn = 0; tn < FP; ++tn) {
            const uint32_t off = LIN ? voff[tn] + step : ((bad[tn] << step) & 0x80000000u) | voff[tn];
            const int soff = LIN ? 0 : xs;
            if constexpr (B16)
                B[u / 2][tn] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)off, soff, 0);
            else if constexpr (BITS == 4)
                B[u][tn] = __builtin_amdgcn_raw_buffer_load_b64(rx, (int)off, soff, 0);
            else
                B[u][tn] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)off, soff, 0);
        }
    };
    auto load_a = [&](int u) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, lane_w + (f & 1) * 256, wpair[f >> 1] + ws, 0);
            A[u][f] = v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
        }
    };
    // RESIDENT: LDS holds the fragments step by step, NF KiB a step
    auto read_a = [&](int set, const uint8_t *p) {
#pragma unroll
        for (int f = 0; f < NF; ++f) A[set][f] = *reinterpret_cast<const v4i *>(p + f * 1024);
    };

    v4i acc[NBK][FP][FE];
    // (a resident kernel of one round starts from the biases; in those of several
    // the registers cost more than the additions: 79 -> 85 us for two 7x7 bottleneck
    // blocks)
    constexpr bool BIAS0 = EXT && WRES && !MULTI;
    v4i sum0[BIAS0 ? NF : 1];
    // (the first step of a tile starts the sums: no clearing)
    auto multiply = [&](int aset, int u, auto start) {
#pragma unroll
        for (int tn = 0; tn < FP; ++tn) {
            v4i bv;
            if constexpr (BITS == 4) {
                const uint32_t x0 = B[B16 ? u / 2 : u][tn][B16 ? u % 2 * 2 : 0];
                const uint32_t x1 = B[B16 ? u / 2 : u][tn][B16 ? u % 2 * 2 + 1 : 1];
                bv = v4i{(int)(x0 & 0x0F0F0F0Fu), (int)((x0 >> 4) & 0x0F0F0F0Fu), (int)(x1 & 0x0F0F0F0Fu),
                         (int)((x1 >> 4) & 0x0F0F0F0Fu)};
            } else {
                bv = v4i{(int)B[u][tn][0], (int)B[u][tn][1], (int)B[u][tn][2], (int)B[u][tn][3]};
            }
#pragma unroll
            for (int f = 0; f < NF; ++f)
                acc[f / FE][tn][f % FE] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                    A[aset][f], bv,
                    !decltype(start)::value ? acc[f / FE][tn][f % FE] : BIAS0 ? sum0[f] : v4i{0, 0, 0, 0}, 0, 0, 0);
        }
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};

    // ---- epilogue: multipliers and biases of the lane's channels (channels
    // past k repeat the last one and are never stored)
    const DirectEpilogue de{a.mode, a.acc_shift, jb.shift, jb.lo, jb.hi, a.res_signed, a.k, a.m,
                            ji ? nullptr : a.res, jb.yptr};
    int32_t mult[NBK][4 * FE], bias[EXT ? NBK : 1][EXT ? 4 * FE : 1];
    auto load_params = [&] {
        if (a.mode != QCONV_OUT_REQUANT) return;
#pragma unroll
        for (int b = 0; b < NBK; ++b)
#pragma unroll
            for (int i = 0; i < 4 * FE; ++i) {
                const int ch = min(chan[b] + i, a.k - 1);
                mult[b][i] = jb.mult[ch];
                if constexpr (EXT) bias[b][i] = jb.bias ? jb.bias[ch] : 0;
            }
    };
    // which form: f32 where the launch allows it and the lane's multipliers and
    // biases do (decided for the wave)
    bool f32 = false;
    auto prepare_params = [&] {
        bool ok = jb.fe.kind != 0 && a.mode == QCONV_OUT_REQUANT;
        if (!ok) return;
        const uint32_t room = jb.fe.bias_room;
#pragma unroll
        for (int b = 0; b < NBK; ++b)
#pragma unroll
            for (int i = 0; i < 4 * FE; ++i) {
                ok = ok && within(mult[b][i], 1u << 24);
                if constexpr (EXT) ok = ok && within(bias[b][i], room);
            }
        f32 = __all(ok);
        if (!f32) return;
#pragma unroll
        for (int b = 0; b < NBK; ++b)
#pragma unroll
            for (int i = 0; i < 4 * FE; ++i)
                mult[b][i] = (int32_t)__builtin_bit_cast(uint32_t, (float)mult[b][i] * jb.fe.scale);
    };
    // P fragments of run b (its multipliers mu, biases bi) at pixel mbase
    constexpr int NWD = 4 * FE * BITS / 32;   // words of a pixel's run
    auto load_residual = [&](auto &rw, int mbase, int cb) {
        if constexpr (EXT) {
            if (de.res && f32) {
#pragma unroll
                for (int tn = 0; tn < (int)(sizeof(rw) / sizeof(rw[0])); ++tn)
                    load_run<BITS, FE>(de, mbase + tn * 16 + l16, cb, rw[tn]);
            }
        }
    };
    // (the residual's words `rw` are loaded ahead for the f32 form only)
    auto finish = [&](auto &v, int mbase, int cb, const int32_t(&mu)[4 * FE], const int32_t *bi, const auto &rw) {
        constexpr int P = sizeof(v) / sizeof(v[0]);
        if constexpr (EXT && !BIAS0) {
            if (a.mode == QCONV_OUT_REQUANT) {
#pragma unroll
                for (int tn = 0; tn < P; ++tn)
#pragma unroll
                    for (int i = 0; i < 4 * FE; ++i)
                        v[tn][i / 4][i % 4] = (int)((uint32_t)v[tn][i / 4][i % 4] + ((uint32_t)bi[i] << (uint32_t)a.acc_shift));
            }
        }
        if (f32) {
            float mf[4 * FE];
#pragma unroll
            for (int i = 0; i < 4 * FE; ++i) mf[i] = __builtin_bit_cast(float, (uint32_t)mu[i]);
            if (EXT && de.res)
                epilogue_f32<BITS, P, FE, true>(de, jb.fe, v, mbase, cb, l16, mf, rw);
            else
                epilogue_f32<BITS, P, FE, false>(de, jb.fe, v, mbase, cb, l16, mf, rw);
            return;
        }
        EpiParams<FE> ep;
        ep.fast = false;
        if (a.mode == QCONV_OUT_REQUANT) make_epilogue_params<FE>(de, mu, ep);
        epilogue<BITS, P, FE, EXT>(de, v, mbase, cb, l16, ep);
    };

    if constexpr (WRES) {
        // ---- the filter block to LDS: 1 KiB fragments, dealt to the waves
        const u32x4 rimg = make_rsrc(a.w, a.wbytes);
        const int frags = steps * NF;
        for (int i = wave; i < frags; i += a.wt) {
            const int st = i / NF, f = i - st * NF;
            const int j = (int)fdiv((uint32_t)(st / US), jb.div_taps), tp = st / US - j * taps;
            const int off = wpair[NP == 2 ? f >> 1 : 0] + (j * 4 * US + st % US) * a.psw + tp * ws_tap + (f & 1) * 256;
            dma16(smem + i * 1024, (uint32_t)(lane_w + off), rimg);
        }
        set_pixels(min(mt, a.mtiles - 1));
        first_step();
        auto fetch = [&](int u) {   // after step u: the loads its registers are free for
            if (u % US != US - 1) return;
            load_b(u);
            next_step();
        };
#pragma unroll
        for (int u = 0; u < LA; ++u) fetch(u);
        load_params();
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        prepare_params();
        if constexpr (BIAS0) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    sum0[f][i] = a.mode == QCONV_OUT_REQUANT
                                     ? (int)((uint32_t)bias[f / FE][4 * (f % FE) + i] << (uint32_t)a.acc_shift) : 0;
        }
        // one round: LA steps, each loading its set again for the round after
        auto round = [&](const uint8_t *p, auto first, auto last) {
#pragma unroll
            for (int u = 0; u < LA; ++u) {
                if (!decltype(last)::value || u + 1 < LA) read_a((u + 1) % AS, p + (u + 1) * NF * 1024);
                if constexpr (decltype(first)::value) {
                    if (u == 0)
                        multiply(0, 0, yes);
                    else
                        multiply(u % AS, u, no);
                } else {
                    multiply(u % AS, u, no);
                }
                fetch(u);
            }
        };
        for (; mt < a.mtiles; mt += a.walk) {
            const uint8_t *p = smem + lane * 16;
            read_a(0, p);
            uint32_t rw[NBK][FP][NWD];
#pragma unroll
            for (int b = 0; b < NBK; ++b) load_residual(rw[b], mt * (FP * 16), chan[b]);
            // (the last round's loads are the next tile's first steps)
            if constexpr (MULTI) {
                round(p, yes, no);
                p += LA * NF * 1024;
                for (int it = 2; it < rounds; ++it) {
                    round(p, no, no);
                    p += LA * NF * 1024;
                }
                set_pixels(min(mt + a.walk, a.mtiles - 1));
                first_step();
                round(p, no, yes);
            } else {
                set_pixels(min(mt + a.walk, a.mtiles - 1));
                first_step();
                round(p, yes, yes);
            }
#pragma unroll
            for (int b = 0; b < NBK; ++b) finish(acc[b], mt * (FP * 16), chan[b], mult[b], bias[EXT ? b : 0], rw[b]);
        }
    } else {
        set_pixels(mt);
        first_step();
#pragma unroll
        for (int u = 0; u < LA; ++u) {
            load_a(u);
            load_b(u);
            next_step();
        }
        load_params();
        if constexpr (MULTI) {
            auto round = [&](auto first) {
#pragma unroll
                for (int u = 0; u < LA; ++u) {
                    if (decltype(first)::value && u == 0)
                        multiply(0, 0, yes);
                    else
                        multiply(u, u, no);
                    load_a(u);
                    load_b(u);
                    next_step();
                }
            };
            round(yes);
            for (int it = 2; it < rounds; ++it) round(no);
#pragma unroll
            for (int u = 0; u < LA; ++u) multiply(u, u, no);
        } else {
            multiply(0, 0, yes);
#pragma unroll
            for (int u = 1; u < LA; ++u) multiply(u, u, no);
        }
        prepare_params();
        if (a.wd == 1) {
            uint32_t rw[NBK][FP][NWD];
#pragma unroll
            for (int b = 0; b < NBK; ++b) load_residual(rw[b], mt * (FP * 16), chan[b]);
#pragma unroll
            for (int b = 0; b < NBK; ++b) finish(acc[b], mt * (FP * 16), chan[b], mult[b], bias[EXT ? b : 0], rw[b]);
            return;
        }
        // ---- the waves of a tile add their sums: unit (run b, fragment tn)
        // belongs to wave unit % wd (a power of two); the others leave theirs in LDS
        constexpr int UNITS = NBK * FP;
        const int owner = a.wd - 1;
        auto slot = [&](int unit, int d) {   // wave d's sums of a unit
            return smem + (size_t)((unit * a.wd + d) * FE) * 1024 + lane * 16;
        };
#pragma unroll
        for (int unit = 0; unit < UNITS; ++unit) {
            if ((unit & owner) == wd_i) continue;
            uint8_t *p = slot(unit, wd_i);
#pragma unroll
            for (int f = 0; f < FE; ++f) *reinterpret_cast<v4i *>(p + f * 1024) = acc[unit / FP][unit % FP][f];
        }
        __syncthreads();
#pragma unroll
        for (int unit = 0; unit < UNITS; ++unit) {
            if ((unit & owner) != wd_i) continue;
            v4i sum[1][FE];
            uint32_t rw[1][NWD];
            load_residual(rw, mt * (FP * 16) + (unit % FP) * 16, chan[unit / FP]);
#pragma unroll
            for (int f = 0; f < FE; ++f) sum[0][f] = acc[unit / FP][unit % FP][f];
            for (int d = 0; d < a.wd; ++d) {
                if (d == wd_i) continue;
                const uint8_t *p = slot(unit, d);
#pragma unroll
                for (int f = 0; f < FE; ++f) sum[0][f] += *reinterpret_cast<const v4i *>(p + f * 1024);
            }
            finish(sum, mt * (FP * 16) + (unit % FP) * 16, chan[unit / FP], mult[unit / FP], bias[EXT ? unit / FP : 0], rw);
        }
    }
}

template <int BITS, int FKB, int NP, int FP, bool EXT, int LA, bool MULTI, bool LIN, bool WRES, bool B16>
static hipError_t launch_direct(const DirectArgs &a, dim3 grid, int threads, size_t lds, hipStream_t stream) {
    hipLaunchKernelGGL((conv_direct<BITS, FKB, NP, FP, EXT, LA, MULTI, LIN, WRES, B16>), grid, dim3(threads), lds, stream, a);
    return hipGetLastError();
}

#define QCONV_DIRECT_ONE(B, FKB, NP, FP, E, LA, MU, LIN, WR, B16)                                                \
    {B, FKB, NP, FP, E, LA, MU, LIN, WR, B16,                                                                     \
     &launch_direct<B, FKB, NP, FP, (E != 0), LA, (MU != 0), (LIN != 0), (WR != 0), (B16 != 0)>,                  \
     reinterpret_cast<const void *>(                                                                              \
         &conv_direct<B, FKB, NP, FP, (E != 0), LA, (MU != 0), (LIN != 0), (WR != 0), (B16 != 0)>)},
#define QCONV_DIRECT_EXT(B, FKB, NP, FP, LA, MU, LIN, WR) \
    QCONV_DIRECT_ONE(B, FKB, NP, FP, 0, LA, MU, LIN, WR, 0) QCONV_DIRECT_ONE(B, FKB, NP, FP, 1, LA, MU, LIN, WR, 0)
#define QCONV_DIRECT_B16(FKB, NP, FP, LA, MU, LIN) \
    QCONV_DIRECT_ONE(4, FKB, NP, FP, 0, LA, MU, LIN, 1, 1) QCONV_DIRECT_ONE(4, FKB, NP, FP, 1, LA, MU, LIN, 1, 1)
// depth: any filter, then 1x1; resident: 1x1, then any filter
#define QCONV_DIRECT_SET(B, FKB)                                                              \
    QCONV_DIRECT_EXT(B, FKB, 1, 1, 9, 0, 0, 0) QCONV_DIRECT_EXT(B, FKB, 1, 1, 9, 1, 0, 0)     \
    QCONV_DIRECT_EXT(B, FKB, 1, 2, 3, 1, 0, 0) QCONV_DIRECT_EXT(B, FKB, 2, 2, 3, 1, 0, 0)     \
    QCONV_DIRECT_EXT(B, FKB, 1, 1, 4, 0, 1, 0) QCONV_DIRECT_EXT(B, FKB, 1, 2, 4, 0, 1, 0)     \
    QCONV_DIRECT_EXT(B, FKB, 1, 1, 8, 0, 1, 0) QCONV_DIRECT_EXT(B, FKB, 1, 2, 8, 0, 1, 0)     \
    QCONV_DIRECT_EXT(B, FKB, 1, 1, 8, 1, 1, 0) QCONV_DIRECT_EXT(B, FKB, 1, 2, 8, 1, 1, 0)     \
    QCONV_DIRECT_EXT(B, FKB, 2, 2, 4, 0, 1, 0) QCONV_DIRECT_EXT(B, FKB, 2, 2, 4, 1, 1, 0)     \
    QCONV_DIRECT_EXT(B, FKB, 2, 4, 4, 0, 1, 0) QCONV_DIRECT_EXT(B, FKB, 2, 4, 4, 1, 1, 0)     \
    QCONV_DIRECT_EXT(B, FKB, 2, 2, 1, 0, 1, 1) QCONV_DIRECT_EXT(B, FKB, 2, 2, 2, 0, 1, 1)     \
    QCONV_DIRECT_EXT(B, FKB, 2, 4, 1, 0, 1, 1) QCONV_DIRECT_EXT(B, FKB, 2, 4, 2, 0, 1, 1)     \
    QCONV_DIRECT_EXT(B, FKB, 2, 2, 4, 0, 1, 1) QCONV_DIRECT_EXT(B, FKB, 2, 2, 4, 1, 1, 1)     \
    QCONV_DIRECT_EXT(B, FKB, 2, 2, 3, 1, 0, 1)
#define QCONV_DIRECT_SET16(FKB)                                                               \
    QCONV_DIRECT_B16(FKB, 2, 2, 2, 0, 1) QCONV_DIRECT_B16(FKB, 2, 4, 2, 0, 1)                 \
    QCONV_DIRECT_B16(FKB, 2, 2, 4, 0, 1) QCONV_DIRECT_B16(FKB, 2, 2, 4, 1, 1)

}  // namespace qconv
