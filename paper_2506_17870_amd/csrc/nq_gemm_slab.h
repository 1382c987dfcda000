// Nested-integer GEMM / implicit-GEMM convolution for layers whose output is too small to fill the chip with the large
// kernel's tiles: one image through a CNN, a few hundred tokens through a transformer layer (paper Sec. 3.3: full-bit
// w_high * 2^l + w_low, Eq. 4; part-bit w_high with s * 2^l, Eq. 8).
//
// What bounds such a layer is the serial chain of one block, not bytes or matrix cores: with 64 x 256 tiles a
// 196 x 2304 -> 256 layer is four blocks that walk all of K.  Here a block owns 32 rows x 32 columns and its NWS waves
// split the reduction as in nq_gemm_skinny.h (wave w: K steps w, w + NWS, ...), so the same layer is 56 blocks and a wave
// walks five of its 36 steps.  Weights and activations go straight into the matrix core's operand registers, SL_PD
// steps ahead: there is too little reuse inside a block to pay for a trip through LDS.  The partial sums meet in LDS
// (integers: any order), wave 0 runs the epilogue, whose constants and residual codes it has requested before the
// reduction.  A step past the end of K requests the last real weights again; its activations are requested out of the
// tensor's range, by their vector offset (the range check does not cover the scalar one), and are zero.
//
// Activations are fetched with dword-aligned 16-byte buffer loads: any K that is a multiple of four serves as a GEMM.
// What a row's last piece reads past K belongs to the next row (or is out of range) and meets the zero weights the
// pages are padded with.  CONV: any filter over a multiple of 32 input channels: the 32 bytes a lane needs of a K step
// are one run of one tap's pixel.  blockIdx.x is the column tile, so that with a multiple of eight column tiles the
// blocks that read the same weights run on the same XCD.
//
// Measured, K-loop kernels before and this one: 196 x 2304 -> 256 (3x3) 14.8 -> 7.2 us, 49 x 4608 -> 512 (3x3) 61 -> 9.4 us,
// 197 x 3072 -> 768 16.7 -> 7.7 us, 64 x 512 -> 512 4.8 -> 4.1 us; a launch that does nothing is about 3.5 us of that.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nq_codec.h"
#include "nq_epilogue.h"
#include "nq_gemm_big.h"

namespace nq {

template <int H, int L, int FULL, int EPI, int NWS, bool CONV>
__global__ void __launch_bounds__(64 * NWS, 2) k_nested_gemm_slab(const GemmParams p, const int x_bytes, const unsigned cin_magic)
{
    constexpr int S = 8 - H;
    constexpr int SHIFT = FULL ? (8 - H - L) : S;
    using LP = LowPage<L, S, FULL>;
    constexpr int SL_PD = 4;
    constexpr int NOWHERE = 0x7fff0000;
    static_assert(EPI != EPI_ANY, "vector epilogues only");

    __shared__ __attribute__((aligned(16))) e_v4i red[NWS - 1][4][64];

    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = blockIdx.x;
    const int m0 = blockIdx.y * 32;
    const int M = (int)p.M;
    const int wslot = epi_weight_slot<EPI>(lane);

    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(p.x), 0, x_bytes, 0x00020000);
    const int64_t tile0 = (int64_t)nb * p.KB;
    const __amdgpu_buffer_rsrc_t hrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.ph + tile0 * (H * 64)), 0,
                                                                         p.KB * (H * 256), 0x00020000);
    const __amdgpu_buffer_rsrc_t lrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t *>(FULL ? p.pl + tile0 * (LP::DW * 64) : p.ph), 0, p.KB * (LP::DW * 256), 0x00020000);

    // the lane's row of the GEMM: its byte offset, and for a filter the input pixel of tap (0, 0)
    const int m = m0 + (lane & 31);
    int x_row, ih0 = 0, iw0 = 0;
    if constexpr (CONV) {
        const int mm = m < M ? m : 0;
        const int HoWo = p.Ho * p.Wo;
        const int b = mm / HoWo, rem = mm - b * HoWo;
        const int oh = rem / p.Wo, ow = rem - oh * p.Wo;
        ih0 = m < M ? oh * p.stride - p.pad : -(1 << 20);          // a row past M: no tap lands in the image
        iw0 = ow * p.stride - p.pad;
        x_row = ((b * p.H + oh * p.stride - p.pad) * p.W + iw0) * p.Cin;
    } else {
        x_row = m < M ? m * p.K : NOWHERE;
    }

    uint32_t P[SL_PD][H];
    uint32_t Q[SL_PD][LP::ARR];
    e_v4i A[SL_PD][2];
    auto request = [&](int slot, int kb) {
        const int kbc = min(kb, p.KB - 1);
        const int hoff = kbc * (H * 256);
#pragma unroll
        for (int c = 0; c < (H + 3) / 4; ++c) gb_fetch(P[slot], hrs, H, c, wslot * (4 * H), hoff);
        if constexpr (FULL != 0) {
            const int loff = kbc * (LP::DW * 256);
#pragma unroll
            for (int c = 0; c < (LP::DW + 3) / 4; ++c) gb_fetch(Q[slot], lrs, LP::DW, c, wslot * (4 * LP::DW), loff);
        }
        const int k0 = 64 * kb + 32 * g;
        int at;
        if constexpr (CONV) {
            const int tap = p.Cin == p.K ? 0 : (int)__umulhi((unsigned)k0, cin_magic);
            const int kh = (tap * p.kw_magic) >> 16, kw = tap - kh * p.KW;
            const int ih = ih0 + kh, iw = iw0 + kw;
            const bool in = k0 < p.K && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
            at = in ? x_row + (kh * p.W + kw) * p.Cin + (k0 - tap * p.Cin) : NOWHERE;
        } else {
            at = kb < p.KB && x_row != NOWHERE ? x_row + k0 : NOWHERE;
        }
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(xrs, at + 16 * hf, 0, 0);
            A[slot][hf] = e_v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
        }
    };

#pragma unroll
    for (int d = 0; d < SL_PD; ++d) request(d, wave + NWS * d);

    // wave 0 asks for what its epilogue needs now
    const int rows = M - m0 < 32 ? M - m0 : 32;
    const int nl0 = nb * 32 + 16 * g;
    EpiRaw16 raw;
    EpiCols<EPI> e;
    e_v4i res = e_v4i{0, 0, 0, 0};
    if (wave == 0) {
        if constexpr (EPI == EPI_I8) {
            epi_cols16_fetch(p, nl0, raw);
            epi_resid_load<EPI>(p, m0, rows, nb * 32, lane, res);
        } else {
            epi_cols<EPI>(p, nb * 32, lane, FULL != 0, e);
        }
    }

    e_v16i acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
    const int rounds = (p.KB + NWS - 1) / NWS;
    for (int j0 = 0; j0 < rounds; j0 += SL_PD) {
#pragma unroll
        for (int d = 0; d < SL_PD; ++d) {
            uint32_t D[8];
            HighCodec<H>::decode(P[d], D);
            LP::apply(Q[d], D);
            const e_v4i a0 = A[d][0], a1 = A[d][1];
            request(d, wave + NWS * (j0 + d + SL_PD));
            acc = epi_mfma<EPI>(e_v4i{(int)D[0], (int)D[1], (int)D[2], (int)D[3]}, a0, acc);
            acc = epi_mfma<EPI>(e_v4i{(int)D[4], (int)D[5], (int)D[6], (int)D[7]}, a1, acc);
        }
    }

    // ---- add the partial sums of the waves -----------------------------------------------------------------------
    if (wave > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            red[wave - 1][q][lane] = e_v4i{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < NWS - 1; ++w)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const e_v4i v = red[w][q][lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[4 * q + i] += v[i];
        }

    // ---- epilogue (Eq. 2 / Eq. 8) -----------------------------------------------------------------------------
    if constexpr (EPI == EPI_I8) epi_cols16_finish(p, FULL != 0, raw, e);
    epi_tile<EPI>(p, acc, SHIFT, e, m0, rows, nb * 32, lane, res);
}

// Defined here, instantiated once per (h, l) by nq_gemm_slab.hip.  The caller has checked the shape (slab_ok in
// nq_gemm.hip) and that the problem takes a vector epilogue.
template <int H, int L>
void launch_nested_gemm_slab(bool full, const GemmParams &p, int x_bytes, hipStream_t st, void *ev_start, void *ev_stop)
{
    const dim3 grid((unsigned)p.NB, (unsigned)((p.M + 31) / 32));
    const bool conv = p.KH != 1 || p.KW != 1 || p.stride != 1 || p.pad != 0;
    const unsigned cin_magic = (unsigned)(((uint64_t(1) << 32) + p.Cin - 1) / p.Cin);
    // Eight waves per block where four would leave a compute unit's SIMDs idle and there are steps to share.
    const bool wide = (int64_t)grid.x * grid.y <= 512 && p.KB >= 12;
#define NQ_SL_ONE(FULLV, EPIV, NWSV, CONVV)                                                               \
    launch_timed(k_nested_gemm_slab<H, L, FULLV, EPIV, NWSV, CONVV>, grid, dim3(64 * NWSV), 0, st, ev_start, ev_stop, p, \
                 x_bytes, cin_magic)
#define NQ_SL_LAUNCH(FULLV, EPIV)                                  \
    do {                                                           \
        if (wide && conv) NQ_SL_ONE(FULLV, EPIV, 8, true);         \
        else if (wide) NQ_SL_ONE(FULLV, EPIV, 8, false);           \
        else if (conv) NQ_SL_ONE(FULLV, EPIV, 4, true);            \
        else NQ_SL_ONE(FULLV, EPIV, 4, false);                     \
    } while (0)
#define NQ_SL_MODES(FULLV)                                             \
    do {                                                               \
        if (epi_mode(p) == EPI_I8) NQ_SL_LAUNCH(FULLV, EPI_I8);        \
        else NQ_SL_LAUNCH(FULLV, EPI_F32);                             \
    } while (0)
    if (full && p.low_signed) NQ_SL_MODES(2); else if (full) NQ_SL_MODES(1); else NQ_SL_MODES(0);
}

}  // namespace nq
