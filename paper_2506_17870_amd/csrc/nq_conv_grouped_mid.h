// Nested-integer grouped convolution with groups of up to 32 channels on the matrix cores (the 3x3 layers of
// ResNeXt, the grouped 1x1 layers of ShuffleNet: lightweight CNNs of the paper's Sec. 4; modes of Sec. 3.3, Eq. 4 /
// Eq. 8).  Input and output widths of a group may differ.
//
// v_mfma_i32_32x32x32_i8 contracts one filter tap: 32 input channels x 32 pixels against a 32 x 32 weight operand
// that is block diagonal over the G = 32 / max(gs_in, gs_out) whole groups it covers (a "half tile": G * gs_in input
// and G * gs_out output channels; a block owns two).  At eight channels per group three quarters of the matrix core
// are multiplied by zero, and it is still far from being the limit: the layer is a stream, bound by the window loads
// and the epilogue.
//
// As in nq_conv_grouped.h a persistent block takes patches of R x CW output pixels; the input window of the next
// patch travels to registers while the present one is computed from LDS (80 bytes per pixel: eight neighbouring pixels
// hit distinct banks with 16-byte reads, at stride 2 as well).  Two waves share a half tile and deal its 32-pixel
// tiles; a wave keeps its half tile's weights, all taps, in registers (four per tap).  The matrix core's row operand is
// the weights in epi_weight_slot() order, so a lane ends up with sixteen consecutive channels of one pixel.
//
// The piece of 16 bytes at the end of a pixel may reach past its channels (12 channels per group, a channel count that
// is no multiple of 32): what follows it in memory, or the zeros of the range check behind the last pixel, which works
// dword by dword, meets zero weights.
//
// 32 x 56 x 56 x 256, 32 groups of 8, 3x3, int8 out: the kernel of nq_conv_grouped_any.h takes 218 us,
// this one 24 us (51 MB in and out: 2.1 TB/s); what is left is the window's trip through registers and LDS and the epilogue.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "nq_codec.h"
#include "nq_conv_grouped.h"
#include "nq_gemm_kernel.h"

namespace nq {

// NT: filter taps the registers hold (1 or 9); missing ones have zero weights.
template <int H, int L, int FULL, int EPI, int NT>
__global__ void __launch_bounds__(256, 2) k_nested_conv_grouped_mid(const GemmParams p, const GroupGeom g)
{
    constexpr int S = 8 - H;
    constexpr int SHIFT = FULL ? (8 - H - L) : S;
    using LP = LowPage<L, S, FULL>;
    static_assert(EPI != EPI_F32, "a lane owns 16 channels of a pixel: swapped layouts only");

    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];     // the decoded weights first, then the window

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave & 1, kg = lane >> 5;
    const int ct = blockIdx.y;

    // ---- window staging plan: piece i = tid + 256*j is 16-byte piece i & 3 of window pixel i >> 2; pieces 0, 1 are
    // the input channels of the first half tile, 2, 3 those of the second ------------------------------------------
    const int sq = tid & 3;
    const int ch0 = (2 * ct + (sq >> 1)) * g.hin + 16 * (sq & 1);     // first channel of the thread's pieces
    const bool ch_ok = ch0 < p.Cin && 16 * (sq & 1) < g.hin;
    int st_lds[GC_NP], st_rc[GC_NP];
#pragma unroll
    for (int j = 0; j < GC_NP; ++j) {
        const int pi = (tid + 256 * j) >> 2;
        const int r = (int)(((unsigned)pi * (unsigned)g.icp_magic) >> 20), c = pi - r * g.ICp;
        st_lds[j] = pi < g.IRp * g.ICp ? pi * GC_PIX + 16 * sq : -1;
        st_rc[j] = (r << 16) | c;
    }
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(p.x), 0,
                                                                           (int)g.x_bytes, 0x00020000);
    g_v4i stage[GC_NP];
    auto request = [&](int b, int rb, int cb) {
        const int ih0 = rb * g.R * p.stride - p.pad, iw0 = cb * g.CW * p.stride - p.pad;
#pragma unroll
        for (int j = 0; j < GC_NP; ++j) {
            if (j < g.np) {
                const int ih = ih0 + (st_rc[j] >> 16), iw = iw0 + (st_rc[j] & 0xffff);
                const bool ok = ch_ok && st_lds[j] >= 0 && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
                const int at = ((b * p.H + ih) * p.W + iw) * p.Cin + ch0;
                // outside the image: an offset past the tensor, which reads as zero
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, ok ? at : 0x7fff0000, 0, 0);
                stage[j] = g_v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
            }
        }
    };
    int u = blockIdx.x;
    int b = u / (g.CB * g.RB), rb = (u - b * g.CB * g.RB) / g.CB, cb = u - (b * g.RB + rb) * g.CB;
    auto advance = [&](int &b_, int &rb_, int &cb_) {
        cb_ += g.step_cb;
        if (cb_ >= g.CB) { cb_ -= g.CB; ++rb_; }
        rb_ += g.step_rb;
        if (rb_ >= g.RB) { rb_ -= g.RB; ++b_; }
        b_ += g.step_b;
    };
    if (u < g.units) request(b, rb, cb);             // travels while the weights are set up

    // ---- weights of the two half tiles -> plain byte matrix in LDS, one row per output channel ------------------
    const int wst = 64 * p.KB + 16;
    for (int idx = tid; idx < 64 * 2 * p.KB; idx += 256) {
        const int row = idx & 63, kk = idx >> 6;     // 32 values of k
        const int c = row & 31, n = (2 * ct + (row >> 5)) * g.hout + c;
        uint32_t D[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) D[j] = 0;
        if (c < g.hout && n < p.N) {
            const int64_t tile = (int64_t)(n >> 5) * p.KB + (kk >> 1);
            const int slot = 32 * (kk & 1) + (n & 31);
            uint32_t P[H];
#pragma unroll
            for (int i = 0; i < H; ++i) P[i] = p.ph[tile * (H * 64) + slot * H + i];
            HighCodec<H>::decode(P, D);
            if constexpr (FULL != 0) {
                uint32_t Q[LP::ARR];
#pragma unroll
                for (int i = 0; i < LP::DW; ++i) Q[i] = p.pl[tile * (LP::DW * 64) + slot * LP::DW + i];
                LP::apply(Q, D);
            }
        }
        uint8_t *dst = lds + row * wst + 32 * kk;
        *reinterpret_cast<g_v4i *>(dst) = g_v4i{(int)D[0], (int)D[1], (int)D[2], (int)D[3]};
        *reinterpret_cast<g_v4i *>(dst + 16) = g_v4i{(int)D[4], (int)D[5], (int)D[6], (int)D[7]};
    }
    __syncthreads();

    // ---- weight fragments: operand row lane & 31 is output channel oc of the half tile, its bytes the input channels
    // 16*kg .. 16*kg + 15, non-zero inside the channel's own group (groups are whole dwords) ------------------------
    const int oc = epi_weight_slot<EPI>(lane) & 31;
    const int gi = oc / g.gs_out;
    g_v4i wf[NT];
    int tap_off[NT];
#pragma unroll
    for (int tap = 0; tap < NT; ++tap) {
        const int kh = (tap * p.kw_magic) >> 16;
        tap_off[tap] = tap < g.taps ? (kh * g.ICp + (tap - kh * p.KW)) * GC_PIX : 0;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int i = 16 * kg + 4 * d - gi * g.gs;            // input channel inside the group
            const bool ok = oc < g.hout && i >= 0 && i < g.gs && tap < g.taps;
            wf[tap][d] = ok ? *reinterpret_cast<const int *>(lds + (32 * half + oc) * wst + tap * g.gs + i) : 0;
        }
    }

    // ---- constants of the lane's sixteen output channels; pc: p with the channel count cut at the half tile's end ----
    const int n_half = (2 * ct + half) * g.hout;
    const int nl0 = n_half + 16 * kg;
    GemmParams pc = p;
    pc.N = n_half + g.hout < p.N ? n_half + g.hout : p.N;
    EpiCols<EPI> e;
    epi_cols16<EPI>(pc, nl0, FULL != 0, e);
    __syncthreads();                                 // every wave has its weights: the window may overwrite them

    const int patch = g.R * g.CW;
    for (; u < g.units; u += gridDim.x) {
#pragma unroll
        for (int j = 0; j < GC_NP; ++j)
            if (j < g.np && st_lds[j] >= 0) *reinterpret_cast<g_v4i *>(lds + st_lds[j]) = stage[j];
        __syncthreads();                             // the window of unit u is complete
        int bn = b, rbn = rb, cbn = cb;
        advance(bn, rbn, cbn);
        if (u + (int)gridDim.x < g.units) request(bn, rbn, cbn);     // travels while this unit is computed

        // a loop without a residual has no load in it: a wait for one would be a wait for the window as well
        auto tiles = [&](auto with_resid) {
            for (int tile = wave >> 1; tile < g.ptiles; tile += 2) {
                const int idx = tile * 32 + (lane & 31);             // the lane's pixel
                const int idc = idx < patch ? idx : patch - 1;
                const int r = (int)(((unsigned)idc * (unsigned)g.cw_magic) >> 20), c = idc - r * g.CW;
                const int oh = rb * g.R + r, ow = cb * g.CW + c;
                const bool live = idx < patch && oh < p.Ho && ow < p.Wo;
                const uint8_t *src = lds + (r * g.ICp + c) * (p.stride * GC_PIX) + 32 * half + 16 * kg;
                const int64_t o = (((int64_t)b * p.Ho + oh) * p.Wo + ow) * p.N + nl0;
                e_v4i res = e_v4i{0, 0, 0, 0};
                if constexpr (EPI == EPI_I8 && decltype(with_resid)::value) {
                    if (live && nl0 < pc.N) res = *reinterpret_cast<const e_v4i *>(p.resid + o);
                }
                g_v4i V[NT];
#pragma unroll
                for (int tap = 0; tap < NT; ++tap) V[tap] = *reinterpret_cast<const g_v4i *>(src + tap_off[tap]);
                e_v16i acc;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] = 0;
#pragma unroll
                for (int tap = 0; tap < NT; ++tap) acc = epi_mfma<EPI>(wf[tap], V[tap], acc);
                if (live) epi_row16<EPI>(pc, acc, SHIFT, e, o, nl0, res);
            }
        };
        if (p.resid) tiles(std::true_type{});
        else tiles(std::false_type{});
        __syncthreads();                             // every wave is done with the window
        b = bn; rb = rbn; cb = cbn;
    }
}

template <int H, int L>
void launch_nested_conv_grouped_mid(bool full, const GemmParams &p, const GroupGeom &g, hipStream_t st, void *ev_start,
                                    void *ev_stop)
{
    const dim3 grid((unsigned)g.grid_x, (unsigned)g.CT), block(256);
    const size_t lds = (size_t)g.lds_bytes;
    // 16-byte stores need half tiles that start on multiples of 16 channels
    const bool vec = epi_mode(p) == EPI_I8 && g.hout % 16 == 0;
#define NQ_GM_LAUNCH(FULLV, EPIV, NTV) \
    launch_timed(k_nested_conv_grouped_mid<H, L, FULLV, EPIV, NTV>, grid, block, lds, st, ev_start, ev_stop, p, g)
    // (a single tap comes here with 16-byte stores only: the caller leaves the others to the direct kernel)
#define NQ_GM_MODES(FULLV)                               \
    do {                                                 \
        if (g.taps == 1) NQ_GM_LAUNCH(FULLV, EPI_I8, 1); \
        else if (vec) NQ_GM_LAUNCH(FULLV, EPI_I8, 9);    \
        else NQ_GM_LAUNCH(FULLV, EPI_ANY, 9);            \
    } while (0)
    if (full && p.low_signed) NQ_GM_MODES(2); else if (full) NQ_GM_MODES(1); else NQ_GM_MODES(0);
}

}  // namespace nq
