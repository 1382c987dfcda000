// Nested-integer GEMM / implicit-GEMM convolution for layers whose output is too small to fill the chip with the large
// kernel's tiles: one image through a CNN, a few hundred tokens through a transformer layer (paper Sec. 3.3: full-bit
// w_high * 2^l + w_low, Eq. 4; part-bit w_high with s * 2^l, Eq. 8).
//
// What bounds such a layer is the serial chain of one block, not bytes or matrix cores: with 64 x 256 tiles a
// 196 x 2304 -> 256 layer is four blocks that walk all of K.  Here a block owns 32 rows x 32 columns (16 columns where even
// those leave compute units idle, 64 rows where there are blocks enough) and its four waves split the reduction (wave w:
// units w, w + 4, ...).  Weights and activations go straight into the matrix core's operand registers, PD units ahead:
// there is too little reuse inside a block to pay for a trip through LDS.  The partial sums meet in LDS (integers: any
// order) and every wave finishes a quarter of the tile, its constants and residual codes requested before the reduction.
//
// The links of that chain, a launch that does nothing being 2.3 us of it: every wave's first requests are ahead of all
// arithmetic, and a wave's decoding is itself a serial chain (8 clocks an instruction with one wave per SIMD), so four waves and a loop
// of rounds beat eight or sixteen waves with a straight line per count, where the compiler moved the later requests down to their
// use (256 x 8192 -> 256 12.9 us against 14.5); requests for units that do not exist are waited for at the end like any
// other, so a wave of few units makes none; the waits count requests, so nothing that branches stands between them.
//
// Activations are fetched with dword-aligned 16-byte buffer loads: any K that is a multiple of four serves as a GEMM.
// What a row's last piece reads past K belongs to the next row (or is out of range) and meets the zero weights the
// pages are padded with.  CONV: any filter over a multiple of four input channels: the 32 bytes a lane needs of a K step are
// one run of one tap's pixel (1: multiples of 32 channels), two of 16 bytes (2), four of 8 (3) or eight of 4 (4), each with the
// tap it lies in: more requests per step, but no staging (7 images of 20 x 20 x 40 -> 464 3x3 stride 2 11.9 us in the
// generic kernel, which walks such rows in pieces, 3.8 here; 52 of 11 x 11 x 36 -> 48 102 and 4.1).  blockIdx.x is the column tile, so that
// with a multiple of eight column tiles the blocks that read the same weights run on the same XCD.
//
// Measured in a replayed graph, eight waves with rounds padded to four before and this: 196 x 1024 -> 256 5.4 -> 3.4 us, 14 x 14 x
// 256 -> 256 3x3 7.7 -> 5.2, 7 x 7 x 512 -> 512 3x3 9.9 -> 7.2, 197 x 3072 -> 768 8.4 -> 6.4, 28 x 28 x 128 -> 512 with a residual
// 5.2 -> 2.8, 64 x 512 -> 512 3.7 -> 2.8; against the kernels that had these: 197 x 768 -> 3072 11.4 -> 5.9 (large), 4000 x 128 ->
// 256 6.3 -> 3.4 (stationary), 8 x 28 x 28 x 128 -> 64 3x3 18.8 -> 6.4 (windowed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "nq_codec.h"
#include "nq_epilogue.h"
#include "nq_gemm_big.h"

namespace nq {

// The same for four channels of one row, y being final but for ReLU and requantisation (the arithmetic of epi_codes16).
__device__ __forceinline__ int epi_codes4(const GemmParams &p, const float (&y)[4])
{
    unsigned d = 0;
    if (p.relu && p.inv_out_scale > 0.0f) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            d = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(y[i] * p.inv_out_scale, 0.0f, 127.0f), i, d);
        return (int)d;
    }
    const float lo = p.relu ? 0.0f : -__builtin_inff();
#pragma unroll
    for (int i = 0; i < 4; ++i)
        d = __builtin_amdgcn_cvt_pk_u8_f32(rintf(fmaxf(y[i], lo) * p.inv_out_scale) + 128.0f, i, d);
    return (int)(d ^ 0x80808080u);
}

// NC: columns of the block's tile, 32 (32x32x32 matrix steps, one K step per unit of work) or 16 (16x16x64 steps, two K
// steps per unit: lanes 0-31 hold the first one's weights, lanes 32-63 the second one's).  RG: row groups of NC rows, all
// multiplied with the same decoded weights.  PD: units in flight per wave.  Four waves per SIMD (the compensated format's
// longer decoding takes the registers of a fourth).
template <int H, int L, int FULL, int NC, int RG, int PD, int CONV>
__global__ void __launch_bounds__(256, FULL == 2 ? 3 : 4) k_nested_gemm_slab(const GemmParams p, const int x_bytes, const unsigned cin_magic)
{
    constexpr int NWS = 4;                         // waves
    constexpr int S = 8 - H;
    constexpr int SHIFT = FULL ? (8 - H - L) : S;
    using LP = LowPage<L, S, FULL>;
    constexpr int NOWHERE = 0x7fff0000;
    constexpr int BM = NC * RG;                    // rows of the block
    constexpr int NQ = NC == 32 ? 4 : 1;           // runs of four channels a lane holds of a row group
    constexpr int SPU = NC == 32 ? 1 : 2;          // K steps per unit

    __shared__ __attribute__((aligned(16))) e_v4i red[NWS][RG * NQ][64];

    const int tid = threadIdx.x, lane = tid & 63, g = (lane / NC) & 1;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = blockIdx.x;                     // tile of NC columns
    const int m0 = blockIdx.y * BM;
    const int M = (int)p.M;
    // the weights are the matrix core's row operand whatever the output type: a lane's sums are runs of four channels
    const int wslot = NC == 32 ? epi_weight_slot<EPI_I8>(lane) : 32 * g + 16 * (nb & 1) + (lane & 15);
    const int pair = NC == 32 ? 0 : lane >> 5;     // which of the unit's K steps the lane works on

    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(p.x), 0, x_bytes, 0x00020000);
    const int64_t tile0 = (int64_t)(NC == 32 ? nb : nb >> 1) * p.KB;
    const __amdgpu_buffer_rsrc_t hrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p.ph + tile0 * (H * 64)), 0,
                                                                         p.KB * (H * 256), 0x00020000);
    const __amdgpu_buffer_rsrc_t lrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t *>(FULL ? p.pl + tile0 * (LP::DW * 64) : p.ph), 0, p.KB * (LP::DW * 256), 0x00020000);

    // the lane's rows of the GEMM: their byte offsets, and for a filter the input pixels of tap (0, 0)
    int x_row[RG], ih0[RG], iw0[RG];
#pragma unroll
    for (int r = 0; r < RG; ++r) {
        const int m = m0 + NC * r + (lane & (NC - 1));
        if constexpr (CONV != 0) {
            const int mm = m < M ? m : 0;
            const int HoWo = p.Ho * p.Wo;
            const int b = mm / HoWo, rem = mm - b * HoWo;
            const int oh = rem / p.Wo, ow = rem - oh * p.Wo;
            ih0[r] = m < M ? oh * p.stride - p.pad : -(1 << 20);          // a row past M: no tap lands in the image
            iw0[r] = ow * p.stride - p.pad;
            x_row[r] = ((b * p.H + oh * p.stride - p.pad) * p.W + iw0[r]) * p.Cin;
        } else {
            x_row[r] = m < M ? m * p.K : NOWHERE;
            ih0[r] = iw0[r] = 0;
        }
    }

    uint32_t P[PD][H];
    uint32_t Q[PD][LP::ARR];
    e_v4i A[PD][RG][2];
    // unit u into slot `slot`; a K step past the last one is requested out of range
    auto request = [&](int slot, int u) {
        const int kb = SPU * u + pair;
        const bool real = kb < p.KB;
        // (the scalar offset of one K step per unit stays inside the page: the range check does not cover it)
        const int hv = real ? wslot * (4 * H) + (SPU == 1 ? 0 : kb * (H * 256)) : NOWHERE;
        const int hs = SPU == 1 ? min(kb, p.KB - 1) * (H * 256) : 0;
#pragma unroll
        for (int c = 0; c < (H + 3) / 4; ++c) gb_fetch(P[slot], hrs, H, c, hv, hs);
        if constexpr (FULL != 0) {
            const int lv = real ? wslot * (4 * LP::DW) + (SPU == 1 ? 0 : kb * (LP::DW * 256)) : NOWHERE;
            const int ls = SPU == 1 ? min(kb, p.KB - 1) * (LP::DW * 256) : 0;
#pragma unroll
            for (int c = 0; c < (LP::DW + 3) / 4; ++c) gb_fetch(Q[slot], lrs, LP::DW, c, lv, ls);
        }
        const int k0 = 64 * kb + 32 * g;
        if constexpr (CONV != 0) {
            // the lane's 32 bytes as one, two, four or eight runs that each lie inside a tap
            constexpr int RUNS = 1 << (CONV - 1);
#pragma unroll
            for (int q = 0; q < RUNS; ++q) {
                const int k = k0 + 32 / RUNS * q;
                const int tap = p.Cin == p.K ? 0 : (int)__umulhi((unsigned)k, cin_magic);
                const int kh = (tap * p.kw_magic) >> 16, kw = tap - kh * p.KW;
                const int ci = (kh * p.W + kw) * p.Cin + (k - tap * p.Cin);
#pragma unroll
                for (int r = 0; r < RG; ++r) {
                    const bool in = k < p.K && (unsigned)(ih0[r] + kh) < (unsigned)p.H && (unsigned)(iw0[r] + kw) < (unsigned)p.W;
                    const int at = in ? x_row[r] + ci : NOWHERE;
                    if constexpr (CONV == 4) {
                        A[slot][r][q >> 2][q & 3] = (int)__builtin_amdgcn_raw_buffer_load_b32(xrs, at, 0, 0);
                    } else if constexpr (CONV == 3) {
                        const auto v = __builtin_amdgcn_raw_buffer_load_b64(xrs, at, 0, 0);
                        A[slot][r][q >> 1][2 * (q & 1)] = (int)v[0];
                        A[slot][r][q >> 1][2 * (q & 1) + 1] = (int)v[1];
                    } else {
#pragma unroll
                        for (int hf = q; hf < q + 2 / RUNS; ++hf) {
                            const auto v = __builtin_amdgcn_raw_buffer_load_b128(xrs, at + 16 * (hf - q), 0, 0);
                            A[slot][r][hf] = e_v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
                        }
                    }
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                const int at = real && x_row[r] != NOWHERE ? x_row[r] + k0 : NOWHERE;
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(xrs, at + 16 * hf, 0, 0);
                    A[slot][r][hf] = e_v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);         // requests stay in order: the waits count them
    };

    // The first waves finish the tile: NC / 4 lanes a row, a lane four channels.  Their constants and residual codes are
    // buffer accesses that are out of range where there is nothing (no bias: a range of zero), so no branch joins in
    // between the requests and the waits that count them.
    const int rows = M - m0 < BM ? M - m0 : BM;
    const int orow = tid / (NC / 4), cq = tid & (NC / 4 - 1), n = nb * NC + 4 * cq;
    constexpr int QUADS = BM * NC / 4, THREADS = 64 * NWS;
    constexpr int QPT = QUADS > THREADS ? QUADS / THREADS : 1, ROW_STEP = THREADS / (NC / 4);   // a lane's rows
    e_v4f cs, cb;
    int cr[QPT];
    auto request_cols = [&]() {
        const __amdgpu_buffer_rsrc_t srs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.scale), 0, p.N * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.bias), 0, p.bias ? p.N * 4 : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t rrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(p.resid + (int64_t)m0 * p.N), 0,
                                                                             p.resid ? rows * p.N : 0, 0x00020000);
        const bool live = orow < rows;
        const auto s4 = __builtin_amdgcn_raw_buffer_load_b128(srs, live ? 4 * n : NOWHERE, 0, 0);
        const auto b4 = __builtin_amdgcn_raw_buffer_load_b128(brs, live ? 4 * n : NOWHERE, 0, 0);
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            const int r = orow + i * ROW_STEP;
            cr[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(rrs, r < rows && n < p.N ? r * p.N + n : NOWHERE, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            cs[i] = __uint_as_float(s4[i]);
            cb[i] = __uint_as_float(b4[i]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    using acc_t = std::conditional_t<NC == 32, e_v16i, e_v4i>;
    acc_t acc[RG];
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
        for (int i = 0; i < 4 * NQ; ++i) acc[r][i] = 0;
    auto multiply = [&](int d) {
        uint32_t D[8];
        HighCodec<H>::decode(P[d], D);
        LP::apply(Q[d], D);
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const e_v4i w = e_v4i{(int)D[4 * hf], (int)D[4 * hf + 1], (int)D[4 * hf + 2], (int)D[4 * hf + 3]};
                if constexpr (NC == 32) acc[r] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, A[d][r][hf], acc[r], 0, 0, 0);
                else acc[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, A[d][r][hf], acc[r], 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);         // no decoding ahead: it would take the registers of the requests
    };

    // Up to PD units per wave are straight-line code: everything is requested at once, every wait is an exact count, and
    // nothing is requested or decoded that does not exist.  Longer ones are a loop of whole
    // rounds: in a straight line per count the later requests ended up right before their use.
    const int units = ((p.KB + SPU - 1) / SPU - wave + NWS - 1) / NWS;
    auto few = [&](auto count) {
#pragma unroll
        for (int d = 0; d < decltype(count)::value; ++d) request(d, wave + NWS * d);
        request_cols();
#pragma unroll
        for (int d = 0; d < decltype(count)::value; ++d) multiply(d);
    };
    if (units <= 0) request_cols();
    else if (units == 1) few(std::integral_constant<int, 1>{});
    else if (units == 2) few(std::integral_constant<int, 2>{});
    else if (PD > 2 && units == 3) few(std::integral_constant<int, PD < 3 ? PD : 3>{});
    else {
#pragma unroll
        for (int d = 0; d < PD; ++d) request(d, wave + NWS * d);
        request_cols();
        int j0 = PD;
        for (; j0 < units; j0 += PD) {
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                multiply(d);
                request(d, wave + NWS * (j0 + d));
            }
        }
        const int left = units - j0 + PD;          // of the last round; what it requested beyond was out of range
#pragma unroll
        for (int d = 0; d < PD; ++d)
            if (d < left) multiply(d);
    }

    // ---- add the partial sums of the waves.  The place of a lane's sixteen bytes is turned by a multiple of the number of
    // its run of four channels, so that the lanes that read one row's runs find them on different banks -----------------
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            red[wave][r * NQ + q][lane ^ (NC == 32 ? 2 * (q + 4 * g) : 4 * (lane >> 4))] =
                e_v4i{acc[r][4 * q], acc[r][4 * q + 1], acc[r][4 * q + 2], acc[r][4 * q + 3]};
    __syncthreads();
    if (n >= p.N) return;

    // ---- epilogue (Eq. 2 / Eq. 8) -----------------------------------------------------------------------------
    const float lo = p.relu ? 0.0f : -__builtin_inff();
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
        const int row = orow + j * ROW_STEP;
        if (row >= rows) return;
        const int rr = row / NC, rl = row & (NC - 1);
        const int part = NC == 32 ? rr * NQ + (cq & 3) : rr;
        const int at = NC == 32 ? (rl + 32 * (cq >> 2)) ^ (2 * cq) : (rl + 16 * cq) ^ (4 * cq);
        e_v4i sum = e_v4i{0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < NWS; ++w) sum += red[w][part][at];
        const int64_t o = (int64_t)(m0 + row) * p.N + n;
        float y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float c = p.act_scale * cs[i];
            if (FULL == 0) c = c * p.part_mul;
            y[i] = (float)(sum[i] >> SHIFT) * c;
            y[i] = y[i] + cb[i];
        }
        if (p.out_int8) {
            if (p.resid) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float rv = p.resid_scale * (float)(int)(int8_t)((unsigned)cr[j] >> (8 * i));
                    y[i] = y[i] + rv;
                }
            }
            *reinterpret_cast<int *>(reinterpret_cast<int8_t *>(p.y) + o) = epi_codes4(p, y);
        } else {
            float *yf = reinterpret_cast<float *>(p.y) + o;
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = fmaxf(y[i], lo);
            if ((reinterpret_cast<uintptr_t>(p.y) & 15u) == 0 && (p.N & 3) == 0) {
                *reinterpret_cast<e_v4f *>(yf) = e_v4f{y[0], y[1], y[2], y[3]};
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n + i < p.N) yf[i] = y[i];
            }
        }
    }
}

// Defined here, instantiated once per (h, l) by nq_gemm_slab.hip.  The caller has checked the shape (slab_ok in
// nq_gemm.hip) and that the problem takes a vector epilogue.
template <int H, int L>
void launch_nested_gemm_slab(bool full, const GemmParams &p, int x_bytes, hipStream_t st, void *ev_start, void *ev_stop)
{
    const bool conv = p.KH != 1 || p.KW != 1 || p.stride != 1 || p.pad != 0;
    const unsigned cin_magic = (unsigned)(((uint64_t(1) << 32) + p.Cin - 1) / p.Cin);
    const int64_t row_tiles = (p.M + 31) / 32, blocks = row_tiles * p.NB;
    const int units = (p.KB + 3) / 4;              // K steps of a wave of a 32-column block
    // Columns of 16 while they find idle compute units: twice the blocks, half the weights each (us, 32 columns against 16: 14 x
    // 14 x 256 -> 256 3x3 5.4, 5.2; 7 x 7 x 512 -> 512 3x3 7.9, 7.2; 256 x 8192 -> 256 12.6, 11.2; with 112 blocks 5.8 and 5.7,
    // with 168 6.3 and 9.2; with 128 blocks K = 1024 3.7 and 3.8, K = 4096 8.5 and 7.6).  Not for gathers in smaller steps than 32
    // channels, whose requests each block makes again: 0.98, 0.94 and 0.89 times as fast in steps of 16, 8 and 4 (1,100 drawn shapes).
    const bool narrow = blocks <= 112 || (blocks <= 128 && p.K >= 2048);
    // Two row tiles per block, which decode the weights once for both, where that halves the blocks of the busiest unit exactly and rows are
    // long: 1.07 to 1.14 times as fast as one on 2,000 drawn shapes (32 x 7 x 7 x 512 -> 512 3x3 23.1, 20.4; 1000 x 1024 -> 1024 8.5, 8.0;
    // 800 x 4096 -> 1024 22.9, 20.6), where it does not 0.87 to 0.97 (4003 x 4856 -> 168 24.6, 27.5; 700 blocks take three rounds of
    // units, half as many blocks two of twice the length).  A last block with one row tile is no loss from sixteen row tiles on (197 x
    // 1024 -> 4096, seven of them, 7.5, 7.7).  The gathers in steps of 8 and 4 channels are 0.73 to 0.98 times as fast with two, that in
    // steps of 16 is from K = 2048 on (0.91; below 1.05), and over rows beyond 8192 so is the filter's (0.94).
    const int64_t per_unit = (blocks + 255) / 256, per_unit_two = ((row_tiles + 1) / 2 * p.NB + 255) / 256;
    const bool halves = blocks > 640 && p.K >= 1024 && (row_tiles % 2 == 0 || row_tiles >= 16) &&
                        (2 * per_unit_two <= per_unit || per_unit > 8);
    // Three or four units in flight per wave, whichever leaves whole rounds (K = 1024: 8.6 with three, 7.5 with four; K = 1536:
    // 8.7 and 9.5: more registers, fewer blocks on a unit).
    const bool three = units % 3 == 0 || units < 3;
#define NQ_SL_ONE(FULLV, NCV, RGV, PDV, CONVV)                                                                          \
    launch_timed(k_nested_gemm_slab<H, L, FULLV, NCV, RGV, PDV, CONVV>,                                             \
                 dim3((unsigned)((p.N + NCV - 1) / NCV), (unsigned)((p.M + NCV * RGV - 1) / (NCV * RGV))), dim3(256), 0, st, \
                 ev_start, ev_stop, p, x_bytes, cin_magic)
#define NQ_SL_LAUNCH(FULLV, CONVV)                           \
    do {                                                     \
        if constexpr (CONVV <= 1) {                          \
            if (narrow) {                                    \
                NQ_SL_ONE(FULLV, 16, 2, 3, CONVV);           \
                break;                                       \
            }                                                \
        }                                                    \
        if constexpr (CONVV <= 2) {                          \
            if (halves && p.K < (CONVV == 0 ? 0x7fffffff : CONVV == 1 ? 8192 : 2048)) { \
                NQ_SL_ONE(FULLV, 32, 2, 2, CONVV);           \
                break;                                       \
            }                                                \
        }                                                    \
        if (three) NQ_SL_ONE(FULLV, 32, 1, 3, CONVV);        \
        else NQ_SL_ONE(FULLV, 32, 1, 4, CONVV);              \
    } while (0)
#define NQ_SL_MODES(FULLV)                       \
    do {                                         \
        if (!conv) NQ_SL_LAUNCH(FULLV, 0);       \
        else if (p.Cin % 32 == 0 || p.Cin == p.K) NQ_SL_LAUNCH(FULLV, 1); \
        else if (p.Cin % 16 == 0) NQ_SL_LAUNCH(FULLV, 2); \
        else if (p.Cin % 8 == 0) NQ_SL_LAUNCH(FULLV, 3); \
        else NQ_SL_LAUNCH(FULLV, 4);             \
    } while (0)
    if (full && p.low_signed) NQ_SL_MODES(2); else if (full) NQ_SL_MODES(1); else NQ_SL_MODES(0);
}

}  // namespace nq
