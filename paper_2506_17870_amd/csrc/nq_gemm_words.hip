// Launcher of the GEMM over the paper's word pages (nq_gemm_words.h); one translation unit per nesting (-DNQ_INST_H=<h>
// -DNQ_INST_L=<l>).
#include "nq_gemm_words.h"

namespace nq {

template <typename K>
static void words_grant_lds(K kernel, size_t lds)
{
    static bool granted = false;   // one per kernel instantiation
    if (!granted && lds > 64 * 1024) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        granted = true;
    }
}

template <int HB, int LB, int MODE, int NW, int RT, int CS, int CONV, int EPI>
static void launch_words_as(const GemmParams &p, int WH, int WL, hipStream_t st, void *ev_start, void *ev_stop)
{
    auto k = k_nested_gemm_words<HB, LB, MODE, NW, RT, CS, CONV, EPI>;
    constexpr size_t lds = words_lds_bytes<HB, MODE == 0 ? 0 : LB, NW, RT, CS>();
    words_grant_lds(k, lds);
    launch_timed(k, dim3((unsigned)p.NB, (unsigned)((p.M + 32 * RT - 1) / (32 * RT))), dim3(64 * NW), lds, st, ev_start, ev_stop, p,
                 WH, WL);
}

template <int HB, int LB, int MODE>
static void launch_words(const GemmParams &p, int WH, int WL, int *row_tiles_of_a_block, hipStream_t st, void *ev_start, void *ev_stop)
{
    const int64_t blocks = (int64_t)p.NB * ((p.M + 31) / 32);
    // Eight waves share a page's steps where there is at most a block per unit (16 x 8192 -> 8192 30.7 us, with four 42.5; 32 x
    // 1574 -> 5510 9.9, 11.2; with 246 blocks and K = 570 5.4, 5.2; K = 300 5.7, 5.4; with 484 blocks 28.7, 26.3).
    const bool wide = blocks <= 256 && p.K >= 400;
    // Two row tiles share the decoding of both pages of long rows: a unit's block of them takes 1.7 times as long as one of four waves and
    // one row tile (full-bit, 9,200 drawn shapes), so they pay where they halve the number of blocks per unit, exactly: not with a
    // single row tile, whose partner is empty, and not with an odd number that leaves a block over (one row tile, then two, us: 700 x
    // 4000 -> 700 26.3, 21.4; 186 x 5292 -> 4643 55.6, 49.8; but 4 x 5813 -> 36206 86.8, 144.0; 81 x 7781 -> 5236 66.8, 79.0; the higher-bit page
    // alone 276 x 2220 -> 3295 18.1, 21.6).  Above four blocks per unit it takes rows of 4000 (two tiles 0.98 of the time at 2000).
    const int64_t row_tiles = (p.M + 31) / 32;
    const int64_t per_unit = (blocks + 255) / 256, per_unit_two = ((row_tiles + 1) / 2 * p.NB + 255) / 256;
    const bool tall = MODE != 0 && 2 * per_unit_two <= per_unit && p.K >= (per_unit <= 4 ? 2000 : 4000);
#define NQ_WD(NW, RT, CS)                                                                                     \
    do {                                                                                                      \
        if (epi_mode(p) == EPI_F32) launch_words_as<HB, LB, MODE, NW, RT, CS, 0, EPI_F32>(p, WH, WL, st, ev_start, ev_stop); \
        else launch_words_as<HB, LB, MODE, NW, RT, CS, 0, EPI_ANY>(p, WH, WL, st, ev_start, ev_stop);     \
    } while (0)
    const bool gather = p.KH != 1 || p.KW != 1 || p.stride != 1 || p.pad != 0;
    if (!gather) {
        if (wide) {
            NQ_WD(8, 1, 4);
            return;
        }
        if constexpr (MODE != 0) {
            if (tall) {
                *row_tiles_of_a_block = 2;
                NQ_WD(8, 2, 2);
                return;
            }
        }
        NQ_WD(4, 1, 4);
        return;
    }
#undef NQ_WD
    // a filter other than 1x1 stride 1 gathers its rows from the NHWC input (four waves, chunks of eight steps: a gather pays for
    // itself over longer runs, 56 x 56 x 64 3x3 16.3 us, with four steps 18.6).  Whole-row epilogues as for a GEMM: the element-wise
    // one's sixteen branches a lane are a third of a small layer (13 x 13 x 20 -> 352 3x3, INT(8|5), fp32: the higher-bit page 10.6 us
    // with it and 7.0, both pages 14.5 and 11.0).
#define NQ_WD_CONV(CONV)                                                                                      \
    do {                                                                                                      \
        const int mode = epi_mode(p);                                                                         \
        if (mode == EPI_F32) launch_words_as<HB, LB, MODE, 4, 1, 8, CONV, EPI_F32>(p, WH, WL, st, ev_start, ev_stop); \
        else if (mode == EPI_I8) launch_words_as<HB, LB, MODE, 4, 1, 8, CONV, EPI_I8>(p, WH, WL, st, ev_start, ev_stop); \
        else launch_words_as<HB, LB, MODE, 4, 1, 8, CONV, EPI_ANY>(p, WH, WL, st, ev_start, ev_stop);         \
    } while (0)
    if (p.Cin % 16 == 0) NQ_WD_CONV(2);
    else NQ_WD_CONV(1);
#undef NQ_WD_CONV
}

template <int H, int L>
void launch_nested_gemm_words(bool full, const GemmParams &p, int WH, int WL, int *row_tiles, hipStream_t st, void *ev_start, void *ev_stop)
{
    *row_tiles = 1;
    if (!full) launch_words<H, L, 0>(p, WH, WL, row_tiles, st, ev_start, ev_stop);
    else if (p.low_signed) launch_words<H, L + 1, 2>(p, WH, WL, row_tiles, st, ev_start, ev_stop);
    else launch_words<H, L, 1>(p, WH, WL, row_tiles, st, ev_start, ev_stop);
}
template void launch_nested_gemm_words<NQ_INST_H, NQ_INST_L>(bool, const GemmParams &, int, int, int *, hipStream_t, void *, void *);

}  // namespace nq
