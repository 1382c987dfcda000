"""GPU parity, against the CPU oracle, of the kernels and dispatch branches for layers between the large tiles: outputs
too small to fill the chip (32 x 32 blocks, the reduction split over the waves), short reductions that are no power of
two, activations in steps of eight channels, groups of up to 32 channels, and the one-launch quantiser + packer.  Integer
sums in a fixed fp32 epilogue: everything is compared for equality."""
import numpy as np
import pytest
import torch

import nq_testlib as tl
from nq_testlib import Case, check_outputs, dev, epi_pair, host, run_gconv_both, set_choice
from oracle import nq_oracle as oracle
from paper_2506_17870_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nq():
    import paper_2506_17870_amd as nq
    assert torch.cuda.is_available()
    return nq


def make_case(nq, N, K, n, l, seed, compensated=False):
    w_int, scale = tl.weights(N, K, inputs.he_sigma(K), n, seed)
    c = Case(nq, w_int, scale, n, l)
    if compensated:
        c.cfg = nq.make_cfg(n, l, nq.NQ_LOW_SIGNED_L1)
        c.W = nq.NestedWeight.from_int8(dev(w_int), dev(scale), c.cfg)
        c.ow_part = oracle.decompose(w_int, n, l, "rtn")[0].astype(np.int16)
        c.ow_full = w_int.astype(np.int16)
    return c


def forced(nq, case, x, shape, choice, family=None):
    """A GEMM (x [M, K], shape None) or a convolution with one kernel forced: fp32 with bias, int8 with and without a
    residual where 16-channel stores apply, full-bit and part-bit."""
    conv = shape is not None
    if conv:
        B, H, W, Cin = x.shape
        KH, KW, stride, pad = shape
        Ho, Wo = oracle.conv_out_hw(H, W, KH, KW, stride, pad)
        lead = (B, Ho, Wo)
        cs = nq.nq_conv_shape(B, H, W, Cin, case.N, KH, KW, stride, pad)
    else:
        lead = (x.shape[0],)
    dx, N = dev(x), case.N
    bias = inputs.small_floats(N, 0.2, seed=N)
    res = inputs.uniform_activations(lead + (N,), seed=N + 1)
    runs = [dict(s_a=0.02, bias=bias)]
    if N % 16 == 0:
        runs += [dict(s_a=0.02, out_int8=True, inv_s_out=4.0),
                 dict(s_a=0.02, bias=bias, residual=res, s_r=0.05, relu=True, out_int8=True, inv_s_out=4.0)]
    for full in (True, False):
        w = case.ow_full if full else case.ow_part
        acc = oracle.conv_acc(x, w.reshape(N, KH, KW, Cin), stride, pad) if conv else oracle.gemm_acc(x, w)
        for kw in runs:
            epi, keep, okw = epi_pair(nq, case, full, lead, dump=False, **kw)
            i8 = kw.get("out_int8", False)
            y = torch.full(lead + (N,), 77, dtype=torch.int8 if i8 else torch.float32, device="cuda")
            set_choice(choice)
            try:
                if conv:
                    (nq.nq_conv_full if full else nq.nq_conv_part)(dx, cs, case.W.desc, epi, y)
                else:
                    (nq.nq_gemm_full if full else nq.nq_gemm_part)(dx, x.shape[0], case.W.desc, epi, y)
            finally:
                set_choice("")
            torch.cuda.synchronize()
            if family is not None:
                assert nq.nq_profile_last_kernel()[0] == family
            check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, i8)


# ---- small outputs: 32 x 32 blocks ------------------------------------------------------------------------------
@pytest.mark.parametrize("M,N,K", [(1, 1, 4), (33, 40, 60), (32, 32, 64), (31, 48, 68), (197, 96, 1000), (65, 80, 768),
                                   (64, 2048, 2052), (300, 16, 4096), (5, 31, 8192)])
def test_small_outputs_gemm(nq, M, N, K):
    # rows and columns off the tile, K steps fewer than waves, ends of K inside a lane's 32 bytes, eight and four waves
    forced(nq, make_case(nq, N, K, 8, 2, seed=M + N + K), inputs.uniform_activations((M, K), seed=K), None, "11", 11)


@pytest.mark.parametrize("B,H,W,Cin,N,k,stride,pad", [
    (1, 7, 7, 512, 64, 3, 1, 1), (2, 5, 6, 32, 48, 3, 1, 1), (1, 9, 8, 96, 33, 3, 2, 1), (1, 8, 8, 64, 32, 5, 1, 2),
    (3, 6, 5, 128, 64, 1, 2, 0), (1, 5, 5, 36, 32, 1, 2, 0), (1, 4, 4, 64, 32, 1, 1, 1), (1, 3, 3, 32, 16, 3, 1, 0)])
def test_small_outputs_filters(nq, B, H, W, Cin, N, k, stride, pad):
    forced(nq, make_case(nq, N, k * k * Cin, 8, 3, seed=Cin + N + k), inputs.uniform_activations((B, H, W, Cin), seed=H),
           (k, k, stride, pad), "11", 11)


@pytest.mark.parametrize("n,l", [(8, l) for l in range(1, 7)] + [(6, l) for l in range(1, 5)])
@pytest.mark.parametrize("compensated", [False, True])
def test_small_outputs_every_nesting(nq, n, l, compensated):
    x = inputs.uniform_activations((70, 1152), seed=l) >> (8 - n)
    forced(nq, make_case(nq, 48, 1152, n, l, seed=n + l, compensated=compensated), x, None, "11", 11)
    x = inputs.uniform_activations((1, 6, 6, 64), seed=l) >> (8 - n)
    forced(nq, make_case(nq, 48, 576, n, l, seed=n * l, compensated=compensated), x, (3, 3, 1, 1), "11", 11)


@pytest.mark.parametrize("M,N,K", [
    (200, 600, 64), (199, 604, 260), (197, 592, 580), (193, 608, 1020),      # 32 columns: one to four units per wave, waves with none
    (200, 600, 1100), (224, 592, 1536), (200, 596, 1796),                    # rounds of three and four, a last one of one to four
    (113, 1024, 2048), (2047, 352, 1024), (2048, 340, 1284), (2033, 352, 1540),   # 16 columns of 128 blocks; two row tiles
    (1544, 512, 1028), (480, 1440, 1300), (4003, 168, 1200)])                # ... the last block's second one empty; blocks that do not halve
def test_small_outputs_every_block_form(nq, M, N, K):
    forced(nq, make_case(nq, N, K, 8, 2, seed=M + K), inputs.uniform_activations((M, K), seed=K), None, "11", 11)


@pytest.mark.parametrize("B,H,W,Cin,N,k,stride,pad,comp", [
    (2, 11, 10, 64, 600, 3, 1, 1, False), (5, 9, 9, 160, 320, 3, 2, 0, True), (8, 16, 16, 128, 352, 3, 1, 1, True)])
def test_small_outputs_every_block_form_filters(nq, B, H, W, Cin, N, k, stride, pad, comp):
    forced(nq, make_case(nq, N, k * k * Cin, 8, 3, seed=Cin + N, compensated=comp), inputs.uniform_activations((B, H, W, Cin), seed=H),
           (k, k, stride, pad), "11", 11)


@pytest.mark.parametrize("M,N,K,kernel", [
    (1, 64, 256, (11, 0)), (16, 4128, 4096, (11, 0)), (17, 4128, 4096, (6, 0)), (17, 4096, 4096, (11, 0)), (17, 4128, 4080, (11, 0)),
    (300, 1040, 768, (11, 0)), (1040, 1024, 1024, (4, 2)), (700, 512, 256, (11, 0)), (2080, 1024, 256, (9, 4)), (640, 128, 1024, (11, 0)),
    (5152, 128, 1024, (4, 7)), (1400, 1008, 120, (11, 0)), (3104, 1024, 120, (1, 1))])
def test_small_outputs_or_the_kernel_they_replace(nq, M, N, K, kernel):
    # either side of the limits against the kernels for few rows, large tiles, stationary weights and the generic one
    case = make_case(nq, N, K, 8, 2, seed=M + K)
    x = inputs.uniform_activations((M, K), seed=K)
    epi, _, okw = epi_pair(nq, case, True, (M,), dump=False, s_a=0.02, out_int8=True, inv_s_out=4.0)
    y = torch.full((M, N), 77, dtype=torch.int8, device="cuda")
    nq.nq_gemm_full(dev(x), M, case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel() == kernel
    acc = oracle.gemm_acc(x, case.ow_full)
    check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, True)


def test_small_outputs_by_the_library(nq):
    """The dispatch itself takes these to the small-output kernel, and to it alone."""
    forced(nq, make_case(nq, 768, 3072, 8, 3, seed=1), inputs.uniform_activations((197, 3072), seed=1), None, "", 11)
    forced(nq, make_case(nq, 256, 2304, 8, 2, seed=2), inputs.uniform_activations((1, 14, 14, 256), seed=2), (3, 3, 1, 1), "", 11)


@pytest.mark.parametrize("M,N,K,i8,family", [
    # what no other kernel wants: small blocks up to the number at which the generic kernel takes as long, per length of K
    (8192, 64, 48, True, 11), (8224, 64, 48, True, 1), (3136, 256, 32, False, 1), (16384, 32, 96, False, 11),
    (12256, 64, 144, True, 11), (12320, 64, 144, True, 1), (29008, 32, 192, True, 1),
    (16384, 64, 320, True, 11), (16416, 64, 320, False, 1), (20480, 64, 520, False, 11),
    (20512, 64, 520, False, 1), (32768, 64, 776, True, 11), (32800, 64, 776, True, 1),
    # fp32 columns of one 128-wide block of the stationary kernel: one block per unit
    (2048, 128, 128, False, 11), (2080, 128, 128, False, 9), (2080, 128, 128, True, 11), (2080, 132, 128, False, 11),
    # up to 64 rows, whatever the length of the reduction; the kernel for few rows has wide layers over long rows
    (33, 256, 704, False, 11), (33, 256, 720, False, 11), (64, 96, 1024, True, 11), (40, 96, 1040, False, 11), (32, 96, 512, False, 11),
    (33, 12320, 2064, True, 6), (33, 12288, 2064, True, 11),
    # fp32 rows that leave element by element: the stationary kernel and, for short rows, the generic one sooner
    (1280, 1021, 128, False, 11), (1312, 1021, 128, False, 9), (1312, 1024, 128, False, 11), (2560, 1021, 72, False, 11), (2592, 1021, 72, False, 1),
    (2592, 1024, 72, False, 11),
    # the large kernel sooner where the activations are more than the caches hold, from K = 1280 on, and for its narrow tiles
    (4400, 192, 2048, True, 4), (4400, 192, 1792, True, 11), (4064, 192, 2080, True, 11), (4352, 112, 2048, True, 4), (4080, 112, 2080, True, 11),
    (4352, 112, 1920, True, 11), (1280, 1024, 512, True, 11), (1312, 1024, 512, True, 4), (1728, 1024, 320, True, 11), (1824, 1024, 320, True, 4)])
def test_small_outputs_where_they_are_the_faster_kernel(nq, M, N, K, i8, family):
    case = make_case(nq, N, K, 8, 2, seed=M + K)
    x = inputs.uniform_activations((M, K), seed=K)
    epi, _, okw = epi_pair(nq, case, True, (M,), dump=False, s_a=0.02, out_int8=i8, inv_s_out=4.0)
    y = torch.full((M, N), 77, dtype=torch.int8 if i8 else torch.float32, device="cuda")
    nq.nq_gemm_full(dev(x), M, case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    acc = oracle.gemm_acc(x, case.ow_full)
    check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, i8)


@pytest.mark.parametrize("B,H,Cin,k,N,int8,family", [
    (1, 8, 64, 3, 460, False, 3), (1, 16, 64, 3, 96, True, 3), (1, 17, 64, 3, 96, False, 11),     # few pixels
    (1, 8, 64, 2, 96, False, 11), (1, 18, 128, 2, 96, True, 11), (1, 17, 128, 2, 32, True, 3),    # 17 x 17 and 16 x 16 outputs
    (4, 33, 128, 2, 64, True, 11), (5, 33, 128, 2, 64, True, 3), (5, 33, 64, 2, 64, False, 3)])   # one block per unit
def test_small_outputs_or_stationary_rows(nq, B, H, Cin, k, N, int8, family):
    pad = k // 2 if k == 3 else 0
    ho = H + 2 * pad - k + 1
    x = inputs.uniform_activations((B, H, H, Cin), seed=N)
    case = make_case(nq, N, k * k * Cin, 8, 2, seed=H)
    epi, _, okw = epi_pair(nq, case, True, (B, ho, ho), dump=False, s_a=0.02, out_int8=int8, inv_s_out=4.0)
    y = torch.full((B, ho, ho, N), 77, dtype=torch.int8 if int8 else torch.float32, device="cuda")
    nq.nq_conv_full(dev(x), nq.nq_conv_shape(B, H, H, Cin, N, k, k, 1, pad), case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    acc = oracle.conv_acc(x, case.ow_full.reshape(N, k, k, Cin), 1, pad)
    check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, int8)


@pytest.mark.parametrize("k,stride,pad,Cin,N,int8,family", [(2, 1, 0, 32, 96, False, 11), (1, 1, 1, 128, 96, False, 11), (1, 2, 1, 128, 72, False, 11),
                                                            (1, 1, 0, 128, 96, False, 9), (1, 1, 0, 128, 96, True, 11)])
def test_small_outputs_at_128_long_reductions(nq, k, stride, pad, Cin, N, int8, family):
    # the stationary kernel's limit for one block of columns is for what it can take: neither filters nor padding
    H = 32 if stride == 1 else 66
    x = inputs.uniform_activations((8, H, H, Cin), seed=N)
    case = make_case(nq, N, k * k * Cin, 8, 2, seed=N + k)
    lead = (8,) + oracle.conv_out_hw(H, H, k, k, stride, pad)
    epi, _, okw = epi_pair(nq, case, True, lead, dump=False, s_a=0.02, out_int8=int8, inv_s_out=4.0)
    y = torch.full(lead + (N,), 77, dtype=torch.int8 if int8 else torch.float32, device="cuda")
    nq.nq_conv_full(dev(x), nq.nq_conv_shape(8, H, H, Cin, N, k, k, stride, pad), case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    acc = oracle.conv_acc(x, case.ow_full.reshape(N, k, k, Cin), stride, pad)
    check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, int8)


# ---- short reductions in steps of 16, activations in steps of 8 ------------------------------------------------
@pytest.mark.parametrize("M,N,K", [(100, 64, 16), (333, 96, 32), (333, 144, 48), (4097, 192, 96), (129, 272, 144),
                                   (700, 64, 192), (257, 40, 240)])
def test_stationary_weights_any_short_reduction(nq, M, N, K):
    for n, l, comp in ((8, 2, False), (6, 3, False), (8, 5, True)):
        x = inputs.uniform_activations((M, K), seed=K) >> (8 - n)
        forced(nq, make_case(nq, N, K, n, l, seed=M + K + l, compensated=comp), x, None, "9", 9)


def test_stationary_weights_strided_short_reduction(nq):
    x = inputs.uniform_activations((3, 13, 11, 48), seed=3)
    forced(nq, make_case(nq, 96, 48, 8, 3, seed=3), x, (1, 1, 2, 0), "9", 9)


@pytest.mark.parametrize("M,N,K,family", [(40000, 80, 48, 9), (39999, 80, 48, 1), (40000, 72, 48, 1), (90000, 80, 144, 1),
                                          (100000, 80, 144, 9), (40000, 72, 64, 9)])
def test_stationary_weights_by_the_library(nq, M, N, K, family):
    # lengths that are no power of two: many rows, more of them above K = 128, and sixteen channels per store
    case = make_case(nq, N, K, 8, 2, seed=K)
    x = inputs.uniform_activations((M, K), seed=N)
    epi, _, okw = epi_pair(nq, case, True, (M,), dump=False, s_a=0.02, out_int8=True, inv_s_out=4.0)
    y = torch.full((M, N), 77, dtype=torch.int8, device="cuda")
    nq.nq_gemm_full(dev(x), M, case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    acc = oracle.gemm_acc(x, case.ow_full)
    check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, True)


@pytest.mark.parametrize("Cin,k,stride,pad", [(8, 3, 1, 1), (24, 3, 2, 1), (40, 1, 1, 0), (72, 5, 1, 2)])
def test_activations_in_steps_of_eight(nq, Cin, k, stride, pad):
    x = inputs.uniform_activations((2, 9, 10, Cin), seed=Cin)
    forced(nq, make_case(nq, 80, k * k * Cin, 8, 2, seed=Cin), x, (k, k, stride, pad), "1", 1)


# ---- the large kernel: channel counts and reductions that are no power of two --------------------------------------
@pytest.mark.parametrize("choice", ["4", "4/tm2", "4/tm3", "4/tm5", "4/tm6", "4/tm7"])
def test_large_kernel_any_multiple_of_sixteen(nq, choice):
    # K one piece past a panel, one piece short of one, shorter than one; rows off the tile
    for M, N, K in ((300, 320, 272), (130, 272, 1008), (333, 96, 48), (200, 528, 2032)):
        forced(nq, make_case(nq, N, K, 8, 2, seed=K), inputs.uniform_activations((M, K), seed=M), None, choice, 4)
    for B, H, W, Cin, N, k, stride, pad in ((2, 9, 8, 48, 144, 3, 1, 1), (1, 13, 11, 80, 272, 5, 2, 2), (3, 12, 9, 208, 96, 1, 2, 0),
                                            (2, 7, 7, 112, 320, 2, 1, 0)):
        forced(nq, make_case(nq, N, k * k * Cin, 8, 3, seed=Cin), inputs.uniform_activations((B, H, W, Cin), seed=H),
               (k, k, stride, pad), choice, 4)


@pytest.mark.parametrize("M,N,K,family", [
    (300, 130, 624, 1), (300, 130, 656, 4), (200, 258, 1008, 1), (200, 258, 1040, 4), (12416, 258, 1040, 1), (300, 500, 656, 4), (300, 450, 656, 1), (300, 470, 656, 4),
    (300, 130, 1024, 4)])
def test_large_kernel_with_ragged_outputs(nq, M, N, K, family):
    # the element-wise epilogue: long reductions, filled column tiles or few blocks; K = 1024 is the plain form
    case = make_case(nq, N, K, 8, 2, seed=K)
    x = inputs.uniform_activations((M, K), seed=M)
    epi, _, okw = epi_pair(nq, case, True, (M,), dump=False, s_a=0.02, out_int8=True, inv_s_out=4.0)
    y = torch.full((M, N), 77, dtype=torch.int8, device="cuda")
    nq.nq_gemm_full(dev(x), M, case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    acc = oracle.gemm_acc(x, case.ow_full)
    check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, True)


@pytest.mark.parametrize("M,N,K,family", [(8192, 400, 320, 4), (8320, 400, 320, 1), (16384, 400, 320, 1), (16512, 400, 320, 4),
                                          (8320, 400, 400, 4)])
def test_large_kernel_on_short_reductions(nq, M, N, K, family):
    # the generic kernel keeps what fills the units once with its 128 x 256 tiles
    case = make_case(nq, N, K, 8, 2, seed=K)
    x = inputs.uniform_activations((M, K), seed=M)
    epi, _, okw = epi_pair(nq, case, True, (M,), dump=False, s_a=0.02, out_int8=True, inv_s_out=4.0)
    y = torch.full((M, N), 77, dtype=torch.int8, device="cuda")
    nq.nq_gemm_full(dev(x), M, case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    acc = oracle.gemm_acc(x, case.ow_full)
    check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, True)


@pytest.mark.parametrize("Cin,family", [(192, 2), (320, 4), (384, 2), (448, 4), (176, 4)])
def test_large_kernel_or_windows_with_ragged_outputs(nq, Cin, family):
    x = inputs.uniform_activations((1, 12, 13, Cin), seed=Cin)
    case = make_case(nq, 72, 9 * Cin, 8, 2, seed=Cin)
    cs = nq.nq_conv_shape(1, 12, 13, Cin, 72, 3, 3, 1, 1)
    epi, _, okw = epi_pair(nq, case, True, (1, 12, 13), dump=False, s_a=0.02, out_int8=True, inv_s_out=4.0)
    y = torch.full((1, 12, 13, 72), 77, dtype=torch.int8, device="cuda")
    nq.nq_conv_full(dev(x), cs, case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    acc = oracle.conv_acc(x, case.ow_full.reshape(72, 3, 3, Cin), 1, 1)
    check_outputs(host(y), None, oracle.epilogue(acc, **okw), acc, True)


# ---- groups of up to 32 channels ------------------------------------------------------------------------------
@pytest.mark.parametrize("geom", [
    # B, H, W, Cin, Cout, groups, KH, stride, pad
    (1, 9, 9, 24, 24, 3, 3, 1, 1),        # 8 per group; a pixel's second piece reaches past its channels
    (2, 7, 6, 36, 36, 3, 3, 1, 1),        # 12 per group: half tiles of 24 channels, the last one of 12
    (1, 11, 9, 96, 96, 8, 3, 2, 1),       # 12 per group, two channel tiles, stride 2
    (1, 56, 33, 256, 256, 32, 3, 1, 1),   # patches of several tiles, ragged in both directions
    (2, 5, 5, 48, 48, 3, 3, 1, 1),        # 16 per group, the second half tile half empty
    (1, 8, 8, 96, 96, 3, 1, 1, 0),        # 32 per group, 1x1
    (1, 6, 7, 64, 16, 4, 2, 1, 0),        # 16 in, 4 out; 2x2
    (1, 6, 7, 16, 64, 4, 3, 1, 1),        # 4 in, 16 out
])
def test_groups_on_the_matrix_cores(nq, geom):
    B, H, W, Cin, Cout, groups, KH, stride, pad = geom
    K = KH * KH * (Cin // groups)
    Ho, Wo = (H + 2 * pad - KH) // stride + 1, (W + 2 * pad - KH) // stride + 1
    x = inputs.uniform_activations((B, H, W, Cin), seed=Cin + H)
    bias = inputs.small_floats(Cout, 0.1, seed=3)
    res = inputs.uniform_activations((B, Ho, Wo, Cout), seed=Cout)
    for n, l, comp in ((8, 2, False), (6, 3, True)):
        case = make_case(nq, Cout, K, n, l, seed=sum(geom) + l, compensated=comp)
        for full in (True, False):
            run_gconv_both(nq, case, x, (KH, KH, stride, pad), groups, full, s_a=0.02, bias=bias)
            run_gconv_both(nq, case, x, (KH, KH, stride, pad), groups, full, s_a=0.02, bias=bias, out_int8=True, inv_s_out=5.0)
            run_gconv_both(nq, case, x, (KH, KH, stride, pad), groups, full, s_a=0.02, bias=bias, residual=res, s_r=0.04,
                           relu=True, out_int8=True, inv_s_out=5.0)
    assert nq.nq_profile_last_kernel() == (10, 2)


# ---- quantise and pack in one launch ----------------------------------------------------------------------------
@pytest.mark.parametrize("N,K", [(1, 4), (8, 60), (31, 64), (33, 68), (65, 1024), (40, 1028), (9, 2048), (32, 2052), (7, 4096),
                                 (7, 4100), (5, 63)])
def test_quantise_and_pack_one_launch(nq, N, K):
    w = inputs.float_weights(N, K, 0.02, seed=N + K)
    w[0] = 0.0                            # an all-zero channel: scale 1
    if N > 4:
        w[3, K // 2] = 3.0e38             # one value decides the scale, the others become zero
    for n, l, signed in ((8, 2, False), (8, 3, True), (6, 1, False)):
        wi, s = oracle.quantize(w, n)
        hi, res = oracle.decompose(wi, n, l, "rtn") if signed else (None, None)
        if signed:
            ph_ref = oracle.pack_dense(hi, n - l, oracle.KIND_CARRIER)
            pl_ref = oracle.pack_dense(oracle.low_encode(res, l, oracle.LOW_SIGNED_L1), l + 1, oracle.KIND_BITSTRING)
        else:
            ph_ref, pl_ref = oracle.decompose_pack(wi, n, l)
        cfg = nq.make_cfg(n, l, nq.NQ_LOW_SIGNED_L1 if signed else nq.NQ_LOW_UNSIGNED_L)
        ph = torch.full((ph_ref.size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        pl = torch.full((pl_ref.size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        sc = torch.zeros(N + 1, dtype=torch.float32, device="cuda")
        nq.nq_quantize_decompose_pack(dev(w), N, K, cfg, sc, ph, pl)
        torch.cuda.synchronize()
        assert np.array_equal(host(sc)[:N].view(np.uint32), s.view(np.uint32)) and host(sc)[N] == 0.0
        assert np.array_equal(host(ph)[:ph_ref.size], ph_ref) and np.all(host(ph)[ph_ref.size:] == 0xA5)
        assert np.array_equal(host(pl)[:pl_ref.size], pl_ref) and np.all(host(pl)[pl_ref.size:] == 0xA5)


@pytest.mark.parametrize("N,K", [(33, 512), (263, 516), (300, 1024), (290, 2044), (513, 256), (34, 3076), (257, 4096)])
@pytest.mark.parametrize("n,l", [(8, 2), (8, 5), (6, 1)])
def test_quantise_and_pack_near_ties(nq, N, K, n, l):
    # Values at a half step and up to 40 units in the last place either side, for steps that are and are not powers of two: where the
    # product with the reciprocal cannot decide, the quotient must.  More than eight tiles of rows, rows off the tile.
    rng = np.random.default_rng(N + K + n)
    qmax = 127 if n == 8 else 31
    step = np.where(rng.random(N) < 0.5, 0.25, rng.uniform(1e-3, 2.0, N)).astype(np.float32)
    w = ((rng.integers(-qmax, qmax, (N, K)) + 0.5).astype(np.float32) * step[:, None])
    w = (w.view(np.int32) + rng.integers(-40, 41, (N, K))).astype(np.int32).view(np.float32)
    w[:, 0] = step * qmax
    wi, s = oracle.quantize(w, n)
    ph_ref, pl_ref = oracle.decompose_pack(wi, n, l)
    ph = torch.full((ph_ref.size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    pl = torch.full((pl_ref.size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    sc = torch.zeros(N + 1, dtype=torch.float32, device="cuda")
    nq.nq_quantize_decompose_pack(dev(w), N, K, nq.make_cfg(n, l), sc, ph, pl)
    torch.cuda.synchronize()
    assert np.array_equal(host(sc)[:N].view(np.uint32), s.view(np.uint32)) and host(sc)[N] == 0.0
    assert np.array_equal(host(ph)[:ph_ref.size], ph_ref) and np.all(host(ph)[ph_ref.size:] == 0xA5)
    assert np.array_equal(host(pl)[:pl_ref.size], pl_ref) and np.all(host(pl)[pl_ref.size:] == 0xA5)


# ---- the stem of a CNN and its last pool on few images --------------------------------------------------------------
@pytest.mark.parametrize("B,H,W,Cin,N,k,stride,pad", [(1, 56, 60, 3, 64, 7, 2, 3), (2, 40, 200, 1, 80, 3, 1, 1), (1, 33, 36, 8, 40, 3, 1, 0),
                                                     (3, 19, 12, 4, 33, 7, 1, 3), (1, 12, 8, 10, 32, 3, 2, 1), (24, 64, 64, 3, 48, 7, 2, 3),
                                                     # a unit has fewer rows only as long as every block has a compute unit of its own
                                                     (11, 46, 46, 4, 128, 3, 1, 1), (40, 32, 32, 2, 96, 7, 2, 3), (2, 64, 64, 3, 400, 3, 1, 1)])
def test_few_input_channels_on_few_images(nq, B, H, W, Cin, N, k, stride, pad):
    for n, l, comp in ((8, 2, False), (6, 2, True)):
        x = inputs.uniform_activations((B, H, W, Cin), seed=W) >> (8 - n)
        forced(nq, make_case(nq, N, k * k * Cin, n, l, seed=H + N, compensated=comp), x, (k, k, stride, pad), "5", 5)


@pytest.mark.parametrize("B,HW,C,off", [(1, 49, 2048, 0), (3, 1, 64, 0), (2, 17, 68, 0), (2, 15, 30, 0), (2, 33, 64, 1), (70, 16, 4, 0),
    # either side of the limits against one thread per channel: pixels, blocks, pixels and channels of many blocks
    (2, 11, 64, 0), (2, 12, 64, 0), (1024, 12, 68, 0), (512, 12, 68, 0), (513, 31, 68, 0), (1025, 31, 64, 0), (1025, 32, 64, 0),
    (1025, 128, 16, 0), (1025, 127, 16, 0), (1025, 200, 12, 0), (20000, 1, 64, 0)])
def test_average_pool_in_slices(nq, B, HW, C, off):
    x = inputs.uniform_activations((B, HW, 1, C), seed=C + HW)
    buf = torch.zeros(x.size + 4, dtype=torch.int8, device="cuda")
    buf[off:off + x.size] = dev(x).reshape(-1)
    y = torch.full((B, C), 77, dtype=torch.int8, device="cuda")
    nq.nq_avgpool_i8(buf[off:off + x.size], B, HW, C, 0.05, 11.0, y)
    assert np.array_equal(host(y), oracle.avgpool(x, 0.05, 11.0))


# ---- filters over channels in steps of 16, 8 and 4 --------------------------------------------------------------------
@pytest.mark.parametrize("B,H,W,Cin,N,k,stride,pad,comp", [
    # taps in two, four and eight runs of a lane's 32 bytes: 16 columns, 32 columns and two row tiles, K ending inside a run's tap
    (1, 7, 6, 16, 33, 3, 1, 1, False), (2, 9, 9, 48, 64, 3, 2, 1, True), (2, 12, 10, 80, 592, 3, 1, 1, False), (8, 16, 16, 144, 352, 3, 1, 1, True),
    (1, 7, 6, 8, 33, 3, 1, 1, True), (3, 6, 5, 24, 48, 5, 1, 2, False), (2, 12, 10, 72, 592, 3, 1, 1, True), (8, 16, 16, 120, 352, 3, 1, 1, False),
    (1, 8, 8, 4, 16, 2, 1, 0, False), (1, 7, 5, 12, 33, 7, 2, 3, True), (1, 5, 4, 36, 32, 1, 1, 1, False), (2, 5, 4, 40, 33, 1, 2, 1, True), (2, 12, 10, 36, 592, 3, 1, 1, False), (8, 16, 16, 116, 352, 3, 1, 1, False)])
def test_filters_of_channels_in_small_steps(nq, B, H, W, Cin, N, k, stride, pad, comp):
    forced(nq, make_case(nq, N, k * k * Cin, 8, 3, seed=Cin + N, compensated=comp), inputs.uniform_activations((B, H, W, Cin), seed=H),
           (k, k, stride, pad), "11", 11)


@pytest.mark.parametrize("B,H,Cin,N,k,family", [
    # either side of the limits against the generic kernel, the large one and the one for few channels
    (1, 56, 36, 40, 3, 11), (20, 112, 36, 32, 3, 11), (46, 56, 24, 32, 3, 11), (47, 56, 24, 32, 3, 1), (34, 56, 56, 32, 3, 11),
    (35, 56, 56, 32, 3, 1), (18, 56, 120, 32, 3, 11), (19, 56, 120, 32, 3, 1), (32, 14, 272, 160, 3, 11), (33, 14, 272, 192, 3, 4),
    (66, 56, 8, 32, 3, 11), (67, 56, 8, 32, 3, 5), (3, 56, 2, 32, 3, 5), (31, 56, 32, 32, 3, 11), (32, 56, 32, 32, 3, 1)])
def test_filters_in_small_steps_or_the_kernel_they_replace(nq, B, H, Cin, N, k, family):
    # routes alone, on images of zeros: outputs of each kernel are compared elsewhere
    case = make_case(nq, N, k * k * Cin, 8, 2, seed=Cin + N)
    cs = nq.nq_conv_shape(B, H, H, Cin, N, k, k, 1, k // 2)
    bias = inputs.small_floats(N, 0.2, seed=N)
    epi, _, _ = epi_pair(nq, case, True, (B, H, H), dump=False, s_a=0.02, bias=bias)
    y = torch.full((B, H, H, N), 77, dtype=torch.float32, device="cuda")
    nq.nq_conv_full(torch.zeros(B, H, H, Cin, dtype=torch.int8, device="cuda"), cs, case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    assert torch.equal(y, torch.from_numpy(bias).to(y).expand_as(y))


@pytest.mark.parametrize(*test_filters_in_small_steps_or_the_kernel_they_replace.pytestmark[0].args)
def test_values_of_filters_in_small_steps_on_large_grids(nq, B, H, Cin, N, k, family):
    # values on the grids above: every image against the generic kernel's, the first and the last against the oracle's
    case = make_case(nq, N, k * k * Cin, 8, 2, seed=Cin + N)
    cs = nq.nq_conv_shape(B, H, H, Cin, N, k, k, 1, k // 2)
    bias = inputs.small_floats(N, 0.2, seed=N)
    x = inputs.uniform_activations((B, H, H, Cin), seed=B + Cin)
    ends = sorted({0, B - 1})
    epi, _, okw = epi_pair(nq, case, True, (len(ends), H, H), dump=False, s_a=0.02, bias=bias)
    y, generic = (torch.full((B, H, H, N), 77, dtype=torch.float32, device="cuda") for _ in range(2))
    nq.nq_conv_full(dev(x), cs, case.W.desc, epi, y)
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == family
    set_choice("1")
    try:
        nq.nq_conv_full(dev(x), cs, case.W.desc, epi, generic)
    finally:
        set_choice("")
    torch.cuda.synchronize()
    assert nq.nq_profile_last_kernel()[0] == 1
    assert torch.equal(y, generic)
    acc = oracle.conv_acc(x[ends], case.ow_full.reshape(N, k, k, Cin), 1, k // 2)
    check_outputs(host(y[ends]), None, oracle.epilogue(acc, **okw), acc, False)
