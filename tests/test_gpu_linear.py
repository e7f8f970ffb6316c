"""GPU parity: linear layers on LabelTensors (dense, conv with padding / stride, sum-pool, bias)
through the C ABI against the oracle, bit-exact."""
import numpy as np
import pytest
import torch

import workloads
from gpu_util import both, upload_bundle, assert_bundle_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["by shape", "mfma"])
def mfma(request, monkeypatch):
    """once with the kernel that the layer's shape asks for and once with the MFMA kernel forced (form 4; layers below its smallest size
    keep the choice by shape)"""
    monkeypatch.setenv("DASH_LINEAR_FORM", "4" if request.param == "mfma" else "0")


def run_linear(k, batch, in_h, in_w, in_c, out_c, kh, stride, pad, wlo, whi, bias, seed, garble=True, pool=False, shift=0):
    from paper_2302_06361_amd import Labels, Layer, DENSE, CONV2D, SUMPOOL
    ctx, orc = both(k)
    g = np.random.default_rng(seed)
    n_in = batch * in_h * in_w * in_c
    x = [workloads.uniform_labels(g, n_in, orc.lam(p), p) for p in orc.primes]
    tin = upload_bundle(ctx, x)
    if pool:
        ref = [orc.sumpool2(i, x[i], batch, in_h, in_w, in_c) for i in range(k)]
        lay = Layer(SUMPOOL, 1, batch, in_h=in_h, in_w=in_w, in_c=in_c)
    else:
        W = g.integers(wlo, whi + 1, (out_c, kh, kh, in_c)).astype(np.int32)
        b = g.integers(-1000, 1000, out_c).astype(np.int32) if bias else None
        ones = [orc.one0(i) if garble else orc.one(i) for i in range(k)]
        ref = [orc.conv2d(i, x[i], batch, in_h, in_w, in_c, out_c, kh, kh, stride, pad, W, b, ones[i]) for i in range(k)]
        wp = ctx.weights_prepare(W.reshape(out_c, -1))
        if shift:                                   # a copy that starts `shift` bytes past an aligned address
            wp = torch.cat([wp.new_zeros(shift), wp.reshape(-1)])[shift:]
        bd = torch.as_tensor(b).to(ctx.device) if bias else None
        dense = in_h == 1 and in_w == 1 and kh == 1
        lay = Layer(DENSE if dense else CONV2D, 1, batch, in_h=in_h, in_w=in_w, in_c=in_c, out_c=out_c, kh=kh, kw=kh,
                    stride=stride, pad=pad, weights=wp, bias=bd)
    oe, tb, sb = ctx.layer_sizes(lay)
    assert tb == 0 and oe * batch == ref[0].shape[0]
    tout = Labels(ctx, oe * batch, zero=True)
    if garble:
        ctx.garble_layer(lay, tin, tout)
    else:
        ctx.eval_layer(lay, tin, None, tout)
    torch.cuda.synchronize()
    assert_bundle_equal(tout, ref, "linear output")


@pytest.mark.parametrize("garble", [True, False])
def test_dense_small_with_bias(garble):
    run_linear(8, 3, 1, 1, 50, 7, 1, 1, 0, -8, 7, True, 1, garble)


def test_dense_mlp_shapes():
    run_linear(8, 1, 1, 1, 784, 128, 1, 1, 0, -8, 7, False, 2)
    run_linear(8, 1, 1, 1, 128, 10, 1, 1, 0, -8, 7, False, 3)


def test_dense_12_primes_wide_weights():
    run_linear(12, 5, 1, 1, 300, 33, 1, 1, 0, -64, 63, True, 4)


def test_conv_lenet_shapes():
    run_linear(8, 2, 28, 28, 1, 6, 5, 1, 2, -8, 7, False, 5)
    run_linear(8, 2, 14, 14, 6, 16, 5, 1, 0, -8, 7, True, 6)


def test_conv_stride_and_padding():
    run_linear(5, 2, 9, 9, 3, 4, 3, 2, 1, -3, 3, True, 7)
    run_linear(5, 1, 8, 8, 2, 5, 4, 2, 0, -3, 3, False, 8)
    # few outputs and a long reduction (the form with a wave per output pixel and eight channels), taps outside the image, odd channel count
    run_linear(5, 1, 6, 6, 8, 3, 3, 1, 1, -3, 3, True, 12)
    run_linear(8, 2, 5, 5, 7, 2, 5, 2, 2, -8, 7, True, 13, garble=False)


def test_conv_vgg_block_shape():
    run_linear(12, 1, 8, 8, 16, 32, 3, 1, 1, -16, 15, False, 9)


def test_sumpool():
    run_linear(8, 3, 10, 10, 16, 16, 1, 1, 0, 0, 0, False, 10, pool=True)
    run_linear(12, 2, 6, 4, 5, 5, 1, 1, 0, 0, 0, False, 11, pool=True)


def test_dense_mfma_ragged_tiles_and_bias(mfma):
    """dense layers large enough for the MFMA kernel: several K stages, ragged M, K and group tails"""
    run_linear(12, 5, 1, 1, 500, 300, 1, 1, 0, -64, 63, True, 21)
    run_linear(8, 7, 1, 1, 128, 257, 1, 1, 0, -8, 7, False, 22, garble=False)
    run_linear(12, 3, 1, 1, 1030, 70, 1, 1, 0, -64, 63, True, 23, garble=False)


def test_dense_mfma_config4_sample(mfma):
    """config 4 shape on a slice: K = 4096 inputs, 96 output rows, batch 2, all 12 primes, weights in [-64, 63]"""
    run_linear(12, 2, 1, 1, 4096, 96, 1, 1, 0, -64, 63, False, 24)


def test_dense_mfma_large_accumulators_and_stage_counts(mfma):
    """K = 13000: (p - 1)^2 K passes 2^24 for p = 37, so the two-step reduction of the accumulators runs (with and
    without bias); K = 250 and 192: four and three K stages (every exit of the software pipeline)"""
    run_linear(12, 1, 1, 1, 13000, 70, 1, 1, 0, -64, 63, True, 25)
    run_linear(12, 2, 1, 1, 13000, 40, 1, 1, 0, -64, 63, False, 26, garble=False)
    run_linear(8, 3, 1, 1, 250, 130, 1, 1, 0, -8, 7, False, 27)
    run_linear(8, 3, 1, 1, 192, 130, 1, 1, 0, -8, 7, True, 28)


def test_conv_mfma_shapes(mfma):
    """convolutions that take the MFMA kernel as an implicit GEMM (channels a multiple of 4): stride, padding,
    bias, batches, a 1x1 kernel, pixel counts that leave ragged group tiles, K not a multiple of 64"""
    run_linear(12, 2, 9, 7, 8, 40, 3, 2, 1, -16, 15, True, 31)
    run_linear(8, 3, 6, 6, 4, 70, 5, 1, 2, -8, 7, False, 32)
    run_linear(8, 1, 5, 5, 64, 64, 1, 1, 0, -8, 7, True, 33, garble=False)
    run_linear(12, 1, 16, 16, 12, 48, 3, 1, 1, -16, 15, False, 34)
    run_linear(5, 2, 7, 7, 20, 33, 3, 1, 0, -3, 3, True, 35)
    run_linear(12, 2, 9, 7, 12, 40, 3, 2, 1, -16, 15, True, 36)       # (stride and padding in a layer of the smallest size and above)


def test_dense_mfma_both_tile_shapes(monkeypatch, mfma):
    """the 256 x 256 and the 128 x 512 block tiles of the MFMA kernel, forced in turn"""
    for shape in ("big", "wide"):
        monkeypatch.setenv("DASH_GEMM_TILE", shape)
        run_linear(12, 5, 1, 1, 500, 300, 1, 1, 0, -64, 63, True, 41)
        run_linear(8, 40, 1, 1, 192, 100, 1, 1, 0, -8, 7, False, 42, garble=False)
        run_linear(12, 2, 9, 7, 8, 40, 3, 2, 1, -16, 15, True, 43)
        run_linear(12, 2, 9, 7, 12, 40, 3, 2, 1, -16, 15, True, 44)


@pytest.mark.parametrize("form", ["1", "2", "3", "5", "6", "7", "8"])
def test_linear_forms(monkeypatch, form):
    """each kernel at the edges of its blocks: 1, 2, 4 and 8 output channels, 4, 64 and 256 entries of the reduction, taps in the padding"""
    monkeypatch.setenv("DASH_LINEAR_FORM", form)
    for i, (K, out_c) in enumerate(((1, 1), (3, 4), (4, 5), (255, 8), (257, 9), (513, 33))):
        run_linear(7, 3, 1, 1, K, out_c, 1, 1, 0, -64, 63, i % 2 == 0, 50 + i, garble=i % 3 == 0)
    run_linear(5, 1, 1, 1, 70, 3, 1, 1, 0, -8, 7, True, 60)
    run_linear(5, 2, 6, 7, 3, 9, 3, 2, 1, -8, 7, True, 61)
    run_linear(8, 1, 5, 5, 7, 2, 5, 1, 2, -8, 7, True, 62, garble=False)
    run_linear(8, 3, 9, 8, 5, 17, 4, 3, 0, -8, 7, False, 63)
    run_linear(12, 1, 4, 4, 65, 7, 2, 2, 0, -8, 7, False, 64)
    for i, (K, out_c) in enumerate(((5, 2), (63, 3), (64, 1), (65, 2), (129, 4))):
        run_linear(7, 21, 1, 1, K, out_c, 1, 1, 0, -64, 63, i % 2 == 0, 65 + i)


@pytest.mark.parametrize("form", ["1", "2", "3", "4", "5", "6", "7", "8"])
def test_linear_weights_at_odd_address(monkeypatch, form):
    """prepared weights have no alignment of their own"""
    monkeypatch.setenv("DASH_LINEAR_FORM", form)
    if form == "4":                                  # (layers of at least the MFMA kernel's smallest size)
        run_linear(7, 3, 1, 1, 70, 130, 1, 1, 0, -8, 7, True, 74, shift=1)
        run_linear(8, 2, 6, 6, 12, 40, 3, 1, 1, -8, 7, False, 75, shift=6)
        return
    run_linear(5, 2, 6, 7, 3, 9, 3, 2, 1, -8, 7, True, 71, shift=1)
    run_linear(7, 3, 1, 1, 70, 5, 1, 1, 0, -8, 7, False, 72, shift=2)


@pytest.mark.parametrize("form", ["1", "2"])
def test_linear_more_channel_blocks_than_a_grid_holds(monkeypatch, form):
    """blocks of 4 and 8 channels past 65535"""
    monkeypatch.setenv("DASH_LINEAR_FORM", form)
    run_linear(2, 1, 1, 1, 2, (4 if form == "1" else 8) * 65535 + 5, 1, 1, 0, -8, 7, False, 73)
