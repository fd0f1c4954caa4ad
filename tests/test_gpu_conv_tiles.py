"""The tiles and gathers of the bf16 convolutions that copy their operands straight
into LDS (csrc/k_conv.hip, k_wgrad.hip) and of the image kernels (k_image.hip), and
which calls each of them takes, each through a small stage whose sizes reach it with
a ragged last tile: every tile of k_conv_gemm_lds by its launch name against 64-bit
autograd, and cases against the oracle's bf16 model (and the exact one where no ReLU
is present) at the bf16 bar, 2e-2, with the launches that they are there for; and
the fp32 tiles of csrc/k_gemm.hip against the exact oracle.

A case is picked by rows (micro-batch x H x W), output channels and input
channels: channels that are no multiple of the 64-channel step take a filter
tap per 16-byte chunk; strided data gradients take their rows by residue class,
also classes that no tap reaches (1 x 1, stride 2)."""
import numpy as np
import pytest

import oracle
import paper_1911_04610_amd as xp
import workloads as wl
from conftest import rel_l2
from gpu_harness import run_stage
from test_gpu_layers import _errs, bn, conv

pytestmark = pytest.mark.gpu


def relu(x):
    return dict(kind="relu", inputs=[x])


CASES = {
    # name: (layers, per-sample input shape, micro-batch)
    "64x64": ([conv(-1, 64, 256, 3)], (29, 27, 64), 4),
    "64x64_chunk_taps": ([conv(-1, 72, 256, 3)], (29, 27, 72), 4),
    "64x64_8_channels_1x7": ([conv(-1, 8, 256, 1, kw=7)], (29, 27, 8), 4),
    "64x128": ([conv(-1, 64, 256, 1)], (57, 57, 64), 4),
    "128x128_chunk_taps": ([conv(-1, 40, 512, 1)], (57, 57, 40), 4),
    "128x64_bias_relu": ([conv(-1, 48, 64, 3, True), relu(0)], (129, 128, 48), 4),
    "96x96": ([conv(-1, 32, 96, 3), bn(0, 96)], (91, 91, 32), 4),
    "96x96_chunk_taps": ([conv(-1, 24, 88, 5)], (91, 91, 24), 4),
    "few_tiles_24_channels": ([conv(-1, 64, 24, 3, True)], (57, 57, 64), 4),
    "strided": ([conv(-1, 64, 256, 3, stride=2)], (57, 55, 64), 4),
    "strided_1x1": ([conv(-1, 256, 512, 1, stride=2)], (81, 80, 256), 4),
    "strided_7x7_chunk_taps": ([conv(-1, 40, 256, 7, stride=2)], (57, 56, 40), 4),
    "unpadded": ([conv(-1, 64, 256, 5, pad="valid")], (33, 32, 64), 4),
    # few tiles: 32 x 32, four or eight buffers
    "few_tiles": ([conv(-1, 64, 64, 3, True), relu(0)], (7, 7, 64), 3),
    "few_tiles_long": ([conv(-1, 512, 48, 3, True), relu(0)], (7, 7, 512), 3),
    "few_tiles_chunk_taps": ([conv(-1, 24, 40, 7), bn(0, 40)], (9, 11, 24), 3),
    "few_tiles_one_step": ([conv(-1, 40, 8, 1)], (9, 11, 40), 3),
    "general_bn_partials": ([conv(-1, 64, 128, 1), bn(0, 128), relu(1), conv(2, 128, 64, 5)], (9, 10, 64), 3),
    "few_tiles_strided": ([conv(-1, 64, 64, 3, stride=2)], (23, 25, 64), 2),
    # output channels that are no multiple of 8: the general kernel's large tiles
    "general_128x128": ([conv(-1, 32, 132, 1)], (129, 128, 32), 4),
    "general_128x64": ([conv(-1, 32, 60, 3)], (129, 128, 32), 4),
    "general_64x96": ([conv(-1, 64, 92, 3)], (27, 29, 64), 4),
    "general_odd_channels": ([conv(-1, 512, 73, 1, kw=3)], (16, 15, 512), 4),
    "general_odd_channels_1x1": ([conv(-1, 256, 155, 1)], (16, 15, 256), 4),
    "general_64x64_1x1": ([conv(-1, 64, 100, 1)], (65, 64, 64), 4),
    "general_64x64_5x5": ([conv(-1, 128, 68, 5)], (19, 17, 128), 4),
    "general_strided_128x128": ([conv(-1, 32, 132, 1, stride=2)], (257, 256, 32), 4),
    "general_strided_128x64": ([conv(-1, 32, 60, 1, stride=2)], (257, 256, 32), 4),
    "general_strided_64x96": ([conv(-1, 32, 92, 1, stride=2)], (257, 256, 32), 4),
    # images (csrc/k_image.hip): ragged rows and columns, a second block of
    # channels, one output row per workgroup, unpadded
    "image_7x7_s2": ([conv(-1, 3, 64, 7, stride=2), bn(0, 64), relu(1)], (75, 131, 3), 4),
    "image_7x7_s2_channels_72": ([conv(-1, 3, 72, 7, True, stride=2), relu(0)], (40, 30, 3), 1),
    "image_3x3": ([conv(-1, 3, 64, 3, True), relu(0)], (32, 32, 3), 3),
    "image_3x3_odd": ([conv(-1, 3, 24, 3)], (37, 41, 3), 2),
    "image_3x3_small": ([conv(-1, 3, 32, 3), bn(0, 32)], (5, 3, 3), 2),
    "image_3x3_s2_unpadded": ([conv(-1, 3, 32, 3, stride=2, pad="valid"), bn(0, 32)], (99, 97, 3), 8),
    "image_5x5": ([conv(-1, 3, 40, 5)], (33, 70, 3), 60),
    "image_least_map": ([conv(-1, 3, 40, 5, True), relu(0)], (12, 12, 3), 3),
    "image_least_map_s2": ([conv(-1, 3, 72, 7, stride=2), bn(0, 72)], (35, 15, 3), 3),
    "image_least_wgrad_map": ([conv(-1, 12, 72, 3)], (8, 8, 12), 5),
    "image_wgrad_150_channels": ([conv(-1, 150, 88, 1)], (13, 12, 150), 5),
    "image_wgrad_44_channels_s2": ([conv(-1, 44, 24, 1, stride=2)], (17, 15, 44), 5),
    "odd_linear": ([dict(kind="linear", inputs=[-1], cin=100, cout=200, bias=True)], (100,), 37),
    "image_one_channel": ([conv(-1, 1, 16, 5)], (28, 28, 1), 8),
    # data gradients with mask, accumulation and batch-norm backward partials
    "bn_partials": ([conv(-1, 64, 256, 1), bn(0, 256), relu(1), conv(2, 256, 64, 3), bn(3, 64), conv(2, 256, 72, 1),
                     dict(kind="concat", inputs=[4, 5])], (57, 57, 64), 4),
    "bn_partials_96": ([conv(-1, 32, 88, 1), bn(0, 88), relu(1), conv(2, 88, 32, 3)], (91, 91, 32), 4),
    "bn_partials_strided": ([conv(-1, 32, 128, 1), bn(0, 128), relu(1), conv(2, 128, 64, 3, stride=2)],
                            (65, 63, 32), 4),
}


# launches that a case is there for
REACHES = {
    "64x64": ["k_conv_gemm_lds<64,64,2,2,64,2,false,0,false,false>", "k_wgrad_lds<128,64,4,2,64,false>"],
    "64x64_chunk_taps": ["k_conv_gemm_lds<64,64,2,2,64,2,true,0,false,false>", "k_wgrad_lds<128,64,4,2,64,false>"],
    "64x64_8_channels_1x7": ["k_conv_gemm_lds<64,64,2,2,64,2,true,0,false,false>", "k_wgrad_lds<128,64,4,2,64,true>"],
    "64x128": ["k_conv_gemm_lds<64,128,2,2,64,2,false,0,false,false>", "k_wgrad_lds<128,64,4,2,64,false>"],
    "128x128_chunk_taps": ["k_conv_gemm_lds<128,128,4,2,64,2,true,0,false,false>",
                           "k_wgrad_lds<128,64,4,2,64,false>"],
    "128x64_bias_relu": ["k_conv_gemm_lds<128,64,4,2,64,2,true,0,false,false>", "k_wgrad_lds<64,64,2,2,64,false>"],
    "96x96": ["k_conv_gemm_lds<96,96,1,3,32,3,false,0,false,false>", "k_wgrad_lds<128,64,4,2,64,false>"],
    "96x96_chunk_taps": ["k_conv_gemm_lds<96,96,1,3,32,3,true,0,false,false>", "k_wgrad_lds<128,64,4,2,64,false>"],
    "few_tiles_24_channels": ["k_conv_gemm_lds<32,32,1,1,64,4,false,0,false,true>",
                              "k_wgrad_lds<64,64,2,2,64,false>"],
    "strided": ["k_conv_gemm_lds<64,64,2,2,64,2,false,1,false,false>", "k_wgrad_lds<128,64,4,2,64,true>"],
    "strided_1x1": ["k_conv_gemm_lds<64,128,2,2,64,2,false,1,false,false>", "k_wgrad_lds<128,64,4,2,64,true>"],
    "strided_7x7_chunk_taps": ["k_conv_gemm_lds<64,64,2,2,64,2,true,1,false,false>",
                               "k_wgrad_lds<128,64,4,2,64,true>"],
    "unpadded": ["k_conv_gemm_lds<64,64,2,2,64,2,false,1,false,false>", "k_wgrad_lds<128,64,4,2,64,true>"],
    "few_tiles": ["k_conv_gemm_lds<32,32,1,1,64,4,false,0,false,true>", "k_wgrad_lds<64,64,2,2,64,false>"],
    "few_tiles_long": ["k_conv_gemm_lds<32,32,1,1,64,8,false,0,false,true>", "k_wgrad_lds<64,64,2,2,64,false>"],
    "few_tiles_chunk_taps": ["k_conv_gemm_lds<32,32,1,1,64,4,true,0,false,true>", "k_wgrad_lds<64,64,2,2,64,false>"],
    "few_tiles_one_step": ["k_conv_gemm_lds<32,32,1,1,64,4,true,0,false,true>", "k_wgrad_lds<64,64,2,2,64,false>"],
    "general_bn_partials": ["k_conv_gemm<bf16,64,64,2,2,false,4,2>"],
    "few_tiles_strided": ["k_conv_gemm_lds<32,32,1,1,64,4,false,1,false,true>", "k_wgrad_lds<64,64,2,2,64,true>"],
    "general_128x128": ["k_conv_gemm<bf16,128,128,2,4,false,2,2>", "k_wgrad<bf16,128,64,2,2,false>"],
    "general_128x64": ["k_conv_gemm<bf16,128,64,2,2,false,2,2>", "k_wgrad<bf16,64,128,2,2,false>"],
    "general_64x96": ["k_conv_gemm<bf16,64,96,2,2,false,1,2>", "k_wgrad<bf16,128,128,2,2,false>"],
    "general_odd_channels": ["k_conv_gemm<bf16,64,96,2,2,false,1,2>", "k_wgrad<bf16,128,128,2,2,false>"],
    "general_odd_channels_1x1": ["k_conv_gemm<bf16,32,64,2,2,false,2,2>", "k_wgrad<bf16,128,128,2,2,false>"],
    "general_64x64_1x1": ["k_conv_gemm<bf16,64,64,2,2,false,2,2>", "k_wgrad<bf16,128,64,2,2,false>"],
    "general_64x64_5x5": ["k_conv_gemm<bf16,64,64,2,2,false,8,2>", "k_wgrad<bf16,128,128,2,2,false>"],
    "general_strided_128x128": ["k_conv_gemm<bf16,128,128,2,4,false,2,2,strided>", "k_wgrad<bf16,128,64,2,2,false>"],
    "general_strided_128x64": ["k_conv_gemm<bf16,128,64,2,2,false,2,2,strided>", "k_wgrad<bf16,64,64,2,2,false>"],
    "general_strided_64x96": ["k_conv_gemm<bf16,64,96,2,2,false,1,2,strided>", "k_wgrad<bf16,128,64,2,2,false>"],
    "image_7x7_s2": ["k_conv_gemm_image<7>", "k_wgrad_image<5>"],
    "image_7x7_s2_channels_72": ["k_conv_gemm_image<7>", "k_wgrad_image<5>"],
    "image_3x3": ["k_conv_gemm_image<3>", "k_wgrad_image<1>"],
    "image_3x3_odd": ["k_conv_gemm_image<3>", "k_wgrad_image<1>"],
    "image_3x3_small": ["k_conv_gemm<bf16,64,32,2,2,true,1,2>", "k_wgrad<bf16,64,64,2,2,true>"],
    "image_3x3_s2_unpadded": ["k_conv_gemm_image<3>", "k_wgrad_image<1>"],
    "image_5x5": ["k_conv_gemm_image<5>", "k_wgrad_image<3>"],
    "image_least_map": ["k_conv_gemm_image<5>", "k_wgrad_image<3>"],
    "image_least_map_s2": ["k_conv_gemm_image<7>", "k_wgrad_image<5>"],
    "image_least_wgrad_map": ["k_conv_gemm<bf16,64,64,2,2,true,2,2>", "k_wgrad<bf16,128,128,2,2,true>"],
    "image_wgrad_150_channels": ["k_conv_gemm<bf16,64,64,2,2,true,2,2>", "k_wgrad_image<5>"],
    "image_wgrad_44_channels_s2": ["k_conv_gemm<bf16,64,32,2,2,true,1,2,strided>", "k_wgrad_image<3>"],
    "odd_linear": ["k_conv_gemm<bf16,64,64,2,2,true,2,2>", "k_wgrad<bf16,128,128,2,2,true>"],
    "image_one_channel": ["k_conv_gemm<bf16,64,32,2,2,true,1,2>", "k_wgrad_image<1>"],
    "bn_partials": ["k_conv_gemm_lds<128,128,4,2,64,2,false,0,true,false>"],
    "bn_partials_96": ["k_conv_gemm_lds<96,96,1,3,32,3,false,0,false,false>",
                       "k_conv_gemm<bf16,64,96,2,2,false,1,2>"],
    "bn_partials_strided": ["k_conv_gemm_lds<64,128,2,2,64,2,false,2,true,false>"],
}


@pytest.mark.parametrize("name", list(CASES))
def test_conv_tiles_match_oracle(name):
    layers, shape, mb = CASES[name]
    launched = sum(_launches(xp.Stage(layers, mb, 1, shape, xp.BF16), shape, mb), [])
    assert set(REACHES[name]) <= set(launched), launched
    w = wl.StageWorkload(name, layers, mb, 1, shape, 1, 0, 0, 0, minibatches=1, seed=131)
    inp = wl.stage_inputs(w, act_dtype="bf16")
    gpu, _ = run_stage(w, inp, xp.BF16, xp.Hyper(), 0, 0, minibatches=1)
    modes = ["bf16"] if any(L["kind"] == "relu" for L in layers) else ["bf16", "f64"]
    for mode in modes:
        ref = oracle.train_stage(oracle.Stage(layers, mode), inp.params, inp.m, inp.v, inp.xs, 0, 0,
                                 oracle.Hyper(), labels=inp.labels, dys=inp.dys)[0]
        e = _errs(gpu[0], ref)
        worst = max(e, key=e.get)
        print(f"{name} vs oracle-{mode}: worst {worst} = {e[worst]:.2e}")
        bad = {k: v for k, v in e.items() if not v <= 2e-2}
        assert not bad, f"vs oracle-{mode}: " + ", ".join(f"{k}={v:.2e}" for k, v in bad.items())


# fp32 storage: the general kernel's tiles by the count of 64 x 64 tiles, each with
# ragged rows and columns; their weight gradients' tiles by workgroups
F32_CASES = {
    "32x32_deep": ([conv(-1, 64, 72, 3, True), relu(0)], (7, 9, 64), 3),
    "32x32_24_channels": ([conv(-1, 24, 40, 7), bn(0, 40)], (9, 11, 24), 3),
    "32x32_48_channels": ([conv(-1, 48, 20, 5), bn(0, 20)], (9, 11, 48), 3),
    "32x32_odd_channels": ([conv(-1, 10, 33, 3)], (9, 11, 10), 3),
    "32x32_odd_columns": ([conv(-1, 64, 96, 1), bn(0, 96)], (65, 64, 64), 4),
    "32x64": ([conv(-1, 32, 120, 3), bn(0, 120), relu(1)], (47, 45, 32), 4),
    "64x64": ([conv(-1, 32, 128, 1), bn(0, 128)], (91, 90, 32), 4),
    "strided": ([conv(-1, 32, 72, 3, stride=2), bn(0, 72)], (23, 25, 32), 2),
    "strided_1x1": ([conv(-1, 64, 40, 1, stride=2)], (15, 16, 64), 2),
    "wgrad_64x64": ([conv(-1, 132, 68, 3)], (16, 17, 132), 16),
    "wgrad_narrow": ([conv(-1, 40, 24, 3)], (14, 14, 40), 32),
    "linear": ([dict(kind="linear", inputs=[-1], cin=200, cout=72, bias=True), relu(0),
                dict(kind="linear", inputs=[1], cin=72, cout=10, bias=True)], (200,), 33),
}


@pytest.mark.parametrize("dtype", [xp.F32, xp.BF16])
@pytest.mark.parametrize("channels", [8, 264, 1032, 2080])
@pytest.mark.parametrize("rows", [(1, 3), (5, 7), (61, 67)])
def test_column_sums(dtype, channels, rows):
    """Batch-norm sums over columns taken by 1 to 17 workgroups of up to 32 chunks, rows
    fewer than a block's groups and many trips, against fp64: a batch norm's output
    is rounded once, its gradients are 64-bit sums rounded once to fp32, of products
    with the same bf16 or fp32 inputs; dx is one rounding too."""
    import torch
    st = xp.Stage([bn(-1, channels)], 2, 1, rows + (channels,), dtype)
    tdt = torch.bfloat16 if dtype == xp.BF16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(5)
    for off, cnt in st.layout:
        st.W[off:off + cnt] = 1 + torch.rand(cnt, generator=g, device="cuda")
    for d in (xp.FWD, xp.BWD):
        st.xpipe_predict_weights(d, 0, xp.Hyper(), 0)
    x = (torch.randn(2, *rows, channels, generator=g, device="cuda") + 1).to(tdt)
    dy = torch.randn(2, *rows, channels, generator=g, device="cuda").to(tdt)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    st.xpipe_stage_fwd(x, y)
    st.xpipe_stage_bwd(x, dy, None, dx)
    X = x.double().reshape(-1, channels).requires_grad_(True)
    gam, bet = (st.W[off:off + cnt].double().requires_grad_(True) for off, cnt in st.layout)
    rstd = (X.var(0, unbiased=False) + 1e-5).rsqrt()
    Y = (X - X.mean(0)) * rstd * gam + bet
    Y.backward(dy.double().reshape(-1, channels))
    one = 2.0 ** -8 if dtype == xp.BF16 else 2.0 ** -23
    for a, b, tol in [(y, Y, one), (dx, X.grad, one)] + [
            (st.grad[off:off + cnt], p.grad, 2.0 ** -23) for (off, cnt), p in zip(st.layout, (gam, bet))]:
        assert rel_l2(a.double().cpu().numpy().ravel(), b.detach().cpu().numpy().ravel()) <= tol


@pytest.mark.parametrize("channels", [8, 264, 1032, 2080])
@pytest.mark.parametrize("hw", [(1, 2), (4, 8), (32, 64)])
def test_column_sums_of_the_pool_gradient(channels, hw):
    """The same sums taken by the global average pool's backward.  A power of two of
    pixels makes its gradient exact; 64-bit sums stored in fp32."""
    import torch
    st = xp.Stage([bn(-1, channels), relu(0), dict(kind="gap", inputs=[1])], 3, 1, hw + (channels,), xp.BF16)
    g = torch.Generator(device="cuda").manual_seed(5)
    (go, gn), (bo, bc) = st.layout
    st.W[go:go + gn] = 1 + torch.rand(channels, generator=g, device="cuda")
    st.W[bo:bo + bc] = torch.randn(channels, generator=g, device="cuda")
    for d in (xp.FWD, xp.BWD):
        st.xpipe_predict_weights(d, 0, xp.Hyper(), 0)
    x = (torch.randn(3, *hw, channels, generator=g, device="cuda") + 1).to(torch.bfloat16)
    dy = torch.randn(3, 1, 1, channels, generator=g, device="cuda").to(torch.bfloat16)
    st.set_timing(True)
    st.xpipe_stage_bwd(x, dy, None, torch.empty_like(x))
    torch.cuda.synchronize()
    assert "k_gap_bwd_bn_v<bf16>" in st.timing(), list(st.timing())
    X = x.double().reshape(-1, channels)
    xhat = (X - X.mean(0)) * (X.var(0, unbiased=False) + 1e-5).rsqrt()
    z = xhat * st.W[go:go + gn].double() + st.W[bo:bo + bc].double()
    G = (dy.double() / (hw[0] * hw[1])).expand(3, *hw, channels).reshape(-1, channels) * (z > 0)
    for off, cnt, ref in ((go, gn, (G * xhat).sum(0)), (bo, bc, G.sum(0))):
        assert rel_l2(st.grad[off:off + cnt].double().cpu().numpy(), ref.cpu().numpy()) <= 2.0 ** -23


@pytest.mark.parametrize("channels", [64, 264])
def test_column_sums_of_many_f32_rows(channels):
    """16 million values and more in fp32: twice the workgroups."""
    test_column_sums(xp.F32, channels, (181, 4 * 64 * 182 // channels))


@pytest.mark.parametrize("name", list(F32_CASES))
def test_f32_tiles_match_oracle(name):
    """Sums are kept in 64 bits and rounded once on store; a chain of at most three
    stored tensors, each 2^-24 off per value, and batch-norm gradients that subtract
    means (a factor below 10 here) stay below 1e-5 of the exact oracle."""
    layers, shape, mb = F32_CASES[name]
    w = wl.StageWorkload(name, layers, mb, 1, shape, 1, 0, 0, 0, minibatches=1, seed=137)
    inp = wl.stage_inputs(w, act_dtype="f32")
    gpu, _ = run_stage(w, inp, xp.F32, xp.Hyper(), 0, 0, minibatches=1)
    ref = oracle.train_stage(oracle.Stage(layers, "f64"), inp.params, inp.m, inp.v, inp.xs, 0, 0,
                             oracle.Hyper(), labels=inp.labels, dys=inp.dys)[0]
    e = _errs(gpu[0], ref)
    worst = max(e, key=e.get)
    print(f"{name}: worst {worst} = {e[worst]:.2e}")
    bad = {k: v for k, v in e.items() if not v <= 1e-5}
    assert not bad, ", ".join(f"{k}={v:.2e}" for k, v in bad.items())


def _launches(st, shape, mb, dtype=xp.BF16):
    """Launch names of one forward, and of one backward, of a stage."""
    import torch
    tdt = torch.bfloat16 if dtype == xp.BF16 else torch.float32
    x = torch.ones((mb,) + shape, dtype=tdt, device="cuda")
    dy = torch.ones(st.out_shape, dtype=tdt, device="cuda").reshape((mb, -1) if len(shape) == 1 else st.out_shape)
    y, dx = torch.empty_like(dy), torch.empty_like(x)
    for d in (xp.FWD, xp.BWD):
        st.xpipe_predict_weights(d, 0, xp.Hyper(), 0)
    out = []
    for run in (lambda: st.xpipe_stage_fwd(x, y), lambda: st.xpipe_stage_bwd(x, dy, None, dx)):
        st.set_timing(True)
        run()
        torch.cuda.synchronize()
        out.append(list(st.timing()))
        st.set_timing(False)
    return out


# One call for each tile, step (whole 64 channels, or a filter tap per 16-byte chunk),
# grid and direction of k_conv_gemm_lds, by its launch name's arguments:
# (filter, input channels, output channels, rows, columns, micro-batch, stride)
LDS_CASES = {
    "128,32,4,1,64,2,false,0,false,false": (3, 64, 32, 79, 78, 4, 1),
    "128,32,4,1,64,2,true,0,false,false": (3, 40, 24, 79, 78, 4, 1),
    "64,64,2,2,64,2,false,0,false,false": (1, 64, 200, 57, 55, 2, 1),
    "64,64,2,2,64,2,true,0,false,false": (1, 72, 200, 57, 55, 2, 1),
    "64,128,2,2,64,2,false,0,false,false": (1, 64, 256, 57, 57, 4, 1),
    "64,128,2,2,64,2,true,0,false,false": (1, 72, 256, 57, 57, 4, 1),
    "128,128,4,2,64,2,false,0,false,false": (1, 64, 512, 57, 57, 4, 1),
    "128,128,4,2,64,2,true,0,false,false": (1, 40, 512, 57, 57, 4, 1),
    "96,96,1,3,32,3,false,0,false,false": (1, 32, 96, 91, 91, 4, 1),
    "96,96,1,3,32,3,true,0,false,false": (1, 40, 88, 91, 91, 4, 1),
    "128,64,4,2,64,2,false,0,false,false": (1, 64, 64, 129, 128, 4, 1),
    "128,64,4,2,64,2,true,0,false,false": (1, 72, 64, 129, 128, 4, 1),
    "32,32,1,1,64,4,false,0,false,true": (3, 64, 40, 7, 9, 3, 1),
    "32,32,1,1,64,4,true,0,false,true": (5, 24, 40, 7, 9, 3, 1),
    "32,32,1,1,64,8,false,0,false,true": (3, 512, 40, 7, 9, 3, 1),
    "128,32,4,1,64,2,false,1,false,false": (3, 64, 32, 113, 111, 4, 2),
    "128,32,4,1,64,2,true,1,false,false": (3, 40, 24, 113, 111, 4, 2),
    "64,64,2,2,64,2,false,1,false,false": (1, 64, 256, 57, 55, 4, 2),
    "64,64,2,2,64,2,true,1,false,false": (1, 72, 256, 57, 55, 4, 2),
    "64,128,2,2,64,2,false,1,false,false": (1, 64, 512, 81, 80, 4, 2),
    "64,128,2,2,64,2,true,1,false,false": (1, 72, 512, 81, 80, 4, 2),
    "128,128,4,2,64,2,false,1,false,false": (1, 64, 512, 113, 112, 4, 2),
    "128,128,4,2,64,2,true,1,false,false": (1, 72, 512, 113, 112, 4, 2),
    "96,96,1,3,32,3,false,1,false,false": (1, 64, 96, 182, 181, 4, 2),
    "96,96,1,3,32,3,true,1,false,false": (1, 40, 88, 182, 181, 4, 2),
    "128,64,4,2,64,2,false,1,false,false": (1, 64, 64, 257, 255, 4, 2),
    "128,64,4,2,64,2,true,1,false,false": (1, 72, 64, 257, 255, 4, 2),
    "32,32,1,1,64,4,false,1,false,true": (3, 64, 40, 13, 15, 3, 2),
    "32,32,1,1,64,4,true,1,false,true": (5, 24, 40, 13, 15, 3, 2),
    "32,32,1,1,64,8,false,1,false,true": (3, 512, 40, 13, 15, 3, 2),
    "64,64,2,2,64,2,false,0,true,false": (3, 64, 256, 65, 64, 4, 1),
    "64,64,2,2,64,2,true,0,true,false": (3, 64, 232, 65, 64, 4, 1),
    "64,128,2,2,64,2,false,0,true,false": (1, 128, 1024, 57, 55, 4, 1),
    "64,128,2,2,64,2,true,0,true,false": (1, 128, 1032, 57, 55, 4, 1),
    "128,128,4,2,64,2,false,0,true,false": (1, 128, 64, 79, 79, 4, 1),
    "128,128,4,2,64,2,true,0,true,false": (1, 128, 136, 79, 79, 4, 1),
    "96,96,1,3,32,3,false,0,true,false": (1, 96, 256, 91, 91, 2, 1),
    "96,96,1,3,32,3,true,0,true,false": (1, 88, 264, 91, 91, 2, 1),
    "128,64,4,2,64,2,false,0,true,false": (1, 64, 64, 91, 91, 4, 1),
    "128,64,4,2,64,2,true,0,true,false": (1, 56, 136, 91, 91, 4, 1),
    "32,32,1,1,64,4,true,0,true,true": (3, 64, 488, 7, 9, 3, 1),
    "32,32,1,1,64,8,false,0,true,true": (3, 64, 512, 7, 9, 3, 1),
    "128,32,4,1,64,2,false,2,true,false": (3, 32, 128, 19, 17, 3, 2),
    "128,32,4,1,64,2,true,2,true,false": (3, 24, 120, 19, 17, 3, 2),
    "64,64,2,2,64,2,false,2,true,false": (3, 64, 64, 19, 17, 3, 2),
    "64,64,2,2,64,2,true,2,true,false": (3, 72, 40, 19, 17, 3, 2),
    "64,128,2,2,64,2,false,2,true,false": (1, 128, 320, 57, 55, 4, 2),
    "64,128,2,2,64,2,true,2,true,false": (1, 128, 264, 57, 55, 4, 2),
    "128,128,4,2,64,2,false,2,true,false": (1, 128, 64, 79, 79, 4, 2),
    "128,128,4,2,64,2,true,2,true,false": (1, 128, 72, 79, 79, 4, 2),
    "96,96,1,3,32,3,false,2,true,false": (1, 96, 288, 91, 91, 2, 2),
    "96,96,1,3,32,3,true,2,true,false": (1, 88, 264, 91, 91, 2, 2),
    "128,64,4,2,64,2,false,2,true,false": (1, 64, 320, 91, 91, 4, 2),
    "128,64,4,2,64,2,true,2,true,false": (1, 56, 264, 91, 91, 4, 2),
}


def _conv64(x, w, stride):
    """[n, h, w, c] by [n, r, s, c], same padding: one product per filter tap."""
    import torch
    k, (h, wd) = w.shape[1], x.shape[1:3]
    x = torch.nn.functional.pad(x, (0, 0, k // 2, k // 2, k // 2, k // 2))
    y = 0
    for r in range(k):
        for q in range(k):
            t = x[:, r:r + h:stride, q:q + wd:stride]
            y = y + t.reshape(-1, t.shape[3]) @ w[:, r, q].t()
    return y.reshape(x.shape[0], (h - 1) // stride + 1, (wd - 1) // stride + 1, -1)


def _bn_relu_conv_case(convs, x_shape, seed, expect):
    """A batch norm, a ReLU and convolutions (k, cout, stride) of it whose outputs are
    concatenated, forward and backward against 64-bit autograd.  Every tensor between
    the layers is rounded to bf16 (2^-9 of a value at most, 1.1e-3 rms, three of them in a
    row for dx and the batch norm's gradients) and a flipped ReLU mask is as rare as an
    output within that of zero: 1e-2 of each result's norm."""
    import torch
    mb, h, w, cin = x_shape
    layers = [bn(-1, cin), relu(0)] + [conv(1, cin, co, k, stride=s) for k, co, s in convs]
    if len(convs) > 1:
        layers.append(dict(kind="concat", inputs=list(range(2, 2 + len(convs)))))
    st = xp.Stage(layers, mb, 1, (h, w, cin), xp.BF16)
    fwd, bwd = _launches(st, (h, w, cin), mb)
    assert expect in (fwd if expect.split(",")[8] == "false" else bwd), (expect, fwd, bwd)
    st.grad.zero_()
    g = torch.Generator(device="cuda").manual_seed(seed)
    params = [1 + torch.rand(cin, generator=g, device="cuda"), torch.randn(cin, generator=g, device="cuda")]
    params += [(torch.randn(co, k, k, cin, generator=g, device="cuda") / (k * k * cin) ** 0.5).to(torch.bfloat16).float()
               for k, co, s in convs]
    for (off, cnt), t in zip(st.layout, params):
        st.W[off:off + cnt] = t.reshape(-1)
    for d in (xp.FWD, xp.BWD):
        st.xpipe_predict_weights(d, 0, xp.Hyper(), 0)
    x = torch.randn(x_shape, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(st.out_shape, generator=g, device="cuda").to(torch.bfloat16)
    y, dx = torch.empty_like(dy), torch.empty_like(x)
    st.xpipe_stage_fwd(x, y)
    st.xpipe_stage_bwd(x, dy, None, dx)
    X = x.double().requires_grad_(True)
    P = [t.double().requires_grad_(True) for t in params]
    var, mean = torch.var_mean(X, (0, 1, 2), unbiased=False)
    A = ((X - mean) * (var + 1e-5).rsqrt() * P[0] + P[1]).relu()
    Y = torch.cat([_conv64(A, wt, s) for wt, (k, co, s) in zip(P[2:], convs)], 3)
    Y.backward(dy.double())
    pairs = {"y": (y, Y.detach()), "dx": (dx, X.grad)}
    pairs.update({f"grad[{i}]": (st.grad[off:off + cnt], p.grad.reshape(-1))
                  for i, ((off, cnt), p) in enumerate(zip(st.layout, P))})
    e = {k: float((a.double() - b).norm() / b.norm()) for k, (a, b) in pairs.items()}
    assert all(v <= 1e-2 for v in e.values()), e


@pytest.mark.parametrize("args", list(LDS_CASES))
def test_lds_copy_tiles(args):
    k, cin, cout, h, w, mb, stride = LDS_CASES[args]
    _bn_relu_conv_case([(k, cout, stride)], (mb, h, w, cin), 7, f"k_conv_gemm_lds<{args}>")


@pytest.mark.parametrize("cout,chunks", [(64, "false"), (136, "true")])
def test_lds_copy_widest_tile_accumulates(cout, chunks):
    """256 x 256 tiles: the second of two data gradients adds to the first's and takes the
    batch norm's partials (with the first's tile also its own stores)."""
    _bn_relu_conv_case([(1, cout, 1), (3, cout, 1)], (5, 214, 245, 256), 9,
                       f"k_conv_gemm_lds<256,256,2,4,64,2,{chunks},0,true,false>")


@pytest.mark.parametrize("k,cin,cout,h,w,mb,stride,fwd,wgrad", [
    (7, 3, 64, 25, 43, 2, 2, "k_conv_gemm_image<7>", "k_wgrad_image<5>"),
    (3, 3, 72, 17, 19, 3, 1, "k_conv_gemm_image<3>", "k_wgrad_image<1>"),
    (3, 9, 24, 11, 13, 3, 1, "k_conv_gemm<", "k_wgrad_image<3>"),
    (1, 20, 16, 23, 19, 3, 2, "k_conv_gemm<", "k_wgrad_image<1>"),
    (3, 64, 200, 57, 55, 2, 1, "k_conv_gemm_lds<64,64,", "k_wgrad_lds<128,64,"),
    (5, 24, 200, 57, 55, 2, 1, "k_conv_gemm_lds<64,64,", "k_wgrad_lds<128,64,"),
    (3, 64, 40, 7, 9, 3, 1, "k_conv_gemm_lds<32,32,", "k_wgrad_lds<64,64,"),
    (5, 24, 40, 13, 15, 3, 2, "k_conv_gemm_lds<32,32,", "k_wgrad_lds<64,64,"),
    (1, 128, 136, 57, 55, 4, 2, "k_conv_gemm_lds<64,64,", "k_wgrad_lds<128,64,"),
    (3, 64, 73, 7, 9, 3, 1, "k_conv_gemm<", "k_wgrad<")])
def test_values_that_are_not_finite_stay_in_their_sums(k, cin, cout, h, w, mb, stride, fwd, wgrad):
    """An infinity in the input and a NaN in the output gradient reach the results whose
    sums they are in, and no other changes a bit: what the kernels read past a row, a
    reduction or the last pixel is zero on both sides."""
    import torch
    st = xp.Stage([conv(-1, cin, cout, k, stride=stride)], mb, 1, (h, w, cin), xp.BF16)
    names = _launches(st, (h, w, cin), mb)
    assert any(n.startswith(fwd) for n in names[0]) and any(n.startswith(wgrad) for n in names[1]), names
    g = torch.Generator(device="cuda").manual_seed(3)
    st.W.normal_(generator=g)
    for d in (xp.FWD, xp.BWD):
        st.xpipe_predict_weights(d, 0, xp.Hyper(), 0)
    x = torch.randn(mb, h, w, cin, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(st.out_shape, generator=g, device="cuda").to(torch.bfloat16)

    def run(x, dy):
        y, dx = torch.empty_like(dy), torch.empty_like(x)
        st.grad.zero_()
        st.xpipe_stage_fwd(x, y)
        st.xpipe_stage_bwd(x, dy, None, dx)
        return y, dx, st.grad[:cout * k * k * cin].reshape(cout, k, k, cin).clone()

    def check(got, clean, touched):
        assert not bool(torch.isfinite(got[touched]).any())
        assert bool(torch.equal(got[~touched], clean[~touched]))

    ones = torch.ones(1, k, k, 1, device="cuda", dtype=torch.double)
    clean = run(x, dy)
    assert all(bool(torch.isfinite(t).all()) for t in clean)
    for at in ((mb - 1, h - 1, w - 1), (0, h // 2, w - 1), (0, 0, 0)):
        bad = x.clone()
        bad[at][cin - 1] = float("inf")
        here = torch.zeros(mb, h, w, 1, device="cuda", dtype=torch.double)
        here[at] = 1
        y, _, gw = run(bad, dy)
        check(y, clean[0], (_conv64(here, ones, stride) > 0).expand_as(y))
        taps = torch.zeros(cout, k, k, cin, dtype=torch.bool, device="cuda")
        for r in range(k):
            for q in range(k):
                one = torch.zeros_like(ones)
                one[0, r, q] = 1
                taps[:, r, q, cin - 1] = bool((_conv64(here, one, stride) > 0).any())
        check(gw, clean[2], taps)
    n, ho, wo, _ = st.out_shape
    at = (n - 1, ho // 2, wo // 2)
    bad = dy.clone()
    bad[at][cout - 1] = float("nan")
    _, dx, gw = run(x, bad)
    here = torch.zeros(mb, h, w, 1, device="cuda", dtype=torch.double, requires_grad=True)
    _conv64(here, ones, stride)[at].sum().backward()
    check(dx, clean[1], (here.grad > 0).expand_as(dx))
    rows = torch.zeros(cout, k, k, cin, dtype=torch.bool, device="cuda")
    rows[cout - 1] = True
    check(gw, clean[2], rows)


LINEAR = dict(kind="linear", inputs=[-1], cin=100, cout=200, bias=False)


@pytest.mark.parametrize("layer,shape,mb,fwd,wgrad", [
    (LINEAR, (100,), 128, "k_conv_gemm<", "k_wgrad<"),  # behind a global pool: 128 maps of one pixel
    (conv(-1, 12, 64, 1), (7, 7, 12), 32, "k_conv_gemm<", "k_wgrad<"),
    (conv(-1, 12, 64, 1), (8, 8, 12), 32, "k_conv_gemm<", "k_wgrad_image<"),
    (conv(-1, 3, 64, 3), (7, 9, 3), 8, "k_conv_gemm<", "k_wgrad<"),
    (conv(-1, 3, 64, 3), (11, 13, 3), 8, "k_conv_gemm<", "k_wgrad_image<"),
    (conv(-1, 3, 64, 3), (12, 12, 3), 8, "k_conv_gemm_image<", "k_wgrad_image<"),
    (conv(-1, 3, 64, 7, stride=2), (23, 24, 3), 8, "k_conv_gemm_image<", "k_wgrad_image<"),
    (conv(-1, 3, 64, 5, pad="valid"), (12, 12, 3), 8, "k_conv_gemm<", "k_wgrad_image<"),
    (conv(-1, 3, 32, 3), (15, 15, 3), 8, "k_conv_gemm<", "k_wgrad_image<"),
    (conv(-1, 3, 32, 3), (15, 16, 3), 8, "k_conv_gemm_image<", "k_wgrad_image<"),
    (conv(-1, 3, 64, 7), (11, 13, 3), 8, "k_conv_gemm<", "k_wgrad<"),
    (conv(-1, 111, 16, 1, stride=2), (35, 31, 111), 8, "k_conv_gemm<", "k_wgrad<"),
    (conv(-1, 3, 64, 3), (200, 7, 3), 4, "k_conv_gemm<", "k_wgrad<")])
def test_image_kernels_take_images(layer, shape, mb, fwd, wgrad):
    """A map of a few pixels keeps the general kernels, which batch over images."""
    f, b = _launches(xp.Stage([layer], mb, 1, shape, xp.BF16), shape, mb)
    assert any(n.startswith(fwd) for n in f), f
    assert any(n.startswith(wgrad) for n in b), b


def _lds(names, dg):
    """Tiles of the LDS-copy forwards (dg false) or data gradients among launch names."""
    args = [n[len("k_conv_gemm_lds<"):-1].split(",") for n in names if n.startswith("k_conv_gemm_lds<")]
    return ["x".join(a[:2]) for a in args if a[8] == ("true" if dg else "false")]


@pytest.mark.parametrize("k,cin,cout,hw,mb,stride,dg,tile", [
    # data gradients of up to 32 channels, of short reductions, of 3x3 filters into 65..96
    # channels and of 196 tiles: the general kernel
    (1, 32, 512, 91, 4, 1, True, None), (1, 64, 32, 91, 4, 1, True, None), (1, 64, 64, 91, 4, 1, True, "128x64"),
    (1, 96, 192, 91, 4, 1, True, None), (1, 96, 256, 91, 4, 1, True, "96x96"),
    (3, 96, 96, 91, 4, 1, True, None), (3, 64, 256, 56, 4, 1, True, None), (3, 64, 256, 64, 4, 1, True, "64x64"),
    (3, 128, 512, 28, 4, 1, True, None), (3, 64, 512, 28, 4, 1, True, "32x32"),
    # by residue classes: from 257 products on, up to 32 channels from 1025
    (1, 64, 256, 40, 4, 2, True, None), (1, 64, 264, 40, 4, 2, True, "64x64"), (3, 32, 112, 40, 4, 2, True, None),
    (3, 32, 120, 40, 4, 2, True, "128x32"), (1, 128, 64, 91, 4, 2, True, "128x128"), (1, 128, 32, 91, 4, 2, True, None),
    # forwards of up to 32 channels, of at most 32 products, of 196 tiles with long chains
    (1, 288, 32, 91, 4, 1, False, None), (3, 40, 32, 91, 4, 1, False, "128x32"), (3, 64, 32, 60, 4, 1, False, "32x32"),
    (1, 32, 256, 91, 4, 1, False, None), (1, 40, 256, 91, 4, 1, False, "128x128"),
    (3, 400, 64, 56, 4, 1, False, None), (3, 392, 64, 56, 4, 1, False, "64x64")])
def test_lds_copy_kernel_takes_what_it_does_faster(k, cin, cout, hw, mb, stride, dg, tile):
    layers = [bn(-1, cin), relu(0), conv(1, cin, cout, k, stride=stride)]
    f, b = _launches(xp.Stage(layers, mb, 1, (hw, hw, cin), xp.BF16), (hw, hw, cin), mb)
    assert _lds(b if dg else f, dg) == ([] if tile is None else [tile]), (f, b)


@pytest.mark.parametrize("cin,rows64,tile", [
    (16, 200, "32,32"), (16, 300, "32,32"), (16, 469, "64,32"), (32, 469, "64,32"), (64, 469, "32,32"),
    (16, 600, "32,32"), (16, 700, "64,32"),
    (10, 120, "32,32"), (10, 200, "64,32"), (10, 300, "64,32")])
def test_f32_narrow_tiles(cin, rows64, tile):
    """Up to 32 columns in fp32 storage: 32-row tiles where they shorten the last round."""
    shape = (8, rows64, cin)
    f, _ = _launches(xp.Stage([conv(-1, cin, 32, 1)], 8, 1, shape, xp.F32), shape, 8, xp.F32)
    assert any(n.startswith(f"k_conv_gemm<f32,{tile},") for n in f), f


@pytest.mark.parametrize("view", ["aligned", "odd"])
@pytest.mark.parametrize("k,kw,cin,cout,hw,mb,chain", [
    (3, 3, 256, 512, 8, 32, 512), (1, 1, 1024, 512, 8, 32, 512), (3, 3, 256, 256, 4, 32, 128),
    (3, 3, 256, 256, 14, 32, 832), (7, 1, 160, 192, 12, 100, 768),
    (3, 3, 96, 96, 35, 32, 576)])  # 69 of the 74 planned chains hold pixels
def test_weight_gradient_chains(k, kw, cin, cout, hw, mb, chain, view):
    """How many bits a bf16 weight gradient keeps: pixels are summed in chains of
    `chain`, 16 per fp32 addition, and the chains in fp64.  An addition rounds the
    sum so far by 0.41 x 2^-24 of it (rms over a binade), a sum of random terms
    grows with the square root of their count, and so a chain of n additions ends
    0.41 x 2^-24 sqrt(n / 2) off; 0.6 leaves room for roundings inside an addition.
    The same where the output gradient starts at an odd 16 bytes (a concat member
    behind four channels), which takes another kernel."""
    import torch
    layers = [conv(-1, cin, cout, k, kw=kw)]
    if view == "odd":
        layers = [conv(-1, cin, 4, 1), conv(-1, cin, cout, k, kw=kw), dict(kind="concat", inputs=[0, 1])]
    st = xp.Stage(layers, mb, 1, (hw, hw, cin), xp.BF16)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(mb, hw, hw, cin, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(st.out_shape, generator=g, device="cuda").to(torch.bfloat16)
    st.xpipe_predict_weights(xp.BWD, 0, xp.Hyper(), 0)
    st.xpipe_stage_bwd(x, dy, None, torch.empty_like(x))
    off, cnt = st.layout[-1]
    got = st.grad[off:off + cnt].double().reshape(cout, k, kw, cin)
    d = dy.double()[..., -cout:].reshape(-1, cout).t()
    xd = torch.nn.functional.pad(x.double(), (0, 0, kw // 2, kw // 2, k // 2, k // 2))
    ref = torch.stack([torch.stack([d @ xd[:, r:r + hw, q:q + hw].reshape(-1, cin) for q in range(kw)], 1)
                       for r in range(k)], 1)
    assert float((got - ref).norm() / ref.norm()) <= 0.6 * 2.0 ** -24 * (chain / 16 / 2) ** 0.5


def test_bn_partials_of_near_constant_channels():
    """A channel whose values are equal but in a few rows, its mean 2^7 to 2^14 times
    its deviation: the sum of g (z - mean) rstd that a data gradient's epilogue takes.
    The identity filter makes g the output gradient exactly.  A 64-bit sum centred
    before it is formed, stored in fp32: 2^-23 of it."""
    import torch
    c, mb, hw = 64, 4, 91
    st = xp.Stage([bn(-1, c), relu(0), conv(1, c, c, 1)], mb, 1, (hw, hw, c), xp.BF16)
    g = torch.Generator(device="cuda").manual_seed(11)
    x = (2.0 ** torch.arange(c, device="cuda").remainder(12)).expand(mb, hw, hw, c).clone()
    rows = x.view(-1, c)
    for k in range(c):  # one to 64 rows one unit in the last place up
        at = torch.randint(0, rows.shape[0], (1 + k,), generator=g, device="cuda")
        rows[at, k] *= 1 + 2.0 ** -7
    x = x.to(torch.bfloat16)
    (go, gn), (bo, bc), (wo, wn) = st.layout
    st.W[go:go + gn] = 1.0
    st.W[bo:bo + bc] = 1.0  # every output positive
    st.W[wo:wo + wn] = torch.eye(c, device="cuda").reshape(-1)
    for d in (xp.FWD, xp.BWD):
        st.xpipe_predict_weights(d, 0, xp.Hyper(), 0)
    dy = torch.randn(mb, hw, hw, c, generator=g, device="cuda").to(torch.bfloat16)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    st.xpipe_stage_fwd(x, y)
    st.set_timing(True)
    st.xpipe_stage_bwd(x, dy, None, dx)
    torch.cuda.synchronize()
    assert any(n.startswith("k_conv_gemm_lds<128,64,4,2,64,2,false,0,true") for n in st.timing()), list(st.timing())
    X, G = x.double().reshape(-1, c), dy.double().reshape(-1, c)
    xhat = (X - X.mean(0)) * (X.var(0, unbiased=False) + 1e-5).rsqrt()
    ref = (G * xhat).sum(0)
    assert float(((st.grad[go:go + gn].double() - ref) / ref).abs().max()) <= 2.0 ** -23
    ref = G.sum(0)
    assert float(((st.grad[bo:bo + bc].double() - ref) / ref).abs().max()) <= 2.0 ** -23


@pytest.mark.parametrize("cout", [64, 136])
def test_wide_data_gradient_tile(cout):
    """256 x 256 tiles (rows of 256 columns in one workgroup): the masked data
    gradient of a 1 x 1 convolution over 262 160 rows, against fp64 products.
    Bound per value: half a unit in bf16's last place (8 significant bits: 2^-8 of
    the value) of a sum that `cout` fp32 additions left within cout x 2^-24 of the sum
    of its terms' magnitudes."""
    import torch
    mb, hw, cin = 5, (214, 245), 256
    st = xp.Stage([relu(-1), conv(0, cin, cout, 1)], mb, 1, hw + (cin,), xp.BF16)
    g = torch.Generator(device="cuda").manual_seed(3)
    W = (torch.randn(cout, cin, generator=g, device="cuda") / 16).to(torch.bfloat16).float()
    st.W[:cout * cin] = W.reshape(-1)
    for d in (xp.FWD, xp.BWD):
        st.xpipe_predict_weights(d, 0, xp.Hyper(), 0)
    x = torch.randn(mb, *hw, cin, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(mb, *hw, cout, generator=g, device="cuda").to(torch.bfloat16)
    dx = torch.empty_like(x)
    st.set_timing(True)
    st.xpipe_stage_bwd(x, dy, None, dx)
    torch.cuda.synchronize()
    assert any(n.startswith("k_conv_gemm_lds<256,256,") for n in st.timing()), list(st.timing())
    ref = (dy.double().reshape(-1, cout) @ W.double()) * (x.reshape(-1, cin) > 0)
    summed = cout * 2.0 ** -24 * (dy.double().abs().reshape(-1, cout) @ W.double().abs())
    d = (dx.reshape(-1, cin).double() - ref).abs()
    assert bool((d <= 2.0 ** -8 * (ref.abs() + summed) + summed).all()), float(d.max())
    assert rel_l2(np.asarray(st.get_tensors(st.grad)[0]),
                  (dy.double().reshape(-1, cout).t() @ x.double().relu().reshape(-1, cin)).cpu().numpy().ravel()) <= 2e-3
