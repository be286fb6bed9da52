"""fp16 convs whose results two entry points promise to the bit: a strided conv by itself and with the 1x1 shortcut conv beside it
as a centre-tap segment of its launch, and a network with its shortcut convs beside their sibling convs or behind them."""
import numpy as np
import pytest
import torch

from workloads import inputs, nets

STRIDED = [(n, c, hw) for n in (1, 2, 4, 8) for c, hw in ((64, 57), (128, 28), (256, 14), (384, 9))]


@pytest.mark.parametrize("n,c,hw", STRIDED)
def test_strided_convs_keep_the_order_of_the_merged_launch(n, c, hw):
    """(host only) The merged launch is the staged kernel's at any size, so the conv by itself has to be, too."""
    from paper_1904_08368_amd import binding as B
    for r in (1, 3, 5):
        d = B.conv_desc(n, c, hw, hw, 2 * c, r, r, 2, r // 2, B.RELAY_F16, B.RELAY_NHWC, B.HAS_BN | B.RELU)
        assert "igemm_dma_kernel" in B.relay_conv2d_kernel_name(d)


@pytest.mark.gpu
@pytest.mark.parametrize("n,c,hw", STRIDED)
def test_merged_shortcut_gives_the_bits_of_separate_launches(n, c, hw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as G
    from tests.test_gpu_combine import _run_windows
    of, oc = nets.conv("a", "x", "a", c, 256, 3, 2, 1), nets.conv("d", "x", "d", c, 128, 1, 2, 0, relu=False)
    pf, pc = inputs.layer_params(of, 41, c + n, "f16"), inputs.layer_params(oc, 41, c + n + 1, "f16")
    x = inputs.activation(41, c, (n, c, hw, hw), "f16")
    (ya, yd), _ = _run_windows(G, x, (of, pf), (oc, pc), 2)
    assert np.array_equal(ya.view(np.uint16), G.run_conv_f16(x, pf["w"], 2, 1, scale=pf["scale"], shift=pf["shift"], relu=True).view(np.uint16))
    assert np.array_equal(yd.view(np.uint16), G.run_conv_f16(x, pc["w"], 2, 0, scale=pc["scale"], shift=pc["shift"]).view(np.uint16))


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [1, 3])
def test_shortcuts_on_a_side_stream_give_the_same_bits(batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_08368_amd.stack import FusedNet
    ops = nets.resnet18()
    params = inputs.net_params(ops, 3, "f16")
    x = inputs.image(42, batch, 3, 224, 224, "f16")
    outs = []
    for side in (False, True):
        net = FusedNet(ops, params, batch, 224, 224, "f16", overlap_shortcuts=side)
        assert bool(net.side_calls) == side
        net.load_input(x)
        net.run()
        torch.cuda.synchronize()
        outs.append({n: net.tensor(n) for n in net.bufs if n != "x"})
    assert outs[0].keys() == outs[1].keys()
    for name in outs[0]:
        assert np.array_equal(outs[0][name].view(np.uint16), outs[1][name].view(np.uint16)), name


# 32 x 32 tiles: whole and ragged pixels and channels, one chunk and many, all three chunk lengths, a residual
NARROW = [(1, 128, 13, 9, 64, 3, 2, False), (1, 256, 14, 14, 40, 3, 2, True), (2, 64, 15, 17, 100, 3, 2, False), (1, 384, 7, 7, 33, 1, 1, True),
          (1, 128, 1, 1, 8, 1, 1, False), (3, 96, 9, 10, 72, 3, 1, True), (1, 32, 5, 5, 24, 5, 2, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", NARROW)
def test_narrow_tile_gives_the_bits_of_the_other_tiles(shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as G
    n, c, h, w, k, r, st, res = shape
    g = np.random.default_rng(inputs.BASE_SEED + 98000 + c + k)
    x = g.standard_normal((n, c, h, w)).astype(np.float16)
    wt = (g.standard_normal((k, c, r, r)) * np.sqrt(2.0 / (c * r * r))).astype(np.float16)
    ho, wo = ((e + 2 * (r // 2) - r) // st + 1 for e in (h, w))
    p = dict(scale=(1 + 0.1 * g.standard_normal(k)).astype(np.float32), shift=(0.1 * g.standard_normal(k)).astype(np.float32), relu=True,
             residual=g.standard_normal((n, k, ho, wo)).astype(np.float16) if res else None)
    narrow = G.run_conv_f16(x, wt, st, r // 2, tile=18, **p)
    other = G.run_conv_f16(x, wt, st, r // 2, tile=5, **p)
    assert np.array_equal(narrow.view(np.uint16), other.view(np.uint16))
