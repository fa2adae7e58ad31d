"""Layers whose residual and output are turned into rows in LDS among other lanes' launches (csrc/conv_common.h, bn_row): against the oracle, and beside
the same layers launch after launch, which load and store from the accumulators."""
import numpy as np
import pytest

import oracle
import synth
from synth import nets as N
from synth import weights as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ens():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2208_14049_amd as e
    e.lib()
    return e


def layers(i, h, w, c):
    """1x1 layers of all tiles with and without residual, pre-activated ones, the 3x3 of 64 channels, bottlenecks of 64 and 128 channels; output channels
    that end within a run of rows (c + 200 is no multiple of 32), output into a part of a wider tensor."""
    n = N.Net("rows%d" % i, h, w, 16, dtype="bf16")
    x = n.conv(0, 64, 1)
    y = n.conv(x, c + 200, 1)
    y = n.conv(y, c + 200, 1, res=y)
    y = n.conv(n.conv(y, 232, 1), 232, 1, act="silu")
    y = n.conv(y, 232, 1, res=y)
    cat = n.tensor(h, w, 640 + 32)
    n.conv(y, 640, 1, dst=(cat, 0))
    n.conv(n.conv(cat, 128, 1, pre=True, src_slice=(0, 640)), 32, 3, dst=(cat, 640))   # a dense-block layer, as two launches
    t = n.conv(cat, 64, 1)
    t = n.conv(t, 64, 3, res=t)
    t = n.conv(t, 64, 3)
    for width in (64, 128):
        for r in range(2):
            short = t if r else n.conv(t, 2 * width, 1, act=None)
            t = n.conv(n.conv(n.conv(t, width, 1), width, 3), 2 * width, 1, res=short, gamma=0.25)
    n.fc(n.gap(t), 16)
    return n


def strips(i, h, w):
    """3x3 layers of 64 channels on maps of more than 62 columns, with and without residual, with a second and a half-empty tile of channels."""
    n = N.Net("strips%d" % i, h, w, 16, dtype="bf16")
    t = n.conv(0, 64, 1)
    t = n.conv(t, 64, 3, res=t)
    t = n.conv(t, 64, 3, act="silu")
    t = n.conv(n.conv(t, 96 + 32 * (i % 2), 3), 64, 1)
    t = n.conv(t, 64, 3, res=t, gamma=0.25)
    n.fc(n.gap(t), 16)
    return n


def test_rows_in_strips(ens):
    """Maps that are walked in strips of columns, the last one narrower: residuals and outputs in rows among other lanes' launches, and without."""
    nets = [strips(i, h, w) for i, (h, w) in enumerate([(9, 67), (12, 130), (11, 63), (10, 125)])]
    blobs = [W.quantise_weights_bf16(net, W.make_blob(net, synth.BASE_SEED + 73, i)) for i, net in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(synth.BASE_SEED + 1073, 80, 12, 130, varied=True))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(12, 130)
    E.ens_set_alloc([[40] * 4])
    pooled = [net.ops[-2]["src"] for net in nets]

    def ask():
        y = E.ens_predict(imgs)
        return [y] + [E.ens_member_logits(m, 80) for m in range(4)] + [E.ens_debug_tensor(m, pooled[m], net.tensors[pooled[m]], 40) for m, net in enumerate(nets)]

    among = ask()
    rows = E.ens_debug_stats()["rows"]
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    E.ens_set_profiling(0)
    # four such layers in each of four members' two batches, all of which took their rows, in both requests
    assert ran["conv3x3_wreg_bf16<128,c64>"] == 32 and rows >= 32 and E.ens_debug_stats()["rows"] == 2 * rows, (rows, ran, E.ens_debug_stats())
    E.ens_debug_rows(0)
    apart = ask()
    assert E.ens_debug_stats()["rows"] == 2 * rows
    for a, b in zip(among, apart):
        assert np.array_equal(a, b)
    E.close()
    for m, net in enumerate(nets):
        ref = oracle.forward_logits(net, blobs[m], oracle.resize_bilinear(imgs, net.in_h, net.in_w), real="f32")
        # some eight bf16 roundings of 2^-9 one after the other: less than the members above have
        assert np.abs(among[1 + m] - ref).max() <= 0.08 * ref.std(), net.name


@pytest.mark.parametrize("images", [25, 37], ids=str)             # (pixels that end within a row of a tile, in different places)
def test_rows(ens, images):
    nets = [layers(i, h, w, c) for i, (h, w, c) in enumerate([(29, 27, 8), (27, 31, 40), (30, 26, 56), (25, 33, 72)])]
    blobs = [W.quantise_weights_bf16(net, W.make_blob(net, synth.BASE_SEED + 71, i)) for i, net in enumerate(nets)]
    # two batches: a request of one would run as chains
    imgs = W.round_bf16(W.make_images(synth.BASE_SEED + 1071, 2 * images, 29, 27, varied=True))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(29, 27)
    E.ens_set_alloc([[images] * 4])
    pooled = [net.ops[-2]["src"] for net in nets]

    def ask():
        y = E.ens_predict(imgs)                                   # and the map in front of the pooling
        return [y] + [E.ens_member_logits(m, 2 * images) for m in range(4)] + [E.ens_debug_tensor(m, pooled[m], net.tensors[pooled[m]], images) for m, net in enumerate(nets)]

    among = ask()
    rows = E.ens_debug_stats()["rows"]
    assert E.ens_debug_stats()["chained"] == 0
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    E.ens_set_profiling(0)
    print(ran, flush=True)
    in_rows = ("conv1x1_direct_bf16<128x128>", "conv1x1_direct_bf16<128x256>", "conv1x1_pre_bf16<128x128>", "conv3x3_wreg_bf16<128,c64>",
               "bottleneck_bf16<c64>", "bottleneck_bf16<c128>")
    for name in in_rows:
        assert name in ran, (name, ran)
    # every launch of theirs took its rows, in both requests; with the turn switched off none does, and nothing else changes
    assert rows == sum(ran[name] for name in in_rows) and E.ens_debug_stats()["rows"] == 2 * rows, (rows, E.ens_debug_stats())
    E.ens_debug_rows(0)
    apart = ask()
    assert E.ens_debug_stats()["rows"] == 2 * rows
    E.ens_debug_rows(1)
    for a, b in zip(among, apart):
        assert np.array_equal(a, b)
    E.ens_debug_one_stream(1)
    alone = ask()
    E.close()
    for m, net in enumerate(nets):
        ref = oracle.forward_logits(net, blobs[m], oracle.resize_bilinear(imgs, net.in_h, net.in_w), real="f32")
        # some 15 bf16 roundings of 2^-9 one after the other, as for the members
        assert np.abs(among[1 + m] - ref).max() <= 0.08 * ref.std(), net.name
    # Alone other kernels may take a layer and add its sums up in another order, which flips roundings of 2^-8 of a value, some 15 layers deep, at values
    # of up to six spreads; 16 bytes in a wrong place are an error of the size of the spread
    for a, b in zip(among[1:], alone[1:]):
        assert np.abs(a - b).max() <= 0.2 * b.std(), (float(np.abs(a - b).max()), float(b.std()))
    assert np.abs(among[0] - alone[0]).max() <= 2e-2
