"""Requests of small fp32 members that run with every tensor in LDS (csrc/resident.hip): against the oracle in float64 and beside the launches."""
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


def windows(classes=7):
    """Convolutions that take 2 x 2 windows or the mean along: fewer and more channels than a tile of 16, a pair of tiles and one channel more, K of
    no whole step, an image of another size than the request's."""
    n = N.Net("windows", 26, 20, classes, dtype="fp32")
    t = n.maxpool(n.conv(0, 5, 5, act="silu"), 2, 2)
    t = n.avgpool(n.conv(t, 33, (1, 7)), 2, 2)                   # 13 rows: the last belongs to no window
    t = n.conv(t, 16, 1, act=None)
    n.fc(n.gap(n.conv(t, 35, 3)), classes)
    return n


def plain(classes=7):
    """What runs by itself: pools of three with padding, strides, a layer without padding, a tensor that two layers read, a mean over a pool."""
    n = N.Net("plain", 19, 23, classes, dtype="fp32")
    t = n.maxpool(n.conv(0, 17, 3, stride=2, bn=False), 3, 2, 1)
    t = n.conv(t, 20, 2, pad="valid", act="silu")
    t = n.avgpool(n.conv(t, 3, 3), 3, 1, 1)
    n.fc(n.gap(n.maxpool(n.conv(t, 40, 1), 2, 1)), classes)
    return n


# one image; fewer than workgroups; pieces of 1024 of a host's images and part of one; several batches a worker and members with two workers
@pytest.mark.parametrize("n,rows", [(1, [[8, 8, 8, 8]]), (37, [[8, 8, 8, 8], [8, 16, 0, 8]]), (1061, [[32, 16, 32, 32]])], ids=str)
def test_members_in_lds(ens, n, rows):
    import torch
    nets = [N.tiny_a(classes=7), N.tiny_b(classes=7), windows(), plain()]
    blobs = [W.make_blob(net, synth.BASE_SEED + 51, i) for i, net in enumerate(nets)]
    imgs = W.make_images(synth.BASE_SEED + 1051, n, 32, 32, varied=True)
    z_ref = [oracle.forward_logits(net, b, oracle.resize_bilinear(imgs, net.in_h, net.in_w), real="f64") for net, b in zip(nets, blobs)]
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(32, 32)
    E.ens_set_alloc(rows)
    d = torch.from_numpy(imgs).cuda()
    first = E.ens_predict(d.clone()).cpu().numpy()
    z = [E.ens_member_logits(m, n) for m in range(len(nets))]
    assert np.array_equal(E.ens_predict(imgs), first)
    out = torch.empty((n, E.classes), device="cuda")
    E.ens_predict_static(d, out)
    assert np.array_equal(out.cpu().numpy(), first)
    assert E.ens_debug_stats()["chained"] == 3, E.ens_debug_stats()
    kept = [op["dst"] for op in nets[3].ops[:-1]]
    got = {t: E.ens_debug_tensor(3, t, nets[3].tensors[t], 1) for t in (0, kept[-1])}
    E.ens_debug_one_stream(1)
    assert np.abs(E.ens_predict(imgs) - first).max() <= 1e-6
    for t in got:
        assert np.abs(E.ens_debug_tensor(3, t, nets[3].tensors[t], 1) - got[t]).max() <= 1e-5, t
    assert E.ens_debug_stats()["chained"] == 3
    for m, net in enumerate(nets):
        # sums of K <= 300 products leave some sqrt(K) 2^-24 = 1e-6 of a value each, over six layers and the largest of many: 4e-5
        std = z_ref[m].std() if n > 1 else 1.0
        err, launches = (float(np.abs(x - z_ref[m]).max() / std) for x in (z[m], E.ens_member_logits(m, n)))
        print("%s: logits max-abs err / std %.2e, by launches %.2e" % (net.name, err, launches), flush=True)
        assert err <= 4e-5, (net.name, err)
    E.close()


def test_values_that_are_no_numbers(ens):
    """An infinity, a NaN and the largest numbers in some images leave the others alone, and what they give is what the launches give."""
    nets = [N.tiny_a(classes=7), windows(), plain()]
    blobs = [W.make_blob(net, synth.BASE_SEED + 53, i) for i, net in enumerate(nets)]
    imgs = W.make_images(synth.BASE_SEED + 1053, 9, 32, 32, varied=True)
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(32, 32)
    E.ens_set_alloc([[8, 8, 8]])
    E.ens_predict(imgs)
    clean = [E.ens_member_logits(m, 9) for m in range(3)]
    imgs[2, 5, 7, 1], imgs[4, 31, 31, :], imgs[6, :, 3, 0] = np.inf, np.nan, -3.4e38
    E.ens_predict(imgs)
    z = [E.ens_member_logits(m, 9) for m in range(3)]
    assert E.ens_debug_stats()["chained"] == 2
    E.ens_debug_one_stream(1)
    E.ens_predict(imgs)
    for m, net in enumerate(nets):
        assert np.array_equal(z[m][[0, 1, 3, 5, 7, 8]], clean[m][[0, 1, 3, 5, 7, 8]]), net.name
        np.testing.assert_allclose(z[m], E.ens_member_logits(m, 9), rtol=1e-4, atol=1e-4, err_msg=net.name)
    E.close()


# Two neighbouring pixels in a tile: 1, 4, 5 and 8 channels, filters of 2 columns and of 7, K a column longer of no whole step and of whole fours, an odd
# number of columns and windows of less than and more than 32; an infinity or a NaN reaches what the filters reach and nothing else.
@pytest.mark.parametrize("size,width,k,act,pool", [((32, 32), 8, 5, "relu", "avg"), ((9, 19), 4, (1, 2), None, "max"), ((13, 30), 5, (4, 3), "silu", "avg"),
                                                   ((23, 8), 1, (2, 7), "relu", "max")], ids=str)
def test_two_pixels_in_a_tile(ens, size, width, k, act, pool):
    net = N.Net("pair", size[0], size[1], 5, dtype="fp32")
    t = net.conv(0, width, k, act=act)
    t = net.avgpool(t, 2, 2) if pool == "avg" else net.maxpool(t, 2, 2)
    net.fc(net.gap(net.conv(t, 9, 1, act=None)), 5)
    blob = W.make_blob(net, synth.BASE_SEED + 57, 0)
    imgs = W.make_images(synth.BASE_SEED + 1057, 12, size[0], size[1], varied=True)
    ref = oracle.forward_logits(net, blob, imgs, real="f64")
    E = ens.Ensemble([net], [blob])
    E.set_base_size(*size)
    E.ens_set_alloc([[8]])
    E.ens_predict(imgs)
    z = E.ens_member_logits(0, 12)
    assert E.ens_debug_stats()["chained"] == 1
    assert np.abs(z - ref).max() <= 4e-5 * ref.std()             # sqrt(K <= 75) 2^-24 of a value, three layers, the largest of many
    bad = imgs.copy()
    bad[1, 0, 1, 0], bad[5, size[0] - 2, size[1] - 2, 2], bad[9, 3, 4, :] = np.inf, np.nan, -np.inf
    E.ens_predict(bad)
    zb = E.ens_member_logits(0, 12)
    pooled = E.ens_debug_tensor(0, t, net.tensors[t], 1)
    E.ens_debug_one_stream(1)
    E.ens_predict(bad)
    rest = [i for i in range(12) if i not in (1, 5, 9)]
    assert np.array_equal(zb[rest], z[rest])
    np.testing.assert_allclose(zb, E.ens_member_logits(0, 12), rtol=1e-4, atol=1e-4)
    np.testing.assert_allclose(pooled, E.ens_debug_tensor(0, t, net.tensors[t], 1), rtol=1e-5, atol=1e-5)
    E.close()


def test_images_drawn_in_turn(ens):
    """More images than two for each workgroup: every one is computed once, request after request, with smaller ones between them, and in pieces of 1 024 from
    host memory, the last one shorter."""
    import torch
    nets = [N.tiny_a(classes=7), N.tiny_b(classes=7)]
    blobs = [W.make_blob(net, synth.BASE_SEED + 59, i) for i, net in enumerate(nets)]
    few = W.make_images(synth.BASE_SEED + 1059, 41, 32, 32, varied=True)
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(32, 32)
    E.ens_set_alloc([[32, 32]])
    want = E.ens_predict(few)
    for n in (1025, 41, 1600, 1600, 513):                        # 512 workgroups
        imgs = torch.from_numpy(np.ascontiguousarray(few[np.arange(n) % 41])).cuda()
        out = torch.empty((n, E.classes), device="cuda")
        for _ in range(3):
            out.fill_(-1)
            E.ens_predict_static(imgs, out)
            assert np.array_equal(out.cpu().numpy(), want[np.arange(n) % 41]), n
    assert E.ens_debug_stats()["chained"] == 16                  # all of them ran in LDS
    for n in (2600, 41, 2049, 2600):
        assert np.array_equal(E.ens_predict(np.ascontiguousarray(few[np.arange(n) % 41])), want[np.arange(n) % 41]), n
    assert E.ens_debug_stats()["chained"] == 20
    E.close()
