"""Parity of the HIP path against the CPU oracle, element by element, through the C interface.

Tolerances (from the workload definition): combined probabilities within 1e-4 (fp32 members) or
2e-2 (bf16 members) max-abs, top-1 agreement >= 99.5 %.  Single bf16 layers are compared against
the oracle with a bound derived from the arithmetic: inputs and weights are bf16-exact on both
sides, products are exact in fp32, so the error is the fp32 accumulation order, the rounding of
the folded weights (relative 2^-9 each, a random walk over the K terms, a few 2^-9 of the output
scale at the tail of 10^5 outputs) and the bf16 rounding of the result (8 significant bits: half
an ulp is 2^-8 relative, and a result that lands across a rounding boundary is a whole ulp, 2^-7).
"""
import numpy as np
import pytest

import oracle
import synth
from synth import nets as N
from synth import weights as W

pytestmark = pytest.mark.gpu

TOL_FP32, TOL_BF16, TOP1 = 1e-4, 2e-2, 0.995


@pytest.fixture(scope="module")
def ens():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2208_14049_amd as e
    e.lib()
    return e


def top1_agreement(y_gpu, y_ref, tol):
    """Strict agreement, and agreement up to ties inside the probability tolerance."""
    a, b = np.argmax(y_gpu, 1), np.argmax(y_ref, 1)
    strict = float((a == b).mean())
    near = float((y_ref[np.arange(len(a)), a] >= y_ref.max(1) - tol).mean())
    return strict, near


def prepared(nets, seed, n, size, bf16, varied_from=None):
    """Seeded parameters and images; images from index `varied_from` on get their own contrast and
    offset so that the members' answers (and the arg-max) differ from image to image."""
    blobs = [W.make_blob(net, seed, i) for i, net in enumerate(nets)]
    imgs = W.make_images(seed + 1000, n, size, size)
    if varied_from is not None:
        imgs[varied_from:] = W.make_images(seed + 1000, n - varied_from, size, size, first=varied_from, varied=True)
    if bf16:
        blobs = [W.quantise_weights_bf16(net, b) for net, b in zip(nets, blobs)]
        imgs = W.round_bf16(imgs)
    return blobs, imgs


# --------------------------------------------------------------------------- config 1 (fp32)
def test_config1_fp32_end_to_end(ens):
    nets = N.config_members(1)
    blobs, imgs = prepared(nets, synth.BASE_SEED, 256, 32, bf16=False)
    y_ref, p_ref = oracle.ensemble_predict(nets, blobs, imgs, real="f32")
    E = ens.Ensemble(nets, blobs)
    E.ens_set_alloc([[8, 8]])
    y = E.ens_predict(imgs)
    assert y.shape == (256, 10) and np.isfinite(y).all()
    assert np.abs(y - y_ref).max() <= TOL_FP32
    np.testing.assert_allclose(y.sum(1), 1.0, atol=1e-5)
    strict, near = top1_agreement(y, y_ref, TOL_FP32)
    assert strict >= TOP1 and near == 1.0
    for m in range(2):
        z = E.ens_member_logits(m, 256)
        z_ref = oracle.forward_logits(nets[m], blobs[m], imgs, real="f64")
        assert np.abs(z - z_ref).max() <= 1e-4 * max(1.0, np.abs(z_ref).max())
    # allocation, segment size and request size change the layout, never the value
    for matrix, seg, n in ([[8, 8]], 16, 256), ([[32, 1]], 128, 255), ([[8, 8], [16, 0]], 64, 100), ([[128, 64]], 128, 1):
        E.ens_set_alloc(matrix, seg)
        y2 = E.ens_predict(imgs[:n])
        assert np.abs(y2 - y_ref[:n]).max() <= TOL_FP32
        assert np.abs(y2 - y[:n]).max() <= 2e-6
    E.close()


def test_empty_and_single_requests(ens):
    nets = N.config_members(1)
    blobs, imgs = prepared(nets, 3, 4, 32, bf16=False)
    E = ens.Ensemble(nets, blobs)
    y0 = E.ens_predict(imgs[:0])
    assert y0.shape == (0, 10)
    y1 = E.ens_predict(imgs[:1])
    ref, _ = oracle.ensemble_predict(nets, blobs, imgs[:1], real="f32")
    assert np.abs(y1 - ref).max() <= TOL_FP32
    with pytest.raises(ens.EnsError) as e:
        E.ens_set_alloc([[8, 0]])            # a column of zeros is illegal
    assert e.value.status == ens.ENS_E_INVALID
    E.close()


def test_ensemble_of_one_is_member_softmax(ens):
    nets = N.config_members(1)[:1]
    blobs, imgs = prepared(nets, 5, 16, 32, bf16=False)
    E = ens.Ensemble(nets, blobs)
    y = E.ens_predict(imgs)
    z = E.ens_member_logits(0, 16).astype(np.float64)
    np.testing.assert_allclose(y, oracle.softmax(z), atol=2e-7)
    E.close()


def test_weights_drawn_from_seed_match_the_shared_generator(ens):
    nets = N.config_members(1)
    blobs, imgs = prepared(nets, 77, 16, 32, bf16=False)
    E1 = ens.Ensemble(nets, blobs)
    E2 = ens.Ensemble(nets, None, seed=77)
    y1, y2 = E1.ens_predict(imgs), E2.ens_predict(imgs)
    assert np.abs(y1 - y2).max() <= 1e-6
    E1.close()
    E2.close()


# --------------------------------------------------------------------------- single layers
def layer_net(h, w, cin, build, dtype):
    """[pad conv to cin] -> layer under test -> gap -> fc, so that the layer's output tensor can
    be read back; returns (net, tensor id of the layer output)."""
    n = N.Net("layer", h, w, 8, dtype=dtype)
    t = n.conv(0, cin, 1, bn=False, act=None) if cin != 3 else 0
    t = build(n, t)
    n.fc(n.gap(t), 8)
    return n, t


def oracle_tensor(net, blob, imgs, t):
    outs = []
    for i in range(imgs.shape[0]):
        _, d = oracle.forward_logits(net, blob, imgs[i:i + 1], real="f32", dump_tensor=t)
        outs.append(d)
    return np.stack(outs)


def assert_after_bf16_layers(got, ref, what):
    """Element-wise bound for a tensor that lies two to four bf16 layers behind the last tensor both sides share.
    Each layer rounds its output to bf16 (relative error uniform in +-2^-9, rms 1.1e-3); through random weights
    of unit gain the errors of a layer's inputs add up like a random walk, so an element's error has a standard
    deviation of about sqrt(layers) * 1.1e-3 * rms(ref), doubled where sums cancel: 4e-3 * rms for three layers.
    The largest of 1e5 to 1e6 elements lies five to six deviations out (2.4e-2 * rms), and the element's own
    rounding adds 2^-9 of its size.  Bounds: max <= 3e-2 * rms + 2^-8 * max|ref|, mean <= 2^-7 * rms."""
    scale = np.sqrt(np.mean(ref ** 2)) + 1e-6
    err = np.abs(got - ref)
    assert err.max() <= 0.03 * scale + 2.0 ** -8 * np.abs(ref).max(), (what, err.max(), scale)
    assert err.mean() <= 2.0 ** -7 * scale, (what, err.mean(), scale)


CONV_LAYERS = [
    # (H, W, cin, cout, k, stride, pad, extra)       shapes span several tiles and ragged tails
    (56, 56, 64, 64, 3, 1, "same", {}),
    (64, 64, 3, 64, 7, 2, "same", {}),                         # input stems: run space-to-depth at stride 1
    (35, 35, 3, 32, 3, 2, "valid", {}),
    (32, 48, 3, 24, 3, 2, "same", {"act": "silu"}),
    (28, 28, 128, 128, 3, 1, "same", {}),
    (56, 56, 128, 512, 3, 1, "same", {}),                      # enough tiles for the one-halo-buffer variant
    (150, 150, 64, 32, 3, 1, "same", {}),                      # narrow output, many tiles: the 256x32 tile
    (100, 220, 128, 32, 3, 1, "same", {"act": None}),          # ... with two channel blocks through one halo buffer
    (28, 28, 64, 64, 3, 1, "same", {"res": True}),             # residual read from the layer's own input
    (24, 40, 64, 96, 3, 1, "same", {"act": None}),             # filter-in-registers kernel: half-empty last channel tile
    (12, 12, 64, 128, 3, 1, "same", {"act": "silu"}),          # ... fewer tiles than workgroups
    (62, 62, 64, 32, 3, 1, "same", {}),                        # ... widest rows it takes, one channel group
    (28, 28, 128, 128, 3, 1, "same", {"groups": 32}),          # grouped: 4 channels per group, 8 groups per dense block
    (28, 28, 256, 256, 3, 2, "same", {"groups": 32}),          # ... 8 per group, stride 2
    (14, 14, 512, 512, 3, 1, "same", {"groups": 32, "res": True}),
    (7, 7, 1024, 1024, 3, 1, "same", {"groups": 32}),          # ... a group is a whole 32-channel block
    (14, 14, 128, 256, 3, 1, "same", {"groups": 2}),           # ... groups wider than a block: 64 -> 128 each
    (14, 14, 256, 256, 1, 1, "same", {"res": True}),
    (14, 14, 256, 96, 3, 1, "same", {}),
    (20, 37, 64, 72, 3, 1, "same", {"act": None}),
    (56, 56, 64, 256, 1, 1, "same", {}),
    (28, 28, 128, 128, 3, 2, "same", {}),
    (14, 14, 256, 512, 1, 2, "same", {"act": None}),
    (17, 17, 128, 192, (1, 7), 1, "same", {"ran": "conv1x7_halo_bf16<128,64,c64>"}),   # window-in-LDS kernel, filters along one axis
    (17, 17, 128, 160, (7, 1), 1, "same", {"ran": "conv7x1_halo_bf16<128,64,c64>"}),
    (17, 17, 160, 192, (7, 1), 1, "same", {"ran": "conv7x1_halo_bf16<128,64,c32>"}),   # ... 32-channel blocks
    (17, 17, 160, 160, (1, 7), 1, "same", {"ran": "conv1x7_halo_bf16<128,64,c32>"}),
    (9, 30, 64, 72, (1, 7), 1, "same", {"ran": "conv1x7_halo_bf16<128,64,c64>", "act": None}),   # ... one channel block, wide rows
    (30, 9, 96, 64, (7, 1), 1, "same", {"ran": "conv7x1_halo_bf16<128,64,c32>", "res": False}),
    (35, 35, 48, 64, 5, 1, "same", {}),
    (35, 35, 96, 96, 3, 2, "valid", {}),
    (8, 8, 384, 384, (1, 3), 1, "same", {"ran": "conv1x3_halo_bf16<128,64,c64>"}),
    (8, 8, 448, 384, (3, 1), 1, "same", {"ran": "conv3x1_halo_bf16<128,64,c64>"}),
    (11, 13, 96, 40, (3, 1), 1, "same", {"ran": "conv3x1_halo_bf16<128,64,c32>"}),
    (11, 13, 224, 136, (1, 3), 1, "same", {"ran": "conv1x3_halo_bf16<128,64,c32>"}),
    (28, 28, 40, 240, 1, 1, "same", {"act": "silu"}),
    (28, 28, 192, 32, 3, 1, "same", {"bn": False, "act": None, "bias": False}),
    (28, 28, 160, 128, 1, 1, "same", {"pre": True}),
    (7, 7, 512, 512, 3, 1, "same", {}),
    (7, 7, 2048, 512, 1, 1, "same", {}),
    (9, 9, 24, 1000, 1, 1, "same", {}),
    (13, 13, 192, 96, 1, 1, "same", {"act": "silu"}),          # weights-from-memory 1x1 kernel: three input chunks, half-empty channel tile
    (10, 10, 64, 32, 1, 1, "same", {"act": None}),             # ... one chunk, one block of channels
    (14, 14, 80, 80, 1, 1, "same", {"res": True, "act": None}),    # ... channels in 8s: half-empty last chunk and last block, residual
    (19, 19, 728, 728, 1, 1, "same", {}),                      # ... the pointwise half of a 728-channel separable layer
    (15, 15, 64, 128, 1, 2, "same", {"act": None}),            # ... a strided shortcut on an odd map: every other pixel of every other row
    (28, 28, 512, 1024, 1, 2, "same", {"act": None}),          # ... eight input chunks, 128-wide channel tiles
]


# (case, images): the persistent kernels (input stem, 64-channel 3x3) only walk several tiles per
# workgroup, on the per-XCD runs, when a batch has more tiles than the chip holds workgroups
MANY_TILES = [
    ((56, 56, 64, 128, 3, 1, "same", {}), 24),                  # 610 tiles for 256 workgroups per channel tile
    ((56, 56, 64, 64, 3, 1, "same", {"res": True}), 40),        # 1016 tiles for 512 workgroups, residual
    ((96, 96, 3, 64, 7, 2, "same", {}), 64),                    # stem: 601 tiles of 256 positions for 512 workgroups
    ((56, 56, 64, 160, 1, 1, "same", {}), 6),                   # 1x1 from operand-ordered weights, 128x128 tiles, 32 channels in the last
    ((28, 28, 128, 128, 1, 1, "same", {"res": True}), 48),      # ... with the residual
    ((56, 56, 256, 512, 1, 2, "same", {"act": None}), 6),       # ... strided: tiles that span rows and images of the output
    ((28, 28, 128, 256, 3, 1, "same", {}), 64),                 # window-in-LDS 3x3 kernel with 128 x 128 tiles: 842 of them
    ((17, 17, 192, 192, (1, 7), 1, "same", {"ran": "conv1x7_halo_bf16<128,64,c64>"}), 96),   # ... 1x7 and 7x1: 765 tiles, one halo buffer
    ((17, 17, 192, 192, (7, 1), 1, "same", {"ran": "conv7x1_halo_bf16<128,64,c64>"}), 96),
    ((8, 8, 384, 384, (3, 1), 1, "same", {"ran": "conv3x1_halo_bf16<128,64,c64>"}), 160),    # ... 3x1: 540 tiles
]


@pytest.mark.parametrize("case,nb", [(c, 3) for c in CONV_LAYERS] + MANY_TILES,
                         ids=lambda c: "%dx%dx%d-%d-k%s-s%d" % (c[0], c[1], c[2], c[3], c[4], c[5]) if isinstance(c, tuple) else "n%d" % c)
def test_conv_layer_bf16(ens, case, nb):
    h, w, cin, cout, k, stride, pad, extra = case
    extra = dict(extra)
    with_res = extra.pop("res", False)
    ran = extra.pop("ran", None)                                # the kernel class that has to run the layer
    net, t = layer_net(h, w, cin, lambda n, s: n.conv(s, cout, k, stride=stride, pad=pad,
                                                      res=s if with_res else None, **extra), "bf16")
    blobs, imgs = prepared([net], 11, nb, h, bf16=True)
    imgs = W.round_bf16(W.make_images(4, nb, h, w))
    E = ens.Ensemble([net], blobs)
    E.set_base_size(h, w)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[max(4, nb)]])
    E.ens_set_profiling(1 if ran else 0)
    E.ens_predict(imgs)
    if ran:
        classes = [kk["name"] for kk in E.ens_profile() if kk["launches"]]
        assert ran in classes, classes
    got = E.ens_debug_tensor(0, t, net.tensors[t], nb)
    # feed the oracle the bf16 tensor the GPU layer actually read, so only this layer is compared
    src = net.ops[-3]["src"]
    if src != 0:
        x_in = E.ens_debug_tensor(0, src, net.tensors[src], nb)
        # that tensor itself (the 1x1 lift of the image to cin channels) against the oracle's from the image
        x_ref = oracle_tensor(net, blobs[0], imgs, src)
        x_scale = np.sqrt(np.mean(x_ref ** 2))
        assert x_scale > 0.1 and (np.abs(x_in - x_ref) <= 2.0 ** -7 * np.abs(x_ref) + x_scale * 2.0 ** -5 + 1e-6).all()
        sub = N.Net("sub", h, w, 8, dtype="bf16", in_c=cin)
        sub.ops, sub.params, sub.blob_size = [dict(net.ops[-3])], net.params, net.blob_size
        sub.tensors = [net.tensors[src], net.tensors[t]]
        sub.ops[0].update(src=0, dst=1)
        if with_res:
            sub.ops[0].update(res=0)
        sub.out_tensor = 1
        ref = oracle.forward_logits(sub, blobs[0], x_in, real="f64").reshape(got.shape)
    else:
        ref = oracle_tensor(net, blobs[0], imgs, t)
    E.close()
    kk = (k * k if isinstance(k, int) else k[0] * k[1]) * cin
    scale = np.sqrt(np.mean(ref ** 2)) + 1e-6
    err = np.abs(got - ref)
    bound = 2.0 ** -7 * np.abs(ref) + scale * 2.0 ** -5 + 1e-6     # one bf16 ulp + accumulated weight rounding
    assert (err <= bound).all(), (err.max(), scale, float((err / bound).max()))
    assert err.mean() <= 2.0 ** -8 * scale, (err.mean(), scale, kk)


# Layers from 32 channels to 32, as grouped convolutions are cut into, with the filter in registers: more tiles of 256 positions than workgroups (on
# the per-XCD runs and without), a last tile that is partly empty, rows of one pixel and the widest that the window's table holds, maps of odd
# sides whose tiles span images, parts of 4, 8 and 32 groups, and rows a pixel wider, which the generic kernel keeps.
NARROW = "conv3x3_narrow_bf16<256,c32>"


@pytest.mark.parametrize("case,nb", [
    ((56, 56, 128, 128, 3, 1, "same", {"groups": 32, "ran": NARROW}), 24),
    ((28, 28, 64, 64, 3, 1, "same", {"groups": 16, "ran": NARROW, "act": "silu"}), 130),
    ((14, 13, 512, 512, 3, 1, "same", {"groups": 64, "ran": NARROW, "act": None}), 21),
    ((7, 7, 1024, 1024, 3, 1, "same", {"groups": 32, "ran": NARROW, "bn": False}), 33),
    ((40, 126, 32, 32, 3, 1, "same", {"ran": NARROW}), 24),
    ((300, 1, 32, 32, 3, 1, "same", {"ran": NARROW}), 400),
    ((40, 127, 32, 32, 3, 1, "same", {"ran": "conv_igemm_bf16<128,32,k64>"}), 24),
], ids=lambda c: "%dx%dx%d" % c[:3] if isinstance(c, tuple) else "n%d" % c)
def test_filter_in_registers_32_channels(ens, case, nb):
    test_conv_layer_bf16(ens, case, nb)


# 64-channel layers in strips of columns: the widest rows that need none, two strips of 32 and 31, three with a last one that is narrower, rows of whole
# strips, a second and a half-empty channel tile, a residual, and one image (fewer tiles than workgroups).
WREG = "conv3x3_wreg_bf16<128,c64>"


@pytest.mark.parametrize("case,nb", [
    ((33, 62, 64, 64, 3, 1, "same", {"ran": WREG}), 9),
    ((33, 63, 64, 64, 3, 1, "same", {"ran": WREG, "res": True}), 9),
    ((20, 143, 64, 96, 3, 1, "same", {"ran": WREG, "act": "silu"}), 7),
    ((9, 122, 64, 160, 3, 1, "same", {"ran": WREG, "act": None}), 40),
    ((224, 224, 64, 64, 3, 1, "same", {"ran": WREG}), 1),
], ids=lambda c: "%dx%dx%d" % c[:3] if isinstance(c, tuple) else "n%d" % c)
def test_filter_in_registers_strips(ens, case, nb):
    test_conv_layer_bf16(ens, case, nb)


def test_two_convolutions_in_one_launch(ens):
    """A residual block's strided 3x3 convolution and its 1x1 shortcut read the same tensor and write
    same-sized outputs: the engine runs them as one launch (argument blocks of both).  Both outputs
    are read back and compared with the oracle; so is a pair the engine must not put together (the
    second reads the first)."""
    n = N.Net("pair", 28, 28, 8, dtype="bf16")
    t = n.conv(0, 64, 3)
    a = n.conv(t, 128, 1, stride=2, act=None)                    # shortcut
    b = n.conv(t, 128, 3, stride=2)                              # branch, same input: one launch with a
    c = n.conv(b, 128, 3, res=a)
    d = n.conv(c, 128, 1, act=None)
    e = n.conv(d, 128, 1)                                        # reads d: not a pair
    cat = n.tensor(14, 14, 64 + 96)                              # two branch heads into slices of one tensor,
    n.conv(e, 64, 1, dst=(cat, 0))                               # different widths: a pair again
    n.conv(e, 96, 1, dst=(cat, 64), act=None)
    e = n.conv(cat, 128, 1)
    n.fc(n.gap(e), 8)
    nb = 5
    blobs, _ = prepared([n], 13, nb, 28, bf16=True)
    imgs = W.round_bf16(W.make_images(6, nb, 28, 28))
    E = ens.Ensemble([n], blobs)
    E.set_base_size(28, 28)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[8]])
    E.ens_predict(imgs)
    got = {x: E.ens_debug_tensor(0, x, n.tensors[x], nb) for x in (a, b, c, cat, e)}
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    conv_launches = sum(k["launches"] for k in E.ens_profile() if k["name"].startswith("conv"))
    E.close()
    assert conv_launches == 7, conv_launches                   # nine convolutions, two pairs
    for x in (a, b, c, cat, e):
        ref = oracle_tensor(n, blobs[0], imgs, x)
        assert_after_bf16_layers(got[x], ref, (x,))


def test_pointwise_layers_of_a_gang(ens):
    """Two members of the same shape run every layer as one launch with two argument blocks; their 1x1
    layers (64 -> 128 with 128-channel tiles, 128 -> 64 with 64-channel tiles and a residual) go to the
    kernel that reads operand-ordered weights.  Each member's tensors are compared with the oracle."""
    nets = []
    for g in range(2):
        n = N.Net("pw%d" % g, 20, 20, 8, dtype="bf16")
        x = n.conv(0, 64, 3)
        a = n.conv(x, 128, 1, act="silu")
        b = n.conv(a, 64, 1, res=x)
        n.fc(n.gap(b), 8)
        nets.append(n)
    nb = 7
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 41, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(42, nb, 20, 20))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(20, 20)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[8, 8]])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    got = [[E.ens_debug_tensor(g, t, nets[g].tensors[t], nb) for t in (a, b)] for g in range(2)]
    E.close()
    assert ran.get("conv1x1_direct_bf16<128x64>") == 2, ran        # both layers: 22 tiles of 128 x 128 are fewer than the compute units
    for g in range(2):
        for t, y in zip((a, b), got[g]):
            ref = oracle_tensor(nets[g], blobs[g], imgs, t)
            assert_after_bf16_layers(y, ref, (g, t,))


@pytest.mark.parametrize("h,w,cout,G,nb", [(64, 64, 64, 1, 5), (70, 54, 64, 1, 7), (96, 96, 64, 2, 40), (60, 60, 96, 1, 9), (224, 224, 64, 1, 3)],
                         ids=["64x64", "70x54_odd_maps", "96x96_gang2_many_bands", "60x60_96_channels", "224x224"])
def test_stem_and_max_pool_in_one_kernel(ens, h, w, cout, G, nb):
    """The 7x7 / stride-2 stem with ReLU and the 3x3 / stride-2 / padding-1 max-pool behind it run as one
    kernel that keeps the stem's output in LDS.  The pooled map is read back and compared with the oracle
    element by element, for each member of the gang; the profile says that the fused kernel ran and that
    no separate pooling kernel did.  Shapes: odd stem output sizes (35 x 27: the last pooled row and column
    reach past the map), more bands than workgroups, a second, half-empty channel tile, the full 224 x 224."""
    nets = []
    for g in range(G):
        n = N.Net("sp%d" % g, h, w, 8, dtype="bf16")
        x = n.conv(0, cout, 7, stride=2)
        pooled = n.maxpool(x, 3, 2, 1)
        n.fc(n.gap(pooled), 8)
        nets.append(n)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 91, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(92, nb, h, w))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(h, w)
    E.ens_set_alloc([[nb] * G])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    got = [E.ens_debug_tensor(g, pooled, nets[g].tensors[pooled], nb) for g in range(G)]   # alive until the global pooling
    E.close()
    assert ran.get("stem_pool_bf16<4x4>") == 1 and "window_kernel<maxpool>" not in ran, ran
    for g in range(G):
        ref = oracle_tensor(nets[g], blobs[g], imgs, pooled)
        scale = np.sqrt(np.mean(ref ** 2)) + 1e-6
        err = np.abs(got[g] - ref)
        bound = 2.0 ** -7 * np.abs(ref) + scale * 2.0 ** -5 + 1e-6     # one bf16 ulp + accumulation order, as for a single convolution
        assert (err <= bound).all(), (g, float(err.max()), float(scale), float((err / bound).max()))
        assert err.mean() <= 2.0 ** -8 * scale


@pytest.mark.parametrize("h,w,nb", [(2016, 224, 1), (2500, 46, 2)], ids=["2016x224", "2500x46_two_images"])
def test_stem_and_max_pool_of_tall_images(ens, h, w, nb):
    """Stem maps of more than a thousand rows: the gap columns between rows are padding in every band of the image, the last
    ones among them.  Compared row by row, since a fault of one band would drown in a mean over the map."""
    n = N.Net("tall", h, w, 8, dtype="bf16")
    pooled = n.maxpool(n.conv(0, 64, 7, stride=2), 3, 2, 1)
    n.fc(n.gap(pooled), 8)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 93, 0))]
    imgs = W.round_bf16(W.make_images(94, nb, h, w))
    E = ens.Ensemble([n], blobs)
    E.set_base_size(h, w)
    E.ens_set_alloc([[nb]])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    got = E.ens_debug_tensor(0, pooled, n.tensors[pooled], nb)
    E.close()
    assert ran.get("stem_pool_bf16<4x4>") == 1, ran
    ref = oracle_tensor(n, blobs[0], imgs, pooled)
    scale = np.sqrt(np.mean(ref ** 2)) + 1e-6
    ratio = np.abs(got - ref) / (2.0 ** -7 * np.abs(ref) + scale * 2.0 ** -5 + 1e-6)   # the bound of the test above
    assert (ratio <= 1.0).all(), np.argwhere(ratio.max(axis=(2, 3)) > 1.0)[:10]


# (C, H, W, cin, cout, residual, activation of the last convolution, members in the gang, images, batch)
BOTTLENECKS = [
    (64, 24, 24, 256, 256, "input", "relu", 1, 56, 64),        # identity block, short last batch
    (64, 24, 24, 256, 256, "input", "relu", 2, 28, 28),        # two members in one launch
    (64, 20, 30, 64, 128, "branch", "relu", 1, 51, 51),        # projection shortcut, non-square, one channel pass
    (64, 9, 62, 96, 384, None, None, 1, 53, 53),               # widest raster the window holds, no residual, no activation
    (128, 28, 28, 128, 128, "input", "relu", 1, 40, 40),
    (128, 30, 30, 64, 256, "branch", "silu", 1, 35, 35),
    (128, 13, 17, 256, 256, "input", None, 2, 66, 66),
]


@pytest.mark.parametrize("case", BOTTLENECKS, ids=lambda c: "c%d_%dx%d_%d-%d_%s_g%d" % (c[0], c[1], c[2], c[3], c[4], c[5], c[7]))
def test_bottleneck_in_one_kernel(ens, case):
    """A residual bottleneck (1x1, 3x3, 1x1 with the residual) runs as one kernel that keeps the two
    tensors in between on chip.  The block's output is read back and compared with the oracle element
    by element, for each member of the gang; the profile says that the fused kernel ran."""
    C, H, Wd, cin, cout, res, act3, G, n_img, batch = case
    nets = []
    for g in range(G):
        n = N.Net("bneck%d" % g, H, Wd, 8, dtype="bf16")
        x = n.conv(0, cin, 3)
        idt = None
        if res == "input":
            idt = x
        elif res == "branch":
            idt = n.conv(x, cout, 1, act=None)
            x = n.conv(x, cin, 1)                                # keeps the shortcut and the block's head apart
        u = n.conv(x, C, 1)
        u = n.conv(u, C, 3)
        y = n.conv(u, cout, 1, res=idt, act=act3)
        n.fc(n.gap(y), 8)
        nets.append(n)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 31, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(32, n_img, H, Wd))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(H, Wd)
    E.ens_set_alloc([[batch] * G])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    # the block's output is alive until the pooling that ends the network: still there after the pass
    got = [E.ens_debug_tensor(g, y, nets[g].tensors[y], n_img) for g in range(G)]
    E.close()
    assert ran.get("bottleneck_bf16<c%d>" % C) == 1, ran
    for g in range(G):
        ref = oracle_tensor(nets[g], blobs[g], imgs, y)
        # three bf16 layers in a row: roundings of the two middle tensors carry into the third
        assert_after_bf16_layers(got[g], ref, (g,))


@pytest.mark.parametrize("h,w,c0,layers,G,nb", [(14, 14, 64, 3, 1, 16), (10, 40, 96, 2, 2, 5), (7, 7, 256, 2, 1, 50),
                                                (20, 20, 64, 2, 1, 6), (14, 14, 32, 1, 1, 150)],
                         ids=["14x14", "10x40_gang2", "7x7_256", "20x20_tiles_of_64", "14x14_many_tiles"])
def test_dense_block_layers_in_one_kernel(ens, h, w, c0, layers, G, nb):
    """A layer of a dense block (pre-activated 1x1 to 128 channels, then 3x3 to 32 channels appended to the
    block's tensor) runs as one kernel with the 128-channel tensor in LDS.  The block's tensor is read
    back after the pass and compared with the oracle element by element, for each member of the gang.
    The cases cover the kernel's tiles of 32 positions (14x14, 7x7), 64 (20x20) and 128 (window of 256
    rows: 10x40; of 192 rows: 14x14 with enough tiles for every compute unit)."""
    nets = []
    for g in range(G):
        n = N.Net("dense%d" % g, h, w, 8, dtype="bf16")
        blk = n.tensor(h, w, c0 + 32 * layers)
        n.conv(0, c0, 3, dst=(blk, 0))
        c = c0
        for _ in range(layers):
            u = n.conv(blk, 128, 1, pre=True, src_slice=(0, c))
            n.conv(u, 32, 3, bn=False, act=None, bias=False, dst=(blk, c))
            c += 32
        n.fc(n.gap(blk, pre=True), 8)
        nets.append(n)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 51, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(52, nb, h, w))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(h, w)
    E.ens_set_alloc([[nb] * G])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    got = [E.ens_debug_tensor(g, blk, nets[g].tensors[blk], nb) for g in range(G)]   # alive until the pooling that ends the network
    E.close()
    assert ran.get("dense_layer_bf16") == layers, ran
    for g in range(G):
        ref = oracle_tensor(nets[g], blobs[g], imgs, blk)
        assert_after_bf16_layers(got[g], ref, (g,))


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_memory_bound_layers(ens, dtype):
    """Depthwise 3x3 / 5x5 (strides 1 and 2), squeeze-excite, max / average pooling into channel
    slices, pre-activated global pooling: one network that chains them, read back per tensor."""
    bf = dtype == "bf16"
    n = N.Net("mb", 30, 30, 16, dtype=dtype)
    t1 = n.conv(0, 32, 3, act="silu")
    t2 = n.dwconv(t1, 3, 1)
    t3 = n.se(t2, 8)
    t4 = n.dwconv(t3, 5, 2)                      # 15 x 15
    cat = n.tensor(7, 7, 32 + 32 + 16)
    n.maxpool(t4, 3, 2, 0, dst=(cat, 0))
    n.avgpool(t4, 3, 2, 0, dst=(cat, 32))
    t5 = n.avgpool(t4, 3, 1, 1)                  # 15 x 15, windows clipped at the border
    t6 = n.maxpool(t5, 3, 2, 1)                  # 8 x 8
    n.conv(t6, 16, 2, pad="valid", dst=(cat, 64))
    g = n.gap(cat, pre=True)
    n.fc(g, 16)
    nb = 5
    blobs, imgs = prepared([n], 21, nb, 30, bf16=bf)
    E = ens.Ensemble([n], blobs)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[8]])
    y = E.ens_predict(imgs)
    tol = 2.0 ** -7 if bf else 2e-5
    for t in (t1, t2, t3, t4, t5, t6, cat, g):
        got = E.ens_debug_tensor(0, t, n.tensors[t], nb)
        ref = oracle_tensor(n, blobs[0], imgs, t)
        scale = np.sqrt(np.mean(ref ** 2)) + 1e-6
        err = np.abs(got - ref).max()
        assert err <= tol * (scale + np.abs(ref).max()) * (4 if bf else 1), (t, err, scale)
    y_ref, _ = oracle.ensemble_predict([n], blobs, imgs, real="f32")
    assert np.abs(y - y_ref).max() <= (TOL_BF16 if bf else TOL_FP32)
    E.close()


@pytest.mark.parametrize("dtype,h,c,pre", [("bf16", 7, 2048, False), ("bf16", 1, 328, True), ("fp32", 5, 100, True), ("bf16", 13, 40, False)],
                         ids=["bf16_7x7x2048", "bf16_1x1x328_pre", "fp32_5x5x100_pre", "bf16_13x13x40"])
def test_global_pool_shapes(ens, dtype, h, c, pre):
    """Global average pooling over the shapes its grid distinguishes: several channel tiles per image
    (2048 channels), a last tile that is partly empty (328 and 40 channels in groups of 8; 100 fp32
    channels), fewer pixels than thread rows (1x1) and more (13x13), with and without pre-activation.
    The pooled vector is read back and compared with the oracle element by element."""
    bf = dtype == "bf16"
    n = N.Net("gp", h, h, 8, dtype=dtype)
    t = n.conv(0, c, 1)
    g = n.gap(t, pre=pre)
    n.fc(g, 8)
    nb = 6
    blobs, imgs = prepared([n], 61, nb, h, bf16=bf)
    E = ens.Ensemble([n], blobs)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[8]])
    E.ens_predict(imgs)
    got = E.ens_debug_tensor(0, g, n.tensors[g], nb)
    E.close()
    ref = oracle_tensor(n, blobs[0], imgs, g)
    scale = np.sqrt(np.mean(ref ** 2)) + 1e-6
    # the inputs of the pooling are the same bf16 (or fp32) values on both sides: only the order of the sum differs
    tol = 2.0 ** -7 if bf else 2e-5
    assert np.abs(got - ref).max() <= tol * (scale + np.abs(ref).max()), (np.abs(got - ref).max(), scale)


@pytest.mark.parametrize("dtype,h,c,r,nb", [("bf16", 28, 96, 4, 3), ("bf16", 7, 1152, 48, 6), ("bf16", 2, 16, 4, 600), ("fp32", 9, 40, 10, 4)],
                         ids=["bf16_28x28x96", "bf16_7x7x1152", "bf16_2x2x16_600_images", "fp32_9x9x40"])
def test_squeeze_excite_shapes(ens, dtype, h, c, r, nb):
    """Squeeze-excite over the shapes its two kernels distinguish: several workgroups share an image in
    the channel sums and in the rescale (28x28x96, 7x7x1152), one workgroup per image in the rescale
    when the batch alone fills the chip (600 images), fp32 with a channel count that is no multiple of
    8.  The rescaled tensor is read back and compared with the oracle element by element."""
    bf = dtype == "bf16"
    n = N.Net("se", h, h, 8, dtype=dtype)
    t = n.conv(0, c, 1, act="silu")
    u = n.se(t, r)
    n.fc(n.gap(u), 8)
    blobs, imgs = prepared([n], 71, nb, h, bf16=bf)
    E = ens.Ensemble([n], blobs)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[nb]])
    E.ens_predict(imgs)
    got = E.ens_debug_tensor(0, u, n.tensors[u], nb)
    E.close()
    ref = oracle_tensor(n, blobs[0], imgs, u)
    scale = np.sqrt(np.mean(ref ** 2)) + 1e-6
    tol = 2.0 ** -7 if bf else 2e-5
    assert np.abs(got - ref).max() <= tol * (scale + np.abs(ref).max()) * (4 if bf else 1), (np.abs(got - ref).max(), scale)


@pytest.mark.parametrize("F,classes,nb,G", [(2048, 1000, 128, 1), (1280, 1000, 37, 1), (1408, 1000, 64, 1), (512, 200, 96, 2), (72, 24, 5, 1)],
                         ids=["2048-1000_n128", "1280-1000_n37", "1408-1000_n64", "512-200_n96_gang2", "72-24_n5"])
def test_fc_head_on_matrix_cores(ens, F, classes, nb, G):
    """The FC head of a bf16 member (fp32 pooled features split into two bf16 parts, bf16 weights, matrix
    cores): the pooled features the GPU computed are read back and fed to the oracle's FC, so that only
    this layer is compared.  Shapes: four image blocks and a ragged one, a K range that is no multiple of
    64 (1408 = 88 steps of 16), a last class block with 8 of 32 classes (200, 1000), two members in one
    launch, a head smaller than one block.  The error left is the 2^-17 of each feature that two bf16
    parts do not hold and the order of the fp32 sums."""
    nets = []
    for g in range(G):
        n = N.Net("fc%d" % g, 4, 4, classes, dtype="bf16")
        t = n.conv(0, F, 1)
        n.fc(n.gap(t), classes)
        nets.append(n)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 81, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(82, nb, 4, 4))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(4, 4)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[nb] * G])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    assert ran.get("fc_mfma_bf16") == 1 and "fc_kernel" not in ran, ran
    for g in range(G):
        net = nets[g]
        pooled = net.ops[-1]["src"]
        x = E.ens_debug_tensor(g, pooled, net.tensors[pooled], nb)          # nb x 1 x 1 x F fp32, as the FC kernel read it
        z = E.ens_member_logits(g, nb)
        sub = N.Net("sub", 1, 1, classes, dtype="bf16", in_c=F)
        sub.ops, sub.params, sub.blob_size = [dict(net.ops[-1])], net.params, net.blob_size
        sub.tensors = [net.tensors[pooled], net.tensors[net.out_tensor]]
        sub.ops[0].update(src=0, dst=1)
        sub.out_tensor = 1
        ref = oracle.forward_logits(sub, blobs[g], x, real="f64")
        assert np.abs(x).max() > 0.1 and ref.std() > 0.05
        bound = 1e-4 * (np.abs(ref) + ref.std())
        assert (np.abs(z - ref) <= bound).all(), (g, float((np.abs(z - ref) / bound).max()))
    E.close()


@pytest.mark.parametrize("h,c,r,cout,res,G,nb", [(28, 144, 6, 24, False, 1, 5), (7, 1152, 48, 192, False, 1, 37), (14, 480, 20, 80, True, 2, 9),
                                                  (56, 96, 4, 24, False, 1, 3), (5, 2688, 112, 448, False, 1, 6)],
                         ids=["28x28x144-24", "7x7x1152-192_n37", "14x14x480-80_res_gang2", "56x56x96-24", "5x5x2688-448"])
def test_squeeze_excite_gate_in_the_projection(ens, h, c, r, cout, res, G, nb):
    """A squeeze-excite block followed by a 1x1 projection (the tail of an inverted-residual block): the
    block stops at its gates and the projection multiplies its input by them, so the rescaled tensor is
    never written.  The projection's output is compared with the oracle element by element and, bit for
    bit, with the same network run layer by layer (every tensor kept: no fusion); the profile says which
    kernels ran.  Shapes: tiles inside one image (56x56, 28x28), tiles over three to six images (7x7,
    5x5), input channels that are no multiple of 64 (144, 480), a residual, two members in one launch."""
    nets = []
    for g in range(G):
        n = N.Net("mb%d" % g, h, h, 8, dtype="bf16")
        x = n.conv(0, cout, 3, act=None) if res else 0
        t = n.conv(x, c, 1, act="silu")
        u = n.se(t, r)
        y = n.conv(u, cout, 1, act=None, res=x if res else None)
        n.fc(n.gap(y), 8)
        nets.append(n)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 101, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(102, nb, h, h))
    outs = []
    for keep in (False, True):
        E = ens.Ensemble(nets, blobs)
        E.set_base_size(h, h)
        if keep:
            E.ens_debug_keep_tensors()
        E.ens_set_alloc([[nb] * G])
        E.ens_set_profiling(1)
        E.ens_predict(imgs)
        ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
        gate_ran = sum(v for k, v in ran.items() if k.endswith(",gate>"))
        assert gate_ran == (0 if keep else 1), ran
        outs.append([E.ens_debug_tensor(g, y, nets[g].tensors[y], nb) for g in range(G)])   # alive until the global pooling
        E.close()
    for g in range(G):
        assert np.array_equal(outs[0][g], outs[1][g])              # same products, same roundings, same sums
        ref = oracle_tensor(nets[g], blobs[g], imgs, y)
        # three bf16 layers in a row (expansion, rescaling, projection)
        assert_after_bf16_layers(outs[0][g], ref, (g,))


@pytest.mark.parametrize("h,c,k,s,r,nb,G,proj", [(28, 144, 3, 1, 6, 5, 1, 0), (57, 96, 3, 2, 4, 3, 1, 24), (14, 480, 5, 1, 20, 9, 2, 80),
                                                  (5, 2688, 5, 1, 112, 6, 1, 0), (112, 32, 3, 1, 8, 2, 1, 16), (3, 8, 3, 2, 2, 4, 1, 0),
                                                  (17, 672, 5, 2, 28, 37, 1, 112)],
                         ids=["28x28x144_k3", "57x57x96_k3s2_proj", "14x14x480_k5_gang2_proj", "5x5x2688_k5", "112x112x32_k3_proj",
                              "3x3x8_k3s2", "17x17x672_k5s2_n37_proj"])
def test_depthwise_leaves_the_channel_sums(ens, h, c, k, s, r, nb, G, proj):
    """A depthwise convolution followed by a squeeze-excite block (the middle of an inverted-residual block):
    the depthwise kernel leaves the channel sums of its output, one row per workgroup, and the block starts
    from them instead of reading the tensor.  What the block (or the 1x1 projection behind it that applies
    its gates) writes is compared with the oracle element by element and with the same network run layer by
    layer, where the block takes its own sums (in another order: equal up to the rounding of the gates);
    the profile says which kernels ran.  Shapes: 14 and 49 workgroups per image (more rows than the block's
    own kernel writes), a ragged last run of columns (29 wide), a last workgroup that is partly idle, more
    channel groups than a workgroup has lanes (2688 channels), an image smaller than one workgroup (3x3x8),
    two members in one launch, stride 2, 37 images."""
    nets = []
    for g in range(G):
        n = N.Net("dwse%d" % g, h, h, 8, dtype="bf16")
        t = n.conv(0, c, 1, act="silu")
        d = n.dwconv(t, k, s)
        u = n.se(d, r)
        y = n.conv(u, proj, 1, act=None) if proj else u
        n.fc(n.gap(y), 8)
        nets.append(n)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 111, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(112, nb, h, h))
    outs = []
    for keep in (False, True):
        E = ens.Ensemble(nets, blobs)
        E.set_base_size(h, h)
        if keep:
            E.ens_debug_keep_tensors()
        E.ens_set_alloc([[nb] * G])
        E.ens_set_profiling(1)
        E.ens_predict(imgs)
        ran = {kk["name"]: kk["launches"] for kk in E.ens_profile() if kk["launches"]}
        assert ran.get("window_kernel<dwconv,sums>", 0) == (0 if keep else 1), ran
        assert ran.get("window_kernel<dwconv>", 0) == (1 if keep else 0), ran
        outs.append([E.ens_debug_tensor(g, y, nets[g].tensors[y], nb) for g in range(G)])   # alive until the global pooling
        E.close()
    for g in range(G):
        ref = oracle_tensor(nets[g], blobs[g], imgs, y)
        # three or four bf16 layers in a row (expansion, depthwise, rescaling, projection)
        assert_after_bf16_layers(outs[0][g], ref, (g, "sums from the depthwise kernel"))
        assert_after_bf16_layers(outs[1][g], ref, (g, "layer by layer"))
        # the two runs differ by the order of the fp32 sums behind the gates only: a bf16 step here and there
        d = np.abs(outs[0][g] - outs[1][g])
        assert d.max() <= 2.0 ** -7 * np.abs(outs[1][g]).max() and (d > 0).mean() < 0.02, (g, float(d.max()), float((d > 0).mean()))


@pytest.mark.parametrize("h,w,cin,cout,act,G,nb", [(35, 35, 192, 32, "relu", 1, 3), (17, 17, 768, 192, "relu", 1, 5), (8, 8, 1280, 192, "relu", 2, 9),
                                                    (9, 13, 64, 64, "silu", 1, 4), (12, 7, 96, 8, None, 1, 2)],
                         ids=["35x35x192-32", "17x17x768-192", "8x8x1280-192_gang2", "9x13x64-64_silu", "12x7x96-8_linear"])
def test_average_pool_changes_places_with_the_projection(ens, h, w, cin, cout, act, G, nb):
    """The pool branch of an inception module: a 3x3 / stride-1 average pool (over the in-bounds part of its window)
    and a 1x1 convolution with batch-norm and activation.  Both are linear up to the activation and the weights of
    an average add up to one, so the library runs convolution and batch-norm first (into the pool's output memory,
    cout channels wide) and the pool, which then applies the activation, on that narrower tensor.  The module's
    output slice is compared with the oracle (which pools first, as the network says) element by element and with
    the library run layer by layer; the profile says which kernels ran."""
    nets = []
    for g in range(G):
        n = N.Net("pb%d" % g, h, w, 8, dtype="bf16")
        x = n.conv(0, cin, 1, act="relu")
        o = n.tensor(h, w, 16 + cout)
        n.conv(x, 16, 1, dst=(o, 0))
        u = n.avgpool(x, 3, 1, 1)
        n.conv(u, cout, 1, act=act, dst=(o, 16))
        n.fc(n.gap(o), 8)
        nets.append(n)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 121, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(122, nb, h, w))
    outs = []
    for keep in (False, True):
        E = ens.Ensemble(nets, blobs)
        E.set_base_size(h, w)
        if keep:
            E.ens_debug_keep_tensors()
        E.ens_set_alloc([[nb] * G])
        E.ens_set_profiling(1)
        E.ens_predict(imgs)
        ran = {kk["name"]: kk["launches"] for kk in E.ens_profile() if kk["launches"]}
        assert ran.get("window_kernel<avgpool,act>", 0) == (0 if keep else 1), ran
        assert ran.get("window_kernel<avgpool>", 0) == (1 if keep else 0), ran
        outs.append([E.ens_debug_tensor(g, o, nets[g].tensors[o], nb) for g in range(G)])
        E.close()
    for g in range(G):
        ref = oracle_tensor(nets[g], blobs[g], imgs, o)
        assert np.abs(ref[..., 16:]).max() > 0.1
        assert_after_bf16_layers(outs[0][g], ref, (g, "convolution first"))
        assert_after_bf16_layers(outs[1][g], ref, (g, "layer by layer"))
        assert np.array_equal(outs[0][g][..., :16], outs[1][g][..., :16])      # the other branch is the same launch either way


@pytest.mark.parametrize("h,w,cin,cout,bn,G,nb", [(56, 56, 256, 128, False, 1, 3), (15, 15, 64, 32, False, 1, 5), (14, 14, 1024, 512, False, 2, 7),
                                                   (9, 12, 1792, 896, False, 1, 4), (28, 28, 96, 64, True, 1, 2)],
                         ids=["56x56x256-128", "15x15x64-32_odd", "14x14x1024-512_gang2", "9x12x1792-896", "28x28x96-64_affine"])
def test_transition_pools_before_its_convolution(ens, h, w, cin, cout, bn, G, nb):
    """The transition between two dense blocks: a pre-activated 1x1 convolution with no activation behind it and a
    2x2 / stride-2 average pool.  The convolution is linear (with a batch-norm of its own: affine, which an average
    commutes with as well), so the library averages the pre-activated input first, into the convolution's output
    memory, and runs the convolution on a quarter of the pixels.  The pooled output is compared with the oracle
    (which convolves first, as the network says) element by element and with the library run layer by layer; the
    profile says which kernels ran.  An odd map (15x15: the pool drops the last row and column either way), two
    members in one launch, a convolution with batch-norm."""
    nets = []
    for g in range(G):
        n = N.Net("tr%d" % g, h, w, 8, dtype="bf16")
        x = n.conv(0, cin, 1, act=None)
        u = n.conv(x, cout, 1, pre=True, bn=bn, act=None, bias=False)
        nxt = n.tensor(h // 2, w // 2, cout + 32)
        n.avgpool(u, 2, 2, dst=(nxt, 0))
        n.conv(nxt, 32, 3, src_slice=(0, cout), dst=(nxt, cout))
        n.fc(n.gap(nxt), 8)
        nets.append(n)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 131, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(132, nb, h, w))
    outs = []
    for keep in (False, True):
        E = ens.Ensemble(nets, blobs)
        E.set_base_size(h, w)
        if keep:
            E.ens_debug_keep_tensors()
        E.ens_set_alloc([[nb] * G])
        E.ens_set_profiling(1)
        E.ens_predict(imgs)
        ran = {kk["name"]: kk["launches"] for kk in E.ens_profile() if kk["launches"]}
        assert ran.get("window_kernel<avgpool,pre>", 0) == (0 if keep else 1), ran
        assert ran.get("window_kernel<avgpool>", 0) == (1 if keep else 0), ran
        outs.append([E.ens_debug_tensor(g, nxt, nets[g].tensors[nxt], nb)[..., :cout] for g in range(G)])
        E.close()
    for g in range(G):
        ref = oracle_tensor(nets[g], blobs[g], imgs, nxt)[..., :cout]
        assert np.abs(ref).max() > 0.1
        assert_after_bf16_layers(outs[0][g], ref, (g, "pool first"))
        assert_after_bf16_layers(outs[1][g], ref, (g, "layer by layer"))


def test_resize_staging(ens):
    """A member at 45 x 45 fed from 32 x 32 requests: bilinear resize inside the library."""
    for dtype in ("fp32", "bf16"):
        n = N.Net("rs", 45, 45, 8, dtype=dtype)
        t = n.conv(0, 8, 3)
        n.fc(n.gap(t), 8)
        blobs, imgs = prepared([n], 31, 6, 32, bf16=(dtype == "bf16"))
        E = ens.Ensemble([n], blobs)
        E.set_base_size(32, 32)
        E.ens_debug_keep_tensors()
        E.ens_set_alloc([[4]])
        E.ens_predict(imgs)
        got = E.ens_debug_tensor(0, 0, (45, 45, 3), 2)       # worker's last batch = images 4, 5
        ref = oracle.resize_bilinear(imgs[4:6], 45, 45)
        tol = 2.0 ** -8 * 4.5 if dtype == "bf16" else 2e-5     # fp32 sample coordinates: ~1e-6 * 32 pixels * |gradient|
        assert np.abs(got - ref).max() <= tol
        E.close()


# --------------------------------------------------------------------------- config 2 (bf16)
@pytest.fixture(scope="module")
def config2():
    nets = N.config_members(2)
    n = 64
    blobs, imgs = prepared(nets, synth.BASE_SEED, n, 224, bf16=True, varied_from=24)
    y_ref, p_ref = oracle.ensemble_predict(nets, blobs, imgs, real="f32")
    assert len(set(np.argmax(y_ref, 1))) >= 8                # the arg-max is not one constant class
    z_ref = [oracle.forward_logits(net, b, imgs[:8], real="f32") for net, b in zip(nets, blobs)]
    return nets, blobs, imgs, y_ref, z_ref


def test_config2_resnet18_ensemble_bf16(ens, config2):
    nets, blobs, imgs, y_ref, z_ref = config2
    E = ens.Ensemble(nets, blobs)
    E.ens_set_alloc([[32, 32, 32]])                       # the benchmark's launch configuration
    y = E.ens_predict(imgs)
    assert np.isfinite(y).all()
    np.testing.assert_allclose(y.sum(1), 1.0, atol=1e-5)
    err = np.abs(y - y_ref).max()
    strict, near = top1_agreement(y, y_ref, TOL_BF16)
    print("config 2: max-abs prob err %.3e, top-1 strict %.4f, within tolerance band %.4f" % (err, strict, near))
    assert err <= TOL_BF16
    # Several arg-maxes are correct when the oracle's top classes lie closer together than the
    # probability tolerance: agreement is counted up to such ties; the strict rate is reported.
    assert near >= TOP1 and (strict >= TOP1 or int(round((1.0 - strict) * len(y))) <= 1)    # at most one of the 64 images
    for m in range(3):
        z = E.ens_member_logits(m, 8)
        rel = np.abs(z - z_ref[m]).max() / z_ref[m].std()
        assert rel <= 0.05, (m, rel)
    # other allocations: data-parallel workers of a member, ragged batches, short request
    for matrix, seg, n in ([[8, 16, 128]], 128, 64), ([[32, 32, 32], [32, 0, 8]], 128, 50), ([[64, 64, 64]], 16, 33):
        E.ens_set_alloc(matrix, seg)
        y2 = E.ens_predict(imgs[:n])
        assert np.abs(y2 - y_ref[:n]).max() <= TOL_BF16
        assert np.abs(y2 - y[:n]).max() <= 5e-3
    E.close()


def test_device_resident_buffers(ens, config2):
    import torch
    nets, blobs, imgs, y_ref, _ = config2
    E = ens.Ensemble(nets, blobs)
    E.ens_set_alloc([[32, 32, 32]])
    d_img = torch.from_numpy(imgs[:40]).cuda()
    y = E.ens_predict(d_img)
    torch.cuda.synchronize()
    assert y.is_cuda and np.abs(y.cpu().numpy() - y_ref[:40]).max() <= TOL_BF16
    E.close()


def test_benchmark_mode_and_memory_budget(ens, config2):
    nets, blobs, _, _, _ = config2
    E = ens.Ensemble(nets, blobs)
    ips = E.ens_bench([[32, 32, 32]], n_calib=256, repeats=2)
    assert ips > 0
    w, a = E.ens_member_bytes(0, 32)
    assert w > 2 * 11e6 and a > 32 * 112 * 112 * 64 * 2
    out = E.ens_plan(3 * w + 3 * a // 4 * 2 + 256 * (224 * 224 * 3 + 4000) * 4, strategy=1, n_calib=256, repeats=1)
    assert out.matrix() == [[8, 8, 8]] and out.score > 0
    with pytest.raises(ens.EnsError) as e:
        E.ens_plan(2 * w, strategy=1, n_calib=8)
    assert e.value.status == ens.ENS_E_NOFIT
    E.close()
