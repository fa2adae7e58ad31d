"""Requests that do not fill a worker's batch size, and requests that come again.

The first run their layers on the kernel for few output pixels (and their bottlenecks and dense layers one by
one), so each shape where its tiles, its split of K or its tables can go wrong is compared with the oracle; the second
are replayed from recorded graphs, so replays are compared with the first, launch-by-launch answer bit for bit."""
import numpy as np
import pytest

import oracle
import synth
from synth import nets as N
from synth import weights as W

from .test_gpu_parity import assert_after_bf16_layers, layer_net, oracle_tensor, prepared

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ens():
    import torch
    assert torch.cuda.is_available(), "this test needs the GPU"
    import paper_2208_14049_amd as ens
    ens.lib()
    return ens


# (H, W, cin, cout, k, stride, extra, images)
FEW = [
    (14, 14, 256, 256, 3, 1, {"res": True}, 1),                # 7 tiles, the last with 4 pixels; 36 chunks over 8 wavefronts
    (7, 7, 512, 512, 3, 1, {}, 3),                             # 72 chunks: nine per wavefront, two in flight
    (5, 5, 8, 72, 3, 1, {"act": None}, 1),                     # 8 channels in the last tile, K = 72: a chunk of 64 and one of 8
    (9, 11, 24, 40, 3, 2, {}, 2),                              # taps that change inside a chunk, half-empty channel tile, odd strided map
    (12, 12, 160, 192, (1, 7), 1, {}, 2),
    (12, 12, 48, 72, (7, 1), 1, {"act": "silu"}, 3),
    (13, 13, 16, 64, 5, 1, {}, 1),
    (14, 14, 1024, 256, 1, 1, {}, 2),                          # two chunks per wavefront
    (28, 28, 512, 128, 1, 1, {"act": "silu"}, 4),              # 392 tiles: one chunk at a time
    (15, 15, 264, 520, 1, 2, {"act": None}, 3),                # strided shortcut, last chunk of 8 channels
    (14, 14, 512, 128, 1, 1, {"pre": True}, 3),                # pre-activated
    (7, 7, 904, 128, 1, 1, {"pre": True}, 7),
    (28, 28, 128, 128, 3, 1, {}, 6),                           # 588 tiles of 32 x 32: four wavefronts
    (14, 14, 512, 512, 1, 1, {"res": True}, 8),                # 784 tiles: 64 x 64 instead
    (14, 14, 128, 256, 3, 1, {"groups": 2}, 2),
]


@pytest.mark.parametrize("case", FEW, ids=lambda c: "%dx%dx%d-%d-k%s-s%d_n%d" % (c[0], c[1], c[2], c[3], c[4], c[5], c[7]))
def test_layers_on_few_images(ens, case):
    h, w, cin, cout, k, stride, extra, nb = case
    extra = dict(extra)
    with_res = extra.pop("res", False)
    net, t = layer_net(h, w, cin, lambda n, s: n.conv(s, cout, k, stride=stride, res=s if with_res else None, **extra), "bf16")
    blobs, _ = prepared([net], 11, nb, h, bf16=True)
    imgs = W.round_bf16(W.make_images(4, nb, h, w))
    E = ens.Ensemble([net], blobs)
    E.set_base_size(h, w)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[2 * nb]])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {kk["name"]: kk["launches"] for kk in E.ens_profile() if kk["launches"]}
    assert ran.get("conv_small_bf16", 0) >= 1, ran
    src = net.ops[-3]["src"]
    got, x = E.ens_debug_tensor(0, t, net.tensors[t], nb), E.ens_debug_tensor(0, src, net.tensors[src], nb)
    E.close()
    sub = N.Net("sub", h, w, 8, dtype="bf16", in_c=cin)
    sub.ops, sub.params, sub.blob_size = [dict(net.ops[-3])], net.params, net.blob_size
    sub.tensors = [net.tensors[src], net.tensors[t]]
    sub.ops[0].update(src=0, dst=1)
    if with_res:
        sub.ops[0].update(res=0)
    sub.out_tensor = 1
    ref = oracle.forward_logits(sub, blobs[0], x, real="f64").reshape(got.shape)
    scale = np.sqrt(np.mean(ref ** 2)) + 1e-6
    err = np.abs(got - ref)
    bound = 2.0 ** -7 * np.abs(ref) + scale * 2.0 ** -5 + 1e-6     # as for the same layers on full batches
    assert (err <= bound).all(), (float(err.max()), float(scale), float((err / bound).max()))
    assert err.mean() <= 2.0 ** -8 * scale


@pytest.mark.parametrize("G", [1, 2])
def test_blocks_on_few_images(ens, G):
    """What runs fused or in pairs on full batches, on two images of a batch of 16: a bottleneck and a dense layer one by one, a strided
    convolution and its shortcut as one launch, a gated projection."""
    nets = []
    for g in range(G):
        n = N.Net("few%d" % g, 28, 28, 8, dtype="bf16")
        x = n.conv(0, 256, 3)
        u = n.conv(n.conv(x, 64, 1), 64, 3)
        y = n.conv(u, 256, 1, res=x)                             # bottleneck
        s = n.conv(y, 96, 1, stride=2, act=None)
        b = n.conv(y, 96, 3, stride=2, act=None)                 # a pair
        z = n.conv(b, 96, 1, res=s)
        e = n.conv(n.se(n.dwconv(n.conv(z, 144, 1, act="silu"), 3), 6), 64, 1, act=None)   # gated projection
        blk = n.tensor(14, 14, 64 + 32)
        n.conv(e, 64, 1, dst=(blk, 0))
        n.conv(n.conv(blk, 128, 1, pre=True, src_slice=(0, 64)), 32, 3, bn=False, act=None, bias=False, dst=(blk, 64))   # dense layer
        n.fc(n.gap(blk, pre=True), 8)
        nets.append(n)
    nb = 2
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 151, i)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(152, nb, 28, 28))
    E = ens.Ensemble(nets, blobs)
    E.ens_set_alloc([[16] * G])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    got = [E.ens_debug_tensor(g, blk, nets[g].tensors[blk], nb) for g in range(G)]   # alive until the global pooling
    E.close()
    assert "bottleneck_bf16<c64>" not in ran and "dense_layer_bf16" not in ran and "conv_small_bf16<32x32,gate>" in ran, ran
    for g in range(G):
        ref = oracle_tensor(nets[g], blobs[g], imgs, blk)
        # eleven bf16 layers from the image: twice the bound of three (errors grow with the root of the number)
        err, scale = np.abs(got[g] - ref), np.sqrt(np.mean(ref ** 2))
        assert err.max() <= 0.06 * scale + 2.0 ** -7 * np.abs(ref).max() and err.mean() <= 2.0 ** -6 * scale, (g, float(err.max()), float(scale))


@pytest.mark.parametrize("cin,cout,k,stride,extra", [(3, 16, 3, 1, {}), (3, 8, 5, 1, {"act": "silu"}), (16, 32, 3, 1, {}), (5, 10, 3, 2, {"act": None}),
                                                     (8, 20, (1, 7), 1, {}), (12, 3, 5, 1, {"res": True}), (6, 33, 1, 1, {"pre": True}), (20, 24, 3, 1, {"pre": True})])
def test_fp32_convolutions(ens, cin, cout, k, stride, extra):
    """The fp32 kernel: channel counts in fours, threes and neither, partly empty channel tiles, filters with and without an unrolled size."""
    extra = dict(extra)
    cout = cin if extra.get("res") else cout
    with_res = extra.pop("res", False)
    for h, nb in ((9, 1), (32, 70)):                             # four channels per lane, and eight or sixteen
        net, t = layer_net(h, h + 2, cin, lambda n, s: n.conv(s, cout, k, stride=stride, res=s if with_res else None, **extra), "fp32")
        blobs, _ = prepared([net], 17, nb, h, bf16=False)
        imgs = W.make_images(5, nb, h, h + 2)
        E = ens.Ensemble([net], blobs)
        E.set_base_size(h, h + 2)
        E.ens_debug_keep_tensors()
        E.ens_set_alloc([[nb]])
        E.ens_predict(imgs)
        m = min(nb, 4)
        got = E.ens_debug_tensor(0, t, net.tensors[t], nb)[-m:]
        E.close()
        ref = oracle_tensor(net, blobs[0], imgs[-m:], t)
        assert np.abs(got - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max()), (h, float(np.abs(got - ref).max()))


def test_repeated_requests_are_replayed(ens):
    """Sizes that come again are replayed as graphs on several lanes: every answer equals the first one of its size, from device and
    host buffers that change from call to call, between other sizes, eager GPU work and changes of the combination rule."""
    import torch
    nets = [N.resnet18(size=64, classes=100), N.efficientnet(0, size=64, classes=100), N.densenet121(size=64, classes=100), N.resnet18(size=48, classes=100)]
    blobs = [W.quantise_weights_bf16(net, W.make_blob(net, synth.BASE_SEED + 3, i)) for i, net in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(synth.BASE_SEED + 1000, 70, 64, 64, varied=True))
    d = torch.from_numpy(imgs).cuda()
    E = ens.Ensemble(nets, blobs)
    E.ens_set_alloc([[16, 8, 32, 16], [8, 0, 0, 16]], 32)
    sizes = (1, 3, 70, 17)
    first = {n: E.ens_predict(d[:n].contiguous()).cpu().numpy() for n in sizes}
    junk = torch.randn(512, 512, device="cuda")
    for rep in range(6):
        for n in sizes:
            x = d[:n].clone() if rep % 2 else imgs[:n].copy()
            junk = junk @ junk * 1e-3
            y = E.ens_predict(x)
            y = y.cpu().numpy() if rep % 2 else y
            assert np.array_equal(y, first[n]), (rep, n)
    # the small sizes were recorded the second time they came after the logits buffers had grown for the largest; the large ones have
    # several batches for more gangs than lanes and are handed out batch by batch
    ran = E.ens_debug_stats()
    assert ran["recorded"] == ran["graphs"] >= 2 and ran["replayed"] == 5 * ran["recorded"] and ran["handed_out"] > 0, ran
    z = E.ens_member_logits(2, sizes[-1])
    E.ens_set_combination("weighted", [0.7, 0.1, 0.1, 0.1])
    w = [E.ens_predict(d[:3].contiguous()).cpu().numpy() for _ in range(3)]
    assert np.array_equal(w[0], w[1]) and np.array_equal(w[0], w[2]) and np.abs(w[0] - first[3]).max() > 1e-4
    E.ens_set_combination("mean")
    assert np.array_equal(E.ens_predict(d[:17].contiguous()).cpu().numpy(), first[17])
    assert np.array_equal(E.ens_member_logits(2, 17), z)
    E.close()


@pytest.mark.parametrize("h,w,cin,nb", [(14, 14, 32, 50), (14, 14, 96, 50), (7, 9, 640, 160), (28, 28, 288, 13), (14, 14, 1888, 51)])
def test_preactivated_layers_on_full_batches(ens, h, w, cin, nb):
    """The pre-activated 1x1 layer of a dense block as a launch of its own: one input chunk (half of it padding) up to thirty, a ragged last tile."""
    n = N.Net("pre", h, w, 8, dtype="bf16")
    blk = n.tensor(h, w, cin + 32)
    n.conv(0, cin, 1, dst=(blk, 0))
    u = n.conv(blk, 128, 1, pre=True, src_slice=(0, cin))
    n.conv(u, 32, 3, bn=False, act=None, bias=False, dst=(blk, cin))
    n.fc(n.gap(blk, pre=True), 8)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 161, 0))]
    imgs = W.round_bf16(W.make_images(162, nb, h, w))
    E = ens.Ensemble([n], blobs)
    E.set_base_size(h, w)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[nb]])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    got = E.ens_debug_tensor(0, u, n.tensors[u], nb)
    E.close()
    assert ran.get("conv1x1_pre_bf16<128x128>") == 1, ran
    for i in (0, nb - 1):                                        # the first tile, and the ragged one
        ref = oracle_tensor(n, blobs[0], imgs[i:i + 1], u)
        assert_after_bf16_layers(got[i:i + 1], ref, (i,))


@pytest.mark.parametrize("h,w,cin,cout,stride,res,nb", [
    (39, 30, 136, 208, 1, False, 112),     # last chunk of 8 channels, last 48 of 256 columns missing, wavefront with 16 of its 64 channels
    (31, 33, 320, 768, 1, False, 43),      # odd number of chunks, ragged last tile
    (14, 14, 256, 1024, 1, True, 64),      # one round of tiles; residual behind an even number of chunks
    (14, 15, 328, 984, 1, True, 57),       # residual behind an odd one, partly missing columns
    (27, 29, 192, 1000, 2, False, 64),     # strided shortcut
])
def test_wide_pointwise_layers(ens, h, w, cin, cout, stride, res, nb):
    """1x1 layers on tiles of 256 output channels."""
    n = N.Net("wide", h, w, 8, dtype="bf16")
    u = n.conv(0, cin, 1)
    r = n.conv(0, cout, 1) if res else None
    y = n.conv(u, cout, 1, stride=stride, res=r)
    n.fc(n.gap(y), 8)
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 171, 0))]
    imgs = W.round_bf16(W.make_images(172, nb, h, w))
    E = ens.Ensemble([n], blobs)
    E.set_base_size(h, w)
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[nb]])
    E.ens_set_profiling(1)
    E.ens_predict(imgs)
    ran = {k["name"]: k["launches"] for k in E.ens_profile() if k["launches"]}
    got = E.ens_debug_tensor(0, y, n.tensors[y], nb)
    E.close()
    assert ran.get("conv1x1_direct_bf16<128x256>") == 1, ran
    for i in (0, nb // 2, nb - 1):
        ref = oracle_tensor(n, blobs[0], imgs[i:i + 1], y)
        assert_after_bf16_layers(got[i:i + 1], ref, (i,))


def test_fp32_layer_wider_than_a_grid(ens):
    """An fp32 convolution with more than 65535 tiles of four output channels takes two launches.  Sums of three products in fp32."""
    net = N.Net("wide", 2, 2, 8, dtype="fp32")
    t = net.conv(0, 262160, 1, act=None)
    net.fc(net.gap(t), 8)
    blob = W.make_blob(net, 245, 0)
    imgs = W.make_images(246, 2, 2, 2)
    E = ens.Ensemble([net], [blob])
    E.ens_debug_keep_tensors()
    E.ens_set_alloc([[2]])
    E.ens_predict(imgs)
    got = E.ens_debug_tensor(0, t, net.tensors[t], 2)
    E.close()
    ref = oracle_tensor(net, blob, imgs, t)
    # scale folded into the weight, three products and sums, the shift: six roundings of 2^-24 of terms of a few times the tensor's rms
    assert np.abs(got - ref).max() <= 8 * 2.0 ** -24 * np.abs(ref).max() * 4


def test_recorded_requests_outlive_the_allocation_free_entry_point(ens):
    """ens_predict_static frees nothing: requests recorded before it are replayed after it, with the answers they gave."""
    import torch
    nets = [tiny_member(i) for i in range(4)]
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 177 + i, 0)) for i, n in enumerate(nets)]
    x = torch.from_numpy(W.round_bf16(W.make_images(178, 24, 12, 12, varied=True))).cuda()
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(12, 12)
    E.ens_set_alloc([[8] * 4])
    parts = {n: x[:n].contiguous() for n in (24, 3, 7)}
    first = {n: E.ens_predict(v).clone() for n, v in parts.items()}
    outs = {n: torch.empty_like(v) for n, v in first.items()}
    for _ in range(2):
        for n, v in parts.items():
            assert torch.equal(E.ens_predict(v, outs[n]), first[n])
    E.ens_predict_static(parts[24], outs[24])
    a = E.ens_debug_stats()
    assert a["recorded"] == a["graphs"] >= 2, a
    for rep in range(4):
        for n, v in parts.items():
            m = (24, 3, 7)[rep % 3]
            outs[m].zero_()
            free = torch.cuda.mem_get_info()[0]
            E.ens_predict_static(parts[m], outs[m])
            assert rep == 0 or torch.cuda.mem_get_info()[0] == free, (rep, m)      # (the runtime's own buffers come with the first calls)
            assert torch.equal(outs[m], first[m]), (rep, m)
            outs[n].zero_()
            assert torch.equal(E.ens_predict(v, outs[n]), first[n]), (rep, n)
    z = E.ens_member_logits(1, 7)
    E.ens_predict_static(parts[7], outs[7])
    assert np.array_equal(E.ens_member_logits(1, 7), z)
    b = E.ens_debug_stats()
    assert b["recorded"] == a["recorded"] and b["graphs"] == a["graphs"] and b["replayed"] == a["replayed"] + 4 * a["graphs"], (a, b)
    E.close()


def test_sizes_in_turn_are_recorded_within_bounds(ens):
    """More request sizes in turn than recorded requests are kept: what is kept is replayed, the others are issued, and a recording takes
    another's place at most once in 32 requests; sizes that come instead of the first ones are recorded in the end."""
    nets = [tiny_member(i) for i in range(4)]
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 175 + i, 0)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(176, 64, 12, 12, varied=True))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(12, 12)
    E.ens_set_alloc([[64] * 4])                                  # four gangs with one batch: four lanes
    first = {n: E.ens_predict(imgs[:n]) for n in range(1, 25)}
    requests = 24
    for rep in range(6):
        for n in range(1, 25):
            assert np.array_equal(E.ens_predict(imgs[:n]), first[n]), (rep, n)
            requests += 1
    a = E.ens_debug_stats()
    assert a["graphs"] == 16 and a["recorded"] <= 16 + requests // 32, a
    assert a["replayed"] >= 6 * 12, a                            # more than half of the requests that came again
    rng = np.random.default_rng(3)
    for n in rng.integers(1, 25, 200):
        assert np.array_equal(E.ens_predict(imgs[:n]), first[n]), n
    b = E.ens_debug_stats()
    assert b["recorded"] - a["recorded"] <= 1 + 200 // 32 and b["graphs"] == 16, (a, b)
    for rep in range(100):                                       # two new sizes and nothing else
        n = 40 + rep % 2
        first.setdefault(n, E.ens_predict(imgs[:n]))
        assert np.array_equal(E.ens_predict(imgs[:n]), first[n]), (rep, n)
    c = E.ens_debug_stats()
    assert c["recorded"] - b["recorded"] >= 2 and c["replayed"] - b["replayed"] >= 20, (b, c)
    E.close()


@pytest.mark.parametrize("rows,images", [([[8, 8, 8, 8], [8, 0, 0, 16]], 75), ([[8, 8, 8]], 83)], ids=["six_gangs", "copies_of_three"])
def test_handed_out_batches(ens, rows, images):
    """Several batches each for more gangs than lanes, handed out as lanes come free: bit for bit what one stream gives, whether the images are on
    the device or come from pinned or ordinary host memory in pieces beside the kernels."""
    import torch
    nets = [N.resnet18(size=64, classes=100), N.efficientnet(0, size=64, classes=100), N.densenet121(size=64, classes=100), N.resnet18(size=48, classes=100)][:len(rows[0])]
    blobs = [W.quantise_weights_bf16(net, W.make_blob(net, synth.BASE_SEED + 7, i)) for i, net in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(synth.BASE_SEED + 1001, images, 64, 64, varied=True))
    d, pinned = torch.from_numpy(imgs).cuda(), torch.from_numpy(imgs).pin_memory()
    out = torch.empty((images, 100), dtype=torch.float32, pin_memory=True)
    E = ens.Ensemble(nets, blobs)
    E.ens_set_alloc(rows, 16)
    E.ens_debug_one_stream(1)
    want = E.ens_predict(imgs)
    z = [E.ens_member_logits(m, images) for m in range(len(nets))]
    E.ens_debug_one_stream(0)
    assert E.ens_debug_stats()["handed_out"] == 0
    for rep in range(3):
        for k, ask in enumerate((lambda: E.ens_predict(d.clone()).cpu().numpy(), lambda: E.ens_predict(pinned, out).numpy().copy(), lambda: E.ens_predict(imgs.copy()))):
            before = E.ens_debug_stats()["handed_out"]
            assert np.array_equal(ask(), want), (rep, k)
            assert E.ens_debug_stats()["handed_out"] - before >= len(nets) * (images // 16), (rep, k)
            assert all(np.array_equal(E.ens_member_logits(m, images), z[m]) for m in range(len(nets))), (rep, k)
    E.close()


def tiny_member(i):
    n = N.Net("turns%d" % i, 12, 12, 8, dtype="bf16")
    n.fc(n.gap(n.conv(n.conv(0, 16 + 8 * i, 3), 32, 3)), 8)
    return n


@pytest.mark.parametrize("members,rows,batch,images", [
    (1, 1, 4, 23),             # six batches of one gang over four arenas, the last one short
    (1, 2, 4, 23),             # two instances: two arenas each
    (3, 1, 4, 11),             # three gangs with three batches each: one arena each
    (3, 1, 4, 17),             # with five: two arenas each
])
def test_batches_take_turns(ens, members, rows, batch, images):
    """Batches of one gang on arenas of its own and its copies': the answer is that of one stream, which uses no copy, and stays it when
    the logits move to the fixed device array and back."""
    import torch
    nets = [tiny_member(i) for i in range(members)]
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 181 + i, 0)) for i, n in enumerate(nets)]
    x = torch.from_numpy(W.round_bf16(W.make_images(182, images, 12, 12))).cuda()
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(12, 12)
    E.ens_set_alloc([[batch] * members] * rows, 8)
    E.ens_debug_one_stream(1)
    want = E.ens_predict(x)
    E.ens_debug_one_stream(0)
    assert E.ens_debug_stats()["copies"] == {1: 3 if rows == 1 else 2, 3: 3}[members]
    out = torch.empty_like(want)
    for _ in range(4):
        assert torch.equal(E.ens_predict(x), want)
        E.ens_predict_static(x, out)
        assert torch.equal(out, want)
    E.close()


@pytest.mark.parametrize("members", [1, 3])
def test_tensors_of_the_last_batch(ens, members):
    """ens_debug_tensor gives a tensor of the last batch of a request, also where batches are dealt to copies of a gang or replayed."""
    nets = [tiny_member(i) for i in range(members)]
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 231 + i, 0)) for i, n in enumerate(nets)]
    x = W.round_bf16(W.make_images(232, 61, 12, 12, varied=True))
    E = ens.Ensemble(nets, blobs)
    E.ens_set_alloc([[8] * members], 64)
    for n in (29, 61, 16, 29, 2, 29):
        E.ens_predict(x[:n])
        last = (n - 1) % 8 + 1
        got = [E.ens_debug_tensor(m, 3, (1, 1, 32), last) for m in range(members)]
        E.ens_debug_one_stream(1)                                # no copies take part
        E.ens_predict(x[:n])
        E.ens_debug_one_stream(0)
        for m in range(members):
            assert np.array_equal(got[m], E.ens_debug_tensor(m, 3, (1, 1, 32), last)), (n, m)
    E.close()


def test_copies_leave_the_request_buffers_their_room(ens):
    """After ens_plan copies of a group come out of the budget beside the workers and the buffers of a request, and are counted."""
    net = tiny_member(0)
    E = ens.Ensemble([net], [W.quantise_weights_bf16(net, W.make_blob(net, 221, 0))])
    weights, arena = E.ens_member_bytes(0, 8)
    images = 4 * arena // (12 * 12 * 3 * 4)                      # buffers of a calibration request larger than three arenas
    reserve = images * (12 * 12 * 3 + 2 * 8) * 4
    opts = dict(domain=[8], slots=1, strategy=1, n_calib=images, repeats=1)
    for budget, copies in ((weights + arena + reserve, 0), (weights + 4 * arena + reserve - 1, 0), (weights + 4 * arena + reserve, 3)):
        a = E.ens_plan(budget, **opts)
        s = E.ens_debug_stats()
        assert s["copies"] == copies and s["copy_bytes"] == copies * arena and a.bytes == weights + (1 + copies) * arena, (budget, s, a.bytes)
    E.close()


def test_small_host_requests_see_their_own_images(ens):
    """Small requests from host memory go through one pinned buffer, and are waited for without synchronising a stream: requests of one
    size with other images each time give the answers that the same images give from device memory."""
    import torch
    nets = [tiny_member(i) for i in range(3)]
    blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 191 + i, 0)) for i, n in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(192, 40, 12, 12, varied=True))
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(12, 12)
    E.ens_set_alloc([[4] * 3], 8)
    want = [E.ens_predict(torch.from_numpy(imgs[4 * i:4 * i + 4]).cuda()).cpu().numpy() for i in range(10)]
    assert np.abs(want[0] - want[1]).max() > 1e-4
    for rep in range(20):
        i = rep * 7 % 10
        assert np.array_equal(E.ens_predict(imgs[4 * i:4 * i + 4].copy()), want[i]), rep
    E.close()


def run_beside(work):
    """Starts work() on a thread of its own; returns the thread and a list that gets the time of its end."""
    import threading
    import time
    end = []

    def body():
        work()
        end.append(time.perf_counter())
    th = threading.Thread(target=body)
    th.start()
    return th, end


def test_a_request_does_not_wait_for_another_handles_lanes(ens):
    """A request of microseconds on one lane, sent while another handle's request of some hundred milliseconds runs on one lane of its own, is
    answered long before that one.  (Through the C entry point with device buffers: torch's own synchronisation of the null stream, which the
    binding does for device tensors, waits for every lane.)"""
    import time
    import torch
    long = N.Net("long", 128, 128, 8, dtype="fp32")
    t = 0
    for _ in range(16):
        t = long.conv(t, 64, 3)
    long.fc(long.gap(t), 8)
    short = tiny_member(0)
    B = ens.Ensemble([long], [W.make_blob(long, 201, 0)])
    B.ens_set_alloc([[256]], 256)                                # one batch: one lane
    A = ens.Ensemble([short], [W.quantise_weights_bf16(short, W.make_blob(short, 202, 0))])
    A.ens_set_alloc([[8]])
    xb, yb = torch.randn(256, 128, 128, 3, device="cuda"), torch.empty(256, 8, device="cuda")
    xa, ya = torch.randn(4, 12, 12, 3, device="cuda"), torch.empty(4, 8, device="cuda")
    B.ens_predict(xb, yb)
    want = A.ens_predict(xa, ya).clone()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    B.ens_predict(xb, yb)
    alone = time.perf_counter() - t0
    L = ens.lib()
    th, end = run_beside(lambda: L.ens_predict(B._h, xb.data_ptr(), 256, yb.data_ptr()))
    time.sleep(0.1 * alone)
    t0 = time.perf_counter()
    assert L.ens_predict(A._h, xa.data_ptr(), 4, ya.data_ptr()) == 0
    t1 = time.perf_counter()
    th.join()
    assert t0 < end[0] and t1 - t0 < 0.4 * alone and t1 < end[0], (alone, t1 - t0, end[0] - t0)
    assert torch.equal(ya, want)
    A.close()
    B.close()


def test_two_handles_in_two_threads(ens):
    """Two handles that share the lanes, one of them with recorded requests, each in a thread of its own: the answers are those that each gives alone."""
    nets = [[N.resnet18(size=64, classes=100), N.efficientnet(0, size=64, classes=100), N.densenet121(size=64, classes=100)], [tiny_member(i) for i in range(4)]]
    sizes, requests = ((1, 5, 40), (2, 9, 33)), []
    for k, members in enumerate(nets):
        blobs = [W.quantise_weights_bf16(n, W.make_blob(n, 211 + k, i)) for i, n in enumerate(members)]
        imgs = W.round_bf16(W.make_images(213 + k, 40, members[0].in_h, members[0].in_w, varied=True))
        E = ens.Ensemble(members, blobs)
        E.ens_set_alloc([[8] * len(members)], 16)
        requests.append((E, imgs, {n: E.ens_predict(imgs[:n]) for n in sizes[k]}))
    wrong = []

    def serve(k):
        E, imgs, want = requests[k]
        for rep in range(40):
            for n in sizes[k]:
                if not np.array_equal(E.ens_predict(imgs[:n]), want[n]):
                    wrong.append((k, rep, n))
    threads = [run_beside(lambda k=k: serve(k)) for k in range(2)]
    for th, end in threads:
        th.join()
        assert end, "a request failed"
    assert not wrong, wrong[:5]
    for E, _, _ in requests:
        E.close()
