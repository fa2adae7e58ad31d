"""Requests of a few images that run in one launch, a member per XCD (csrc/chain.hip): against the oracle, for every family of members and for
layers at the edges of what the kernel's steps take."""
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


def ask_all_ways(ens, nets, blobs, imgs, base, batch, sizes, bound):
    """Every size of `sizes`, from device and host memory and through the allocation-free entry point, in one order and another, beside the oracle's logits."""
    import torch
    x = [oracle.resize_bilinear(imgs, net.in_h, net.in_w) for net in nets]
    z_ref = [oracle.forward_logits(net, b, xi, real="f32") for net, b, xi in zip(nets, blobs, x)]
    d = torch.from_numpy(imgs).cuda()
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(base[0], base[1])
    E.ens_set_alloc([[batch] * len(nets)])
    first = {}
    for n in sizes:
        first[n] = E.ens_predict(d[:n].clone()).cpu().numpy()
        for m, net in enumerate(nets):
            z, ref = E.ens_member_logits(m, n), z_ref[m][:n]
            err = float(np.abs(z - ref).max() / z_ref[m].std())
            print("%s, %d images: logits max-abs err / std %.4f" % (net.name, n, err), flush=True)
            assert np.isfinite(z).all() and err <= bound, (net.name, n, err)
    assert E.ens_debug_stats()["chained"] == len(sizes) and E.ens_debug_stats()["recorded"] == 0, E.ens_debug_stats()
    out = {n: torch.empty((n, E.classes), device="cuda") for n in sizes}
    for n in tuple(reversed(sizes)) + tuple(sizes):
        assert np.array_equal(E.ens_predict(imgs[:n].copy()), first[n]), n
        E.ens_predict_static(d[:n].contiguous(), out[n])
        assert np.array_equal(out[n].cpu().numpy(), first[n]), n
    ran = E.ens_debug_stats()
    assert ran["chained"] == 5 * len(sizes) and ran["graphs"] == 0, ran
    # the pooled features of the last request, and what launches leave of them
    n = sizes[-1]
    pooled = [net.ops[-1]["src"] for net in nets]
    got = [E.ens_debug_tensor(m, pooled[m], net.tensors[pooled[m]], n) for m, net in enumerate(nets)]
    E.ens_debug_one_stream(1)
    plain = E.ens_predict(imgs[:n].copy())
    E.ens_debug_one_stream(0)
    assert E.ens_debug_stats()["chained"] == ran["chained"] and np.abs(plain - first[n]).max() <= 2e-2
    for m, net in enumerate(nets):
        want = E.ens_debug_tensor(m, pooled[m], net.tensors[pooled[m]], n)
        assert np.abs(got[m] - want).max() <= bound * want.std(), net.name
    E.close()


def test_families_of_members(ens):
    """Residual, dense, inception, inverted-residual, separable, grouped and plain members at reduced size, two of them at another resolution than the
    request; one image, and several per program.  The bound on the logits is that of each family's own test."""
    nets = [N.resnet18(size=64, classes=200), N.resnet50(size=64, classes=200), N.densenet121(size=64, classes=200), N.efficientnet(0, size=64, classes=200),
            N.inception_v3(size=107, classes=200), N.resnext50(size=64, classes=200), N.xception(size=107, classes=200), N.mobilenet_v2(size=64, classes=200),
            N.vgg(16, size=64, classes=200)]
    blobs = [W.quantise_weights_bf16(net, W.make_blob(net, synth.BASE_SEED + 41, i)) for i, net in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(synth.BASE_SEED + 1041, 5, 64, 64, varied=True))
    ask_all_ways(ens, nets, blobs, imgs, (64, 64), 16, (1, 3, 5), 0.08)


def edges(i):
    """Layers at the edges of the chain's steps: K of 8 and of a chunk and 8, taps that change inside a chunk, odd maps, strides, filters along one
    axis, slices of a concatenation, groups, a squeeze-excite block with and without a depthwise layer in front, pools of every kind."""
    n = N.Net("edges%d" % i, 45, 37, 24, dtype="bf16")
    t = n.conv(0, 24 + 8 * i, 3)                                  # the image itself, 8 channels stored
    t = n.conv(t, 40, 3, stride=2, act="silu")
    a = n.conv(t, 72, 1)
    b = n.conv(a, 72, (1, 7), act=None)
    t = n.conv(b, 72, (7, 1), res=a)
    t = n.maxpool(t, 3, 2, 1)
    h, w, _ = n.tensors[t]
    cat = n.tensor(h, w, 40 + 48 + 72)                            # three branches into slices
    n.conv(t, 40, 1, dst=(cat, 0))
    n.conv(n.conv(t, 16, 5), 48, 3, dst=(cat, 40))
    n.avgpool(t, 3, 1, 1, dst=(cat, 88))
    t = n.conv(cat, 136, 1, pre=True)
    t = n.dwconv(t, 5, stride=1)
    t = n.conv(n.se(t, 10), 64, 1, act=None)
    t = n.dwconv(t, 3, stride=2, act="relu")
    t = n.se(n.conv(t, 64, 3, groups=2, act=None), 3)             # no depthwise layer in front of this one
    t = n.avgpool(n.conv(t, 128, 1, pre=True, act=None), 2, 2)
    t = n.conv(t, 200, 1, stride=2)
    n.fc(n.gap(t, pre=True), 24)
    return n


@pytest.mark.parametrize("members,sizes", [(4, (1, 2)), (8, (3, 5, 7))], ids=str)   # (more images take more members for the rule to chain them)
def test_layers_at_the_edges(ens, members, sizes):
    nets = [edges(i) for i in range(members)]
    blobs = [W.quantise_weights_bf16(net, W.make_blob(net, synth.BASE_SEED + 43, i)) for i, net in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(synth.BASE_SEED + 1043, sizes[-1], 45, 37, varied=True))
    # some 20 bf16 roundings of 2^-9 from the image to the logits, as for the members above
    ask_all_ways(ens, nets, blobs, imgs, (45, 37), 16, sizes, 0.08)


def long_filters(i):
    """Filters of 32 taps in a row or in two, in a column, of 31, windows that begin 33 columns outside the image, and 49 taps that are never outside."""
    n = N.Net("long%d" % i, 45, 37, 24, dtype="bf16")
    t = n.conv(0, 16 + 8 * i, 3)
    t = n.conv(t, 32, (1, 32), pad=(0, 15))
    t = n.conv(t, 32, (1, 31))
    t = n.conv(t, 32, (2, 16), pad=(1, 8), act="silu")
    t = n.conv(t, 24, (32, 1), pad=(16, 0), stride=2)
    h, w, _ = n.tensors[t]
    t = n.conv(t, 40, (1, 3), pad=(0, 33))
    n.tensors[t] = (h, w + 31, 40)                                # the last window ends in the image's last columns
    t = n.conv(n.avgpool(t, 2, 2), 32, 7, pad="valid")
    for _ in range(9):
        t = n.conv(t, 32, 1)
    n.fc(n.gap(t), 24)
    return n


def test_long_filters(ens):
    nets = [long_filters(i) for i in range(8)]
    blobs = [W.quantise_weights_bf16(net, W.make_blob(net, synth.BASE_SEED + 45, i)) for i, net in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(synth.BASE_SEED + 1045, 3, 45, 37, varied=True))
    # some 17 bf16 roundings of 2^-9 from the image to the logits, as for the members above; a dropped tap is an error of the size of the values
    ask_all_ways(ens, nets, blobs, imgs, (45, 37), 16, (1, 3), 0.08)


def test_chains_are_as_exact_as_launches(ens):
    """The twelve full-size members on one image and on four: chains add up in another order than the launches, and lie no further from the oracle."""
    import json
    import os
    import torch
    from tests.golden import make_oracle_cache as cache
    nets, blobs, imgs, z_ref = cache.load_or_make(4)
    with open(os.path.join(os.path.dirname(ens.__file__), "allocations.json")) as f:
        plan = json.load(f)["4"]
    E = ens.Ensemble(nets, blobs)
    E.ens_set_alloc(plan["matrix"], plan["segment"])

    def errors(n):
        z = []
        for s in range(0, 12, n):
            E.ens_predict(torch.from_numpy(imgs[s:s + n].copy()).cuda())
            z.append(np.stack([E.ens_member_logits(m, n) for m in range(len(nets))]))
        return np.sqrt(((np.concatenate(z, 1).astype(np.float64) - z_ref[:, :12]) ** 2).mean((1, 2))) / z_ref[:, :12].std((1, 2))
    chains = errors(1), errors(4)
    assert E.ens_debug_stats()["chained"] == 15
    E.ens_debug_one_stream(1)
    launches = errors(1), errors(4)
    assert E.ens_debug_stats()["chained"] == 15
    E.close()
    for c, l in zip(chains, launches):
        print("rms error of the logits / their spread: chains %s, launches %s" % (np.round(c, 5), np.round(l, 5)), flush=True)
        # Two draws of the same roundings: over 12 images and all classes their root mean squares were within 4 % of each other for every member
        assert (c <= 1.15 * l).all(), (c / l)


def test_values_that_are_no_numbers(ens):
    """An infinity, a NaN and the largest numbers in an image leave the others of its programs alone, and what they give is what the launches give:
    numbers where those give numbers (most kernels' ReLU drops a NaN), NaN where those do."""
    import torch
    nets = [N.resnet18(size=64, classes=200), N.densenet121(size=64, classes=200), N.efficientnet(0, size=64, classes=200), N.inception_v3(size=107, classes=200),
            N.resnext50(size=64, classes=200), N.xception(size=107, classes=200), N.mobilenet_v2(size=64, classes=200), N.vgg(16, size=64, classes=200)]
    blobs = [W.quantise_weights_bf16(net, W.make_blob(net, synth.BASE_SEED + 47, i)) for i, net in enumerate(nets)]
    imgs = W.round_bf16(W.make_images(synth.BASE_SEED + 1047, 5, 64, 64, varied=True))
    odd = imgs.copy()
    odd[1, 20, 31, 1], odd[2, 63, 0, :], odd[3] = np.inf, 3e38, np.nan
    E = ens.Ensemble(nets, blobs)
    E.set_base_size(64, 64)
    E.ens_set_alloc([[16] * len(nets)])

    def ask(x):
        E.ens_predict(torch.from_numpy(x).cuda())
        return [E.ens_member_logits(m, 5) for m in range(len(nets))]
    clean, got = ask(imgs), ask(odd)
    assert E.ens_debug_stats()["chained"] == 2
    E.ens_debug_one_stream(1)
    want = ask(odd)
    assert E.ens_debug_stats()["chained"] == 2
    nans = 0
    for m, net in enumerate(nets):
        assert np.array_equal(got[m][[0, 4]], clean[m][[0, 4]]), net.name
        assert np.array_equal(np.isnan(got[m]), np.isnan(want[m])), net.name
        nans += np.isnan(want[m]).sum()
        for i in range(5):
            if not np.isnan(want[m][i]).any():                    # the bound of the members above
                spread = want[m][i].astype(np.float64).std()
                assert np.abs(got[m][i].astype(np.float64) - want[m][i]).max() <= 0.08 * spread, (net.name, i)
    assert nans > 0
    E.close()


def test_chains_beside_other_requests(ens):
    """Requests that run as chains while another handle's request keeps three of the four streams full, and chains of two handles at once: the answers are
    those that each gives alone.  (A chain's group is then made of the compute units that were free when it began, down to one.)"""
    import threading
    import torch
    def deep(i, width):
        n = N.Net("deep%d" % i, 28, 28, 16, dtype="bf16")
        t = n.conv(0, width, 3)
        for k in range(20):
            t = n.conv(t, width, 3 if k % 2 else 1)
        n.fc(n.gap(t), 16)
        return n
    busy = ens.Ensemble([deep(i, 192 + 64 * i) for i in range(3)], [W.make_blob(deep(i, 192 + 64 * i), synth.BASE_SEED + 48, i) for i in range(3)])
    busy.ens_set_alloc([[128] * 3])
    handles = []
    for k in range(2):
        nets = [deep(i, 32 + 16 * i) for i in range(6 + k)]
        E = ens.Ensemble(nets, [W.make_blob(net, synth.BASE_SEED + 49 + k, i) for i, net in enumerate(nets)])
        E.ens_set_alloc([[8] * len(nets)])
        handles.append(E)
    L = ens.lib()
    x = torch.randn(512, 28, 28, 3, device="cuda")
    y = torch.empty(512, 16, device="cuda")
    busy.ens_predict(x, y)
    alone, out = [], []
    for E in handles:
        alone.append([E.ens_predict(x[:n].contiguous()).clone() for n in (1, 2)])
        out.append(torch.empty(2, 16, device="cuda"))
    assert all(E.ens_debug_stats()["chained"] == 2 for E in handles) and busy.ens_debug_stats()["chained"] == 0
    torch.cuda.synchronize()
    wrong = []

    def serve(k, requests):
        for rep in range(requests):
            for n in (1, 2):                                      # (through the C entry point: torch would wait for every stream)
                if L.ens_predict(handles[k]._h, x.data_ptr(), n, out[k].data_ptr()) != 0:
                    wrong.append((k, rep, n))
                answers[k].append((n, out[k][:n].clone()))
    answers = [[], []]
    for threads in ([threading.Thread(target=lambda: [L.ens_predict(busy._h, x.data_ptr(), 512, y.data_ptr()) for _ in range(8)]), threading.Thread(target=serve, args=(0, 30))],
                    [threading.Thread(target=serve, args=(k, 60)) for k in range(2)]):
        for th in threads:
            th.start()
        for th in threads:
            th.join()
    assert not wrong, wrong[:5]
    for k in range(2):
        assert len(answers[k]) >= 120
        for n, a in answers[k]:
            assert torch.equal(a, alone[k][n - 1]), (k, n)
        assert handles[k].ens_debug_stats()["chained"] == 2 + len(answers[k])
    for E in handles + [busy]:
        E.close()
