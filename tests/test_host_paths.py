"""Host paths of the library where device memory runs short, on the CPU: the library runs in a process of its own in front of fake_hip.cpp,
whose device memory is host memory with a limit and whose launches do nothing."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-o", lib, os.path.join(ROOT, "tests", "fake_hip.cpp")])
    return lib


def beside_fake_hip(lib, call):
    """Runs `call` (an expression over this module) in a process with the fake runtime in front."""
    preload = ":".join([lib] + [p for p in (os.environ.get("LD_PRELOAD"),) if p])
    p = subprocess.run([sys.executable, "-c", "import tests.test_host_paths as t; t.%s" % call], cwd=ROOT, env=dict(os.environ, LD_PRELOAD=preload),
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=100)
    assert p.returncode == 0, p.stdout.decode()[-3000:]


def fake():
    L = ctypes.CDLL(None)
    L.fake_limit.argtypes = [ctypes.c_size_t]
    for f in ("fake_used", "fake_launches", "fake_null_copies"):
        getattr(L, f).restype = ctypes.c_size_t
    return L


def tiny_ensemble(members):
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    nets = []
    for i in range(members):
        n = N.Net("tiny%d" % i, 12, 12, 8, dtype="bf16")
        n.fc(n.gap(n.conv(n.conv(0, 16 + 8 * i, 3), 32, 3)), 8)
        nets.append(n)
    return ens.Ensemble(nets, [W.make_blob(n, 231, i) for i, n in enumerate(nets)])


def copies_go(members, rows, copies):
    import paper_2208_14049_amd as ens
    F, x = fake(), np.zeros((64, 12, 12, 3), np.float32)
    E = tiny_ensemble(members)
    arena, start = E.ens_member_bytes(0, 64)[1], F.fake_used()
    limit = start + 16 * members * rows * arena
    F.fake_limit(limit)
    E.ens_set_alloc([[64] * members] * rows, 64)
    for n in (64, 8, 64, 8, 64):
        E.ens_predict(x[:n])
    s = E.ens_debug_stats()
    assert s["copies"] == copies and s["copy_bytes"] > 0, s
    assert s["graphs"] == (2 if members == 4 else 0), s          # four lanes: recorded requests, which run on the copies' lanes too
    # images that fit without the copies only
    n = (limit - F.fake_used() + s["copy_bytes"] // 2) // (12 * 12 * 3 * 4 + (members + 1) * 8 * 4)
    held, before = F.fake_used(), F.fake_launches()
    E.ens_predict(np.zeros((n, 12, 12, 3), np.float32))
    t = E.ens_debug_stats()
    assert t["copies"] == t["copy_bytes"] == t["graphs"] == 0 and F.fake_launches() > before, t
    assert F.fake_used() <= limit and F.fake_used() > held
    for m in (64, 8, 64, 8):
        E.ens_predict(x[:m])
    # images that fit nowhere: refused, and the next request is answered
    E.ens_set_alloc([[64] * members] * rows, 64)
    out = np.empty((8, 8), np.float32)
    assert ens.lib().ens_predict(E._h, x.ctypes.data, 1 << 40, out.ctypes.data) == -2
    for m in (64, 8):
        E.ens_predict(x[:m])
    E.close()
    assert F.fake_used() == 0


@pytest.mark.parametrize("members,rows,copies", [(1, 1, 3), (1, 2, 2), (2, 1, 2), (4, 1, 4)])
def test_copies_go_when_a_request_finds_no_memory(fake_hip, members, rows, copies):
    """A request whose buffers do not fit beside the copies of the gangs is answered without them, as it was before there were copies."""
    beside_fake_hip(fake_hip, "copies_go(%d, %d, %d)" % (members, rows, copies))


def last_batch():
    import paper_2208_14049_amd as ens
    x, out = np.zeros((64, 12, 12, 3), np.float32), np.empty((8, 1, 1, 32), np.float32)
    for members, n in ((1, 29), (4, 29), (1, 8), (4, 61)):       # three copies of the one, one of each of the four
        E = tiny_ensemble(members)
        E.ens_set_alloc([[8] * members], 64)
        for size in (16, n, 2, 16, n, n):                        # what comes again runs from a graph with four members
            E.ens_predict(x[:size])
            in_last = (size - 1) % 8 + 1
            for m in range(members):
                rc = [ens.lib().ens_debug_tensor(E._h, m, 3, k, out.ctypes.data) for k in range(1, 9)]
                assert rc == [0] * in_last + [-1] * (8 - in_last), (members, size, m, rc)
        E.close()


def test_a_worker_tells_of_its_last_batch(fake_hip):
    """ens_debug_tensor is about the last batch of the member's first worker, whichever copy of its gang took it."""
    beside_fake_hip(fake_hip, "last_batch()")


def large_fp32_layers():
    import ctypes as C
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    fake().fake_limit(90 << 30)                                  # nothing is written there; no room for copies
    for side, cout, nb in ((2, 262160, 1), (32768, 1, 2)):       # wider than 65535 tiles of four channels; 2^31 output pixels
        n = N.Net("large", side, side, 8, dtype="fp32")
        n.fc(n.gap(n.conv(0, cout, 1)), 8)
        E = ens.Ensemble([n], [W.make_blob(n, 241, 0)])
        E.ens_set_alloc([[nb]])
        L, some = ens.lib(), np.empty(64, np.float32)
        assert L.ens_set_io(E._h, side, side, 1, 1) == 0
        assert L.ens_predict(E._h, C.c_void_p(some.ctypes.data), nb, C.c_void_p(some.ctypes.data)) == 0, (side, cout)
        E.close()


def test_fp32_layers_of_any_width(fake_hip):
    """The fp32 convolution is launched for every number of output channels, and for as many pixels as a launch can have threads."""
    beside_fake_hip(fake_hip, "large_fp32_layers()")


def graphs_go():
    F, x = fake(), np.zeros((64, 12, 12, 3), np.float32)
    E = tiny_ensemble(6)                                         # more groups than streams: no copies
    E.ens_set_alloc([[64] * 6], 64)
    for n in (64, 8, 3, 8, 3):
        E.ens_predict(x[:n])
    s = E.ens_debug_stats()
    assert s["graphs"] == 2 and s["copies"] == 0, s
    # room for larger buffers of a request once they, or its recordings, are gone
    F.fake_limit(F.fake_used() + (2 << 20))
    n = (5 << 20) // (12 * 12 * 3 * 4 + 7 * 8 * 4)
    E.ens_predict(np.zeros((n, 12, 12, 3), np.float32))
    assert E.ens_debug_stats()["graphs"] == 0
    for n in (64, 8, 3, 8):
        E.ens_predict(x[:n])
    E.close()
    assert F.fake_used() == 0


def test_recorded_requests_go_when_a_request_finds_no_memory(fake_hip):
    """The memory of recorded requests is given back to a request whose buffers do not fit beside them."""
    beside_fake_hip(fake_hip, "graphs_go()")


@pytest.fixture(scope="module")
def chain_view(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("view") / "libchain_view.so")
    subprocess.check_call(["hipcc", "-O1", "-std=c++17", "-fPIC", "-shared", "-x", "hip", "--offload-arch=gfx950", "-I" + os.path.join(ROOT, "paper_2208_14049_amd", "csrc"),
                           "-Wl,-Bsymbolic", "-o", lib, os.path.join(ROOT, "tests", "chain_view.cpp"), "-x", "none",
                           os.path.join(ROOT, "paper_2208_14049_amd", "libens_mi355x.so")])
    return lib


def odd_blocks(view):
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    V, none = ctypes.CDLL(view), 0
    for i, (h, c) in enumerate(((112, 96), (96, 48), (75, 32), (40, 328))):
        n = N.Net("odd%d" % i, h, h, 16, dtype="bf16")
        t = n.conv(n.conv(0, c, 3), 16, 1)
        t = n.conv(n.conv(t, c, 3), 2 * c, 1, pre=True)
        for _ in range(13):
            t = n.conv(t, 32, 3, stride=1 + (n.tensors[t][0] > 16))
        n.fc(n.gap(t), 16)
        E = ens.Ensemble([n], [W.make_blob(n, 251, i)])
        E.ens_set_alloc([[32]])
        assert V.chain_steps(E._h, 0) > 16
        beyond = ctypes.c_int()
        assert V.chain_weights_outside(E._h, 0, ctypes.byref(beyond)) == 0, (h, c)
        none += beyond.value
        E.close()
    assert none > 0                                              # wide tiles of which half has no channels were among them


def test_chains_read_no_weights_behind_a_layers_own(fake_hip, chain_view):
    """Output channels in an odd number of blocks of 32: the second half of the last wide tile has no weights to ask for."""
    beside_fake_hip(fake_hip, "odd_blocks(%r)" % chain_view)


def splits(view):
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    V, nets = ctypes.CDLL(view), []
    for short in (False, True):
        n = N.Net("stage%d" % short, 32, 32, 16, dtype="bf16")
        t = n.conv(n.conv(0, 32, 3, stride=2), 256, 1)
        a = n.conv(t, 512, 3, stride=2)
        t = n.conv(a, 512, 3, res=n.conv(t, 512, 1, stride=2, act=None) if short else None)
        for _ in range(15):
            t = n.conv(t, 32, 3)
        n.fc(n.gap(t), 16)
        nets.append(n)
    E = ens.Ensemble(nets, [W.make_blob(n, 255, i) for i, n in enumerate(nets)])
    E.ens_set_alloc([[32, 32]])
    for K in (9 * 256, 9 * 512):                                 # the layer beside a shortcut, and the one behind both
        s = [[V.chain_split(E._h, m, K, 512, z) for z in range(6)] for m in range(2)]
        assert -1 not in s[0] and s[0] == s[1], (K, s)
    assert V.chain_split(E._h, 0, 256, 512, 0) == -1 and V.chain_split(E._h, 1, 256, 512, 0) >= 0
    E.close()


def test_a_layers_sums_do_not_depend_on_its_neighbours(fake_hip, chain_view):
    """In how many parts a layer's sums are added up, and so its answer's last bits, follows from the layer and the images of a program, not from what
    else runs in its phase."""
    beside_fake_hip(fake_hip, "splits(%r)" % chain_view)


def tiles(view):
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    V, large = ctypes.CDLL(view), N.Net("large", 160, 160, 1000, dtype="bf16")
    t = large.conv(0, 64, 3)
    cat = large.tensor(160, 160, 256 + 256 + 64)                  # three branches; 32 images make 6 400 units of the first two
    for c0, c, k in ((0, 256, 3), (256, 256, 1), (512, 64, 5)):
        large.conv(t, c, k, dst=(cat, c0))
    t = cat
    for _ in range(15):
        t = large.conv(t, 32, 1)
    large.fc(large.gap(t), 1000)
    nets = [N.inception_v3(size=299), N.resnet50(), N.densenet121(), large]
    E = ens.Ensemble(nets, [W.make_blob(n, 257, i) for i, n in enumerate(nets)])
    E.ens_set_alloc([[32] * len(nets)])
    for m, net in enumerate(nets):
        better, most = ctypes.c_int(), ctypes.c_int()
        assert V.chain_tiles_wrong(E._h, m, ctypes.byref(better), ctypes.byref(most)) == 0, net.name
        assert better.value > 0 or net.name not in ("inception_v3", "resnet50"), net.name
    assert most.value > 2048
    E.close()


def test_tiles_of_a_phase(fake_hip, chain_view):
    """The tiles that a phase's convolutions are given together are none worse by the estimate than each one's own and cut K as those do; the estimate of a phase
    of one step is the step's, however many units it has."""
    beside_fake_hip(fake_hip, "tiles(%r)" % chain_view)


def routes():
    import paper_2208_14049_amd as ens
    from synth import nets as N
    # images: is it a chain?  (us as launches and as a chain)
    requests = [([N.resnet50(), N.densenet121()], 16, {1: True, 8: True}),                    # 924 / 631, 1024 / 769
                ([N.efficientnet(0), N.efficientnet(2), N.efficientnet(4)], 16, {1: True, 16: False}),   # 1186 / 993, 2026 / 2741
                ([N.resnet50()], 64, {1: False, 8: True, 45: False}),                         # 332 / 374, 473 / 410, 1217 / 1293
                ([N.inception_v3()], 16, {8: True, 16: True}),                                # 790 / 593, 1156 / 787
                ([N.xception()], 16, {1: False, 4: False}), ([N.vgg(16)], 16, {4: False})]    # 530 / 816, 660 / 895, 465 / 778
    for nets, batch, sizes in requests:
        E = ens.Ensemble(nets)
        E.set_base_size(224, 224)
        E.ens_set_alloc([[batch] * len(nets)])
        for n, chain in sizes.items():
            before = E.ens_debug_stats()["chained"]
            E.ens_predict(np.zeros((n, 224, 224, 3), np.float32))
            assert E.ens_debug_stats()["chained"] - before == chain, (nets[0].name, n)
        E.close()


def test_requests_go_the_faster_way(fake_hip):
    """Requests that were measured both ways, chains and launches at least 6 % apart, go the way that was faster."""
    beside_fake_hip(fake_hip, "routes()")


def wide_programs(view):
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    V = ctypes.CDLL(view)
    fake().fake_limit(90 << 30)                                  # nothing is written there
    # more images in a batch than a program's 16 bits count
    n = N.Net("many", 6, 6, 8, dtype="bf16")
    t = n.conv(0, 8, 3)
    for _ in range(15):
        t = n.conv(t, 8, 3)
    n.fc(n.gap(t), 8)
    E = ens.Ensemble([n], [W.make_blob(n, 261, 0)])
    E.ens_set_alloc([[40000]], 40000)
    assert V.chain_steps(E._h, 0) > 16 and V.chain_cap(E._h, 0) == 32767, V.chain_cap(E._h, 0)
    E.close()
    # 36 tensors of 128 MB at a time: more bytes for an image than 32 bits count
    n = N.Net("large", 1000, 1000, 8, dtype="bf16")
    held = [n.conv(0, 64, 1)]
    for _ in range(36):
        held.append(n.conv(held[-1], 64, 1))
    t = held[-1]
    for a in reversed(held[:-1]):
        t = n.conv(t, 64, 1, res=a)
    n.fc(n.gap(t), 8)
    E = ens.Ensemble([n], [W.make_blob(n, 262, 0)])
    E.ens_set_alloc([[2]])
    assert V.chain_steps(E._h, 0) == 0
    E.close()


def test_chains_within_the_widths_of_a_program(fake_hip, chain_view):
    """The first image of a program has 16 bits and the bytes of an image 32: larger batches and images are left to the launches."""
    beside_fake_hip(fake_hip, "wide_programs(%r)" % chain_view)


def members_in_lds():
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    F, nets = fake(), [N.tiny_a(classes=8), N.tiny_b(classes=8)]
    x = np.zeros((8, 32, 32, 3), np.float32)
    E = ens.Ensemble(nets, [W.make_blob(n, 281, i) for i, n in enumerate(nets)])
    bytes_of = [E.ens_member_bytes(m, 8) for m in range(2)]
    plain, reserve = sum(w for w, _ in bytes_of) + 2 * sum(a for _, a in bytes_of), 8 * (32 * 32 * 3 + 3 * 8) * 4   # two workers and a copy of each
    opts = dict(domain=[8], slots=1, strategy=1, n_calib=8, repeats=1)
    E.ens_plan(plain + reserve, **opts)                          # a budget for launches only
    assert E.ens_debug_stats()["copies"] == 2
    ran = E.ens_debug_stats()["chained"]
    E.ens_predict(x)
    assert E.ens_debug_stats()["chained"] == ran
    kept = E.ens_plan(1 << 30, **opts).bytes - plain
    assert 0 < kept < 1 << 20, kept
    ran = E.ens_debug_stats()["chained"]
    E.ens_predict(x)
    assert E.ens_debug_stats()["chained"] == ran + 1
    # what a request needs and finds only without them
    F.fake_limit(F.fake_used() + (1 << 20))
    n = ((1 << 20) + E.ens_debug_stats()["copy_bytes"] + kept // 2) // (32 * 32 * 3 * 4 + 3 * 8 * 4)
    E.ens_predict(np.zeros((n, 32, 32, 3), np.float32))
    s = E.ens_debug_stats()
    assert s["chained"] == ran + 1 and s["copies"] == 0, s
    E.ens_predict(x)
    assert E.ens_debug_stats()["chained"] == ran + 1
    E.close()
    assert F.fake_used() == 0


def test_members_in_lds_are_part_of_the_budget(fake_hip):
    """What small fp32 members keep on the device counts in their allocation's bytes and in a budget, and goes when a request finds no memory."""
    beside_fake_hip(fake_hip, "members_in_lds()")


def deep_members(count):
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    nets = []
    for i in range(count):
        n = N.Net("deep%d" % i, 12, 12, 8, dtype="bf16")
        t = n.conv(0, 16 + 8 * i, 3)                              # of shapes of their own: they share no launches
        for _ in range(15):
            t = n.conv(t, 16, 3)
        n.fc(n.gap(t), 8)
        nets.append(n)
    return ens.Ensemble(nets, [W.make_blob(n, 271, i) for i, n in enumerate(nets)])


def groups_give_up(view):
    V, F, x = ctypes.CDLL(view), fake(), np.zeros((4, 12, 12, 3), np.float32)
    E = deep_members(8)
    E.ens_set_alloc([[8] * 8])
    E.ens_predict(x)
    assert E.ens_debug_stats()["chained"] == 1
    before = F.fake_launches()
    V.chain_gave_up(E._h)
    E.ens_predict(x)                                             # a chain, and then the launches of every layer
    assert E.ens_debug_stats()["chained"] == 2 and F.fake_launches() - before > 16, F.fake_launches() - before
    E.ens_predict(x[:1])
    E.ens_predict(x)
    assert E.ens_debug_stats()["chained"] == 2
    E.ens_set_alloc([[8] * 8])
    E.ens_predict(x)
    assert E.ens_debug_stats()["chained"] == 3
    E.close()
    assert F.fake_used() == 0


def test_a_chain_that_gives_up_is_answered_by_launches(fake_hip, chain_view):
    """A group of compute units that waited in vain fails no request: its launches answer it, and those that follow until the next allocation."""
    beside_fake_hip(fake_hip, "groups_give_up(%r)" % chain_view)


def copies_first(view):
    V, E = ctypes.CDLL(view), deep_members(1)
    weights, arena = E.ens_member_bytes(0, 8)
    reserve = 8 * (12 * 12 * 3 + 2 * 8) * 4
    opts = dict(domain=[8], slots=1, strategy=1, n_calib=8, repeats=1)
    for extra, copies, chains in ((0, 3, False), (-1, 0, True), (1 << 20, 3, True)):
        a = E.ens_plan(weights + 4 * arena + reserve + extra, **opts)
        s = E.ens_debug_stats()
        assert s["copies"] == copies and (V.chain_steps(E._h, 0) > 0) == chains, (extra, s, V.chain_steps(E._h, 0))
        assert (a.bytes > weights + (1 + copies) * arena) == chains, (extra, a.bytes)
    E.close()


def test_copies_come_before_chains_in_a_budget(fake_hip, chain_view):
    """What is kept for requests of a few images takes nothing of a budget that copies of the workers would have fitted into."""
    beside_fake_hip(fake_hip, "copies_first(%r)" % chain_view)


def plans():
    import paper_2208_14049_amd as ens
    from synth import nets as N, weights as W
    small = [N.tiny_a(classes=8), N.tiny_b(classes=8)]
    for E, side in ((deep_members(8), 12), (ens.Ensemble(small, [W.make_blob(n, 281, i) for i, n in enumerate(small)]), 32)):
        for strategy in (0, 1, 2):
            a = E.ens_plan(0, domain=[8, 16], slots=1, strategy=strategy, n_calib=4, repeats=1, max_neighs=3, max_iter=1)
            assert a.score > 0 and E.ens_debug_stats()["chained"] == 0, (strategy, E.ens_debug_stats())
        E.ens_predict(np.zeros((4, side, side, 3), np.float32))
        E.ens_bench([[8] * E.n_members], n_calib=4, repeats=1)
        assert E.ens_debug_stats()["chained"] == 3, E.ens_debug_stats()   # the request, and the benchmark's warm-up and run
        E.close()


def test_plans_are_made_launch_by_launch(fake_hip):
    """The optimizer compares matrices by their workers' batches, members alone and all of them by the same path; requests and single benchmarks take theirs."""
    beside_fake_hip(fake_hip, "plans()")


def unequal_workers(view):
    V, E = ctypes.CDLL(view), deep_members(2)
    for matrix, chains in (([[8, 16]], True), ([[8, 16], [8, 16]], True), ([[8, 16], [8, 0]], True), ([[8, 8], [16, 8]], False), ([[8, 16], [0, 8]], False), ([[16, 8], [0, 16]], False)):
        E.ens_set_alloc(matrix)
        assert [V.chain_steps(E._h, m) > 0 for m in range(2)] == [chains] * 2, matrix
    E.close()


def test_chains_leave_unequal_workers_alone(fake_hip, chain_view):
    """Workers of one member with different batch sizes: which of them takes a batch is what such a matrix is about, so that its requests go launch by launch."""
    beside_fake_hip(fake_hip, "unequal_workers(%r)" % chain_view)
