"""What a program that serves ensembles with this library has it do, as cases to be timed.

A case is one request: an ensemble that is loaded and laid out on the GPU, and `images` images that are
predicted in one call of `ens_predict` (or `ens_predict_static`), from the images as the caller holds them
to the combined class probabilities where the caller wants them.  A serving program loads an ensemble and
installs its allocation once and then answers request after request, each in a buffer of its own; so the
ensembles are kept here between states, with fixed weights, and a state is a request's images.

Fields of a case:
  ensemble   which members (see ENSEMBLES)
  images     images of the request
  batch      batch size of every worker; 0 = the allocation kept for this workload in allocations.json
  rows       worker rows of the allocation matrix (instances per member); ignored with batch 0
  base       height and width of the request's images (members of another resolution get them resized)
  input      "device": fp32 tensor on the GPU, answer on the GPU; "pinned": pinned host tensors;
             "numpy": ordinary host arrays, as a request decoder or a data loader leaves them
  entry      "predict", or "static" for the entry point that allocates nothing (device tensors only)
  rule       combination: "mean" of the members' softmax outputs or "weighted" average
"""
import json
import math
import os

import numpy as np
import torch

import paper_2208_14049_amd as ens
from synth import nets as N

TABLE_BYTES = 4096              # bytes of the static entry point's pointer table

# workload configurations 1-5 and the paper's four-member ensemble, and the light members of configuration 6
ENSEMBLES = {
    "tiny_fp32": lambda: N.config_members(1),
    "resnet18x3": lambda: N.config_members(2),
    "hetero4": lambda: N.config_members(3),
    "heavy12": lambda: N.config_members(4),
    "resnet50": lambda: N.config_members(5),
    "imn4": lambda: N.config_members(8),
    "light3": lambda: [N.resnext50(), N.xception(size=299), N.mobilenet_v2()],
}
KEPT = {"resnet18x3": "2", "hetero4": "3", "heavy12": "4", "resnet50": "5"}
BATCHES = (8, 16, 32, 64, 128)  # the planner's default domain
PARAM_SEED = 220814049

_nets, _handles, _costs = {}, {}, {}


def _case(name, ensemble, images, batch=0, rows=1, base=224, input="device", entry="predict", rule="mean"):
    return dict(name=name, ensemble=ensemble, images=images, batch=batch, rows=rows, base=base, input=input, entry=entry,
                rule=rule)


def listed():
    return [
        # one user's image sent to a small fp32 ensemble: launches and host work only
        _case("tiny_fp32_online", "tiny_fp32", 8, batch=8, base=32, input="numpy"),
        # the same ensemble over a data set resident on the GPU, last batch short
        _case("tiny_fp32_bulk", "tiny_fp32", 8100, batch=128, base=32),
        # one image, the allocation a handle has when nothing was planned (batch size 8): latency of a light service
        _case("resnet18x3_single", "resnet18x3", 1, batch=8, input="numpy"),
        # a few images for one deep member through the allocation-free entry point of a tight serving loop
        _case("resnet50_few", "resnet50", 4, batch=16, entry="static"),
        # one image through twelve co-located members: hundreds of short launches on twelve streams
        _case("heavy12_single", "heavy12", 1),
        # a micro-batch that an adaptive-batching front end collects
        _case("hetero4_microbatch", "hetero4", 32),
        # a request that fills no batch, images as a decoder leaves them in host memory
        _case("hetero4_ragged_host", "hetero4", 300, input="numpy"),
        # images at another resolution than any member's, weighted combination
        _case("imn4_resized_weighted", "imn4", 100, batch=64, base=256, rule="weighted"),
        # grouped and separable convolutions, batch size of the middle of the range, ragged
        _case("light3_ragged", "light3", 215, batch=64),
        # offline throughput on resident images, small batch size and two instances per member
        _case("resnet18x3_bulk", "resnet18x3", 1024),
        # offline throughput of one member with images streamed from host memory
        _case("resnet50_bulk_host", "resnet50", 1024, input="pinned"),
        # offline throughput of the heavy ensemble (the benchmark's headline)
        _case("heavy12_bulk", "heavy12", 1024),
    ]


def draw(rng):
    name = rng.choice(sorted(ENSEMBLES))
    most = 8192 if name == "tiny_fp32" else 1024
    n = max(1, min(most, int(round(math.exp(rng.uniform(0.0, math.log(most)))))))
    kept = name in KEPT and rng.random() < 0.4
    base = 32 if name == "tiny_fp32" else rng.choice((224, 224, 224, 256))
    where = rng.choice(("device", "device", "pinned", "numpy"))
    entry = "static" if where == "device" and rng.random() < 0.3 and _fits_static(name, n) else "predict"
    # large requests of deep members are planned with the larger batch sizes
    batches = BATCHES if n <= 256 or name == "tiny_fp32" else BATCHES[2:]
    c = _case("", name, n, batch=0 if kept else rng.choice(batches), rows=1 if kept else rng.choice((1, 1, 2)), base=base,
              input=where, entry=entry, rule=rng.choice(("mean", "mean", "mean", "weighted")))
    del c["name"]
    return c


def _members(name):
    if name not in _nets:
        _nets[name] = ENSEMBLES[name]()
    return _nets[name]


def _fits_static(name, n):
    nets = _members(name)
    return n * len(nets) * nets[0].classes * 4 <= ens.lib().ens_static_scratch_bytes() - TABLE_BYTES


def _params(net, index):
    """A member's parameter blob (the distributions of synth.weights, drawn on the GPU), as a trained one would be given."""
    g = torch.Generator(device="cuda").manual_seed(PARAM_SEED + index)
    blob = torch.randn(net.blob_size, generator=g, device="cuda")
    for p in net.params:
        o, s = p["offset"], p["size"]
        if p["role"] == "conv_w":
            blob[o:o + s] *= p["std"]
            if net.dtype == "bf16":
                blob[o:o + s] = blob[o:o + s].bfloat16().float()
        elif p["role"] == "bias":
            blob[o:o + s] *= 0.1
        else:
            c = p["channels"]
            blob[o:o + c] = p["gamma"]
            blob[o + c:o + 2 * c] = 0.0
            blob[o + 2 * c:o + 3 * c] *= 0.1
            blob[o + 3 * c:o + 4 * c] = torch.rand(c, generator=g, device="cuda") + 0.5
    return blob.cpu().numpy()


def _handle(case):
    """The ensemble of a case, loaded and laid out, kept as a serving program keeps it."""
    key = tuple(case[k] for k in ("ensemble", "batch", "rows", "base", "rule"))
    if key not in _handles:
        nets = _members(case["ensemble"])
        E = ens.Ensemble(nets, [_params(net, i) for i, net in enumerate(nets)])
        segment = 128
        if case["batch"]:
            matrix = [[case["batch"]] * len(nets)] * case["rows"]
        else:
            with open(os.path.join(os.path.dirname(os.path.abspath(ens.__file__)), "allocations.json")) as f:
                kept = json.load(f)[KEPT[case["ensemble"]]]
            matrix, segment = kept["matrix"], kept["segment"]
        E.set_base_size(case["base"], case["base"])
        E.ens_set_alloc(matrix, segment)
        if case["rule"] == "weighted":
            w = [1.0 + 0.25 * i for i in range(len(nets))]
            E.ens_set_combination("weighted", [v / sum(w) for v in w])
        _handles[key] = E
    return _handles[key]


def prepare(case, seed):
    E = _handle(case)
    n, s = case["images"], case["base"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    # contrast and colour cast differ from image to image, as in photographs that were normalised by data-set statistics
    x = torch.randn((n, s, s, 3), generator=g, device="cuda")
    x *= torch.rand((n, 1, 1, 1), generator=g, device="cuda") * 1.5 + 0.25
    x += torch.randn((n, 1, 1, 3), generator=g, device="cuda")
    out = None
    if case["input"] == "numpy":
        x = x.cpu().numpy()
    elif case["input"] == "pinned":
        h = torch.empty(x.shape, dtype=torch.float32, pin_memory=True)
        h.copy_(x)
        x = h
        out = torch.empty((n, E.classes), dtype=torch.float32, pin_memory=True)
    elif case["entry"] == "static":
        out = torch.empty((n, E.classes), dtype=torch.float32, device="cuda")
    return dict(E=E, x=x, out=out, static=case["entry"] == "static")


def run(state):
    E = state["E"]
    if state["static"]:
        return E.ens_predict_static(state["x"], state["out"])
    return E.ens_predict(state["x"], state["out"])


def _member_cost(net):
    """(flop per image, parameter bytes) of one member."""
    flop = 0.0
    for o in net.ops:
        h, w, _ = net.tensors[o["dst"]]
        if o["kind"] == N.CONV:
            flop += 2.0 * h * w * o["cout"] * o["kh"] * o["kw"] * o["cin"] / max(1, o["r"])
        elif o["kind"] == N.DWCONV:
            flop += 2.0 * h * w * o["cout"] * o["kh"] * o["kw"]
        elif o["kind"] == N.FC:
            flop += 2.0 * o["cin"] * o["cout"]
        elif o["kind"] == N.SE:
            flop += 4.0 * o["cin"] * o["r"]
    return flop, net.blob_size * (2.0 if net.dtype == "bf16" else 4.0)


def work(case):
    name = case["ensemble"]
    if name not in _costs:
        _costs[name] = [sum(v) for v in zip(*[_member_cost(net) for net in _members(name)])]
    flop, params = _costs[name]
    n = case["images"]
    return {"bytes": params + n * (case["base"] ** 2 * 3 + _members(name)[0].classes) * 4.0, "flops": flop * n}


def tolerance(case):
    if case["ensemble"] == "tiny_fp32":
        return {"rel": 1e-5, "max": 1e-4}
    # probabilities after 20 to 200 layers with bf16 activations: a sum taken in another order flips roundings of 2^-9,
    # and softmax turns a logit's absolute error into a relative one
    return {"rel": 1e-2, "max": 0.1}
