"""The work that users of this library have it do, as timed cases.

A case is one pass through the public ``Net`` calls: a stretch of training
(dense patterns, one-hot windows or sequence streams), which returns the error
sum and the updated weights and momentum, or a forward pass, which returns the
output activations.  Sizes follow the named workloads of
``paper_1801_01554_amd.workloads`` and the paper's NETtalk net, and beside them
generic nets outside those: odd layer widths, short last batches, windows and
hidden layers past the sizes of the named nets.

Inputs are seeded; targets come from a random linear teacher, so that training
has something to learn, and the step size is scaled by batch and layer width
so that units neither saturate nor stand still.
"""
import math

import torch

from paper_1801_01554_amd import bp
from paper_1801_01554_amd import metrics
from paper_1801_01554_amd import workloads as wl

SYMBOLS = 29           # symbols per letter position of a one-hot window
MOMENTUM = 0.9
FAULT_LIMIT = 1.0e6    # range check: far above any sound summed change


def _case(name, kind, sizes, **more):
    c = {"name": name, "kind": kind, "sizes": sizes, "sigmoid": "exact", "checked": False}
    c.update(more)
    return c


def listed():
    return [
        # One word through the text-to-speech net: the smallest call, all latency.
        _case("word_onehot", "forward_onehot", "203-120-26", n=8),
        # A corpus through the same net, table sigmoid (the paper's evaluation).
        _case("corpus_onehot", "forward_onehot", "203-120-26", n=20000, sigmoid="table"),
        # An epoch of the NETtalk-shaped net in batches of 512 (40 updates, the last one short).
        _case("epoch_onehot_512", "train_onehot", "203-120-26", n=20000, batch=512),
        # The same corpus in batches of 16 with the range check on: 250 updates of launch latency.
        _case("epoch_onehot_16", "train_onehot", "203-120-26", n=4000, batch=16, checked=True),
        # A wider window and hidden layer than the paper's, with a pooled batch of thousands.
        _case("epoch_onehot_wide", "train_onehot", "435-512-64", n=10000, batch=4096),
        # The paper's 203-60-26 net fed dense rows (input rows of 812 bytes) in small batches.
        _case("epoch_dense_small", "train", "203-60-26", n=1000, batch=100),
        # Odd widths in every layer, batches that are no multiple of anything, a short last one.
        _case("epoch_dense_odd", "train", "333-1100-701-61", n=7100, batch=1500),
        # The wide and deep nets of the benchmark, half an epoch each.
        _case("epoch_dense_wide", "train", "1024-4096-1024", n=131072, batch=4096),
        _case("epoch_dense_deep", "train", "512-2048-2048-2048-64", n=262144, batch=8192),
        # Scoring a held-out set with the deep net: whole chunks and a remainder.
        _case("score_dense_deep", "forward", "512-2048-2048-2048-64", n=20011),
        # Recurrent nets: an epoch of 1024 parallel streams, an update every 8 steps.
        _case("epoch_sequences", "train_sequences", "320-256-64", n_ctx=256, streams=1024, steps=128, window=8),
        # The same net run forward over streams, no learning.
        _case("run_sequences", "forward_sequences", "320-256-64", n_ctx=256, streams=1000, steps=64),
    ]


# ---------------------------------------------------------------- draws

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: sizes spread over their logarithm, odd ones as often as round ones."""
    while True:
        kind = rng.choice(("forward_onehot", "train_onehot", "train_onehot", "train", "train", "train", "forward",
                           "train_sequences", "forward_sequences"))
        c = {"kind": kind, "sigmoid": rng.choice(("exact", "exact", "table")), "checked": rng.random() < 0.25}
        if kind.endswith("onehot"):
            sizes = [SYMBOLS * rng.randint(3, 15), _log(rng, 20, 1024), _log(rng, 5, 128)]
        elif kind.endswith("sequences"):
            hidden = _log(rng, 16, 512)
            sizes = [_log(rng, 8, 128) + hidden, hidden, _log(rng, 4, 128)]
            c.update(n_ctx=hidden, streams=_log(rng, 16, 2048), steps=_log(rng, 8, 128))
        else:
            sizes = [_log(rng, 32, 2048)] + [_log(rng, 32, 4096) for _ in range(rng.randint(1, 3))] + [_log(rng, 8, 1024)]
        if kind.startswith("forward"):
            c["checked"] = False
            if kind != "forward_sequences":
                c["n"] = _log(rng, 1, 40000)
        elif kind == "train_sequences":
            c["window"] = rng.randint(1, 16)
        else:
            c["batch"] = _log(rng, 8, 8192)
            c["n"] = c["batch"] * _log(rng, 1, 40) - rng.choice((0, 0, c["batch"] // 3))
        c["sizes"] = "-".join(str(v) for v in sizes)
        if work(c)["flops"] <= 3e12:
            return c


# ---------------------------------------------------------------- inputs

def _sizes(case):
    return tuple(int(v) for v in case["sizes"].split("-"))


def _patterns(case):
    return case["steps"] * case["streams"] if case["kind"].endswith("sequences") else case["n"]


def _lr(case):
    """Step of the summed change: a mean over the patterns of an update, smaller for wide layers."""
    rows = case["window"] * case["streams"] if case["kind"] == "train_sequences" else min(case["batch"], case["n"])
    return 2.0 / (rows * max(64, *_sizes(case)[1:]))


def _data(case, seed):
    """The pass's inputs on the GPU: input rows or active indices, targets, flags, and host weights."""
    sizes, kind, n = _sizes(case), case["kind"], _patterns(case)
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    d = {"weights": wl.draw_weights(seed, sizes, "uniform0.3" if kind.endswith("onehot") else "fanin")}
    if kind.endswith("onehot"):
        pos = sizes[0] // SYMBOLS
        sym = torch.randint(0, SYMBOLS, (n, pos), generator=g, device="cuda", dtype=torch.int32)
        d["active"] = sym + SYMBOLS * torch.arange(pos, device="cuda", dtype=torch.int32)
    elif kind.endswith("sequences"):
        T, S, n_ext = case["steps"], case["streams"], sizes[0] - case["n_ctx"]
        d["inputs"] = torch.randn((T, S, n_ext), generator=g, device="cuda")
        # sequences of 40 steps on average, a tenth of the patterns padding
        d["cont"] = (torch.rand((T, S), generator=g, device="cuda") > 0.025).float()
        d["mask"] = (torch.rand((T, S), generator=g, device="cuda") > 0.1).float()
    else:
        d["inputs"] = torch.randn((n, sizes[0]), generator=g, device="cuda")
    if kind.startswith("train"):
        if kind == "train_onehot":
            teacher = torch.randn((sizes[0], sizes[-1]), generator=g, device="cuda")
            score = torch.zeros((n, sizes[-1]), device="cuda")
            for k in range(d["active"].shape[1]):
                score += teacher[d["active"][:, k].long()]
        else:
            x = d["inputs"]
            score = x @ torch.randn((x.shape[-1], sizes[-1]), generator=g, device="cuda")
        d["targets"] = torch.where(score > 0, 0.9, 0.1).float().contiguous()
        del score
    return d


def prepare(case, seed):
    state = _data(case, seed)
    sizes = _sizes(case)
    net = bp.Net(sizes)
    net.set_weights(state.pop("weights"))
    if case["kind"].endswith("sequences"):
        net.set_context([1] * case["n_ctx"], list(range(case["n_ctx"])))
    if case["sigmoid"] == "table":
        net.set_sigmoid(bp.BP_SIGMOID_TABLE)
    if case["checked"]:
        net.set_fault_limit(FAULT_LIMIT)
    state.update(net=net, kind=case["kind"], batch=case.get("batch"), window=case.get("window"))
    if case["kind"].startswith("train"):
        state["lr"] = _lr(case)
    return state


def run(state):
    net, kind = state["net"], state["kind"]
    if kind == "forward":
        return net.forward(inputs=state["inputs"])
    if kind == "forward_onehot":
        return net.forward(active=state["active"])
    if kind == "forward_sequences":
        return net.forward_sequences(state["inputs"], state["cont"])
    if kind == "train_sequences":
        sse = net.train_sequences(state["inputs"], state["targets"], state["cont"], state["mask"], state["window"],
                                  state["lr"], MOMENTUM)
    else:
        sse = net.train_batches(state["targets"], state["batch"], state["lr"], MOMENTUM, inputs=state.get("inputs"),
                                active=state.get("active"))
    return {"sse": sse, "weights": net.get_weights(), "momentum": net.get_momentum()}


# ---------------------------------------------------------------- work and tolerance

def work(case):
    """Bytes: inputs, targets or outputs once, and the state (training: weights and momentum read, written and handed
    over; forward: weights read).  Flops: the products of the method; a one-hot first layer adds its active rows."""
    sizes, kind, n = _sizes(case), case["kind"], _patterns(case)
    W = metrics.num_weights(sizes)
    if kind.endswith("onehot"):
        pos = sizes[0] // SYMBOLS
        dense = W - (sizes[0] + 1) * sizes[1]
        row, fwd, chg = pos, 2.0 * dense + (pos + 1) * sizes[1], 2.0 * dense + (pos + 1) * sizes[1]
    else:
        row = sizes[0] - case.get("n_ctx", 0) + (2 if kind.endswith("sequences") else 0)
        fwd = chg = 2.0 * W
    if kind.startswith("forward"):
        return {"bytes": 4.0 * (n * (row + sizes[-1]) + W), "flops": n * fwd}
    hidden = sum(2.0 * sizes[l] * sizes[l + 1] for l in range(1, len(sizes) - 1))
    return {"bytes": 4.0 * (n * (row + sizes[-1]) + 6 * W), "flops": n * (fwd + hidden + chg)}


def tolerance(case):
    """About four times the largest difference from 64 bits that the fp32 path shows over the listed and some thirty
    drawn cases: forward 3.1e-7 (largest 2.0e-6), training 1.2e-6 in the momentum (largest 1.4e-5)."""
    if case["kind"].startswith("forward"):
        return {"rel": 1.2e-6, "max": 8e-6}
    return {"rel": 5e-6, "max": 6e-5}


# ---------------------------------------------------------------- the same in 64 bits

def _sigma(z, table):
    if not table:
        return torch.sigmoid(z)
    entry = torch.sigmoid(-15.0 + 30.0 * torch.arange(256, dtype=torch.float64, device=z.device) / 255.0)
    x1 = (z.clamp(-15.0, 15.0) + 15.0) * 8.5
    i = x1.floor().clamp(max=254).long()
    lo, hi = entry[i], entry[i + 1]
    return lo + (x1 - i) * (hi - lo)


def exact(case, seed):
    sizes, kind = _sizes(case), case["kind"]
    table = case["sigmoid"] == "table"
    if _updates(case) > 2000:
        return None
    d = _data(case, seed)
    flat = torch.from_numpy(d["weights"]).cuda().double()
    W, o = [], 0
    for a, b in zip(sizes[:-1], sizes[1:]):
        W.append(flat[o:o + (a + 1) * b].view(a + 1, b).clone())
        o += (a + 1) * b
    onehot = kind.endswith("onehot")

    def inputs(lo, hi):
        if not onehot:
            return d["inputs"][lo:hi].double()
        x = torch.zeros((hi - lo, sizes[0]), dtype=torch.float64, device="cuda")
        return x.scatter_(1, d["active"][lo:hi].long(), 1.0)

    def forward(x):
        acts = [x]
        for w in W:
            acts.append(_sigma(acts[-1] @ w[:-1] + w[-1], table))
        return acts

    if kind in ("forward", "forward_onehot"):
        return torch.cat([forward(inputs(lo, min(case["n"], lo + 8192)))[-1] for lo in range(0, case["n"], 8192)])

    V = [torch.zeros_like(w) for w in W]
    lr = float(torch.tensor(_lr(case), dtype=torch.float32)) if kind.startswith("train") else 0.0
    mom = float(torch.tensor(MOMENTUM, dtype=torch.float32))

    def update(acts, delta):
        for l in range(len(W) - 1, -1, -1):
            below = (delta @ W[l][:-1].T) * acts[l] * (1 - acts[l]) if l else None
            V[l].mul_(mom)
            V[l][:-1] += lr * (acts[l].T @ delta)
            V[l][-1] += lr * delta.sum(0)
            W[l] += V[l]
            delta = below

    sse = torch.zeros((), dtype=torch.float64, device="cuda")
    if kind == "train" or kind == "train_onehot":
        for lo in range(0, case["n"], case["batch"]):
            hi = min(case["n"], lo + case["batch"])
            acts = forward(inputs(lo, hi))
            e = d["targets"][lo:hi].double() - acts[-1]
            sse += (e * e).sum()
            update(acts, e * acts[-1] * (1 - acts[-1]))
    else:
        T, S, step = case["steps"], case["streams"], case.get("window", case["steps"])
        hidden = torch.zeros((S, case["n_ctx"]), dtype=torch.float64, device="cuda")
        outs = []
        for w0 in range(0, T, step):
            acts, deltas = [], []
            for t in range(w0, min(T, w0 + step)):
                x = torch.cat([d["inputs"][t].double(), d["cont"][t].double()[:, None] * hidden], 1)
                a = forward(x)
                hidden = a[1][:, :case["n_ctx"]]
                outs.append(a[-1])
                if kind == "train_sequences":
                    e = (d["targets"][t].double() - a[-1]) * d["mask"][t].double()[:, None]
                    sse += (e * e).sum()
                    acts.append(a)
                    deltas.append(e * a[-1] * (1 - a[-1]))
            if kind == "train_sequences":
                update([torch.cat(a) for a in zip(*acts)], torch.cat(deltas))
        if kind == "forward_sequences":
            return torch.stack(outs)
    return {"sse": float(sse), "weights": torch.cat([w.reshape(-1) for w in W]),
            "momentum": torch.cat([v.reshape(-1) for v in V])}


def _updates(case):
    if case["kind"] == "train_sequences":
        return -(-case["steps"] // case["window"])
    return -(-case["n"] // case["batch"]) if case["kind"].startswith("train") else 0
