"""The measured cases of the Zeno aggregation library.

A case is the work of one server iteration through the public entry points of
paper_1805_10032_amd.binding:

  kind "mlp"        zeno_score, then zeno_aggregate_update (or zeno_aggregate), for a chain of linear layers
  kind "cnn"        the same for a convolutional model
  kind "baselines"  zeno_mean, zeno_median and zeno_krum on the candidates of one iteration
  kind "median"     zeno_median alone, for more candidates than zeno_krum takes

Candidates are what a server meets: the workers' minibatch gradients at the current parameters, some of
them replaced by a fault (the honest mean times -4, copied over all such rows, and Gaussian rows three times
as long as an honest one).  Everything is made on the GPU from the seed.  The same plain-torch model gives
the workers' gradients in float32 and the float64 values of exact().
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1805_10032_amd import binding as B

_CNN = {"hw": 32, "c_in": 3, "conv": "32/1 32/2 64/1 64/2", "out": 10}


def listed():
    mlp = {"kind": "mlp", "bias": True, "loss": "softmax_ce", "fwd": "fp32", "align": 1, "static": False, "update": True}
    return [
        # the smallest call: a linear model, eight workers, scratch inside the library; launches and host time count
        dict(mlp, name="linear_64", dims="64 1", bias=False, loss="squared", m=8, b=2, n_r=16, gamma=0.1, rho=5e-4,
             static=True),
        # softmax regression on 28 x 28 images with the paper's twenty workers, eight of them faulty
        dict(mlp, name="softmax_784", dims="784 10", m=20, b=8, n_r=32, gamma=0.1, rho=5e-4),
        # an ordinary small network on 32 x 32 x 3 images, rows of G packed as a plain [m x d] tensor
        dict(mlp, name="mlp_3072_512", dims="3072 512 10", m=20, b=8, n_r=32, gamma=0.05, rho=1e-3),
        # a wide network in float32 (the default precision), rows of G as alloc_candidates places them
        dict(mlp, name="mlp_2048_fp32", dims="3072 2048 2048 2048 10", m=20, b=8, n_r=32, gamma=0.05, rho=1e-3, align=32),
        # the same network for a hundred workers with bf16 operands, rows of G packed (8-byte aligned only)
        dict(mlp, name="mlp_2048_bf16_m100", dims="3072 2048 2048 2048 10", m=100, b=40, n_r=64, gamma=0.05, rho=1e-3,
             fwd="bf16"),
        # the largest: 14 GB of candidates, selection and average as two calls
        dict(mlp, name="mlp_4096_bf16_m64", dims="4096 4096 4096 4096 1000", m=64, b=16, n_r=128, gamma=0.02, rho=1e-4,
             fwd="bf16", align=32, update=False),
        # odd widths, odd row length, more samples than one pass over G takes
        dict(mlp, name="mlp_ragged_nr200", dims="1001 777 333 7", m=33, b=10, n_r=200, gamma=0.05, rho=5e-4, fwd="bf16"),
        # the paper's model class with the paper's server batch of four, and with an ordinary batch
        dict(_CNN, name="cnn_nr4", kind="cnn", m=20, b=8, n_r=4, gamma=0.1, rho=5e-4),
        dict(_CNN, name="cnn_nr32", kind="cnn", m=20, b=8, n_r=32, gamma=0.1, rho=5e-4),
        # the rules Zeno is compared with, on the small network's candidates and on a hundred large ones
        {"name": "baselines_m20", "kind": "baselines", "m": 20, "d": 1578506, "b": 8, "align": 1},
        {"name": "baselines_m100", "kind": "baselines", "m": 100, "d": 14706698, "b": 40, "align": 32},
        # the marginal median over several hundred workers
        {"name": "median_m300", "kind": "median", "m": 300, "d": 1578506, "b": 100, "align": 1},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the listed ranges; at most about half of the largest listed one's time."""
    kind = rng.choice(["mlp", "mlp", "mlp", "mlp", "cnn", "cnn", "baselines", "baselines", "median"])
    align = rng.choice([1, 1, 4, 32])
    if kind == "mlp":
        layers = rng.choice([1, 2, 2, 3, 3, 4])
        widths = [_log(rng, 32, 4096)] + [_log(rng, 16, 4096) for _ in range(layers - 1)]
        if rng.random() < 0.5:
            widths = [max(64, w // 64 * 64) for w in widths]
        loss = rng.choice(["softmax_ce", "softmax_ce", "softmax_ce", "squared"])
        widths.append(1 if loss == "squared" else rng.choice([2, 10, 10, 100, 1000]))
        m, n_r, fwd = _log(rng, 4, 100), _log(rng, 1, 200), rng.choice(["fp32", "bf16"])
        case = {"kind": kind, "bias": rng.random() < 0.8, "loss": loss, "fwd": fwd, "align": align, "static": False,
                "update": rng.random() < 0.7, "dims": "", "m": m, "b": rng.randint(0, m // 2), "n_r": n_r,
                "gamma": rng.choice([0.02, 0.05, 0.1]), "rho": rng.choice([0.0, 1e-4, 5e-4, 1e-3])}
        while True:
            case["dims"] = " ".join(map(str, widths))
            w = work(case)
            if 4.0 * _num_params(case) * m <= 4e9 and w["flops"] <= (1e11 if fwd == "fp32" else 6e11):
                return case
            widths = [max(16, int(v * 0.8)) for v in widths[:-1]] + widths[-1:]
    if kind == "cnn":
        convs = []
        for _ in range(rng.choice([1, 2, 3, 4])):
            convs.append("%d/%d" % (rng.choice([8, 16, 20, 32, 33, 48, 64]), rng.choice([1, 2])))
        m, n_r = _log(rng, 4, 40), _log(rng, 1, 64)
        case = {"kind": kind, "hw": rng.choice([8, 14, 28, 32]), "c_in": rng.choice([1, 3]), "conv": " ".join(convs), "out": 10,
                "m": m, "b": rng.randint(0, m // 2), "n_r": n_r, "gamma": rng.choice([0.05, 0.1]), "rho": rng.choice([0.0, 5e-4])}
        while work(case)["flops"] > 3e10 and case["n_r"] > 1:
            case["n_r"] = max(1, case["n_r"] * 3 // 4)
        return case
    m = _log(rng, 5, 128) if kind == "baselines" else _log(rng, 129, 1024)
    d = _log(rng, 64, 1e7)
    d = max(64, min(d, int((3e9 if kind == "baselines" else 1.5e9) // (4 * m))))
    return {"kind": kind, "m": m, "d": d, "b": (m - 3) // 2 if rng.random() < 0.5 else rng.randint(0, (m - 3) // 2), "align": align}


# ---- models in plain torch

def _dims(case):
    return [int(v) for v in case["dims"].split()]


def _convs(case):
    return [tuple(int(v) for v in c.split("/")) for c in case["conv"].split()]


def _maps(case):
    """[(height = width, channels)] of the input and of every map: 3 x 3 kernels, zero padding 1."""
    maps = [(case["hw"], case["c_in"])]
    for c, stride in _convs(case):
        maps.append(((maps[-1][0] - 1) // stride + 1, c))
    return maps


def _blocks(case):
    """[(rows, columns, has bias)] of the weight matrices in the order of a parameter vector."""
    if case["kind"] == "mlp":
        dims = _dims(case)
        return [(n, k, case["bias"]) for k, n in zip(dims[:-1], dims[1:])]
    maps = _maps(case)
    blocks = [(c, 9 * ci, True) for (_, ci), (_, c) in zip(maps[:-1], maps[1:])]
    return blocks + [(case["out"], maps[-1][0] ** 2 * maps[-1][1], True)]


def _num_params(case):
    return sum(n * k + (n if bias else 0) for n, k, bias in _blocks(case))


def _views(p, case):
    out, off = [], 0
    for n, k, bias in _blocks(case):
        W, off = p[off:off + n * k].view(n, k), off + n * k
        if bias:
            out.append((W, p[off:off + n]))
            off += n
        else:
            out.append((W, None))
    return out


def _affine(h, W, bias):
    z = h @ W.t()
    return z if bias is None else z + bias


def _logits(p, case, features):
    """The model's outputs at the flat parameters p, in p's precision."""
    h = features.to(p.dtype)
    layers = _views(p, case)
    if case["kind"] == "cnn":
        n = h.shape[0]
        h = h.view(n, case["hw"], case["hw"], case["c_in"])
        for (W, bias), (_, stride) in zip(layers, _convs(case)):
            size = (h.shape[1] - 1) // stride + 1
            padded = torch.nn.functional.pad(h, (0, 0, 1, 1, 1, 1))
            last = stride * (size - 1) + 1
            taps = [padded[:, y:y + last:stride, x:x + last:stride] for y in range(3) for x in range(3)]
            h = torch.relu(_affine(torch.cat(taps, -1).reshape(n * size * size, -1), W, bias)).view(n, size, size, -1)
        return _affine(h.reshape(n, -1), *layers[-1])
    for W, bias in layers[:-1]:
        h = torch.relu(_affine(h, W, bias))
    return _affine(h, *layers[-1])


def _loss(case, z, labels, targets):
    if case.get("loss") == "squared":
        return 0.5 * torch.mean((z[:, 0] - targets.to(z.dtype)) ** 2)
    return torch.mean(torch.logsumexp(z, 1) - z.gather(1, labels.long()[:, None])[:, 0])


# ---- inputs

def _rows(m, d, align):
    """An uninitialised [m x d] candidate matrix: packed, or as alloc_candidates lays the rows out."""
    if align == 1:
        return torch.empty((m, d), dtype=torch.float32, device="cuda")
    return B.alloc_candidates(m, d, torch.device("cuda"), align)


def _batch(case, n, gen):
    width = _dims(case)[0] if case["kind"] == "mlp" else case["hw"] ** 2 * case["c_in"]
    features = torch.randn((n, width), generator=gen, device="cuda")
    if case.get("loss") == "squared":
        return features, None, torch.randn(n, generator=gen, device="cuda")
    classes = _blocks(case)[-1][0]
    return features, torch.randint(0, classes, (n,), generator=gen, device="cuda", dtype=torch.int32), None


def _faults(G, rows, gen):
    """Replace the given rows: the first half of them by -4 times the honest mean, the others by noise."""
    if not rows:
        return
    honest = [i for i in range(G.shape[0]) if i not in set(rows)]
    total = torch.zeros(G.shape[1], device="cuda")
    for i in honest:
        total += G[i]
    norm = torch.linalg.vector_norm(G[honest[0]])
    flips = rows[:(len(rows) + 1) // 2]
    for i in rows:
        if i in flips:
            G[i] = total * (-4.0 / len(honest))
        else:
            noise = torch.randn(G.shape[1], generator=gen, device="cuda")
            G[i] = noise * (3.0 * norm / torch.linalg.vector_norm(noise))


def _inputs(case, seed):
    """Parameters, candidates and the server's batch, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    m, b = case["m"], case["b"]
    order = torch.randperm(m, generator=torch.Generator().manual_seed(seed)).tolist()
    if case["kind"] in ("baselines", "median"):
        # rows around one common gradient, each worker's at its own distance from it
        G = _rows(m, case["d"], case["align"])
        common = torch.randn(case["d"], generator=gen, device="cuda") * 0.01
        for i in range(m):
            G[i] = torch.randn(case["d"], generator=gen, device="cuda").mul_(0.01 + 0.01 * (order[i] + 1) / m).add_(common)
        _faults(G, sorted(order[:b]), gen)
        return {"G": G}
    d = _num_params(case)
    x = torch.zeros(d, device="cuda")
    for W, bias in _views(x, case):
        W.copy_(torch.randn(W.shape, generator=gen, device="cuda") * (2.0 / W.shape[1]) ** 0.5)
        if bias is not None:
            bias.copy_(torch.randn(bias.shape, generator=gen, device="cuda") * 0.01)
    G = _rows(m, d, case.get("align", 1))
    faulty = sorted(order[:b])
    for i in range(m):
        if i in faulty:
            continue
        features, labels, targets = _batch(case, 32, gen)
        p = x.clone().requires_grad_(True)
        _loss(case, _logits(p, case, features), labels, targets).backward()
        G[i] = p.grad
    _faults(G, faulty, gen)
    features, labels, targets = _batch(case, case["n_r"], gen)
    return {"x": x, "G": G, "features": features, "labels": labels, "targets": targets}


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    m, d, dev = case["m"], s["G"].shape[1], s["G"].device
    if case["kind"] in ("baselines", "median"):
        s["median"] = torch.empty(d, device=dev)
        if case["kind"] == "baselines":
            s["mean"], s["krum"] = torch.empty(d, device=dev), torch.empty(d, device=dev)
            n = int(B.load_library().zeno_krum_workspace_bytes(m))
            s["workspace"] = torch.empty(n, dtype=torch.uint8, device=dev)
        return s
    if case["kind"] == "mlp":
        s["model"] = B.ZenoModel(_dims(case), case["bias"], case["loss"], case["fwd"])
    else:
        s["model"] = B.ZenoCnnModel(dict(in_h=case["hw"], in_w=case["hw"], in_c=case["c_in"],
                                         conv_c=[c for c, _ in _convs(case)], conv_stride=[t for _, t in _convs(case)],
                                         fc_out=case["out"], has_bias=True))
    if not case.get("static"):
        s["workspace"] = B.alloc_workspace(s["model"], m, case["n_r"], dev)
    s["scores"] = torch.empty(m, device=dev)
    s["selected"] = torch.empty(m - case["b"], dtype=torch.int32, device=dev)
    s["out"] = torch.empty(d, device=dev)
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "median":
        return {"median": B.zeno_median(s["G"], out=s["median"])}
    if case["kind"] == "baselines":
        mean = B.zeno_mean(s["G"], out=s["mean"])
        median = B.zeno_median(s["G"], out=s["median"])
        row, chosen, sums = B.zeno_krum(s["G"], case["b"], out=s["krum"], workspace=s["workspace"])
        return {"mean": mean, "median": median, "krum": row, "krum_chosen": chosen, "krum_scores": sums}
    args = (s["model"], s["x"], s["G"], s["features"], case["gamma"], case["rho"])
    batch = {"labels": s["labels"], "targets": s["targets"], "scores": s["scores"]}
    if case.get("static"):
        scores = B.zeno_score_static(*args, **batch)
    else:
        scores = B.zeno_score(*args, workspace=s["workspace"], **batch)
    if case.get("update", True):
        out, _, selected = B.zeno_aggregate_update(s["G"], scores, case["b"], case["gamma"], s["x"], x_next=s["out"],
                                                   want_out=False, selected=s["selected"])
    else:
        out, selected = B.zeno_aggregate(s["G"], scores, case["b"], out=s["out"], selected=s["selected"])
    return {"scores": scores, "selected": selected, "out": out}


def work(case):
    """Every call reads its inputs and writes its outputs once; the selected rows are an input of the second call."""
    m, b = case["m"], case["b"]
    if case["kind"] == "median":
        return {"bytes": 4.0 * case["d"] * (m + 1), "flops": 1.0 * case["d"] * m}
    if case["kind"] == "baselines":
        return {"bytes": 4.0 * case["d"] * (3 * m + 3), "flops": case["d"] * (m * (m + 1.0) + 2.0 * m)}
    d, n_r = _num_params(case), case["n_r"]
    if case["kind"] == "mlp":
        macs = sum(n * k for n, k, _ in _blocks(case))
    else:
        blocks, maps = _blocks(case), _maps(case)
        macs = sum(n * k * h * h for (n, k, _), (h, _) in zip(blocks[:-1], maps[1:])) + blocks[-1][0] * blocks[-1][1]
    width = _dims(case)[0] if case["kind"] == "mlp" else case["hw"] ** 2 * case["c_in"]
    rows = (m + 1) + (m - b) + (2 if case.get("update", True) else 1)
    return {"bytes": 4.0 * d * rows + 4.0 * n_r * width, "flops": 2.0 * (m + 1) * n_r * macs}


def tolerance(case):
    # four times what the same sums in another order, or other rounding of a 16-bit operand's last bit, were seen to give
    if case["kind"] == "median":
        return "exact"
    if case["kind"] == "baselines" or case["kind"] == "cnn" or case["fwd"] == "fp32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 1e-1, "differ": 0.01}


# ---- float64 values

def _mean(G, rows):
    total = torch.zeros(G.shape[1], dtype=torch.float64, device=G.device)
    for i in rows:
        total += G[i]
    return total / len(rows)


def _median(G):
    m, d = G.shape
    out = torch.empty(d, dtype=torch.float64, device=G.device)
    for lo in range(0, d, 1 << 18):
        v = G[:, lo:lo + (1 << 18)].t().contiguous().sort(dim=1).values.double()
        out[lo:lo + (1 << 18)] = 0.5 * (v[:, (m - 1) // 2] + v[:, m // 2])
    return out


def _krum(G, b):
    m, d = G.shape
    gram = torch.zeros((m, m), dtype=torch.float64, device=G.device)
    for lo in range(0, d, 1 << 18):
        g = G[:, lo:lo + (1 << 18)].double()
        gram += g @ g.t()
    sq = gram.diagonal()
    dist = (sq[:, None] + sq[None, :] - 2.0 * gram).clamp_min(0.0)
    dist.fill_diagonal_(math.inf)
    sums = dist.sort(dim=1).values[:, :m - b - 2].sum(1)
    best = int(sums.argmin())
    return G[best].double(), torch.tensor([best], dtype=torch.int32, device=G.device), sums


def exact(case, seed):
    s = _inputs(case, seed)
    G, m, b = s["G"], case["m"], case["b"]
    if case["kind"] == "median":
        return {"median": _median(G)}
    if case["kind"] == "baselines":
        row, chosen, sums = _krum(G, b)
        return {"mean": _mean(G, range(m)), "median": _median(G), "krum": row, "krum_chosen": chosen, "krum_scores": sums}
    gamma, rho = float(np.float32(case["gamma"])), float(np.float32(case["rho"]))
    x = s["x"].double()

    def f(p):
        return _loss(case, _logits(p, case, s["features"]), s["labels"], s["targets"])

    at_x = f(x)
    scores = torch.stack([at_x - f(x - gamma * G[i].double()) - rho * G[i].double().square().sum() for i in range(m)])
    order = torch.argsort(scores, descending=True, stable=True)
    selected = order[:m - b].sort().values
    out = _mean(G, selected.tolist())
    return {"scores": scores, "selected": selected.to(torch.int32), "out": x - gamma * out if case.get("update", True) else out}
