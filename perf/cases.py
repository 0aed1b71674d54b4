"""The calls whose speed matters to a user of this framework, at the sizes of
its workloads (``synth/workloads.py``) and over the ranges around them:

* the fused Non-blocking step on replicas resident in HBM: launch-bound,
  ordinary and large, on padded and on contiguous rows, with even, odd and
  ragged parameter counts, with each mixing kind and order, and its
  parameter-server form;
* the same update from its three unfused calls;
* the per-mini-batch gradients of the MLP workload (forward and backward) and
  its evaluation (forward only), small and full size;
* one whole training iteration of the MLP workload, host work included.

Every case fixes its straggler schedule (seed 0 at the case's ``iteration``),
so the finished mini-batches, and with them the work, follow from the case;
tensors follow from the seed handed to ``prepare``.
"""

from __future__ import annotations

import dataclasses
import functools
import math

import numpy as np
import torch

from paper_2211_00889_amd import _lib, runner
from synth import workloads

DEV = "cuda:0"
G_STD = math.sqrt(1e-3)  # of the synthetic gradients
KINDS = {"exp": _lib.DELAY_EXP, "lomax": _lib.DELAY_LOMAX, "const": _lib.DELAY_CONST}
ORDERS = {"mix_then_step": _lib.MIX_THEN_STEP, "step_then_mix": _lib.STEP_THEN_MIX}
BATCH = 32


def _step(name, n, m, P, mixing, order, delay, param, slow=1.0, layout="padded", kind="step"):
    return {"name": name, "kind": kind, "n": n, "m": m, "P": P, "mixing": mixing, "order": order,
            "delay": delay, "param": param, "slow": slow, "layout": layout, "iteration": 0}


def _mlp(name, kind, n, m, d_in, hidden, classes, n_samples, entry="strided"):
    return {"name": name, "kind": kind, "n": n, "m": m, "d_in": d_in, "hidden": hidden,
            "classes": classes, "n_samples": n_samples, "entry": entry, "delay": "exp", "param": 1.0,
            "slow": 1.0, "iteration": 0}


def listed():
    return [
        # four learners of a 10,000-parameter model: everything fits a cache,
        # the time is the call and the launch
        _step("step_tiny", 4, 4, 10_000, "uniform", "step_then_mix", "exp", 1.0,
              layout="contiguous"),
        # a small model of odd size as a program allocates it, [n, P]
        _step("step_small_odd", 8, 8, 262_143, "ring", "mix_then_step", "exp", 1.0,
              layout="contiguous"),
        # ResNet-18-sized D-PSGD with one slow learner, padded rows
        _step("step_resnet18_ring", 8, 8, 11_200_000, "ring", "mix_then_step", "exp", 1.0, slow=3.0),
        # the same size less an odd remainder on contiguous rows, so no row
        # but the first is aligned to more than a float
        _step("step_odd_contiguous", 8, 8, 11_181_641, "ring", "mix_then_step", "exp", 1.0,
              slow=3.0, layout="contiguous"),
        # ResNet-50-sized, sixteen learners, few mini-batches, MATCHA
        _step("step_resnet50_matcha", 16, 4, 23_500_000, "matcha", "mix_then_step", "exp", 0.5),
        # one eighth of the columns of the VGG-16-sized all-reduce workload
        # (the step splits by columns), heavy-tailed stragglers
        _step("step_vgg16_shard", 8, 16, 17_250_000, "uniform", "step_then_mix", "lomax", 1.5),
        # parameter server (Alg. 3)
        _step("step_server", 8, 8, 11_200_000, "uniform", "step_then_mix", "exp", 1.0, slow=3.0,
              kind="server"),
        # accumulate, mix and update called one by one
        _step("unfused_resnet18", 8, 8, 11_200_000, "ring", "mix_then_step", "exp", 1.0, slow=3.0,
              layout="contiguous", kind="unfused"),
        # gradients of a small network: the calls and launches count
        _mlp("mlp_grad_small", "mlp_grad", 4, 4, 128, 64, 10, 2_560, entry="noalloc"),
        # gradients of every finished mini-batch of the CIFAR-sized workload
        _mlp("mlp_grad_full", "mlp_grad", 8, 8, 3072, 512, 10, 50_000),
        # evaluation of the average replica on 4,096 samples
        _mlp("mlp_eval", "mlp_loss", 1, 128, 3072, 512, 10, 50_000),
        # a whole training iteration: schedule, shuffling, gradients, step
        _mlp("mlp_iteration", "mlp_iteration", 8, 8, 3072, 512, 10, 50_000),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    if rng.random() < 0.6:
        n, m = _log_int(rng, 1, 16), _log_int(rng, 1, 64)
        # no more than the largest listed cases move, also in three passes with every row finished
        P = _log_int(rng, 10_000, min(24_000_000, 2_000_000_000 // (n * (m + 8))))
        mixing = rng.choice(("ring", "uniform") if n % 2 or n < 4 else ("ring", "uniform", "matcha"))
        delay, param = rng.choice((("exp", 1.0), ("exp", 0.5), ("lomax", 1.5)))
        case = _step("", n, m, P, mixing, rng.choice(sorted(ORDERS)), delay, param,
                     rng.choice((1.0, 3.0)), rng.choice(("padded", "contiguous")),
                     rng.choice(("step", "step", "step", "server", "unfused")))
        if case["kind"] == "unfused":
            case["layout"] = "contiguous"
    else:
        d_in, hidden = 128 * _log_int(rng, 1, 24), 64 * _log_int(rng, 1, 8)
        kind = rng.choice(("mlp_grad", "mlp_grad", "mlp_loss"))
        if kind == "mlp_loss":
            n, m = 1, _log_int(rng, 1, 128)
        else:
            n, m = _log_int(rng, 1, 16), _log_int(rng, 1, 16)
        case = _mlp("", kind, n, m, d_in, hidden, rng.randint(2, 16), _log_int(rng, 1_000, 80_000))
    case["iteration"] = rng.randrange(50)
    del case["name"]
    return case


@functools.lru_cache(maxsize=64)
def _schedule(n, m, delay, param, slow, iteration):
    """(mask, counts) of the case's iteration; the last learner is slowed."""
    mask, counts, _, _ = _lib.sample_mask(0, iteration, n, m, KINDS[delay], 1.0, param,
                                          n - 1 if slow != 1.0 else -1, slow)
    return mask, counts


def _mask(case):
    mask, counts = _schedule(case["n"], case["m"], case["delay"], case["param"], case["slow"],
                             case["iteration"])
    return mask.copy(), counts.copy()


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(shape, std, gen):
    t = torch.empty(shape, dtype=torch.float32, device=DEV)
    return t.normal_(0.0, std, generator=gen)


# ----------------------------------------------------------------- step cases
def _w(case):
    n = case["n"]
    if case["mixing"] == "uniform":
        return _lib.w_allreduce(n)
    if case["mixing"] == "ring":
        return _lib.w_ring(n)
    return _lib.Matcha(0, n, 3).w(case["iteration"])[0]


def _prepare_step(case, seed):
    n, m, P = case["n"], case["m"], case["P"]
    ld = _lib.row_stride(P) if case["layout"] == "padded" else P
    g = _gen(seed)
    mask, counts = _mask(case)
    s = {"case": case, "P": P, "mask": mask, "counts": counts, "W": _w(case),
         "lr": 0.1, "mu": 0.9, "order": ORDERS[case["order"]]}
    # replicas, momentum in mid-training, and each mini-batch's gradient
    s["X"] = _normal((ld,) if case["kind"] == "server" else (n, ld), 1.0, g)
    s["V"] = _normal((n, ld), G_STD, g)
    s["G"] = _normal((n, m, ld), G_STD, g)
    if case["kind"] == "unfused":
        s["Gbar"] = torch.zeros((n, P), dtype=torch.float32, device=DEV)
        s["Y"] = torch.zeros((n, P), dtype=torch.float32, device=DEV)
    return s


def _run_step(s):
    case, P, X, V, G = s["case"], s["P"], s["X"], s["V"], s["G"]
    if case["kind"] == "server":
        _lib.step_server(X, V, G, P, s["mask"], s["lr"], s["mu"])
        return {"x": X[:P], "V": V[:, :P]}
    if case["kind"] == "unfused":
        _lib.accumulate(G, s["mask"], s["Gbar"])
        if s["order"] == _lib.MIX_THEN_STEP:
            _lib.mix(X, s["W"], s["Y"])
            _lib.update(s["Y"], V, s["Gbar"], s["counts"], case["m"], s["lr"], s["mu"])
        else:
            _lib.update(X, V, s["Gbar"], s["counts"], case["m"], s["lr"], s["mu"])
            _lib.mix(X, s["W"], s["Y"])
        return {"X": s["Y"], "V": V, "Gbar": s["Gbar"]}
    if case["layout"] == "contiguous":
        _lib.step(X, V, G, s["mask"], s["W"], s["lr"], s["mu"], s["order"])
    else:
        _lib.step_strided(X, V, G, P, s["mask"], s["W"], s["lr"], s["mu"], s["order"])
    return {"X": X[:, :P], "V": V[:, :P]}


def _exact_step(case, seed):
    s = _prepare_step(case, seed)
    n, m, P = case["n"], case["m"], case["P"]
    mask, mu, lr = s["mask"], float(np.float32(s["mu"])), float(np.float32(s["lr"]))
    V = s["V"][:, :P].double()
    means = []
    for i in range(n):
        done = [j for j in range(m) if mask[i, j]]
        g = torch.zeros(P, dtype=torch.float64, device=DEV)
        for j in done:
            g += s["G"][i, j, :P]
        g /= len(done)
        V[i] *= mu
        V[i] += g
        if case["kind"] == "unfused":
            means.append(g)
    eta = [lr * float(mask[i].sum()) / m for i in range(n)]
    if case["kind"] == "server":
        x = s["X"][:P].double()
        for i in range(n):
            x -= V[i] * (eta[i] / n)
        return {"x": x, "V": V}
    W = torch.from_numpy(s["W"].astype(np.float64)).to(DEV)
    Z = s["X"][:, :P].double()
    if s["order"] == _lib.STEP_THEN_MIX:
        for i in range(n):
            Z[i] -= eta[i] * V[i]
    X = torch.zeros_like(Z)
    for i in range(n):
        for p in range(n):
            if s["W"][i, p] != 0:
                X[i] += W[i, p] * Z[p]
    if s["order"] == _lib.MIX_THEN_STEP:
        for i in range(n):
            X[i] -= eta[i] * V[i]
    out = {"X": X, "V": V}
    if case["kind"] == "unfused":
        out["Gbar"] = torch.stack(means)
    return out


def _work_step(case):
    n, P = case["n"], case["P"]
    total = int(_mask(case)[1].sum())
    adds = total + 4 * n + (0 if case["kind"] == "server" else 3 * n)
    if case["kind"] == "server":
        rows = total + 2 * n + 2
    elif case["kind"] == "unfused":  # three passes: G -> Gbar, X -> Y, (Y, V, Gbar) -> (Y, V)
        rows = total + 8 * n
    else:
        rows = total + 4 * n
    return {"bytes": 4.0 * P * rows, "flops": 1.0 * P * adds}


# ------------------------------------------------------------------ MLP cases
def _dims(case):
    return case["d_in"], case["hidden"], case["classes"]


def _samples(case, g):
    """Standardised samples and the labels a random linear teacher gives."""
    data = _normal((case["n_samples"], case["d_in"]), 1.0, g)
    teacher = _normal((case["d_in"], case["classes"]), 1.0, g)
    return data, (data @ teacher).argmax(1).to(torch.int32)


def _params(case, g, rows):
    """Replicas around a common network: U(+-1/sqrt(fan_in)) weights and biases."""
    d, h, c = _dims(case)
    out = torch.zeros((rows, _lib.mlp_param_count(d, h, c)), dtype=torch.float32, device=DEV)
    off = 0
    for size, fan in ((d * h, d), (h, d), (h * c, h), (c, h)):
        base = torch.empty(size, dtype=torch.float32, device=DEV)
        base.uniform_(-1.0, 1.0, generator=g)
        out[:, off:off + size] = (base + _normal((rows, size), 0.1, g)) / math.sqrt(fan)
        off += size
    return out


def _prepare_mlp(case, seed):
    g = _gen(seed)
    n, m, dims = case["n"], case["m"], _dims(case)
    if case["kind"] == "mlp_iteration":
        wl = dataclasses.replace(workloads.MLP, n=n, m=m, d_in=dims[0], hidden=dims[1],
                                 classes=dims[2], n_samples=case["n_samples"])
        data, labels = _samples(case, g)
        x0 = _params(case, g, 1)[0, :wl.P]
        r = runner.MlpRunner(wl, DEV, data.cpu().numpy(), labels.cpu().numpy(), x0.cpu().numpy())
        return {"case": case, "runner": r, "k": 0}
    data, labels = _samples(case, g)
    P = _lib.mlp_param_count(*dims)
    idx = torch.randint(0, case["n_samples"], (n, m, BATCH), generator=g, device=DEV,
                        dtype=torch.int32).cpu().numpy()
    s = {"case": case, "dims": dims, "data": data, "labels": labels, "idx": idx, "P": P}
    ws = _lib.mlp_workspace_bytes(*dims, n * m * BATCH)
    s["workspace"] = torch.empty((ws + 15) // 16 * 4, dtype=torch.float32, device=DEV)
    if case["kind"] == "mlp_loss":
        s["params"] = _params(case, g, 1)[0].contiguous()
        s["losses"] = torch.zeros(m, dtype=torch.float32, device=DEV)
        return s
    ld = _lib.row_stride(P)
    s["X"] = torch.zeros((n, ld), dtype=torch.float32, device=DEV)
    s["X"][:, :P] = _params(case, g, n)
    s["G"] = torch.zeros((n, m, ld), dtype=torch.float32, device=DEV)
    s["losses"] = torch.zeros(n * m, dtype=torch.float32, device=DEV)
    s["mask"] = _mask(case)[0]
    return s


def _run_mlp(s):
    case = s["case"]
    if case["kind"] == "mlp_iteration":
        r = s["runner"]
        r.step(s["k"])
        s["k"] += 1
        return {"X": r.X, "V": r.V, "G": r.G, "losses": r.losses}
    if case["kind"] == "mlp_loss":
        _lib.mlp_loss(s["params"], s["dims"], s["data"], s["labels"], s["idx"], s["losses"],
                      s["workspace"])
        return {"losses": s["losses"]}
    if case["entry"] == "noalloc":
        _lib.mlp_grad_noalloc(s["X"], case["m"], s["dims"], s["data"], s["labels"], s["idx"],
                              s["mask"], s["G"], s["losses"])
    else:
        _lib.mlp_grad_strided(s["X"], case["m"], s["dims"], s["data"], s["labels"], s["idx"],
                              s["mask"], s["G"], s["losses"], s["workspace"])
    return {"G": s["G"][:, :, :s["P"]], "losses": s["losses"]}


def _exact_grad(prm, dims, A, y):
    """(gradient, mean loss) of one mini-batch in 64 bits, nothing rounded."""
    d, h, c = dims
    A = A.double()
    W1, b1 = prm[:d * h].view(d, h), prm[d * h:d * h + h]
    o = d * h + h
    W2, b2 = prm[o:o + h * c].view(h, c), prm[o + h * c:o + h * c + c]
    z1 = A @ W1 + b1
    hid = z1.clamp_min(0)
    logits = hid @ W2 + b2
    loss = torch.nn.functional.cross_entropy(logits, y.long())
    dz2 = (torch.softmax(logits, 1) - torch.nn.functional.one_hot(y.long(), c)) / A.shape[0]
    dz1 = (dz2 @ W2.T) * (z1 > 0)
    g = torch.cat([(A.T @ dz1).reshape(-1), dz1.sum(0), (hid.T @ dz2).reshape(-1), dz2.sum(0)])
    return g, loss


def _exact_mlp(case, seed):
    s = _prepare_mlp(case, seed)
    n, m, dims = case["n"], case["m"], _dims(case)
    it = case["kind"] == "mlp_iteration"
    if it:
        r = s["runner"]
        wl = r.wl
        mask = r.schedule.mask(0)[0]
        idx = _lib.minibatch_indices(wl.seed, 0, n, m, BATCH, wl.shard)
        data, labels, P, X = r.data, r.labels, r.P, r.X
    else:
        idx, data, labels, P = s["idx"], s["data"], s["labels"], s["P"]
    idx = torch.from_numpy(idx).to(DEV).long()
    losses = torch.zeros(n * m, dtype=torch.float64, device=DEV)
    if case["kind"] == "mlp_loss":
        prm = s["params"].double()
        for k in range(m):
            losses[k] = _exact_grad(prm, dims, data[idx[0, k]], labels[idx[0, k]])[1]
        return {"losses": losses}
    if not it:
        mask, X = s["mask"], s["X"]
    if 8.0 * n * m * P > 8e9:  # the 64-bit gradients alone
        return None
    G = torch.zeros((n, m, P), dtype=torch.float64, device=DEV)
    for i in range(n):
        prm = X[i].double()
        for j in range(m):
            if mask[i, j]:
                g, losses[i * m + j] = _exact_grad(prm, dims, data[idx[i, j]], labels[idx[i, j]])
                G[i, j, :g.numel()] = g
    if not it:
        return {"G": G, "losses": losses}
    W = torch.from_numpy(_lib.w_ring(n).astype(np.float64)).to(DEV)
    V = torch.stack([G[i].sum(0) / float(mask[i].sum()) for i in range(n)])  # from zero momentum
    eta = torch.tensor([float(np.float32(wl.lr)) * float(mask[i].sum()) / m for i in range(n)],
                       dtype=torch.float64, device=DEV)
    Xn = W @ X.double() - eta[:, None] * V
    return {"X": Xn, "V": V, "G": G, "losses": losses}


def _work_mlp(case):
    n, (d, h, c) = case["n"], _dims(case)
    P = d * h + h + h * c + c
    if case["kind"] == "mlp_loss":
        mbs, backward = case["m"], 0
    else:
        mbs, backward = int(_mask(case)[1].sum()), 1
    samples = mbs * BATCH
    # parameters and samples read once, each finished gradient written once
    rows = n + backward * mbs
    if case["kind"] == "mlp_iteration":  # and read by the step, with X and V
        rows += mbs + 4 * n - n
    flops = 2.0 * samples * (d * h + h * c) + backward * 2.0 * samples * (d * h + 2 * h * c)
    return {"bytes": 4.0 * (rows * P + samples * d), "flops": flops}


# ------------------------------------------------------------------ interface
def _is_mlp(case):
    return case["kind"].startswith("mlp")


def prepare(case, seed):
    return (_prepare_mlp if _is_mlp(case) else _prepare_step)(case, seed)


def run(state):
    return (_run_mlp if _is_mlp(state["case"]) else _run_step)(state)


def work(case):
    return (_work_mlp if _is_mlp(case) else _work_step)(case)


def exact(case, seed):
    return (_exact_mlp if _is_mlp(case) else _exact_step)(case, seed)


def tolerance(case):
    if not _is_mlp(case):
        # fp32 sums of up to 64 gradients and 16 replicas in another order:
        # about 1e-7 (measured against 64 bits: 2e-8 to 8e-8)
        return {"rel": 4e-7, "max": 5e-6}
    if case["kind"] == "mlp_loss":
        # bf16 products summed in fp32 in another order: measured 5e-7 over
        # 128 losses, 4e-6 for a single one
        return {"rel": 1.5e-5, "max": 3e-5}
    # The same, but a pre-activation within a rounding of zero may pass the
    # ReLU on one side only, which moves a column of a gradient by one
    # sample's share: measured 4e-5 without and 1.8e-3 with one such unit
    # (largest entry 0.98 of the rms) on the full shape.
    return {"rel": 8e-3, "max": 0.99}
