"""The work users of this framework have it do, as cases that can be timed and compared.

Five kinds, each a dict of plain values:

  rnn_train     one training iteration of the tanh RNN on the bit-stream task (RnnTrainer.step: forward,
                head, backward as a scan, parameter gradients, Adam).  H = 20 is the paper's model, other H
                take the general kernels.  `materialise`: the Jacobians are stored (general H needs that) or
                generated inside the scan.
  rnn_backward  the backward pass as its three calls (build_jacobians, scan, param_grads) for a program
                that does its own forward pass and wants the Jacobians.
  gru_step      forward, head and backward of the GRU classifier; `fused` generates the Jacobians inside
                the scan (H = 128 only); `g0` asks for the gradient of the initial state as well, as a
                program does that learns it or cuts its sequences into windows.
  cnn_step      one retraining iteration's backward pass of a pruned VGG-style network on one image: all
                Jacobians as CSR from the weights, masks and activations, the plan (the pooling
                pattern is another one for every image), the sparse scan.
  cnn_run       the sparse scan alone on a plan that is kept, with `up_levels` levels of CSR products:
                what is repeated when a pattern is studied or reused.

Everything is fp32 with int32 indices: the library has no other type.  Sizes are those of this repository's
configurations, tests and benchmark sweeps; initial weights and inputs follow the same recipes.
"""
from __future__ import annotations

import math

import torch

import paper_1907_10134_amd as bp

DEV = "cuda"
VGG_CHANNELS = (64, 128, 256, 256, 512, 512, 512, 512)
VGG_POOL_AFTER = (1, 2, 4, 6, 8)


def listed():
    return [
        # The shortest sequence of the paper's sweep: seven small launches, nothing else to hide behind.
        {"name": "rnn_train_T10_B16", "kind": "rnn_train", "T": 10, "B": 16, "H": 20, "materialise": False},
        # The paper's ordinary point: T = 1000, B = 16.
        {"name": "rnn_train_T1000_B16", "kind": "rnn_train", "T": 1000, "B": 16, "H": 20, "materialise": False},
        # The widest batch of its batch sweep.
        {"name": "rnn_train_T1000_B256", "kind": "rnn_train", "T": 1000, "B": 256, "H": 20, "materialise": False},
        # A long sequence, ragged on every axis: no multiple of a unit, a batch that no die count divides.
        {"name": "rnn_train_T9999_B13", "kind": "rnn_train", "T": 9999, "B": 13, "H": 20, "materialise": False},
        # The headline step of bench.py: the three calls at T = 1000, B = 16.
        {"name": "rnn_backward_T1000_B16", "kind": "rnn_backward", "T": 1000, "B": 16, "H": 20},
        # The longest sequence of the sweep: 768 MB of Jacobians written and read.
        {"name": "rnn_backward_T30000_B16", "kind": "rnn_backward", "T": 30000, "B": 16, "H": 20},
        # A hidden size the library has no kernel of its own for, on a ragged batch.
        {"name": "rnn_train_H64_T300_B7", "kind": "rnn_train", "T": 300, "B": 7, "H": 64, "materialise": True},
        # The paper's GRU: 20 hidden units on the middle MFCC set (517 frames of 24 features), B = 32.
        {"name": "gru_H20_T517_B32", "kind": "gru_step", "T": 517, "B": 32, "H": 20, "I": 24, "fused": False, "g0": False},
        # The large GRU of the configurations: 4.3 GB of dense Jacobians.
        {"name": "gru_H128_T4096_B16", "kind": "gru_step", "T": 4096, "B": 16, "H": 128, "I": 1, "fused": False,
         "g0": False},
        # The same cell as a user with the long MFCC set and a small odd batch runs it: nothing stored.
        {"name": "gru_H128_T1034_B5_fused", "kind": "gru_step", "T": 1034, "B": 5, "H": 128, "I": 12, "fused": True,
         "g0": True},
        # The pruned VGG-11-style network of the configurations, a whole iteration.
        {"name": "cnn_step_vgg11", "kind": "cnn_step", "image": 32, "width": 64, "convs": 8, "keep": 0.1, "up_levels": 0},
        # The same network with two levels of CSR products on a plan in hand.
        {"name": "cnn_run_vgg11_up2", "kind": "cnn_run", "image": 32, "width": 64, "convs": 8, "keep": 0.1,
         "up_levels": 2},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("rnn_train", "rnn_train", "rnn_backward", "rnn_general", "gru_small", "gru_128", "cnn_step", "cnn_run"))
    if kind in ("rnn_train", "rnn_backward"):
        # the sweeps of the paper: T from 10 to 30000, B from 2 to 256, as much as T = 30000, B = 16 in all
        T = _log_int(rng, 10, 30000)
        B = _log_int(rng, 2, max(2, min(256, 480000 // T)))
        case = {"kind": kind, "T": T, "B": B, "H": 20}
        if kind == "rnn_train":
            case["materialise"] = rng.random() < 0.25
        return case
    if kind == "rnn_general":
        H = rng.choice((5, 8, 16, 24, 32, 33, 48, 64, 80, 96, 100))
        T = _log_int(rng, 30, 1000)
        return {"kind": "rnn_train", "T": T, "B": _log_int(rng, 1, max(1, min(64, 16384 // T))), "H": H, "materialise": True}
    if kind == "gru_small":
        return {"kind": "gru_step", "T": _log_int(rng, 50, 1034), "B": _log_int(rng, 2, 64),
                "H": rng.choice((20, 20, 20, 8, 16, 32, 33, 64)), "I": rng.choice((1, 2, 12, 24, 38)), "fused": False,
                "g0": rng.random() < 0.3}
    if kind == "gru_128":
        T = _log_int(rng, 60, 4096)
        I = rng.choice((1, 2, 3, 8, 12)) if T <= 1034 else rng.choice((1, 2, 3, 8))
        return {"kind": "gru_step", "T": T, "B": _log_int(rng, 1, max(1, min(64, 65536 // T))), "H": 128, "I": I,
                "fused": rng.random() < 0.5, "g0": rng.random() < 0.3}
    image = rng.choice((8, 12, 16, 20, 24, 28, 32))
    return {"kind": kind, "image": image, "width": rng.choice((8, 12, 16, 24, 32, 48, 64)), "convs": rng.randint(3, 8),
            "keep": round(rng.uniform(0.03, 0.1), 3), "up_levels": rng.choice((0, 0, 1) if kind == "cnn_step" else (0, 1, 2))}


# ---- inputs --------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, shape, bound):
    return (torch.rand(shape, generator=g, device=DEV) * 2.0 - 1.0) * bound


def _empty(*shape):
    return torch.empty(shape, dtype=torch.float32, device=DEV)


def _bitstream(g, T, B):
    """Section 4.1's task: a class per sample, and a stream of Bernoulli(0.05 + 0.1 c) bits."""
    labels = torch.randint(0, 10, (B,), generator=g, device=DEV, dtype=torch.int32)
    x = torch.rand((T, B), generator=g, device=DEV) < (0.05 + 0.1 * labels.float())
    return x.float().reshape(T, B, 1).contiguous(), labels


def _prepare_rnn_train(case, g):
    T, B, H = case["T"], case["B"], case["H"]
    k = 1.0 / math.sqrt(H)
    shapes = {"w_ih": (H, 1), "w_hh": (H, H), "b_ih": (H,), "b_hh": (H,), "w_out": (10, H), "b_out": (10,)}
    params = {name: _uniform(g, shapes[name], k) for name in bp.RNN_PARAM_ORDER}
    x, labels = _bitstream(g, T, B)
    trainer = bp.RnnTrainer(T, B, H, 1, 10, params, materialise=case["materialise"])
    return {"kind": "rnn_train", "trainer": trainer, "x": x, "labels": labels}


def _prepare_rnn_backward(case, g):
    T, B, H = case["T"], case["B"], case["H"]
    k = 1.0 / math.sqrt(H)
    x = torch.randn((T, B, 1), generator=g, device=DEV)
    w_ih, w_hh, b = _uniform(g, (H, 1), k), _uniform(g, (H, H), k), _uniform(g, (H,), k)
    h = torch.zeros((T + 1, B, H), device=DEV)
    bp.forward(bp.RNN_TANH, x, w_ih, w_hh, b, None, h)
    labels = torch.randint(0, 10, (B,), generator=g, device=DEV, dtype=torch.int32)
    seed, _ = bp.head_seed(h[T], _uniform(g, (10, H), k), _uniform(g, (10,), k), labels)
    pg_ws = torch.empty(bp.param_grads_workspace_bytes(bp.RNN_TANH, T, B, H, 1), dtype=torch.uint8, device=DEV)
    return {"kind": "rnn_backward", "h": h, "x": x, "w_hh": w_hh, "seed": seed, "Jt": _empty(T, B, H, H),
            "G": _empty(T, B, H), "grads": (_empty(H, 1), _empty(H, H), _empty(H), _empty(H)),
            "scan_ws": torch.empty(bp.scan_workspace_bytes(T, B, H), dtype=torch.uint8, device=DEV), "pg_ws": pg_ws}


def _prepare_gru(case, g):
    T, B, H, I = case["T"], case["B"], case["H"], case["I"]
    k = 1.0 / math.sqrt(H)
    # an audio-like stream: three sinusoids per sample and feature, and noise
    t = torch.arange(T, device=DEV, dtype=torch.float32).reshape(T, 1, 1)
    x = 0.1 * torch.randn((T, B, I), generator=g, device=DEV)
    for _ in range(3):
        f = 0.5 * torch.rand((1, B, I), generator=g, device=DEV)
        x += torch.sin(2.0 * math.pi * (torch.frac(f * t) + torch.rand((1, B, I), generator=g, device=DEV)))
    st = {"kind": "gru_step", "fused": case["fused"], "x": x.contiguous(),
          "w": (_uniform(g, (3 * H, I), k), _uniform(g, (3 * H, H), k), _uniform(g, (3 * H,), k), _uniform(g, (3 * H,), k)),
          "w_out": _uniform(g, (11, H), k), "b_out": _uniform(g, (11,), k),
          "labels": torch.randint(0, 11, (B,), generator=g, device=DEV, dtype=torch.int32),
          "h": torch.zeros((T + 1, B, H), device=DEV), "G": _empty(T, B, H),
          "head": (_empty(B, H), _empty(1), _empty(11, H), _empty(11)),
          "grads": (_empty(3 * H, I), _empty(3 * H, H), _empty(3 * H), _empty(3 * H)),
          "g0": _empty(B, H) if case["g0"] else None, "Jt": None if case["fused"] else _empty(T, B, H, H)}
    scan_bytes = bp.gru_scan_fused_workspace_bytes(T, B, H) if case["fused"] else bp.scan_workspace_bytes(T, B, H)
    st["scan_ws"] = torch.empty(max(scan_bytes, 256), dtype=torch.uint8, device=DEV)
    st["pg_ws"] = torch.empty(bp.param_grads_workspace_bytes(bp.GRU, T, B, H, I), dtype=torch.uint8, device=DEV)
    return st


def _network(case):
    """(kind, channels in, channels out, image size) per layer: the VGG-11-style list of the pruned
    configuration, cut to `convs` convolutions, `width` channels in the first and a pool wherever the
    image can still be halved."""
    layers, c, n = [], 3, case["image"]
    for i in range(case["convs"]):
        co = VGG_CHANNELS[i] * case["width"] // 64
        layers += [("conv", c, co, n), ("relu", co, co, n)]
        c = co
        if i + 1 in VGG_POOL_AFTER and n % 2 == 0:
            layers.append(("pool", c, c, n))
            n //= 2
    d, hidden = c * n * n, 8 * case["width"]
    for j, out in enumerate((hidden, hidden, 10)):
        layers.append(("fc", d, out, 1))
        if j < 2:
            layers.append(("relu", out, out, 1))
        d = out
    return layers


def _pruned(g, pattern, shape, fan_in, keep):
    """He-normal weights, all but the `keep` fraction of largest magnitude masked out; with a pattern
    generator of their own, those weights after some retraining steps that kept the mask."""
    w = math.sqrt(2.0 / fan_in) * torch.randn(shape, generator=pattern or g, device=DEV)
    if pattern:
        drift = 1.0 + 0.1 * torch.randn(shape, generator=g, device=DEV)
    kept = torch.topk(w.abs().reshape(-1), max(1, math.ceil(keep * w.numel()))).indices
    mask = torch.zeros(w.numel(), dtype=torch.uint8, device=DEV)
    mask[kept] = 1
    mask = mask.reshape(shape)
    return (w * drift if pattern else w) * mask, mask


def _layer_inputs(case, g):
    """What the backward pass needs of every layer, last layer first (scan order).  A scan on a kept plan
    meets one pattern (masks and pooling winners) with ever new values."""
    pattern = _gen(5) if case["kind"] == "cnn_run" else None
    out = []
    for kind, ci, co, n in _network(case):
        if kind == "conv":
            out.append((kind, *_pruned(g, pattern, (co, ci, 3, 3), 9 * ci, case["keep"]), n))
        elif kind == "fc":
            out.append((kind, *_pruned(g, pattern, (co, ci), ci, case["keep"]), n))
        elif kind == "relu":
            out.append((kind, torch.randn(ci * n * n, generator=g, device=DEV), None, n))
        else:                       # pooling sees what a ReLU let through: about half zeros, ties among them
            out.append((kind, torch.relu(torch.randn((ci, n, n), generator=pattern or g, device=DEV)), None, n))
    return out[::-1]


def _jacobians(layer_inputs):
    jts = []
    for kind, a, mask, n in layer_inputs:
        if kind == "conv":
            jts.append(bp.csr_conv3x3(a, mask, n, n))
        elif kind == "fc":
            jts.append(bp.csr_linear(a, mask))
        elif kind == "relu":
            jts.append(bp.csr_relu(a))
        else:
            jts.append(bp.csr_maxpool2x2(a))
    return jts


def _prepare_cnn(case, g):
    layer_inputs = _layer_inputs(case, g)
    rows = [ci * n * n for _, ci, _, n in _network(case)][::-1]
    st = {"kind": case["kind"], "layers": layer_inputs, "up_levels": case["up_levels"],
          "seed": torch.randn(10, generator=g, device=DEV), "grads": [_empty(r) for r in rows],
          "arena": torch.empty((1 << 30) if case["up_levels"] else (64 << 20), dtype=torch.uint8, device=DEV)}
    if case["kind"] == "cnn_run":
        st["jts"] = _jacobians(layer_inputs)
        st["plan"] = bp.SpscanPlan(st["jts"], case["up_levels"], st["arena"])
        st["products"] = [st["plan"].product(i)[0].data for i in range(st["plan"].num_products())]
    return st


def prepare(case, seed):
    g = _gen(seed)
    if case["kind"] == "rnn_train":
        return _prepare_rnn_train(case, g)
    if case["kind"] == "rnn_backward":
        return _prepare_rnn_backward(case, g)
    if case["kind"] == "gru_step":
        return _prepare_gru(case, g)
    return _prepare_cnn(case, g)


# ---- one pass ------------------------------------------------------------------------------------

def _run_rnn_train(st):
    tr = st["trainer"]
    loss = tr.step(st["x"], st["labels"])
    return {"loss": loss, "params": tr.params, "grads": tr.grads, "adam_m": tr.adam_m, "adam_v": tr.adam_v, "h": tr.h,
            "G": tr.G, "seed": tr.seed}


def _run_rnn_backward(st):
    bp.build_jacobians(bp.RNN_TANH, st["h"], w_hh=st["w_hh"], Jt=st["Jt"])
    bp.scan(st["Jt"], st["seed"], st["G"], workspace=st["scan_ws"])
    bp.param_grads(bp.RNN_TANH, st["h"], st["x"], st["G"], out=st["grads"], workspace=st["pg_ws"])
    return {"Jt": st["Jt"], "G": st["G"], "grads": st["grads"]}


def _run_gru(st):
    h, x, w, G, g0 = st["h"], st["x"], st["w"], st["G"], st["g0"]
    bp.forward(bp.GRU, x, *w, h)
    seed = st["head"][0]
    bp.head_backward(h[-1], st["w_out"], st["b_out"], st["labels"], *st["head"])
    if st["fused"]:
        bp.gru_scan_fused(h, x, *w, seed, G, g0=g0, workspace=st["scan_ws"])
    else:
        bp.build_jacobians(bp.GRU, h, x, *w, Jt=st["Jt"])
        bp.scan(st["Jt"], seed, G, g0=g0, workspace=st["scan_ws"])
    bp.param_grads(bp.GRU, h, x, G, *w, out=st["grads"], workspace=st["pg_ws"])
    return {"h": h, "head": st["head"], "Jt": st["Jt"], "G": G, "g0": g0, "grads": st["grads"]}


def _run_cnn(st):
    if st["kind"] == "cnn_run":
        st["plan"].run(st["jts"], st["seed"], st["grads"])
        return {"grads": st["grads"], "products": st["products"]}
    jts = _jacobians(st["layers"])
    plan = bp.SpscanPlan(jts, st["up_levels"], st["arena"])
    plan.run(jts, st["seed"], st["grads"])
    return {"grads": st["grads"], "indptr": [m.indptr for m in jts]}


def run(state):
    if state["kind"] == "rnn_train":
        return _run_rnn_train(state)
    if state["kind"] == "rnn_backward":
        return _run_rnn_backward(state)
    if state["kind"] == "gru_step":
        return _run_gru(state)
    return _run_cnn(state)


# ---- what a pass cannot do without ---------------------------------------------------------------

def _cnn_work(case):
    nnz = rows = params = acts = 0
    for kind, ci, co, n in _network(case):
        rows += ci * n * n
        if kind == "conv":
            params += 9 * ci * co
            nnz += case["keep"] * ci * co * (3 * n - 2) ** 2
        elif kind == "fc":
            params += ci * co
            nnz += case["keep"] * ci * co
        else:
            acts += ci * n * n
            nnz += ci * n * n if kind == "relu" else ci * n * n / 4
    csr = 8.0 * nnz + 4.0 * rows
    if case["kind"] == "cnn_run":           # every matrix read once, every gradient written once
        return {"bytes": csr + 4.0 * rows, "flops": 2.0 * nnz}
    # weights and masks read, activations read, the matrices written and read, the gradients written
    return {"bytes": 5.0 * params + 4.0 * acts + 2.0 * csr + 4.0 * rows, "flops": 2.0 * nnz}


def work(case):
    if case["kind"] in ("cnn_step", "cnn_run"):
        return _cnn_work(case)
    T, B, H = case["T"], case["B"], case["H"]
    rows, gates = float(T) * B, 1 if case["kind"] != "gru_step" else 3
    I = case.get("I", 1)
    weights = gates * H * (H + I + 2)
    # forward, the gradient chain and the parameter gradients: one product with a weight-sized matrix each
    flops = 2.0 * rows * (2 * gates * H * (H + I) + H * H)
    data = 4.0 * rows * (2 * H + I) + 8.0 * weights        # x read, h and G written; weights and their gradients
    tiles = 8.0 * rows * H * H                              # the Jacobians, written and read
    if case["kind"] == "rnn_backward":
        return {"bytes": 4.0 * rows * (2 * H + I) + 4.0 * weights + tiles, "flops": flops - 2.0 * rows * H * (H + I)}
    if case["kind"] == "rnn_train":
        n = H * (H + 3) + 10 * (H + 1)
        return {"bytes": data + 24.0 * n + (tiles if case["materialise"] else 0.0), "flops": flops}
    return {"bytes": data + (0.0 if case["fused"] else tiles), "flops": flops}


def tolerance(case):
    # fp32 throughout; sums and the bracketing of the products may be reordered
    return {"rel": 2e-5}
