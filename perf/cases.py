"""The work that a user of this library has it do, as cases that can be timed and compared.

`listed()` names the cases, `draw()` gives more of the same ranges, `prepare()` makes what a user's
program holds before the call (weights packed, workspaces allocated, a decode step captured where a
serving loop would capture it), `run()` makes one pass through the public entry points, `work()`
says what a pass cannot do without and `tolerance()` how far two correct implementations may differ.

Kinds of case:
  linear     one linear layer, called eagerly (rosaq_linear / rosaq_linear_headwise)
  attention  the q/k/v batch and the output projection of `layers` attention blocks
  decoder    the seven linears of `layers` decoder layers: q/k/v batch, o, gated MLP block
  mlp        `layers` gated MLP blocks (rosaq_mlp_swiglu)
  pack       the offline step of one layer: rosaq_pack_weights and the canonical arrays it yields
  pca        calibration: rosaq_pca_headwise or rosaq_pca_full

Weights, activations and rotations are synthetic and made from the seed on the GPU; their
distributions are those of paper_2506_13472_amd.synth (log-normal channel scales, weights of 0.02
with one entry in a thousand ten times as large).  Every layer of a stack has its own copy of its
weights, so that a pass streams them from memory as a model of many layers does.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2506_13472_amd import binding as B
from paper_2506_13472_amd import torch_glue as T

GROUP = 128
HEAD = 128


def listed():
    return [
        # The smallest configuration: one 1024 x 1024 layer and a batch of four rows, called eagerly.
        # Launches and the host path count.
        {"name": "linear_1024_m4", "kind": "linear", "d": 1024, "n": 1024, "m": 4, "bits": 4, "k": 128,
         "rotation": "headwise", "absorbed": False, "pad": 0},
        # Ragged sizes with a padded row stride: rows and output channels that fill no tile, three-bit codes,
        # a layer-wise rotation.
        {"name": "linear_ragged_m37", "kind": "linear", "d": 1408, "n": 1003, "m": 37, "bits": 3, "k": 128,
         "rotation": "full", "absorbed": False, "pad": 8},
        # One user's decode step: a single row through 7B-shaped decoder layers, replayed as a graph.
        {"name": "decode_7b_m1", "kind": "decoder", "d": 4096, "f": 11008, "m": 1, "bits": 4, "layers": 4,
         "absorbed": False, "graph": True},
        # A small batch in the deployment where the rotations are folded into the producing layers and
        # the output projection keeps 32 salient channels per head; three-bit codes.
        {"name": "decode_7b_m16_int3", "kind": "decoder", "d": 4096, "f": 11008, "m": 16, "bits": 3, "layers": 4,
         "absorbed": True, "graph": True},
        # The batch of 64 that the benchmark's decode step runs.
        {"name": "decode_7b_m64", "kind": "decoder", "d": 4096, "f": 11008, "m": 64, "bits": 4, "layers": 4,
         "absorbed": False, "graph": True},
        # The benchmark's headline: the head-wise rotated attention projections at batch 64.
        {"name": "attention_7b_m64", "kind": "attention", "d": 4096, "m": 64, "bits": 4, "layers": 8,
         "absorbed": False, "graph": True},
        # A vocabulary-sized projection for a few rows, without rotation: the widest launch.
        {"name": "linear_vocab_m8", "kind": "linear", "d": 4096, "n": 32000, "m": 8, "bits": 4, "k": 128,
         "rotation": "none", "absorbed": False, "pad": 0},
        # A short prefill (or a large decode batch) of a 13B-shaped MLP behind a layer-wise rotation.
        {"name": "mlp_13b_m256", "kind": "mlp", "d": 5120, "f": 13824, "m": 256, "bits": 4, "layers": 2,
         "absorbed": False, "graph": False},
        # A prefill of 2048 tokens through one decoder layer: bound by arithmetic.
        {"name": "prefill_7b_m2048", "kind": "decoder", "d": 4096, "f": 11008, "m": 2048, "bits": 4, "layers": 1,
         "absorbed": False, "graph": False},
        # The offline step of one gate / up projection behind a layer-wise rotation.
        {"name": "pack_7b_gate_int3", "kind": "pack", "d": 4096, "n": 11008, "bits": 3, "k": 128, "rotation": "full"},
        # Calibration of an attention block's input: one PCA per head.
        {"name": "pca_headwise_4096", "kind": "pca", "d": 4096, "rows": 512, "rotation": "headwise"},
        # Layer-wise calibration of a small layer.
        {"name": "pca_full_1024", "kind": "pca", "d": 1024, "rows": 2048, "rotation": "full"},
    ]


def _log_int(rng, lo, hi):
    """A whole number of [lo, hi], spread over the logarithm."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def _fits(case):
    """No dearer than the largest listed case of its kind of work."""
    w = work(case)
    if case["kind"] in ("pack", "pca"):
        most = max(work(c)["flops"] for c in listed() if c["kind"] == case["kind"] and c["rotation"] == "full")
    else:
        most = work([c for c in listed() if c["name"] == "prefill_7b_m2048"][0])["flops"]
    return w["flops"] <= most


def draw(rng):
    while True:
        kind = rng.choice(("linear", "linear", "linear", "attention", "decoder", "decoder", "mlp", "pack", "pca"))
        bits = rng.choice((4, 4, 3))
        d = GROUP * _log_int(rng, 8, 40)
        # half of the draws are decode batches, half go up to prefill sizes
        m = _log_int(rng, 1, 64) if rng.random() < 0.5 else _log_int(rng, 65, 2048)
        if kind == "linear":
            rotation = rng.choice(("headwise", "full", "none"))
            d = GROUP * _log_int(rng, 8, 40 if rotation == "full" else 108)
            case = {"kind": kind, "d": d, "n": _log_int(rng, 512, 32000), "m": m, "bits": bits,
                    "k": rng.choice((0, 128, 128, 256)), "rotation": rotation, "absorbed": rng.random() < 0.25,
                    "pad": rng.choice((0, 8, 64))}
            if rotation == "none":
                case["absorbed"] = False
        elif kind == "attention":
            case = {"kind": kind, "d": d, "m": m, "bits": bits, "layers": rng.randint(2, 8),
                    "absorbed": rng.random() < 0.25, "graph": m <= 64 and rng.random() < 0.7}
        elif kind in ("decoder", "mlp"):
            case = {"kind": kind, "d": d, "f": GROUP * _log_int(rng, 16, 108), "m": m, "bits": bits,
                    "layers": rng.randint(1, 4), "absorbed": rng.random() < 0.4, "graph": m <= 64 and rng.random() < 0.7}
        elif kind == "pack":
            rotation = rng.choice(("headwise", "full", "none"))
            case = {"kind": kind, "d": d, "n": _log_int(rng, 512, 11008), "bits": bits, "k": rng.choice((128, 128, 256)),
                    "rotation": rotation}
        else:
            rotation = rng.choice(("headwise", "full"))
            d = GROUP * _log_int(rng, 8, 40) if rotation == "headwise" else GROUP * rng.randint(2, 8)
            rows = rng.choice((256, 320, 500, 512, 1000)) if rotation == "headwise" else d + rng.choice((256, 333, 1024))
            case = {"kind": kind, "d": d, "rows": rows, "rotation": rotation}
        if _fits(case):
            return case


# ---- inputs -------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _activations(g, rows, d, pad=0):
    sigma = torch.exp(torch.randn(d, generator=g, device="cuda"))
    x = torch.empty((rows, d + pad), dtype=torch.float16, device="cuda")
    x[:, :d] = (torch.randn((rows, d), generator=g, device="cuda") * sigma).to(torch.float16)
    if pad:
        x[:, d:] = 0
    return x[:, :d]


def _weight(g, n, d):
    w = torch.randn((n, d), generator=g, device="cuda") * 0.02
    w = torch.where(torch.rand((n, d), generator=g, device="cuda") < 1e-3, w * 10.0, w)
    return w.to(torch.float16).cpu().numpy()


def _blocks(g, heads):
    """Random orthogonal 128 x 128 blocks, fp32."""
    a = torch.randn((heads, HEAD, HEAD), generator=g, device="cuda").double().cpu()
    q, r = torch.linalg.qr(a)
    return (q * torch.sign(torch.diagonal(r, dim1=1, dim2=2))[:, None, :]).float().numpy()


def _rotation(g, d, rotation):
    """(Q for rosaq_pack_weights, eigenvalues): random orthogonal blocks, or two block-diagonal
    rotations with a stride permutation between them as a dense one; a log-normal spectrum, sorted
    inside each block."""
    heads = d // HEAD
    runs = heads if rotation == "headwise" else 1
    lam = torch.exp(2.0 * torch.randn(d, generator=g, device="cuda").double().cpu()).reshape(runs, -1)
    lam = torch.sort(lam, dim=1, descending=True).values.reshape(-1).numpy()
    if rotation == "none":
        return None, lam
    q = _blocks(g, heads)
    if rotation == "headwise":
        return q, lam
    first = torch.block_diag(*torch.from_numpy(q).cuda())
    second = torch.block_diag(*torch.from_numpy(_blocks(g, heads)).cuda())
    order = torch.arange(d, device="cuda").reshape(heads, HEAD).t().reshape(-1)
    return (first[:, order] @ second).cpu().numpy(), lam


_MODE = {"none": B.Q_NONE, "full": B.Q_FULL, "headwise": B.Q_HEADWISE}


def _pack(g, n, d, bits, k, rotation, rot, absorbed, rule=B.SELECT_TOP):
    q, lam = rot
    return B.rosaq_pack_weights(_weight(g, n, d), q, lam, k, bits, _MODE[rotation], select_rule=rule,
                                rotation_absorbed=absorbed and rotation != "none")


def _stack(base, layers):
    """`layers` copies of a dict of handles, each with device memory of its own."""
    return [base] + [{name: B.rosaq_packed_clone(p) for name, p in base.items()} for _ in range(layers - 1)]


def prepare(case, seed):
    g = _gen(seed)
    kind, d = case["kind"], case["d"]
    if kind == "pca":
        return {"case": case, "x": _activations(g, case["rows"], d)}
    if kind == "pack":
        q, lam = _rotation(g, d, case["rotation"])
        return {"case": case, "w": _weight(g, case["n"], d), "q": q, "lam": lam}
    m, bits, absorbed = case["m"], case["bits"], case["absorbed"]
    if kind == "linear":
        p = _pack(g, case["n"], d, bits, case["k"], case["rotation"], _rotation(g, d, case["rotation"]), absorbed)
        y = torch.empty((m, case["n"] + case["pad"]), dtype=torch.float16, device="cuda")[:, :case["n"]]
        return {"case": case, "p": p, "x": _activations(g, m, d, case["pad"]), "y": y, "ws": T.alloc_workspace(p, m)}

    layers, base = case["layers"], {}
    if kind != "mlp":
        rot = _rotation(g, d, "headwise")
        for name in "qkv":
            base[name] = _pack(g, d, d, bits, 128, "headwise", rot, absorbed)
        # the output projection: one salient set over all heads, or (rotations folded) 32 channels per head;
        # 32 per head is a whole number of groups only where the head count is a multiple of four
        per_head = absorbed and (d // HEAD) % 4 == 0
        base["o"] = _pack(g, d, d, bits, 32 * (d // HEAD) if per_head else 128, "headwise", _rotation(g, d, "headwise"),
                          absorbed, B.SELECT_TOP_PER_HEAD if per_head else B.SELECT_TOP)
    if kind != "attention":
        f = case["f"]
        rot = _rotation(g, d, "full")
        for name in ("gate", "up"):
            base[name] = _pack(g, f, d, bits, 128, "full", rot, absorbed)
        base["down"] = _pack(g, d, f, bits, 128, "none", _rotation(g, f, "none"), False)
    stack = _stack(base, layers)
    state = {"case": case, "stack": stack, "out": {}}
    need = [B.rosaq_workspace_bytes(p, m) for p in base.values()]
    if kind != "mlp":
        need.append(B.rosaq_workspace_bytes_batch([base[n] for n in "qkv"], m))
        state["x"] = [_activations(g, m, d) for _ in range(layers)]
        state["x_o"] = [_activations(g, m, d) for _ in range(layers)]
        qkv = state["out"]["qkv"] = torch.empty((layers, 3, m, d), dtype=torch.float16, device="cuda")
        state["out"]["o"] = torch.empty((layers, m, d), dtype=torch.float16, device="cuda")
        state["batch"] = [B.BatchArgs([lay[n] for n in "qkv"], [qkv[i, j].data_ptr() for j in range(3)], [d] * 3)
                          for i, lay in enumerate(stack)]
    if kind != "attention":
        need.append(B.rosaq_workspace_bytes_mlp(base["gate"], base["up"], base["down"], m))
        state["x_mlp"] = [_activations(g, m, d) for _ in range(layers)]
        state["out"]["mlp"] = torch.empty((layers, m, d), dtype=torch.float16, device="cuda")
    state["ws"] = torch.empty(max(need), dtype=torch.uint8, device="cuda")
    if case["graph"]:
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            _issue(state)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            _issue(state)
        state["graph"] = graph
    return state


# ---- one pass ------------------------------------------------------------------------------------

def _issue(s):
    """The calls of a stack, on the current stream."""
    m, ws, stream = s["case"]["m"], s["ws"], T.current_stream_ptr()
    for i, lay in enumerate(s["stack"]):
        if "batch" in s:
            x = s["x"][i]
            B.rosaq_linear_batch(s["batch"][i], x.data_ptr(), m, x.stride(0), ws.data_ptr(), ws.numel(), stream)
            T.linear(lay["o"], s["x_o"][i], s["out"]["o"][i], ws)
        if "x_mlp" in s:
            x, y = s["x_mlp"][i], s["out"]["mlp"][i]
            B.rosaq_mlp_swiglu(lay["gate"], lay["up"], lay["down"], x.data_ptr(), m, x.stride(0), y.data_ptr(),
                               y.stride(0), ws.data_ptr(), ws.numel(), stream)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "linear":
        return T.linear(state["p"], state["x"], state["y"], state["ws"])
    if kind == "pca":
        x = state["x"]
        pca = B.rosaq_pca_headwise if case["rotation"] == "headwise" else B.rosaq_pca_full
        q, lam = pca(x.data_ptr(), x.shape[0], x.shape[1], x.stride(0), T.current_stream_ptr())
        return {"q": q, "lam": lam}
    if kind == "pack":
        p = B.rosaq_pack_weights(state["w"], state["q"], state["lam"], case["k"], case["bits"], _MODE[case["rotation"]],
                                 stream=T.current_stream_ptr())
        out = B.rosaq_packed_export(p)
        p.free()
        # bit patterns, so that the whole result is held to exact equality
        return {name: a.view(np.int16) if a.dtype == np.float16 else a for name, a in out.items()}
    if "graph" in state:
        state["graph"].replay()
    else:
        _issue(state)
    return state["out"]


# ---- what a pass cannot do without ----------------------------------------------------------------

def _layer(n, d, bits, k):
    """(bytes of the packed weights, flops per row) of one layer."""
    return n * (2 * k + (d - k) * bits // 8 + 4 * (d - k) // GROUP), 2.0 * n * d


def _rot(d, rotation, absorbed):
    """(bytes of fp16(Q), flops per row) of a run-time rotation."""
    if rotation == "none" or absorbed:
        return 0, 0.0
    width = HEAD if rotation == "headwise" else d
    return 2 * d * width, 2.0 * d * width


def work(case):
    kind, d = case["kind"], case["d"]
    if kind == "pca":
        # read X, write Q and the eigenvalues; the second moment and a symmetric eigenproblem per block
        width = HEAD if case["rotation"] == "headwise" else d
        return {"bytes": 2 * case["rows"] * d + 4 * d * width + 8 * d,
                "flops": 1.0 * case["rows"] * d * width + 9.0 * d * width * width}
    if kind == "pack":
        # read W and Q, write the canonical arrays; the rotation of the weight
        n, k = case["n"], case["k"]
        width = {"none": 0, "headwise": HEAD, "full": d}[case["rotation"]]
        return {"bytes": 2 * n * d + 4 * d * width + 2 * n * k + n * (d - k) + 4 * n * ((d - k) // GROUP),
                "flops": 2.0 * n * d * max(width, 1)}
    m, bits, ab = case["m"], case["bits"], case["absorbed"]
    if kind == "linear":
        wb, wf = _layer(case["n"], d, bits, case["k"])
        rb, rf = _rot(d, case["rotation"], ab)
        return {"bytes": wb + rb + 2 * m * (d + case["n"]), "flops": m * (wf + rf)}
    nbytes, flops = 0, 0.0
    if kind != "mlp":
        per_head = ab and (d // HEAD) % 4 == 0
        for k in (128, 128, 128, 32 * (d // HEAD) if per_head else 128):
            wb, wf = _layer(d, d, bits, k)
            nbytes, flops = nbytes + wb + 2 * m * d, flops + m * wf
        rb, rf = _rot(d, "headwise", ab)
        nbytes, flops = nbytes + 2 * rb + 2 * 2 * m * d, flops + 2 * m * rf
    if kind != "attention":
        f = case["f"]
        for n_, d_ in ((f, d), (f, d), (d, f)):
            wb, wf = _layer(n_, d_, bits, 128)
            nbytes, flops = nbytes + wb, flops + m * wf
        rb, rf = _rot(d, "full", ab)
        nbytes, flops = nbytes + rb + 2 * m * (d + d), flops + m * rf
    return {"bytes": nbytes * case["layers"], "flops": flops * case["layers"]}


def tolerance(case):
    # Offline: the packed arrays are defined bit for bit.
    if case["kind"] == "pack":
        return "exact"
    # Calibration works in fp64 and rounds the rotation to fp32 once: 2.5e-8 against LAPACK.
    if case["kind"] == "pca":
        return {"rel": 1e-7}
    # fp16 inputs and outputs, the rotated input rounded to fp16, fp32 sums.  Measured against the same
    # path in fp64: 2.1e-4 to 3.0e-4 for a linear layer, 4.2e-4 for the gated block.
    return {"rel": 1.7e-3 if case["kind"] in ("decoder", "mlp") else 1.2e-3}
