"""The work this library is measured on: the calls a serving program makes per MoE layer.

Three kinds of call, each through ``paper_2607_23099_amd.moe.Path`` and weights held as a program
would hold them (fragment-packed, in HBM, laid out once):

* ``layer`` with a tuned table: ``route_dispatch`` (histogram, permutation, variant choice on the
  device) then ``fused`` (grouped GEMM1 + SwiGLU, grouped GEMM2, gate-weighted reduce).  bf16 and
  MXFP4 weights of a DeepSeek-V3-shaped layer at decode sizes, one expert-parallel rank of it, and a
  bf16 Kimi-K2-shaped layer from decode to prefill sizes.
* ``layer`` with a named kernel variant: ``route`` then ``fused(force_variant=...)``.  fp8 weights
  (128 x 128 block scales) at prefill sizes, for which no table is shipped.
* ``router``: gating logits, top-k experts and gates of each token.

Routing is drawn as in the benchmark: a Dirichlet(alpha) expert distribution, k distinct experts a
token by Gumbel-top-k, softmax gates.  alpha = 0.05 is a heavily skewed batch, 10 a nearly uniform one.
"""
from __future__ import annotations

import os
from types import SimpleNamespace

import numpy as np
import torch

from paper_2607_23099_amd import damoe, moe

TABLES = os.path.join(os.path.dirname(os.path.abspath(damoe.__file__)), "tables")
DEVICE = "cuda"
W_SIGMA = 0.02  # standard deviation of the expert weights

# model -> experts of the whole layer, experts per token, hidden size, expert intermediate size
MODELS = {"dsv3": (256, 8, 7168, 2048), "kimi-k2": (384, 8, 7168, 2048)}
WDTYPE = {"bf16": damoe.W_BF16, "fp8": damoe.W_FP8_B128, "mxfp4": damoe.W_MXFP4}


def _layer(name, model, weights, T, alpha, table="", variant="", ep=1):
    return {"name": name, "kind": "layer", "model": model, "weights": weights, "T": T, "alpha": alpha,
            "table": table, "variant": variant, "ep": ep}


def _router(name, model, T):
    return {"name": name, "kind": "router", "model": model, "T": T}


def listed():
    return [
        # One token, eight experts: single-stream decode, where launches and latencies weigh most.
        _layer("decode_t1", "dsv3", "bf16", 1, 1.0, table="dsv3"),
        # A common decode batch with moderate skew: the weight stream of ~100 experts.
        _layer("decode_t32", "dsv3", "bf16", 32, 0.3, table="dsv3"),
        # A large ragged decode batch on few hot experts: several token tiles per expert.
        _layer("decode_t117_skewed", "dsv3", "bf16", 117, 0.05, table="dsv3"),
        # Small and large decode batches of a 4-bit layer.
        _layer("decode_mxfp4_t6", "dsv3", "mxfp4", 6, 1.0, table="dsv3-mxfp4"),
        _layer("decode_mxfp4_t128", "dsv3", "mxfp4", 128, 10.0, table="dsv3-mxfp4"),
        # One rank of an 8-way expert-parallel group: 32 local experts, remote slots masked.
        _layer("ep8_rank_t96", "dsv3", "bf16", 96, 1.0, table="dsv3-ep8", ep=8),
        # A chunk of prefill mixed into decode: a handful of tokens on each of ~300 experts.
        _layer("kimi_t300", "kimi-k2", "bf16", 300, 1.0, table="kimi-k2"),
        # Full prefill, bf16: bound by the matrix cores and by the operand feed.
        _layer("kimi_t8192", "kimi-k2", "bf16", 8192, 0.3, table="kimi-k2"),
        # fp8 prefill: a short prompt (a few dozen tokens per expert) and the largest call.
        _layer("fp8_t1024", "dsv3", "fp8", 1024, 1.0, variant="deep8_bm64"),
        _layer("fp8_t16384", "dsv3", "fp8", 16384, 0.3, variant="big8_bm256"),
        # The gate in front of a decode step and of a prefill.
        _router("router_t32", "kimi-k2", 32),
        _router("router_t8192", "dsv3", 8192),
    ]


def draw(rng):
    """One more call of the ranges above; token counts and skews spread over their logarithm."""
    def log_int(lo, hi):
        return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))

    alpha = float("%.3g" % (0.05 * 200.0 ** rng.random()))
    family = rng.choice(["decode", "decode", "mxfp4", "ep8", "kimi", "kimi", "fp8", "fp8", "router"])
    if family == "decode":
        c = _layer("", "dsv3", "bf16", log_int(1, 128), alpha, table="dsv3")
    elif family == "mxfp4":
        c = _layer("", "dsv3", "mxfp4", log_int(1, 128), alpha, table="dsv3-mxfp4")
    elif family == "ep8":
        c = _layer("", "dsv3", "bf16", log_int(8, 256), alpha, table="dsv3-ep8", ep=8)
    elif family == "kimi":
        c = _layer("", "kimi-k2", "bf16", log_int(1, 8192), alpha, table="kimi-k2")
    elif family == "fp8":
        T = log_int(1024, 16384)
        c = _layer("", "dsv3", "fp8", T, alpha, variant="deep8_bm64" if T < 2048 else "big8_bm256")
    else:
        c = _router("", rng.choice(["dsv3", "kimi-k2"]), log_int(1, 8192))
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

def _generator(*key):
    """A device generator seeded from the key (any integers)."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(np.random.SeedSequence([int(v) & 0xFFFFFFFF for v in key]).generate_state(2, np.uint32)
                      .astype(np.uint64).dot(np.array([1, 1 << 31], np.uint64))) & (2 ** 62 - 1))
    return g


def _routing(case, seed):
    """(ids int32 [T][k], gates float32 [T][k]) of a layer call, on the device.  Of an expert-parallel
    rank (the first of `ep`): the tokens with a slot on the rank, remote slots masked with -1."""
    E, k, _, _ = MODELS[case["model"]]
    T, alpha, ep = case["T"], case["alpha"], case["ep"]
    rng = np.random.default_rng([seed, T, 1])
    logp = np.log(rng.gamma(alpha + 1.0, size=E)) + np.log(rng.random(E)) / alpha
    logp = torch.from_numpy(logp - np.logaddexp.reduce(logp)).to(DEVICE)
    g = _generator(seed, T, 2)
    rows = []
    need, local = T, E // ep
    for _ in range(4096):
        n = need if ep == 1 else 4 * T
        u = torch.rand((n, E), generator=g, device=DEVICE, dtype=torch.float64).clamp_min_(1e-300)
        ids = (logp - torch.log(-torch.log(u))).topk(k, dim=1).indices
        if ep > 1:
            ids = torch.where(ids < local, ids, -1)
            ids = ids[(ids >= 0).any(dim=1)]
        rows.append(ids[:need])
        need -= rows[-1].shape[0]
        if need == 0:
            break
    if need:  # a rank that the drawn distribution hardly reaches: one local slot a token
        ids = torch.full((need, k), -1, dtype=torch.int64, device=DEVICE)
        ids[:, 0] = torch.randint(0, local, (need,), generator=g, device=DEVICE)
        rows.append(ids)
    ids = torch.cat(rows).to(torch.int32)
    gates = torch.softmax(torch.randn((T, k), generator=g, device=DEVICE, dtype=torch.float64), dim=1)
    return ids, gates.to(torch.float32)


def _tokens(T, H, seed):
    return torch.randn((T, H), generator=_generator(seed, T, 3), device=DEVICE).to(torch.bfloat16)


def _matrix(case, seed, e, m, dequantised=False):
    """Matrix m (0: W1, 1: W3, 2: W2) of expert e: the stored tensors (values, scales or None), or its
    exact values in float64."""
    _, _, H, I = MODELS[case["model"]]
    r, c = (H, I) if m == 2 else (I, H)
    w = torch.randn((r, c), generator=_generator(seed, e, m, 4), device=DEVICE).mul_(W_SIGMA).to(torch.bfloat16)
    if case["weights"] == "bf16":
        return w.double() if dequantised else (w, None)
    w = w.float()
    if case["weights"] == "fp8":
        b = w.view(r // 128, 128, c // 128, 128)
        s = b.abs().amax(dim=(1, 3)) / 448.0
        q = (b / s[:, None, :, None]).to(torch.float8_e4m3fn)
        if dequantised:
            return (q.double() * s.double()[:, None, :, None]).view(r, c)
        return q.view(torch.uint8).view(r, c), s
    # MXFP4: one power-of-two scale per 32 columns, values on the e2m1 grid 0, .5, 1, 1.5, 2, 3, 4, 6.
    b = w.view(r, c // 32, 32)
    ex = torch.frexp(b.abs().amax(dim=2)).exponent - 3
    v = torch.ldexp(b.abs(), -ex[:, :, None])
    step = torch.where(v < 2, 0.5, torch.where(v < 4, 1.0, 2.0))
    v = torch.round(v / step).mul_(step).clamp_max_(6.0)
    if dequantised:
        return torch.ldexp(v.double(), ex[:, :, None]).mul_(torch.sign(b).double()).view(r, c)
    code = torch.where(v < 2, v * 2, torch.where(v < 4, v + 2, v / 2 + 4)).to(torch.uint8)
    code |= (b < 0).to(torch.uint8) << 3
    code = code.view(r, c // 2, 2)
    return code[:, :, 0] | (code[:, :, 1] << 4), (ex + 127).to(torch.uint8)


def _weights(case, seed):
    """The layer as a program holds it: packed weights in HBM and the descriptor of the library."""
    _, k, H, I = MODELS[case["model"]]
    E = MODELS[case["model"]][0] // case["ep"]
    wd = WDTYPE[case["weights"]]
    w, s, packed = [], [], []
    for m in range(3):
        r, c = (H, I) if m == 2 else (I, H)
        q, sc = _matrix(case, seed, 0, m)
        w.append(torch.empty((E,) + tuple(q.shape), dtype=q.dtype, device=DEVICE))
        s.append(None if sc is None else torch.empty((E,) + tuple(sc.shape), dtype=sc.dtype, device=DEVICE))
        for e in range(E):
            q, sc = _matrix(case, seed, e, m)
            w[m][e] = q
            if sc is not None:
                s[m][e] = sc
        packed.append(torch.empty((E, r * c * 17 // 32), dtype=torch.uint8, device=DEVICE) if wd == damoe.W_MXFP4
                      else torch.empty_like(w[m]))
    damoe.pack_weights(damoe.make_layer(E, k, H, I, wd, *w, *s), *packed)
    torch.cuda.synchronize()
    if wd == damoe.W_MXFP4:
        s = [None] * 3
    layer = damoe.make_layer(E, k, H, I, wd, *packed, *s, layout=damoe.LAYOUT_FRAG16)
    return SimpleNamespace(shape=SimpleNamespace(E=E, k=k, H=H, I=I), layer=layer, w=packed, s=s)


def prepare(case, seed):
    E, k, H, I = MODELS[case["model"]]
    T = case["T"]
    if case["kind"] == "router":
        # The router's buffers belong to a Path; a descriptor without weights is enough for it.
        shape = SimpleNamespace(E=E, k=k, H=H, I=I)
        layer = damoe.make_layer(E, k, H, I, damoe.W_BF16, None, None, None)
        path = moe.Path(SimpleNamespace(shape=shape, layer=layer), T)
        wg, bias = _gate(case, seed)
        path.x.copy_(_tokens(T, H, seed))
        return SimpleNamespace(case=case, path=path, gate=SimpleNamespace(wg=wg, bias=bias))
    dl = _weights(case, seed)
    path = moe.Path(dl, T)
    ids, gates = _routing(case, seed)
    path.ids.copy_(ids.view(-1))
    path.w.copy_(gates.view(-1))
    path.x.copy_(_tokens(T, H, seed))
    table = damoe.Table.load(os.path.join(TABLES, case["table"] + ".damoe")) if case["table"] else None
    names = [damoe.variant_name(v) for v in range(damoe.num_variants())]
    variant = names.index(case["variant"]) if case["variant"] else -1
    return SimpleNamespace(case=case, path=path, table=table, variant=variant)


def _gate(case, seed):
    E, _, H, _ = MODELS[case["model"]]
    g = _generator(seed, 5)
    wg = torch.randn((E, H), generator=g, device=DEVICE).mul_(H ** -0.5).to(torch.bfloat16)
    return wg, torch.randn(E, generator=g, device=DEVICE).mul_(0.1)


def run(state):
    case, path = state.case, state.path
    T = case["T"]
    if case["kind"] == "router":
        k = path.dl.shape.k
        path.router(state.gate, T)
        return {"logits": path.logits[:T], "ids": path.ids[: T * k], "gates": path.w[: T * k]}
    if state.table is not None:
        path.route_dispatch(state.table, T)
        path.fused(T)
    else:
        path.route(T)
        path.fused(T, force_variant=state.variant)
    return {"y": path.y[:T], "counts": path.counts, "perm": path.inv_perm}


# ---------------------------------------------------------------- work, tolerance, reference

def work(case):
    E, k, H, I = MODELS[case["model"]]
    T = case["T"]
    if case["kind"] == "router":
        return {"bytes": (T + E) * H * 2 + T * E * 4 + T * k * 8, "flops": 2 * T * E * H}
    ids, _ = _routing(case, 1)
    touched = int(torch.unique(ids[ids >= 0]).numel())
    slots = int((ids >= 0).sum())
    per = {"bf16": 2.0, "fp8": 1.0 + 4 / 128 ** 2, "mxfp4": 17 / 32}[case["weights"]]
    return {"bytes": touched * 3 * H * I * per + 2 * T * H * 2 + T * k * 8, "flops": 6 * H * I * slots}


def tolerance(case):
    if case["kind"] == "router":
        # fp32 sums of exact bf16 products in another order; ids of logits that close may swap.
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    if case["weights"] == "fp8":
        # h travels as e4m3 (2^-4 steps): a rounding of GEMM1 less or more (the weights' products
        # with their block scale, say) moves some of it by a step.  In a simulation of the layer that
        # is 1.3e-2 of y, where both results are 2.7e-2 off the exact one.
        return {"rel": 3e-2, "max": 3e-1}
    # h, out and y are rounded to bf16.
    return {"rel": 1e-2, "max": 1e-1}


def exact(case, seed):
    E, k, H, I = MODELS[case["model"]]
    T = case["T"]
    if case["kind"] == "router":
        wg, bias = _gate(case, seed)
        logits = _tokens(T, H, seed).double() @ wg.double().t() + bias.double()
        top = torch.sort(logits, dim=1, descending=True, stable=True)
        ids = top.indices[:, :k]
        return {"logits": logits, "ids": ids.reshape(-1), "gates": torch.softmax(top.values[:, :k], dim=1).reshape(-1)}
    E //= case["ep"]
    ids, gates = _routing(case, seed)
    x = _tokens(T, H, seed).double()
    y = torch.zeros((T, H), dtype=torch.float64, device=DEVICE)
    flat = ids.view(-1).long()
    counts = torch.bincount(flat[flat >= 0], minlength=E)
    order = torch.argsort(torch.where(flat >= 0, flat, E), stable=True)
    inv = torch.full_like(flat, -1)
    n_valid = int(counts.sum())
    inv[order[:n_valid]] = torch.arange(n_valid, device=DEVICE)
    for e in torch.nonzero(counts).view(-1).tolist():
        t, j = torch.nonzero(ids == e, as_tuple=True)
        xe = x[t]
        g = xe @ _matrix(case, seed, e, 0, True).t()
        u = xe @ _matrix(case, seed, e, 1, True).t()
        o = (g * torch.sigmoid(g) * u) @ _matrix(case, seed, e, 2, True).t()
        y.index_add_(0, t, o * gates[t, j].double()[:, None])
    return {"y": y, "counts": counts, "perm": inv}
