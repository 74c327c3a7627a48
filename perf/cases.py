"""The work that a MuLoCo training program has this library do, as timed cases.

Every case is one call of a public entry point (or the few calls that one step makes) on state
that such a program keeps: parameters, momenta, replicas, quantiser buffers, the work space.
Shapes follow the workloads of `synth_inputs.py` (transformer-shaped parameter sets from 2 layers
of width 128 to a layer of width 5120), their streaming fragments, and ragged sizes that no tile
divides.  `draw` gives further cases of the same ranges.
"""
import math

import torch

import paper_2505_23725_amd as mlc

DEV = "cuda:0"
COEFFS = (3.4445, -4.7750, 2.0315)      # of the Newton-Schulz polynomial
PARAM_STD, GRAD_STD, DELTA_STD = 0.02, 1e-3, 1e-2        # as in synth_inputs.py
NS_ITERS = 5
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # The smallest optimizer step: 2 layers of width 128, fp32, one replica.  Launches count.
        {"name": "inner_tiny", "kind": "inner", "d": 128, "f": 512, "layers": 2, "K": 1,
         "param": "f32", "grad": "f32"},
        # Muon step of eight resident replicas of the 150M-scale model (768 / 3072 wide).
        {"name": "inner_150m_k8", "kind": "inner", "d": 768, "f": 3072, "layers": 12, "K": 8,
         "param": "bf16", "grad": "bf16"},
        # Muon step of the 1.76B-scale model: the benchmark's own inner step, the largest case.
        {"name": "inner_1.76b", "kind": "inner", "d": 2048, "f": 8192, "layers": 24, "K": 1,
         "param": "bf16", "grad": "bf16"},
        # One layer at 15B scale: few, very large matrices (a step that goes layer by layer).
        {"name": "inner_15b_layer", "kind": "inner", "d": 5120, "f": 20480, "layers": 1, "K": 1,
         "param": "bf16", "grad": "bf16"},
        # Ragged widths (nothing divides a tile), fp32 weights from bf16 gradients.
        {"name": "inner_ragged", "kind": "inner", "d": 1001, "f": 2730, "layers": 4, "K": 2,
         "param": "f32", "grad": "bf16"},
        # Orthogonalising one ordinary matrix: far fewer tiles than compute units.
        {"name": "ns_single", "kind": "ns", "count": 1, "m": 1024, "n": 1024, "io": "bf16", "static": True},
        # A small batch of ragged fp32 matrices, odd row length.
        {"name": "ns_ragged", "kind": "ns", "count": 6, "m": 3001, "n": 1000, "io": "f32", "static": False},
        # Outer step over eight resident replicas of the 150M-scale model, nothing compressed.
        {"name": "outer_150m_k8", "kind": "outer", "d": 768, "f": 3072, "layers": 12, "K": 8,
         "worker": "bf16", "global": "f32", "bits": 0, "ef": False, "offset": False, "per_matrix": False},
        # Streaming fragment: one layer of the 3.1B-scale model, four replicas, 4-bit codes.
        {"name": "outer_q4_layer_k4", "kind": "outer", "d": 2560, "f": 10240, "layers": 1, "K": 4,
         "worker": "bf16", "global": "f32", "bits": 4, "ef": False, "offset": False, "per_matrix": False},
        # Ragged rows (not a multiple of 8), 8-bit offset codes with error feedback.
        {"name": "outer_q8_ef_ragged", "kind": "outer", "d": 1001, "f": 2730, "layers": 6, "K": 2,
         "worker": "bf16", "global": "f32", "bits": 8, "ef": True, "offset": True, "per_matrix": False},
        # The other compressor: top 5 % with error feedback over layers of the 1.76B-scale model.
        {"name": "topk_ef_1.76b", "kind": "topk", "d": 2048, "f": 8192, "layers": 6, "K": 1,
         "fraction": 0.05, "ef": True},
        # What Muon does not cover: a tied embedding, and two norm gains and a bias per layer.
        {"name": "adamw_nonmatrix", "kind": "adamw", "vocab": 32000, "d": 2048, "layers": 24,
         "param": "bf16", "grad": "bf16"},
    ]


# ---------------------------------------------------------------------------------------
def shapes_of(case):
    """(count, m, n) of the three shape groups of `layers` transformer layers."""
    L, d, f = case["layers"], case["d"], case["f"]
    return [(4 * L, d, d), (L, d, f), (L, f, d)]


def elements(case):
    return sum(c * m * n for c, m, n in shapes_of(case))


def ns_flops(count, m, n, iters=NS_ITERS):
    """The iteration as printed: X X^T and its square are symmetric and need half their entries."""
    s, l = min(m, n), max(m, n)
    return float(count) * iters * (3.0 * s * s * l + 1.0 * s ** 3)


def esize(name):
    return 4 if name == "f32" else 2


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A width between lo and hi: as models have them, a multiple of 8, or any number."""
    w = _log_int(rng, lo, hi)
    how = rng.random()
    if how < 0.5:
        step = 128 if w >= 512 else 64
    elif how < 0.75:
        step = 8
    else:
        step = 1
    return max(step, w // step * step)


def draw(rng):
    kind = rng.choice(["inner", "inner", "inner", "ns", "ns", "outer", "outer", "outer", "topk", "adamw"])
    if kind == "inner":
        d = _width(rng, 96, 5120)
        f = _width(rng, d, 4 * d)
        K = rng.choice([1, 1, 2, 4, 8])
        case = {"kind": kind, "d": d, "f": f, "layers": 1, "K": K, "param": rng.choice(["bf16", "bf16", "f32"]),
                "grad": rng.choice(["bf16", "bf16", "f32"])}
        # no more than two thirds of the largest listed case's work
        most = min(2.0e13 / (K * sum(ns_flops(*s) for s in shapes_of(case))), 4.0e8 / (K * elements(case)), 24.0)
        if most < 1.0:
            case["K"] = 1
            most = min(2.0e13 / sum(ns_flops(*s) for s in shapes_of(case)), 24.0)
        case["layers"] = _log_int(rng, 1, max(1.0, most))
        return case
    if kind == "ns":
        m, n = _width(rng, 64, 4096), _width(rng, 64, 4096)
        most = max(1.0, min(5.0e12 / ns_flops(1, m, n), 1.0e8 / (m * n), 256.0))
        return {"kind": kind, "count": _log_int(rng, 1, most), "m": m, "n": n, "io": rng.choice(["bf16", "f32"]),
                "static": m * n <= 2048 * 2048 and max(m, n) <= 2048 and rng.random() < 0.3}
    if kind == "adamw":
        return {"kind": kind, "vocab": _log_int(rng, 1000, 64000), "d": _width(rng, 128, 4096),
                "layers": _log_int(rng, 2, 48), "param": rng.choice(["bf16", "f32"]), "grad": rng.choice(["bf16", "f32"])}
    d = _width(rng, 128, 4096)
    f = _width(rng, d, 4 * d)
    K = rng.choice([1, 2, 4, 8])
    case = {"kind": kind, "d": d, "f": f, "layers": 1, "K": K}
    case["layers"] = _log_int(rng, 1, max(1.0, min(4.0e8 / (K * elements(case)), 24.0)))
    if kind == "topk":
        case.update(fraction=round(math.exp(rng.uniform(math.log(0.005), math.log(0.2))), 4), ef=rng.random() < 0.7)
        return case
    bits = rng.choice([0, 2, 4, 4, 8])
    if bits and (d % (8 // bits) or f % (8 // bits)):
        bits = 8
    case.update(worker=rng.choice(["bf16", "bf16", "f32"]), bits=bits, ef=bits != 0 and rng.random() < 0.4,
                offset=bits != 0 and rng.random() < 0.3, per_matrix=bits != 0 and rng.random() < 0.2)
    case["global"] = "f32" if case["worker"] == "f32" or rng.random() < 0.8 else "bf16"
    return case


# ---------------------------------------------------------------------------------------
def _normal(gen, shape, std, dtype=torch.float32):
    """std * N(0, 1), drawn and rounded slice by slice so that no large temporary is held."""
    out = torch.empty(shape, dtype=dtype, device=DEV)
    flat = out.view(-1)
    step = 1 << 27
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=gen, device=DEV) * std
    return out


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "inner":
        # a step in the middle of training: gradients and a momentum that has built up
        groups = []
        for c, m, n in shapes_of(case):
            shape = (case["K"] * c, m, n)
            groups.append(mlc.InnerGroup(_normal(gen, shape, PARAM_STD, DTYPES[case["param"]]),
                                         _normal(gen, shape, GRAD_STD, DTYPES[case["grad"]]),
                                         _normal(gen, shape, 3 * GRAD_STD), math.sqrt(n / m)))
        ws = torch.empty(mlc.muloco_inner_workspace_bytes(groups), dtype=torch.uint8, device=DEV)
        return {"kind": kind, "groups": groups, "ws": ws,
                "hp": mlc.MuonHParams(eta=6.25e-2, weight_decay=1.25e-3, beta=0.9)}
    if kind == "ns":
        x = _normal(gen, (case["count"], case["m"], case["n"]), GRAD_STD, DTYPES[case["io"]])
        need = 0 if case["static"] else mlc.newton_schulz_workspace_bytes(case["count"], case["m"], case["n"])
        return {"kind": kind, "x": x, "out": torch.empty_like(x), "static": case["static"],
                "ws": torch.empty(need, dtype=torch.uint8, device=DEV)}
    if kind == "adamw":
        d, L = case["d"], case["layers"]
        sizes = [case["vocab"] * d] + [d] * (2 * L + 1) + [3 * d] * L
        # slices of one flat buffer per kind of state, each starting on a 32-byte boundary
        ends = [0]
        for n in sizes:
            ends.append(ends[-1] + (n + 15) // 16 * 16)
        flat = (_normal(gen, (ends[-1],), PARAM_STD, DTYPES[case["param"]]),
                _normal(gen, (ends[-1],), GRAD_STD, DTYPES[case["grad"]]),
                _normal(gen, (ends[-1],), GRAD_STD), _normal(gen, (ends[-1],), GRAD_STD).square_())
        tensors = [tuple(t[e:e + n] for t in flat) for e, n in zip(ends, sizes)]
        return {"kind": kind, "tensors": tensors, "flat": flat,
                "hp": mlc.AdamWHParams(lr=1e-3, weight_decay=0.1, bias_correction=True, step=100)}
    # outer step: replicas that H inner steps have moved away from the global copy
    K, bits = case["K"], case.get("bits", 0)
    wd, gd = DTYPES[case.get("worker", "bf16")], DTYPES[case.get("global", "f32")]
    groups = []
    for c, m, n in shapes_of(case):
        theta = _normal(gen, (c, m, n), PARAM_STD, gd)
        workers = []
        for _ in range(K):
            w = torch.empty((c, m, n), dtype=wd, device=DEV)
            for i in range(c):
                w[i] = theta[i].float() - _normal(gen, (m, n), DELTA_STD)
            workers.append(w)
        g = mlc.OuterGroup(workers, theta, _normal(gen, (c, m, n), GRAD_STD))
        ranges = c if case.get("per_matrix") else c * m
        if bits:
            g.codes = [torch.empty((c * m, n * bits // 8), dtype=torch.uint8, device=DEV) for _ in range(K)]
            g.scales = [torch.empty(ranges, device=DEV) for _ in range(K)]
        if case.get("offset"):
            g.offsets = [torch.empty(ranges, device=DEV) for _ in range(K)]
        if kind == "topk":
            g.scales = [torch.empty(c, device=DEV) for _ in range(K)]
        if case["ef"]:
            g.residuals = [_normal(gen, (c, m, n), 0.3 * DELTA_STD) for _ in range(K)]
        groups.append(g)
    # fp32 replicas that received the fp32 global copy would leave nothing to compress on a second
    # pass over the same state; there the write-back is left out
    state = {"kind": kind, "groups": groups,
             "hp": mlc.OuterHParams(K=K, eta_out=0.7, mu=0.9, quant_bits=bits, write_back=wd != gd or not bits,
                                    error_feedback=case["ef"], ef_beta=0.9,
                                    quant_offset=bool(case.get("offset")),
                                    quant_per_matrix=bool(case.get("per_matrix")))}
    if kind == "topk":
        state["fraction"] = case["fraction"]
        state["ws"] = torch.empty(mlc.muloco_topk_workspace_bytes(groups, K), dtype=torch.uint8, device=DEV)
    return state


def run(state):
    kind = state["kind"]
    if kind == "inner":
        mlc.muloco_inner_step(state["groups"], state["hp"], state["ws"])
        return [(g.param, g.momentum) for g in state["groups"]]
    if kind == "ns":
        if state["static"]:
            return mlc.newton_schulz_static_scratch(state["x"], state["out"])
        return mlc.newton_schulz(state["x"], state["out"], state["ws"])
    if kind == "adamw":
        mlc.muloco_adamw_step(state["tensors"], state["hp"])
        theta, _, m, v = state["flat"]
        return [theta, m, v]
    if kind == "topk":
        mlc.muloco_topk_outer_step(state["groups"], state["hp"], state["fraction"], state["ws"])
    else:
        mlc.muloco_outer_step(state["groups"], state["hp"])
    out = []
    for g in state["groups"]:
        # of the replicas and their buffers two stand for all: 64 outputs are the most that fit
        two = range(0, len(g.worker_params), max(1, len(g.worker_params) - 1))
        out.append([g.global_param, g.outer_momentum] +
                   [[ts[k] for k in two] for ts in (g.worker_params, g.codes, g.scales, g.offsets, g.residuals)
                    if ts is not None])
    return out


# ---- the same in 64 bits --------------------------------------------------------------
def _orthogonalise(u):
    a, b, c = COEFFS
    x = u / (u.norm() + 1e-7)
    wide = x.shape[0] <= x.shape[1]
    for _ in range(NS_ITERS):
        g = x @ x.T if wide else x.T @ x
        p = b * g + c * (g @ g)
        x = a * x + (p @ x if wide else x @ p)
    return x


def _levels(v, bits, offset, per_matrix):
    """(dequantised values, scale, lower end) of [c][m][n] fp32 values.  Which level a value falls
    on is defined in 32 bits (a tensor by a tensor: a true division); everything after that is in
    64."""
    r = v.reshape(v.shape[0], 1, -1) if per_matrix else v
    if offset:
        lo, levels = r.amin(-1, keepdim=True), 2 ** bits - 1
        scale = (r.amax(-1, keepdim=True) - lo) / torch.full_like(lo, levels)
        q = ((r - lo) / scale).round_().clamp_(0, levels)
    else:
        lo, levels = torch.zeros_like(r[..., :1]), 2 ** (bits - 1) - 1
        scale = r.abs().amax(-1, keepdim=True) / torch.full_like(lo, levels)
        q = (r / scale).round_().clamp_(-levels, levels)
    sent = q.double() * scale.double() + lo.double()
    return sent.reshape(v.shape), scale.reshape(-1).double(), lo.reshape(-1).double()


def _exact_outer(state):
    hp, fraction = state["hp"], state.get("fraction")
    out = []
    for g in state["groups"]:
        theta = g.global_param
        c = theta.shape[0]
        mean = torch.zeros(theta.shape, dtype=torch.float64, device=DEV)
        scales, offsets, residuals = [], [], []
        for k, w in enumerate(g.worker_params):
            if not hp.quant_bits and fraction is None:
                mean += theta.double() - w.double()
                continue
            v = theta.float() - w.float()
            if hp.error_feedback:
                v = g.residuals[k] * hp.ef_beta + v
            if fraction is None:
                sent, scale, lo = _levels(v, hp.quant_bits, hp.quant_offset, hp.quant_per_matrix)
                scales.append(scale)
                offsets.append(lo)
            else:
                per = v[0].numel()
                kept = min(per, max(1, math.ceil(fraction * per)))
                tau = torch.stack([m.abs().flatten().sort(descending=True).values[kept - 1] for m in v])
                sent = torch.where(v.abs() >= tau[:, None, None], v, torch.zeros_like(v)).double()
                scales.append(tau.double())
            residuals.append(v.double() - sent)
            mean += sent
        psi = mean / hp.K
        u = hp.mu * g.outer_momentum.double() + hp.eta_out * psi
        new = theta.double() - hp.mu * u - hp.eta_out * psi
        two = range(0, hp.K, max(1, hp.K - 1))
        rows = [[new if hp.write_back else w.double() for w in g.worker_params]]
        if g.codes is not None:
            rows.append([None] * hp.K)                    # whole numbers
        if g.scales is not None:
            rows.append(scales)
        if g.offsets is not None:
            rows.append(offsets)
        if g.residuals is not None:
            rows.append(residuals)
        out.append([new, u] + [[r[k] for k in two] for r in rows])
    return out


def exact(case, seed):
    state = prepare(case, seed)
    kind, hp = state["kind"], state.get("hp")
    if kind == "ns":
        return torch.stack([_orthogonalise(x.double()) for x in state["x"]])
    if kind == "inner":
        out = []
        for g in state["groups"]:
            w, m = g.param.double(), g.momentum.double()
            for i in range(w.shape[0]):
                grad = g.grad[i].double()
                m[i] = hp.beta * m[i] + grad
                o = _orthogonalise(grad + hp.beta * m[i])
                w[i] -= hp.eta * hp.weight_decay * w[i] + hp.eta * g.lr_scale * o
            out.append((w, m))
        return out
    if kind == "adamw":
        theta, grad, m, v = [t.double() for t in state["flat"]]
        new = [theta.clone(), m.clone(), v.clone()]
        ends = 0
        for n in [t[0].numel() for t in state["tensors"]]:
            s = slice(ends, ends + n)
            new[1][s] = hp.beta1 * m[s] + (1 - hp.beta1) * grad[s]
            new[2][s] = hp.beta2 * v[s] + (1 - hp.beta2) * grad[s] ** 2
            mh = new[1][s] / (1 - hp.beta1 ** hp.step)
            vh = new[2][s] / (1 - hp.beta2 ** hp.step)
            new[0][s] -= hp.lr * mh / (vh.sqrt() + hp.eps) + hp.lr * hp.weight_decay * theta[s]
            ends += (n + 15) // 16 * 16
        return new
    return _exact_outer(state)


def work(case):
    kind = case["kind"]
    if kind == "inner":
        n = case["K"] * elements(case)
        return {"bytes": float(n) * (2 * esize(case["param"]) + esize(case["grad"]) + 8),
                "flops": case["K"] * sum(ns_flops(*s) for s in shapes_of(case))}
    if kind == "ns":
        c, m, n = case["count"], case["m"], case["n"]
        return {"bytes": 2.0 * c * m * n * esize(case["io"]), "flops": ns_flops(c, m, n)}
    if kind == "adamw":
        n = case["vocab"] * case["d"] + case["d"] * (2 * case["layers"] + 1) + 3 * case["d"] * case["layers"]
        return {"bytes": float(n) * (2 * esize(case["param"]) + esize(case["grad"]) + 16), "flops": 0.0}
    n, K = elements(case), case["K"]
    wb, gb = case.get("worker", "bf16"), case.get("global", "f32")
    bits = case.get("bits", 0)
    back = wb != gb or not bits
    per = K * esize(wb) * (2 if back else 1) + 2 * esize(gb) + 8 + K * bits / 8.0 + (8 * K if case["ef"] else 0)
    ranges = sum(c if case.get("per_matrix") or kind == "topk" else c * m for c, m, _ in shapes_of(case))
    tables = (1 if bits or kind == "topk" else 0) + (1 if case.get("offset") else 0)
    return {"bytes": n * per + 4.0 * K * ranges * tables, "flops": 0.0}


def tolerance(case):
    kind = case["kind"]
    if kind == "ns":
        # products of bf16 operands, bf16 between products: 0.8e-2 to 1.1e-2 from the same
        # iteration in 64 bits
        return {"rel": 0.03, "max": 0.6}
    if kind == "inner":
        # the error above on the update, which is a twentieth (wide bf16 models) to two fifths
        # (narrow fp32 ones) of the weights, plus a storage rounding of the weights
        return {"rel": 0.01, "max": 0.25}
    # 32-bit elementwise arithmetic; a bf16 copy may fall to the other side of a rounding
    narrow = kind == "topk" or "bf16" in (case.get("worker"), case.get("global"), case.get("param"))
    return {"rel": 1e-4, "max": 1.6e-2} if narrow else {"rel": 1e-5}
