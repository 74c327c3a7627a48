"""Shared helpers for the GPU parity tests: conversions between torch buffers and the
float64 arrays the oracle works on, and the comparison rules.

Comparison rules (derived from the arithmetic):
* fp32 outputs of elementwise paths: relative Frobenius error <= 1e-5 per tensor.
* bf16-stored outputs of elementwise paths: each element must be a correct rounding of a
  value within 1e-5 of the oracle: |gpu - ref| <= ulp_bf16(ref)/2 + 1e-5 * max(|ref|, rms(ref)).
  The rms floor is there because these outputs are sums of terms of the tensor's typical
  magnitude (theta - mu u - eta Psi): the fp32 rounding error of such a sum scales with its
  operands, not with a result that cancellation happened to make small.
* Newton-Schulz outputs (bf16 matrix-core path): relative Frobenius error <= 2e-2 per matrix,
  and so that a wrong block cannot hide in the norm of a large matrix: the same ratio on
  every 256 x 256 block of the output (<= 3e-2: a block averages over fewer elements), and
  the largest element error <= 16 x the rms error and <= a quarter of the largest element
  (bf16 rounding errors scale with the element, and elements reach 5-6 x their rms, so the
  largest error of 1.7e7 elements sits near 10 x the rms error on a correct result).
* quantiser codes and scales: exact equality.
"""
import os
import re

import numpy as np
import torch

from oracle import storage

NS_TOL = 2e-2
EW_TOL = 1e-5


def to_f64(t: torch.Tensor) -> np.ndarray:
    """Exact float64 copy of what a (fp32 / bf16 / integer) tensor holds."""
    t = t.detach().cpu()
    if t.dtype == torch.bfloat16:
        return t.to(torch.float32).numpy().astype(np.float64)
    return t.numpy().astype(np.float64)


def dtype_name(t: torch.Tensor) -> str:
    return {torch.float32: "f32", torch.bfloat16: "bf16"}[t.dtype]


def rel_fro(got: np.ndarray, ref: np.ndarray) -> float:
    den = np.linalg.norm(ref.ravel())
    num = np.linalg.norm((got - ref).ravel())
    return float(num / den) if den > 0 else float(num)


NS_TILE = 256          # block edge of the per-block check (the GEMM's output tile)
NS_TILE_TOL = 3e-2
NS_MAX_OVER_RMS = 16.0
NS_MAX_FRACTION = 0.25


def ns_error_stats(got: np.ndarray, ref: np.ndarray) -> dict:
    """Error figures of one Newton-Schulz output against the oracle's."""
    d = got - ref
    m, n = ref.shape
    worst_tile, where = 0.0, (0, 0)
    for i in range(0, m, NS_TILE):
        for j in range(0, n, NS_TILE):
            den = np.linalg.norm(ref[i:i + NS_TILE, j:j + NS_TILE])
            num = np.linalg.norm(d[i:i + NS_TILE, j:j + NS_TILE])
            r = float(num / den) if den > 0 else float(num)
            if r > worst_tile:
                worst_tile, where = r, (i, j)
    rms = float(np.sqrt(np.mean(d * d)))
    return {"fro": rel_fro(got, ref), "tile": worst_tile, "tile_at": where,
            "max": float(np.max(np.abs(d))), "rms": rms, "ref_max": float(np.max(np.abs(ref)))}


def assert_ns_close(got: np.ndarray, ref: np.ndarray, what: str, tol: float = NS_TOL) -> dict:
    """All comparison rules of a Newton-Schulz output; `tol` scales every bound alike."""
    st = ns_error_stats(got, ref)
    k = tol / NS_TOL
    assert st["fro"] <= tol, f"{what}: relative Frobenius error {st['fro']:.3e} > {tol:.1e}"
    assert st["tile"] <= NS_TILE_TOL * k, (f"{what}: block at {st['tile_at']} has relative Frobenius "
                                           f"error {st['tile']:.3e} > {NS_TILE_TOL * k:.1e}")
    if st["rms"] > 0:
        assert st["max"] <= NS_MAX_OVER_RMS * st["rms"], (
            f"{what}: largest element error {st['max']:.3e} is {st['max'] / st['rms']:.1f}x the rms error")
    assert st["max"] <= NS_MAX_FRACTION * k * st["ref_max"] + 1e-30, (
        f"{what}: largest element error {st['max']:.3e} vs largest element {st['ref_max']:.3e}")
    return st


def assert_fp32_close(got_t: torch.Tensor, ref: np.ndarray, what: str, tol: float = EW_TOL):
    err = rel_fro(to_f64(got_t), ref)
    assert err <= tol, f"{what}: relative Frobenius error {err:.3e} > {tol:.1e}"


def assert_bf16_rounding_of(got_t: torch.Tensor, ref: np.ndarray, what: str, tol: float = EW_TOL):
    got = to_f64(got_t)
    rms = float(np.sqrt(np.mean(ref * ref))) if ref.size else 0.0
    bound = storage.bf16_ulp(ref) * (0.5 + 2.0 ** -12) + tol * np.maximum(np.abs(ref), rms) + 1e-30
    bad = np.abs(got - ref) > bound
    assert not bad.any(), (f"{what}: {int(bad.sum())} of {bad.size} elements are not a rounding of a "
                           f"value within {tol:.0e} of the oracle; worst "
                           f"{np.max(np.abs(got - ref) / bound):.3f}x the bound")


def assert_stored_close(got_t: torch.Tensor, ref: np.ndarray, what: str):
    if got_t.dtype == torch.bfloat16:
        assert_bf16_rounding_of(got_t, ref, what)
    else:
        assert_fp32_close(got_t, ref, what)


def update_error_bf16(W_gpu_t: torch.Tensor, W0: np.ndarray, W_ref: np.ndarray) -> float:
    """Relative Frobenius error of the update when the result was stored in bf16.

    W_gpu - W_ref = (storage rounding, |.| <= ulp/2, mean square ulp^2/12, independent of the
    update) + (error of the update).  The rounding part is removed in quadrature with its
    expectation, which is far tighter than allowing half an ulp per element."""
    d = to_f64(W_gpu_t) - W_ref
    ulp = storage.bf16_ulp(W_ref)
    excess = float(np.sum(d * d) - np.sum(ulp * ulp) / 12.0)
    return float(np.sqrt(max(excess, 0.0)) / np.linalg.norm(W_ref - W0))


UPDATE_ELEMENT_C = 0.05


def assert_update_elements(W_gpu_t: torch.Tensor, W_ref: np.ndarray, O_ref: np.ndarray, step: float,
                           what: str) -> float:
    """Element-wise bound on the parameters after an inner step, so that a wrong block cannot
    hide in the Frobenius norm of the update: every element must be a storage rounding of a
    value whose orthogonalised term is off by at most UPDATE_ELEMENT_C * max|O| (the element
    bound of the Newton-Schulz output: 16 x its rms error of 1e-2, with rms(O) about a fifth
    of max|O|, plus margin).  step = eta * lr_scale.  Returns the worst ratio to the bound."""
    got = to_f64(W_gpu_t)
    half_ulp = storage.bf16_ulp(W_ref) * (0.5 + 2.0 ** -12) if W_gpu_t.dtype == torch.bfloat16 else 0.0
    bound = half_ulp + UPDATE_ELEMENT_C * abs(step) * float(np.max(np.abs(O_ref))) + 1e-6 * np.abs(W_ref)
    ratio = np.abs(got - W_ref) / bound
    worst = float(ratio.max())
    assert worst <= 1.0, (f"{what}: {int((ratio > 1).sum())} of {ratio.size} elements off by more than the "
                          f"element bound, worst {worst:.2f}x")
    return worst


# ---- which output tile a Newton-Schulz product runs ------------------------------------
def _tile_constants():
    """The fitted constants of the tile estimate, from the kernel source."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    text = open(os.path.join(root, "paper_2505_23725_amd", "csrc", "ns_gemm.hip")).read()

    def numbers(name):
        m = re.search(r"\b%s\[3\] = (\{.*?\})[;,] ?(?:R|F|$|\n|constexpr)" % name, text)
        return [float(x) for x in re.findall(r"\d+\.?\d*", m.group(1))]
    return {"E": numbers("E"), "R": numbers("R"), "F": numbers("F"), 128: numbers("F128"), 64: numbers("F64")}


def ns_tiles(groups, cus=256):
    """[(gram, polynomial, apply) tile width per group] that one call of the library over these
    groups (count, m, n) uses, by the rule of csrc/ns_gemm.hip; None for a group on the
    one-workgroup chain.  test_gpu_newton_schulz.py checks it against the executed FLOP."""
    k = _tile_constants()
    jobs = []
    for i, (c, m, n) in enumerate(groups):
        mp, np_ = -(-m // 128) * 128, -(-n // 128) * 128
        s, l = min(mp, np_), max(mp, np_)
        if not (s == 128 and l <= 512):
            jobs.append((i, c, s, l))
    out = [None if i not in [j[0] for j in jobs] else [0, 0, 0] for i in range(len(groups))]
    def estimate(t, form, tiles, kt):
        full, rest = divmod(tiles, cus)
        if t == 256:
            f = rest / cus
            return 3.5 + full * (kt * 1.40 + k["E"][form]) + (
                kt * (1.02 + 0.38 * f) + k["R"][form] + k["F"][form] * f if rest else 0.0)
        base, one, more, epi = k[t][4 * form:4 * form + 4]
        return base + one * kt + (full + (rest > 0) - 1) * (more * kt + epi)

    for form in range(3):
        def shape(j):
            _, c, s, l = j
            return c, s, (l if form == 2 else s), (l if form == 0 else s)       # batch, M, N, K

        def count(some, t):
            return sum(c * (-(-M // t) * (-(-M // t) + 1) // 2 if form < 2 else -(-M // t) * -(-N // t))
                       for c, M, N, K in map(shape, some))

        def large(M, N):     # sides that the 256 x 256 tile divides, or long enough for half a tile twice
            return all(d >= 256 and (d % 256 == 0 or d >= 896) for d in (M, N))
        todo, sets = list(jobs), []
        while todo:
            first = shape(todo[0])
            fits = large(*first[1:3])
            some = [j for j in todo if shape(j)[3] == first[3] and large(*shape(j)[1:3]) == fits][:3]
            todo = [j for j in todo if j not in some]
            kt = first[3] // 64
            nbytes = sum(2 * c * K * (M + (N if form == 2 else 0)) for c, M, N, K in map(shape, some))
            tile, us = 128, estimate(128, form, count(some, 128), kt)
            e64 = estimate(64, form, count(some, 64), kt)
            if kt >= 4 and e64 < 0.95 * us:
                tile, us = 64, e64
            if fits and kt >= 4 and not us < (0.85 if nbytes > 64e6 else 0.95) * estimate(256, form, count(some, 256), kt):
                tile = 256
            sets.append([some, tile, kt])
        # sets that run different small tiles and make one round together take one tile
        sets.sort(key=lambda x: -x[2])
        for i, a in enumerate(sets):
            for b in sets[i + 1:]:
                if not a[0] or not b[0] or len(a[0]) + len(b[0]) > 3 or (a[1] == 256) != (b[1] == 256):
                    continue
                if a[1] == b[1]:
                    ca, cb = count(a[0], a[1]), count(b[0], b[1])
                    q = 2 if a[1] == 64 else 3
                    several = (ca + cb) * 4 > (q + 4) * cus and min(ca, cb) * 4 > q * cus
                    if a[1] != 256 and a[2] != b[2] and shape(a[0][0])[1] != shape(b[0][0])[1] and several:
                        continue
                    tile = a[1]
                else:
                    us = sum(estimate(x[1], form, count(x[0], x[1]), x[2]) for x in (a, b))
                    tile = 0
                    for t in (128, 64):
                        n = count(a[0] + b[0], t)
                        if n <= cus and (t == 128 or b[2] >= 4) and estimate(t, form, n, a[2]) < us:
                            tile, us = t, estimate(t, form, n, a[2])
                    if not tile:
                        continue
                if tile == 128 and b[2] < 4 and a[2] > 10:       # the long ring needs four K tiles
                    continue
                a[0], a[1], b[0] = a[0] + b[0], tile, []
            for j in a[0]:
                out[j[0]][form] = a[1]
    return [None if o is None else tuple(o) for o in out]


def ns_executed_flops(groups, iters=5):
    """Matrix-core FLOP that the library's recorder counts for groups off the one-workgroup chain."""
    total = 0.0
    for (c, m, n), (gram, poly, apply) in zip(groups, ns_tiles(groups)):
        mp, np_ = -(-m // 128) * 128, -(-n // 128) * 128
        s, l = min(mp, np_), max(mp, np_)

        def sym(t):          # of a 256 x 256 tile on the diagonal 144 of 256 MFMAs are executed
            return (-(-s // t) * (-(-s // t) + 1) / 2 - (-(-s // t) * 112 / 256 if t == 256 else 0)) * t * t
        total += iters * c * 2.0 * (sym(gram) * l + sym(poly) * s + -(-s // apply) * -(-l // apply) * apply ** 2 * s)
    return total
