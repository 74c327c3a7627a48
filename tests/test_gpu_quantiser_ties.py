"""Levels of values next to a tie, where the quantiser divides instead of multiplying by a reciprocal, and of rows whose
scale has no ordinary reciprocal; rows and matrices that hold NaN or infinities: codes, scales, offsets and residuals bit for bit."""
import numpy as np
import pytest
import torch

import paper_2505_23725_amd as mlc
from oracle import diloco

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rows(rows, n, bits, offset, seed):
    """Rows whose values are half-integer multiples of the row's scale, up to a few units in the last place off; scales over
    the whole range of fp32, among them subnormal ones, a power of two and one that is zero."""
    rng = np.random.default_rng(seed)
    levels = 2 ** bits - 1 if offset else 2 ** (bits - 1) - 1
    scale = np.float32(2.0) ** rng.uniform(-149, 118, rows).astype(np.float32)
    scale[:8] = np.float32([2.0 ** -149, 2.0 ** -140, 2.0 ** -126, 2.0 ** -100, 2.0 ** -101, 2.0 ** 100, 1.0, 0.0])
    lo = (rng.normal(size=rows) * 3 * scale if offset else np.zeros(rows)).astype(np.float32)
    top = np.float32(levels) * scale
    k = rng.integers(0 if offset else -levels, levels, (rows, n)).astype(np.float32) + np.float32(0.5)
    v = (k * scale[:, None]).astype(np.float32)
    for _ in range(3):
        step = rng.integers(-1, 2, v.shape)
        v = np.where(step == 0, v, np.nextafter(v, np.where(step > 0, np.float32(np.inf), np.float32(-np.inf)))).astype(np.float32)
    if offset:
        v = np.clip(v + lo[:, None], lo[:, None], (lo + top)[:, None]).astype(np.float32)
        v[:, 0], v[:, 1] = lo, lo + top
    else:
        v = np.clip(v, -top[:, None], top[:, None])
        v[:, 0] = top
    return v


@pytest.mark.parametrize("bits,offset", [(2, False), (4, False), (8, False), (2, True), (4, True), (8, True)])
@pytest.mark.parametrize("n,K,ef", [(64, 1, False), (640, 1, True), (1000, 2, False), (1001 * 8, 3, False), (904, 9, False),
                                    (9000, 2, True), (6001 * 4, 1, True)])       # a row a workgroup
def test_ties(bits, offset, n, K, ef):
    rows, m = 64, 32
    v = _rows(rows, n, bits, offset, seed=n + bits)
    q, scale, lo = diloco.quantize_values(v, bits, offset)
    theta = torch.from_numpy(v).view(rows // m, m, n)
    zero = torch.zeros_like(theta)
    groups = []
    for _ in range(2 if K < 9 else 1):               # two groups share a launch, one has its own
        like = lambda dt, *s: [torch.zeros(s, dtype=dt, device=DEV) for _ in range(K)]  # noqa: E731
        g = mlc.OuterGroup([zero.to(DEV) for _ in range(K)], theta.to(DEV), zero.to(DEV), like(torch.uint8, rows, n * bits // 8),
                           like(torch.float32, rows))
        if offset:
            g.offsets = like(torch.float32, rows)
        if ef:
            g.residuals = [zero.to(DEV) for _ in range(K)]
        groups.append(g)
    hp = mlc.OuterHParams(K=K, eta_out=0.0, mu=0.0, quant_bits=bits, write_back=False, error_feedback=ef, ef_beta=1.0,
                          quant_offset=offset)
    mlc.muloco_outer_step(groups, hp)
    torch.cuda.synchronize()
    want = (diloco.pack_codes_unsigned if offset else diloco.pack_codes)(q, bits)
    for g in groups:
        for k in range(K):
            assert np.array_equal(g.codes[k].cpu().numpy(), want)
            assert np.array_equal(g.scales[k].cpu().numpy().view(np.uint32), scale.view(np.uint32))
            if offset:
                assert np.array_equal(g.offsets[k].cpu().numpy(), lo)
            if ef:
                sent = diloco.dequantize_values(q, scale, lo, offset).astype(np.float32)
                assert np.array_equal(g.residuals[k].cpu().numpy().reshape(rows, n), v - sent)


def _no_numbers(m, n, per_matrix):
    """[4, m, n]: among ordinary values NaN, infinities of either sign and both, and a range (row or matrix) of nothing but NaN."""
    rng = np.random.default_rng(n)
    v = rng.normal(size=(4, m, n)).astype(np.float32)
    v = torch.from_numpy(v).bfloat16().float().numpy()
    r = v.reshape(4, -1) if per_matrix else v.reshape(4 * m, n)       # one range each
    at = lambda: rng.integers(0, r.shape[1], 3)  # noqa: E731
    r[0, at()] = np.nan
    r[1, at()] = np.inf
    r[2] = np.nan
    r[3, at()], r[3, 0] = -np.inf, np.inf
    if not per_matrix:
        r[4, at()] = -np.inf
        r[5] = np.inf                               # max - min is no number
        r[6], r[6, 1:4] = 0.0, np.nan
        r[7, at()], r[7, 0] = np.nan, np.inf
        r[8, :-1] = np.nan                          # a single number
    return v


def _rule(v, bits, offset, per_matrix):
    """(levels, scales, lower ends, values sent) of [4, m, n] values: ranges leave NaN out, a NaN takes the lowest level, and
    without a positive scale every level is 0."""
    r = v.reshape(4, 1, -1) if per_matrix else v
    levels = np.float32(2 ** bits - 1 if offset else 2 ** (bits - 1) - 1)
    with np.errstate(all="ignore"):
        mn, mx = np.fmin.reduce(r, -1, keepdims=True), np.fmax.reduce(r, -1, keepdims=True)
        none = np.isnan(mn)
        if per_matrix:
            mn, mx = np.where(none, np.float32(np.nan if offset else 0), mn), np.where(none, np.float32(np.nan if offset else 0), mx)
        else:
            mn, mx = np.where(none, np.float32(np.inf), mn), np.where(none, np.float32(-np.inf), mx)
        scale = ((mx - mn) if offset else np.fmax(mx, -mn)) / levels
        lo = mn if offset else np.zeros_like(mn)
        x = (r - lo if offset else r) / scale
        q = np.rint(x)
        low = np.float32(0) if offset else -levels
        q = np.where(np.isnan(q), low, np.clip(q, low, levels))
        q = np.where(scale > 0, q, np.float32(0))
        sent = q * scale
        if offset:
            sent = sent + lo
    return q.reshape(-1, v.shape[-1]).astype(np.int64), scale.ravel(), lo.ravel(), sent.reshape(v.shape).astype(np.float32)


# Kernels of one worker, of narrow rows, of all lengths, of ragged rows with four vectors, of one group, of one row a workgroup, and
# of two passes (fp32 workers with a bf16 global copy; rows past 24576)
@pytest.mark.parametrize("n,K,wd,gd,two", [
    (64, 1, torch.bfloat16, torch.float32, True), (512, 2, torch.float32, torch.float32, True), (1000, 3, torch.bfloat16, torch.bfloat16, True),
    (1404, 2, torch.bfloat16, torch.float32, True), (2052, 2, torch.float32, torch.float32, True), (4100, 8, torch.bfloat16, torch.float32, True),
    (904, 9, torch.bfloat16, torch.float32, True), (2560, 4, torch.bfloat16, torch.float32, False),
    (9000, 2, torch.bfloat16, torch.float32, False), (264, 2, torch.float32, torch.bfloat16, True), (24584, 2, torch.bfloat16, torch.float32, False)])
@pytest.mark.parametrize("bits,offset,ef,per_matrix", [(4, False, True, False), (8, False, False, False), (2, True, False, False),
                                                       (8, True, True, False), (4, False, False, True), (4, True, True, True)])
def test_values_that_are_no_numbers(n, K, wd, gd, two, bits, offset, ef, per_matrix):
    m = 8
    v = _no_numbers(m, n, per_matrix)
    q, scale, lo, sent = _rule(v, bits, offset, per_matrix)
    codes = (diloco.pack_codes_unsigned if offset else diloco.pack_codes)(q, bits)
    ranges = scale.size
    groups = []
    for _ in range(2 if two else 1):
        like = lambda dt, *s: [torch.zeros(s, dtype=dt, device=DEV) for _ in range(K)]  # noqa: E731
        groups.append(mlc.OuterGroup(like(wd, 4, m, n), torch.from_numpy(v).to(DEV, gd), torch.zeros(4, m, n, device=DEV),
                                     like(torch.uint8, 4 * m, n * bits // 8), like(torch.float32, ranges),
                                     like(torch.float32, 4, m, n) if ef else None, None, None,
                                     like(torch.float32, ranges) if offset else None))
    hp = mlc.OuterHParams(K=K, eta_out=0.5, mu=0.0, quant_bits=bits, write_back=False, error_feedback=ef, ef_beta=1.0,
                          quant_offset=offset, quant_per_matrix=per_matrix)

    def check(g):
        with np.errstate(invalid="ignore"):
            left = v - sent
        for k in range(K):
            assert np.array_equal(g.codes[k].cpu().numpy(), codes), k
            assert np.array_equal(g.scales[k].cpu().numpy(), scale, equal_nan=True), k
            if offset:
                assert np.array_equal(g.offsets[k].cpu().numpy(), lo, equal_nan=True), k
            if ef:
                assert np.array_equal(g.residuals[k].cpu().numpy(), left, equal_nan=True), k
    alone = mlc.OuterGroup(**{f: getattr(groups[0], f) if f in ("worker_params", "global_param") else
                              [torch.zeros_like(t) for t in getattr(groups[0], f)] if getattr(groups[0], f) is not None else None
                              for f in ("worker_params", "global_param", "codes", "scales", "residuals", "offsets")},
                           outer_momentum=None)
    mlc.muloco_quantize_delta([alone], hp)                  # the compressor by itself
    check(alone)
    mlc.muloco_outer_step(groups, hp)
    for g in groups:
        check(g)
        # what all workers sent is the mean: finite where one value is
        u = g.outer_momentum.cpu().numpy()
        assert np.array_equal(np.isnan(u), np.isnan(sent)) and np.array_equal(np.isinf(u), np.isinf(sent))
