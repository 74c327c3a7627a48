"""GPU parity: muloco_topk_outer_step (C-ABI) against the oracle: thresholds and residuals bit
for bit, the outer update within the elementwise tolerances."""
import numpy as np
import pytest
import torch

import paper_2505_23725_amd as mlc
import synth_inputs as S
from oracle import diloco
from helpers import assert_fp32_close, assert_stored_close, to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(cnt, m, n, K, wdtype, gdtype, seed):
    tg = S.normal((cnt, m, n), S.PARAM_STD, seed, 0, dtype=gdtype)
    ws = [(tg.float() - S.normal((cnt, m, n), S.DELTA_STD, seed, 10 + k)).to(wdtype) for k in range(K)]
    u = S.normal((cnt, m, n), 1e-3, seed, 5, dtype=torch.float32)
    return tg, ws, u


CASES = [
    # cnt, m, n, K, worker dtype, global dtype, fraction, error feedback
    (2, 64, 128, 3, torch.bfloat16, torch.float32, 0.05, False),
    (1, 50, 1000, 2, torch.bfloat16, torch.float32, 0.005, True),
    (3, 33, 7, 2, torch.float32, torch.float32, 0.2, True),             # 231 elements: scalar path
    (2, 96, 200, 4, torch.bfloat16, torch.bfloat16, 0.1, False),        # coarse grid of deltas: many ties
    (2, 512, 2048, 2, torch.bfloat16, torch.float32, 0.01, True),
    (1, 128, 128, 1, torch.float32, torch.float32, 1.0, False),         # everything is kept
    (1, 128, 128, 2, torch.bfloat16, torch.float32, 1e-9, False),       # a single entry per matrix
    (1, 40, 64, 2, torch.float32, torch.bfloat16, 0.5, True),
]


@pytest.mark.parametrize("cnt,m,n,K,wd,gd,frac,ef", CASES)
def test_topk_outer_step_matches_oracle(cnt, m, n, K, wd, gd, frac, ef):
    seed = 17 * n + K
    tg0, ws0, u0 = _inputs(cnt, m, n, K, wd, gd, seed)
    tg, u = tg0.to(DEV), u0.to(DEV)
    ws = [w.to(DEV) for w in ws0]
    res0 = [S.normal((cnt, m, n), 2e-3, seed, 40 + k) for k in range(K)] if ef else None
    res = [r.to(DEV) for r in res0] if ef else None
    taus = [torch.full((cnt,), -1.0, dtype=torch.float32, device=DEV) for _ in range(K)]
    grp = mlc.OuterGroup(ws, tg, u, None, taus, res)
    hp = mlc.OuterHParams(K=K, eta_out=0.9, mu=0.8, error_feedback=ef, ef_beta=0.9)
    need = mlc.muloco_topk_workspace_bytes([grp], K)
    assert need == cnt * K * (2048 + 4) * 4     # a 2048-bin histogram and 4 words per (worker, matrix)
    wsp = torch.full((need,), 0xCD, dtype=torch.uint8, device=DEV)          # contents must not matter
    mlc.muloco_topk_outer_step([grp], hp, frac, wsp)
    torch.cuda.synchronize()
    ref = diloco.outer_step(to_f64(tg0).reshape(-1, n), to_f64(u0).reshape(-1, n),
                            [to_f64(w).reshape(-1, n) for w in ws0], eta_out=0.9, mu=0.8,
                            residuals=[r.numpy().reshape(-1, n) for r in res0] if ef else None, ef_beta=0.9,
                            topk_fraction=frac, rows_per_matrix=m)
    for k in range(K):
        assert np.array_equal(taus[k].cpu().numpy().view(np.uint32), ref["thresholds"][k].view(np.uint32)), \
            f"worker {k}: thresholds differ"
        if ef:
            assert np.array_equal(res[k].cpu().numpy().reshape(-1, n).view(np.uint32),
                                  ref["residuals"][k].view(np.uint32)), f"worker {k}: residuals differ"
    assert_fp32_close(u.cpu().reshape(-1, n), ref["u"], "outer momentum")
    assert_stored_close(tg.cpu().reshape(-1, n), ref["theta"], "global parameters")
    for k in range(K):
        assert torch.equal(ws[k].cpu(), tg.cpu().to(wd)), f"worker {k} write-back differs from theta_g"


def test_topk_second_call_reuses_the_workspace():
    cnt, m, n, K = 2, 64, 128, 2
    tg0, ws0, u0 = _inputs(cnt, m, n, K, torch.bfloat16, torch.float32, 5)
    hp = mlc.OuterHParams(K=K, eta_out=0.9, mu=0.8, write_back=False)
    grp0 = mlc.OuterGroup([w.to(DEV) for w in ws0], tg0.to(DEV), u0.to(DEV))
    wsp = torch.empty((mlc.muloco_topk_workspace_bytes([grp0], K),), dtype=torch.uint8, device=DEV)
    outs = []
    for _ in range(2):
        tg, u = tg0.to(DEV), u0.to(DEV)
        mlc.muloco_topk_outer_step([mlc.OuterGroup([w.to(DEV) for w in ws0], tg, u)], hp, 0.03, wsp)
        torch.cuda.synchronize()
        outs.append((tg.cpu(), u.cpu()))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


# sizes that no vector of 8 divides (shorter than one, one over, one short), with the residual
# holding v between the passes and without a residual
@pytest.mark.parametrize("cnt,m,n,K,wd,gd,frac,ef", [
    (3, 1, 5, 2, torch.bfloat16, torch.float32, 0.3, True),
    (2, 3, 3, 1, torch.float32, torch.float32, 0.5, False),
    (2, 77, 1001, 3, torch.bfloat16, torch.bfloat16, 0.05, True),
    (1, 411, 271, 2, torch.bfloat16, torch.float32, 0.02, False),
    (2, 511, 513, 1, torch.float32, torch.bfloat16, 0.01, True),
])
def test_topk_sizes_off_the_vector(cnt, m, n, K, wd, gd, frac, ef):
    test_topk_outer_step_matches_oracle(cnt, m, n, K, wd, gd, frac, ef)


@pytest.mark.parametrize("cnt,m,n,ef", [(2, 64, 64, True), (1, 77, 1001, False), (1, 3, 5, False), (1, 200, 333, True)])
@pytest.mark.parametrize("steps", [(1.0,), (1.0, 16.0), (1.0, 4.0, 64.0, 0.0), (1.0, 1.0, 1.0, 1.0, 1.0, 0.0)])
def test_topk_few_distinct_magnitudes(cnt, m, n, ef, steps):
    """Values whose first digits agree over most of a wavefront (counted together) or fall on two or
    more of them, in sizes that leave lanes idle: thresholds, residuals and update as the oracle."""
    gen = np.random.default_rng(m * n + len(steps))
    mag = np.float32(2.0 ** -8) * np.asarray(steps, np.float32)[gen.integers(0, len(steps), (cnt, m, n))]
    d = torch.from_numpy(mag * gen.choice(np.float32([-1, 1]), (cnt, m, n)))
    tg0 = torch.zeros(cnt, m, n)
    w0 = (tg0 - d).to(torch.bfloat16)           # powers of two: exact
    u0 = S.normal((cnt, m, n), 1e-3, 3, 5)
    tg, w, u = tg0.to(DEV), w0.to(DEV), u0.to(DEV)
    res0 = torch.zeros(cnt, m, n)
    res = res0.to(DEV)
    taus = [torch.full((cnt,), -1.0, device=DEV)]
    grp = mlc.OuterGroup([w], tg, u, None, taus, [res] if ef else None)
    hp = mlc.OuterHParams(K=1, eta_out=0.9, mu=0.8, error_feedback=ef, ef_beta=0.9)
    wsp = torch.empty(mlc.muloco_topk_workspace_bytes([grp], 1), dtype=torch.uint8, device=DEV)
    mlc.muloco_topk_outer_step([grp], hp, 0.3, wsp)
    torch.cuda.synchronize()
    ref = diloco.outer_step(to_f64(tg0).reshape(-1, n), to_f64(u0).reshape(-1, n), [to_f64(w0).reshape(-1, n)],
                            eta_out=0.9, mu=0.8, residuals=[res0.numpy().reshape(-1, n)] if ef else None,
                            ef_beta=0.9, topk_fraction=0.3, rows_per_matrix=m)
    assert np.array_equal(taus[0].cpu().numpy().view(np.uint32), ref["thresholds"][0].view(np.uint32))
    if ef:
        assert np.array_equal(res.cpu().numpy().reshape(-1, n).view(np.uint32), ref["residuals"][0].view(np.uint32))
    assert_fp32_close(u.cpu().reshape(-1, n), ref["u"], "outer momentum")


# Groups of about 4 M values (by the passes; test_topk_from_a_sample_of_larger_groups has those that start from a
# sample) off the vector, many workers, and values that a sample misjudges: `rare` puts the entries that are
# kept into one row, `grid` takes a few distinct magnitudes, `one` a single one.
@pytest.mark.parametrize("cnt,m,n,K,wd,gd,frac,ef,kind", [
    (1, 2048, 2048, 1, torch.bfloat16, torch.float32, 0.05, True, "normal"),
    (32, 256, 256, 2, torch.bfloat16, torch.float32, 0.005, True, "normal"),
    (70, 255, 257, 1, torch.float32, torch.float32, 0.1, False, "normal"),
    (5, 1001, 901, 1, torch.bfloat16, torch.float32, 0.2, True, "normal"),
    (1, 723, 727, 8, torch.bfloat16, torch.bfloat16, 0.02, False, "normal"),
    (1, 1449, 1451, 2, torch.float32, torch.bfloat16, 1.0, True, "normal"),
    (1, 1449, 1451, 2, torch.bfloat16, torch.float32, 1e-9, True, "normal"),
    (4, 1024, 1024, 1, torch.bfloat16, torch.float32, 0.0009, True, "rare"),
    (2, 1024, 1024, 2, torch.bfloat16, torch.float32, 0.05, True, "grid"),
    (2, 1024, 1024, 2, torch.bfloat16, torch.float32, 0.05, False, "one"),
])
def test_topk_from_a_sample(cnt, m, n, K, wd, gd, frac, ef, kind):
    gen = torch.Generator().manual_seed(m + n + K)
    deltas = [S.DELTA_STD * torch.randn(cnt, m, n, generator=gen) for _ in range(K)]
    tg0 = torch.zeros(cnt, m, n, dtype=gd)
    for d in deltas:
        if kind == "rare":
            d[:, 700] *= 1e3
        if kind in ("grid", "one"):
            d.copy_(d.sign() * torch.exp2(torch.randint(-9, -7 if kind == "grid" else -8, d.shape, generator=gen)))
    if kind == "normal":
        tg0 = (S.PARAM_STD * torch.randn(cnt, m, n, generator=gen)).to(gd)
    ws0 = [(tg0.float() - d).to(wd) for d in deltas]
    u0 = 1e-3 * torch.randn(cnt, m, n, generator=gen)
    scale = 0.0 if kind in ("grid", "one") else 2e-3
    res0 = [scale * torch.randn(cnt, m, n, generator=gen) for _ in range(K)] if ef else None
    tg, u, ws = tg0.to(DEV), u0.to(DEV), [w.to(DEV) for w in ws0]
    res = [r.to(DEV) for r in res0] if ef else None
    taus = [torch.full((cnt,), -1.0, device=DEV) for _ in range(K)]
    grp = mlc.OuterGroup(ws, tg, u, None, taus, res)
    hp = mlc.OuterHParams(K=K, eta_out=0.9, mu=0.8, error_feedback=ef, ef_beta=0.9)
    wsp = torch.full((mlc.muloco_topk_workspace_bytes([grp], K),), 0xCD, dtype=torch.uint8, device=DEV)
    mlc.muloco_topk_outer_step([grp], hp, frac, wsp)
    torch.cuda.synchronize()
    ref = diloco.outer_step(to_f64(tg0).reshape(-1, n), to_f64(u0).reshape(-1, n),
                            [to_f64(w).reshape(-1, n) for w in ws0], eta_out=0.9, mu=0.8,
                            residuals=[r.numpy().reshape(-1, n) for r in res0] if ef else None, ef_beta=0.9,
                            topk_fraction=frac, rows_per_matrix=m)
    for k in range(K):
        assert np.array_equal(taus[k].cpu().numpy().view(np.uint32), ref["thresholds"][k].view(np.uint32))
        if ef:
            assert np.array_equal(res[k].cpu().numpy().reshape(-1, n).view(np.uint32),
                                  ref["residuals"][k].view(np.uint32))
    assert_fp32_close(u.cpu().reshape(-1, n), ref["u"], "outer momentum")
    assert_stored_close(tg.cpu().reshape(-1, n), ref["theta"], "global parameters")
    for k in range(K):
        assert torch.equal(ws[k].cpu(), tg.cpu().to(wd))


def _sampled(elems):
    """Elements of a matrix that the sample for the window reads (topk_sample_kernel): the same for every matrix."""
    stretch, at = elems // 8 // 2048, []
    for r in range(2048):
        h = r * 2654435761 & 0xffffffff
        h = (h ^ h >> 15) * 2246822519 & 0xffffffff
        first = 8 * (r * stretch + (h * stretch >> 32))
        at.extend(range(first, first + 8))
    return torch.tensor(at, device=DEV)


def _misled(cnt, m, n, K, wd, gd, ef, open_, seed=1):
    """A group on the device of whose matrices those with open_(worker, matrix) mislead the sample."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    normal = lambda std: std * torch.randn(cnt, m, n, generator=gen, device=DEV)  # noqa: E731
    at = _sampled(m * n)
    tg, ws = normal(S.PARAM_STD).to(gd), []
    for k in range(K):
        d = normal(S.DELTA_STD)
        for i in range(cnt):
            if open_(k, i):
                d[i].view(-1)[at] *= 1e3 if i % 2 else 0.0
        ws.append((tg.float() - d).to(wd))
    taus = [torch.full((cnt,), -1.0, device=DEV) for _ in range(K)]
    return mlc.OuterGroup(ws, tg, normal(1e-3), None, taus, [normal(2e-3) for _ in range(K)] if ef else None)


def _clone(grp, pick=slice(None)):
    c = lambda ts: None if ts is None else [t[pick].clone() for t in ts]  # noqa: E731
    return mlc.OuterGroup(c(grp.worker_params), grp.global_param[pick].clone(), grp.outer_momentum[pick].clone(), None,
                          c(grp.scales), c(grp.residuals))


def _topk(groups, K, frac, ef):
    hp = mlc.OuterHParams(K=K, eta_out=0.9, mu=0.8, error_feedback=ef, ef_beta=0.9)
    wsp = torch.full((mlc.muloco_topk_workspace_bytes(groups, K),), 0xCD, dtype=torch.uint8, device=DEV)
    mlc.muloco_topk_outer_step(groups, hp, frac, wsp)


def _bytes(grp, K, ef, window):
    """What the recorder counts for a group, by its route."""
    w, g = (2 if t.dtype == torch.bfloat16 else 4 for t in (grp.worker_params[0], grp.global_param))
    values = K * (w + g)
    values = (values + 8 * K if ef else values) if window else (values + 16 * K if ef else 3 * values)
    return grp.global_param.numel() * (values + (8 * K if ef else K * w) + K * w + 2 * g + 8)


def _recorded(groups, K, frac, ef):
    mlc.muloco_timing_enable(True)
    try:
        mlc.muloco_timing_read()
        _topk(groups, K, frac, ef)
        torch.cuda.synchronize()
        return mlc.muloco_timing_read()["topk"]["bytes"]
    finally:
        mlc.muloco_timing_enable(False)


def _together_and_alone(grp, K, frac, ef):
    """The matrices of a group that starts from a sample, also one by one, which take the passes."""
    alone = [_clone(grp, slice(i, i + 1)) for i in range(grp.global_param.shape[0])]
    assert _recorded([grp], K, frac, ef) == _bytes(grp, K, ef, True)
    assert _recorded(alone, K, frac, ef) == sum(_bytes(a, K, ef, False) for a in alone)
    return alone


# Groups of which the window leaves some matrices open (one of them, the first, the last, some of more than are listed at a time,
# those of one worker, all), or whose ties do: the same bits as matrix by matrix.
@pytest.mark.parametrize("cnt,m,n,K,wd,gd,frac,ef,which", [
    (8, 1024, 1024, 1, torch.bfloat16, torch.float32, 0.05, True, "one"),
    (300, 512, 512, 1, torch.bfloat16, torch.float32, 0.05, True, "some"),
    (300, 300, 301, 2, torch.bfloat16, torch.float32, 0.05, False, "first"),
    (260, 256, 256, 3, torch.bfloat16, torch.float32, 0.05, True, "last"),
    (12, 513, 517, 3, torch.float32, torch.float32, 0.1, False, "worker"),
    (9, 768, 768, 2, torch.bfloat16, torch.bfloat16, 0.02, False, "all"),
    (4, 1000, 1001, 3, torch.bfloat16, torch.float32, 0.3, True, "all"),
    (12, 1024, 2048, 1, torch.bfloat16, torch.bfloat16, 0.05, False, "ties"),
])
def test_topk_matrices_that_the_window_leaves_open(cnt, m, n, K, wd, gd, frac, ef, which):
    grp = _misled(cnt, m, n, K, wd, gd, ef, lambda k, i: {"one": i == cnt // 2, "first": i == 0, "last": i == cnt - 1, "some": i % 7 == 3, "all": True,
                                                          "worker": k == 1, "ties": False}[which])
    alone = _together_and_alone(grp, K, frac, ef)
    for k in range(K):
        assert torch.equal(grp.scales[k], torch.cat([a.scales[k] for a in alone])), k
        assert torch.equal(grp.worker_params[k], torch.cat([a.worker_params[k] for a in alone])), k
        if ef:
            assert torch.equal(grp.residuals[k], torch.cat([a.residuals[k] for a in alone])), k
    assert torch.equal(grp.global_param, torch.cat([a.global_param for a in alone]))
    assert torch.equal(grp.outer_momentum, torch.cat([a.outer_momentum for a in alone]))


def test_topk_open_matrices_have_the_whole_chip():
    """Three further passes cost at most 12 of 40 bytes an element: a sample that misleads about every matrix takes less
    than half as long again (with a fixed share of a small grid for every matrix 1.9 times as long)."""
    us = {}
    for name in ("settled", "open"):
        first = _misled(6, 2048, 2048, 8, torch.bfloat16, torch.float32, True, lambda k, i: name == "open")
        times = []
        for _ in range(7):
            grp = _clone(first)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            _topk([grp], 8, 0.05, True)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        us[name] = sorted(times)[2]
    assert us["open"] < 1.5 * us["settled"], us


# On either side of the lines of the rule for the window: matrices of few values, few matrices, many workers, ties, one large matrix.
@pytest.mark.parametrize("cnt,m,n,K,wd,gd,ef,window", [
    (400, 256, 256, 1, torch.bfloat16, torch.float32, True, True), (400, 255, 256, 1, torch.bfloat16, torch.float32, True, False),
    (16, 512, 512, 1, torch.bfloat16, torch.float32, True, True), (15, 512, 512, 1, torch.bfloat16, torch.float32, True, False),
    (4, 1024, 1024, 1, torch.bfloat16, torch.float32, True, False), (8, 1024, 1024, 1, torch.bfloat16, torch.float32, True, True),
    (1, 1024, 1024, 8, torch.bfloat16, torch.float32, True, True), (1, 1024, 1024, 8, torch.bfloat16, torch.float32, False, False),
    (2, 1024, 1024, 8, torch.bfloat16, torch.float32, False, True), (2, 1536, 1536, 2, torch.bfloat16, torch.float32, False, False),
    (8, 1024, 1024, 1, torch.bfloat16, torch.bfloat16, False, True), (6, 1024, 1024, 1, torch.bfloat16, torch.bfloat16, False, False),
    (1, 2560, 2560, 1, torch.bfloat16, torch.float32, True, True), (1, 2048, 2560, 1, torch.float32, torch.float32, True, False),
])
def test_topk_route_by_size(cnt, m, n, K, wd, gd, ef, window):
    grp = _misled(cnt, m, n, K, wd, gd, ef, lambda k, i: False)
    some = slice(0, cnt, max(1, cnt // 5))
    alone = [_clone(grp, slice(i, i + 1)) for i in range(cnt)[some]]
    assert _recorded([grp], K, 0.05, ef) == _bytes(grp, K, ef, window)
    _topk(alone, K, 0.05, ef)
    for k in range(K):
        assert torch.equal(grp.scales[k][some], torch.cat([a.scales[k] for a in alone])), k
    assert torch.equal(grp.global_param[some], torch.cat([a.global_param for a in alone]))


# The cases of test_topk_from_a_sample in groups that do start from one
@pytest.mark.parametrize("cnt,m,n,K,wd,gd,frac,ef,kind", [
    (1, 2560, 2560, 1, torch.bfloat16, torch.float32, 0.05, True, "normal"),
    (64, 300, 300, 2, torch.bfloat16, torch.float32, 0.005, True, "normal"),
    (90, 313, 315, 1, torch.float32, torch.float32, 0.1, False, "normal"),
    (9, 1001, 901, 1, torch.bfloat16, torch.float32, 0.2, True, "normal"),
    (3, 723, 727, 8, torch.bfloat16, torch.bfloat16, 0.02, False, "normal"),
    (2, 1449, 1451, 4, torch.float32, torch.bfloat16, 1.0, True, "normal"),
    (2, 1449, 1451, 4, torch.bfloat16, torch.float32, 1e-9, True, "normal"),
    (9, 1024, 1024, 1, torch.bfloat16, torch.float32, 0.0009, True, "rare"),
    (4, 1024, 1024, 3, torch.bfloat16, torch.float32, 0.05, True, "grid"),
    (6, 1024, 1024, 2, torch.bfloat16, torch.float32, 0.05, False, "one"),
])
def test_topk_from_a_sample_of_larger_groups(cnt, m, n, K, wd, gd, frac, ef, kind):
    grp = _misled(cnt, m, n, K, wd, gd, ef, lambda k, i: False)
    assert _recorded([grp], K, frac, ef) == _bytes(grp, K, ef, True)
    test_topk_from_a_sample(cnt, m, n, K, wd, gd, frac, ef, kind)


# Not-a-numbers and infinities compare by their bit patterns, above every number: in groups that start from a sample as in
# those that take the passes.
@pytest.mark.parametrize("cnt,m,n,K,wd,gd,frac,ef,every", [
    (9, 1024, 1024, 1, torch.bfloat16, torch.float32, 0.05, True, (100003, 70001)),    # few: all of them are sent
    (6, 1000, 1001, 2, torch.float32, torch.float32, 0.01, False, (64, 31)),            # more than are sent: the threshold is one
    (12, 1024, 2048, 1, torch.bfloat16, torch.bfloat16, 0.3, True, (0, 3)),              # infinities tie
])
def test_topk_not_a_number_from_a_sample(cnt, m, n, K, wd, gd, frac, ef, every):
    grp = _misled(cnt, m, n, K, wd, gd, ef, lambda k, i: False)
    for w in grp.worker_params:
        if every[0]:
            w.view(-1)[::every[0]] = float("nan")
        w.view(-1)[5::every[1]] = float("inf")
        w.view(-1)[6::2 * every[1]] = -float("inf")
    alone = _together_and_alone(grp, K, frac, ef)
    bits = lambda t: t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)  # noqa: E731
    for k in range(K):
        assert torch.equal(bits(grp.scales[k]), bits(torch.cat([a.scales[k] for a in alone]))), k
        if ef:
            assert torch.equal(bits(grp.residuals[k]), bits(torch.cat([a.residuals[k] for a in alone]))), k
    for got, ref in [(grp.global_param, [a.global_param for a in alone]), (grp.outer_momentum, [a.outer_momentum for a in alone])]:
        ref = torch.cat(ref)
        assert torch.equal(torch.isnan(got), torch.isnan(ref))
        assert torch.equal(bits(torch.nan_to_num(got)), bits(torch.nan_to_num(ref)))


# Matrices too large for the window's bins (67 M values, 20 %: some 2000 in the bin of the threshold), against the oracle's rule
# on the device: the k-th largest magnitude, and everything from it on sent.
def test_topk_matrix_too_large_to_settle():
    gen = torch.Generator(device=DEV).manual_seed(3)
    m, n, frac = 4096, 16384, 0.2
    tg0 = S.PARAM_STD * torch.randn(1, m, n, generator=gen, device=DEV)
    w0 = (tg0 - S.DELTA_STD * torch.randn(1, m, n, generator=gen, device=DEV)).bfloat16()
    e0 = 2e-3 * torch.randn(1, m, n, generator=gen, device=DEV)
    u0 = 1e-3 * torch.randn(1, m, n, generator=gen, device=DEV)
    grp = mlc.OuterGroup([w0.clone()], tg0.clone(), u0.clone(), None, [torch.zeros(1, device=DEV)], [e0.clone()])
    _topk([grp], 1, frac, True)
    v = 0.9 * e0 + (tg0 - w0.float())        # rounded after the product and after each sum, as in the kernel
    k = -(-m * n * 2 // 10)
    tau = v.abs().view(-1).kthvalue(m * n - k + 1).values
    assert torch.equal(grp.scales[0], tau.view(1))
    sent = v.abs() >= tau
    assert torch.equal(grp.residuals[0], torch.where(sent, torch.zeros_like(v), v))
    u1 = 0.8 * u0.double() + 0.9 * torch.where(sent, v, torch.zeros_like(v)).double()
    assert ((grp.outer_momentum.double() - u1).norm() / u1.norm()).item() < 1e-5


def _terabytes_per_second(first, K, frac, ef):
    """Recorded bytes of a call over its median time."""
    rates = []
    mlc.muloco_timing_enable(True)
    try:
        for _ in range(7):
            grp = _clone(first)
            torch.cuda.synchronize()
            mlc.muloco_timing_read()
            _topk([grp], K, frac, ef)
            torch.cuda.synchronize()
            t = mlc.muloco_timing_read()["topk"]
            rates.append(t["bytes"] / t["total_ms"] * 1e-9)
    finally:
        mlc.muloco_timing_enable(False)
    return sorted(rates)[3]


def test_topk_many_small_matrices_run_at_memory_speed():
    """4000 matrices of 128 x 128, four workers: 4.2 of the 5 TB/s that a stream reaches.  (Where the last workgroup
    of every state picked the digit, all 128000 took a ticket and waited for it: 2.3.)"""
    grp = _misled(4000, 128, 128, 4, torch.bfloat16, torch.float32, True, lambda k, i: False)
    assert _terabytes_per_second(grp, 4, 0.05, True) > 3.0


# as many workgroups a pass as the last picks among, and more
@pytest.mark.parametrize("cnt,m,n,K", [(88, 128, 128, 1), (89, 128, 128, 1), (4, 1024, 512, 1), (2, 1024, 513, 2), (5, 1024, 512, 1), (705, 8, 16, 1)])
@pytest.mark.parametrize("ef", [False, True])
def test_topk_digits_picked_last_and_in_launches(cnt, m, n, K, ef):
    test_topk_outer_step_matches_oracle(cnt, m, n, K, torch.bfloat16, torch.float32, 0.03, ef)


def _crowded(cnt, m, n, K, wd, gd, ef, seed=5):
    """Values of which a tenth lies close about one magnitude, the threshold's at 5 %: long lists."""
    grp = _misled(cnt, m, n, K, wd, gd, ef, lambda k, i: False, seed)
    gen = torch.Generator(device=DEV).manual_seed(seed + 1)
    for k in range(K):
        d = 1e-3 * torch.randn(cnt, m, n, generator=gen, device=DEV)
        at = torch.rand(cnt, m, n, generator=gen, device=DEV) < 0.1
        d[at] = (0.02 + 2e-4 * torch.randn(int(at.sum()), generator=gen, device=DEV)) * torch.sign(d[at])
        if ef:
            grp.residuals[k].zero_()
        grp.worker_params[k].copy_(grp.global_param.float() - d)
    return grp


# Lists of many entries and of many workers, elements that several workers' lists hold, more matrices than
# workgroups for them: the same bits as matrix by matrix.
@pytest.mark.parametrize("cnt,m,n,K,wd,gd,ef", [
    (17, 1024, 1024, 3, torch.float32, torch.float32, False), (9, 768, 768, 6, torch.float32, torch.float32, True),
    (150, 300, 300, 3, torch.float32, torch.bfloat16, True), (7, 500, 1001, 8, torch.bfloat16, torch.float32, True),
    (40, 257, 1023, 7, torch.bfloat16, torch.bfloat16, False),
])
def test_topk_long_lists(cnt, m, n, K, wd, gd, ef):
    grp = _crowded(cnt, m, n, K, wd, gd, ef)
    alone = _together_and_alone(grp, K, 0.05, ef)
    for k in range(K):
        assert torch.equal(grp.scales[k], torch.cat([a.scales[k] for a in alone])), k
        assert torch.equal(grp.worker_params[k], torch.cat([a.worker_params[k] for a in alone])), k
        if ef:
            assert torch.equal(grp.residuals[k], torch.cat([a.residuals[k] for a in alone])), k
    assert torch.equal(grp.global_param, torch.cat([a.global_param for a in alone]))
    assert torch.equal(grp.outer_momentum, torch.cat([a.outer_momentum for a in alone]))


def test_topk_long_lists_do_not_hold_a_call_up():
    """768 x 3072, sixteen bf16 workers of a bf16 global copy, whose ties make lists of hundreds: 2 TB/s of the recorded bytes
    (0.7 when one workgroup settled all of them)."""
    grp = _misled(1, 768, 3072, 16, torch.bfloat16, torch.bfloat16, False, lambda k, i: False)
    assert _terabytes_per_second(grp, 16, 0.05, False) > 1.3


# Two groups of equally large matrices share launches where the work space holds the states of both (here a third group's), and give
# the bits of a call each: by the passes, from a sample, with odd sizes, and where the pass of the window takes the workers in turn
# (both groups past the memory-side cache).  Groups that share memory, of other sizes or types, or whose states do not fit, follow
# each other.
@pytest.mark.parametrize("c0,c1,m,n,K,wd,gd,ef,together", [
    (2, 1, 64, 128, 3, torch.bfloat16, torch.float32, True, True),
    (1, 3, 33, 7, 2, torch.float32, torch.float32, False, True),
    (5, 3, 512, 1024, 2, torch.bfloat16, torch.bfloat16, True, True),
    (2, 2, 2048, 4096, 2, torch.bfloat16, torch.float32, True, True),
    (2, 2, 1449, 1451, 8, torch.bfloat16, torch.float32, False, True),
    (40, 40, 313, 315, 3, torch.float32, torch.float32, True, True),
    (3, 3, 1811, 1813, 2, torch.bfloat16, torch.float32, True, True),           # in turn, element by element
    (2, 2, 64, 128, 2, torch.bfloat16, torch.float32, True, "shared memory"),
    (2, 2, 64, 128, 2, torch.bfloat16, torch.float32, True, "states"),
    (2, 2, 64, 128, 2, torch.bfloat16, torch.float32, False, "size"),
    (2, 2, 64, 128, 2, torch.bfloat16, torch.float32, False, "type"),
])
def test_topk_groups_of_equal_matrices_share_launches(c0, c1, m, n, K, wd, gd, ef, together):
    quiet = lambda k, i: False  # noqa: E731
    first = _misled(c0, m, n, K, wd, gd, ef, quiet)
    second = _misled(c1, n, m + (together == "size"), K, wd, torch.bfloat16 if together == "type" else gd, ef, quiet)
    for t in second.worker_params:                                  # not the first group's values over again
        t.mul_(1.01)
    if together == "shared memory":
        first.residuals, second.residuals = ([t for t in first.residuals],
                                             [t.reshape(c1, n, m) for t in first.residuals])
    groups = [first, second]
    if together != "states":
        groups.append(_misled(c0 + c1, 16, 24, K, wd, gd, ef, quiet))
    shared = _clone(first), _clone(second)
    if together == "shared memory":
        shared[1].residuals = [t.reshape(c1, n, m) for t in shared[0].residuals]
    for grp in shared:
        _topk([grp], K, 0.05, ef)
    mlc.muloco_timing_enable(True)
    try:
        mlc.muloco_timing_read()
        _topk(groups, K, 0.05, ef)
        torch.cuda.synchronize()
        assert mlc.muloco_timing_read()["topk"]["launches"] == len(groups) - (together is True)
    finally:
        mlc.muloco_timing_enable(False)
    for got, want in zip(groups, shared):
        assert torch.equal(got.global_param, want.global_param) and torch.equal(got.outer_momentum, want.outer_momentum)
        for k in range(K):
            assert torch.equal(got.scales[k], want.scales[k]) and torch.equal(got.worker_params[k], want.worker_params[k])
            assert not ef or torch.equal(got.residuals[k], want.residuals[k])


def test_topk_pair_shares_launches_in_a_work_space_for_both():
    """Two groups and nothing else: the query's bytes serve them one after the other, those of one group with the matrices of
    both together, the same bits."""
    K, first = 2, _misled(2, 64, 128, 2, torch.bfloat16, torch.float32, True, lambda k, i: False)
    second = _misled(3, 128, 64, K, torch.bfloat16, torch.float32, True, lambda k, i: False)
    whole = mlc.OuterGroup([torch.cat([a.flatten(1), b.flatten(1)]).view(5, 64, 128) for a, b in
                            zip(first.worker_params, second.worker_params)], torch.empty(5, 64, 128, device=DEV), None)
    least = mlc.muloco_topk_workspace_bytes([first, second], K)
    both = mlc.muloco_topk_workspace_bytes([whole], K)
    assert both == least // 3 * 5
    hp = mlc.OuterHParams(K=K, eta_out=0.9, mu=0.8, error_feedback=True, ef_beta=0.9)
    done = []
    for size, launches in ((least, 2), (both - 1, 2), (both, 1)):
        groups = [_clone(first), _clone(second)]
        mlc.muloco_timing_enable(True)
        try:
            mlc.muloco_timing_read()
            mlc.muloco_topk_outer_step(groups, hp, 0.05, torch.full((size,), 0xCD, dtype=torch.uint8, device=DEV))
            torch.cuda.synchronize()
            assert mlc.muloco_timing_read()["topk"]["launches"] == launches
        finally:
            mlc.muloco_timing_enable(False)
        done.append([t for g in groups for t in [g.global_param, g.outer_momentum, *g.worker_params, *g.scales, *g.residuals]])
    for other in done[1:]:
        assert all(torch.equal(a, b) for a, b in zip(done[0], other))
