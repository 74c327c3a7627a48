"""GPU parity: muloco_inner_step (C-ABI) against the fp64 oracle on seeded inputs."""
import math

import numpy as np
import pytest
import torch

import paper_2505_23725_amd as mlc
import synth_inputs as S
from oracle import muon, storage
from helpers import (EW_TOL, NS_TOL, assert_fp32_close, assert_update_elements, dtype_name, ns_tiles, rel_fro,
                     to_f64, update_error_bf16)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _make_group(cnt, m, n, pdtype, gdtype, seed, zero_momentum=False):
    W = S.normal((cnt, m, n), S.PARAM_STD, seed, 1, dtype=pdtype)
    g = S.normal((cnt, m, n), S.GRAD_STD, seed, 2, dtype=gdtype)
    mom = S.normal((cnt, m, n), 3 * S.GRAD_STD, seed, 3, dtype=torch.float32)
    if zero_momentum:
        mom.zero_()
    return W, g, mom


def _oracle_group(W, g, mom, hp: mlc.MuonHParams, lr_scale):
    Wn, mn, On = [], [], []
    for i in range(W.shape[0]):
        w1, m1, o1 = muon.inner_step(to_f64(W[i]), to_f64(mom[i]), to_f64(g[i]), eta=hp.eta,
                                     weight_decay=hp.weight_decay, beta=hp.beta, nesterov=hp.nesterov,
                                     ns_iters=hp.ns_iters, coeffs=(hp.ns_a, hp.ns_b, hp.ns_c),
                                     eps=hp.ns_eps, lr_scale=lr_scale)
        Wn.append(w1); mn.append(m1); On.append(o1)
    return np.stack(Wn), np.stack(mn), np.stack(On)


def _check_group(W0, g, mom0, W1, mom1, hp, lr_scale, what):
    Wr, mr, Or = _oracle_group(W0, g, mom0, hp, lr_scale)
    assert_fp32_close(mom1, mr, f"{what}: momentum")
    W0f, W1f = to_f64(W0), to_f64(W1)
    for i in range(W0.shape[0]):
        # compare the update, never the weights (the weights would hide any error); for
        # bf16-stored weights the storage rounding is removed in quadrature
        if W1.dtype == torch.bfloat16:
            err = update_error_bf16(W1[i], W0f[i], Wr[i])
        else:
            err = rel_fro(W1f[i] - W0f[i], Wr[i] - W0f[i])
        assert err <= NS_TOL, f"{what}: matrix {i} update error {err:.3e}"
        assert_update_elements(W1[i], Wr[i], Or[i], hp.eta * lr_scale, f"{what}: matrix {i}")


CASES = [
    # cnt, m, n, param dtype, grad dtype
    (2, 128, 128, torch.float32, torch.float32),
    (2, 128, 512, torch.float32, torch.float32),
    (2, 512, 128, torch.float32, torch.float32),
    (3, 100, 380, torch.bfloat16, torch.float32),      # ragged, one-launch path, L = 384
    (2, 128, 640, torch.bfloat16, torch.bfloat16),      # short side 128, too long for that path
    (3, 256, 384, torch.bfloat16, torch.bfloat16),
    (2, 200, 136, torch.bfloat16, torch.float32),
    (1, 333, 77, torch.float32, torch.bfloat16),
    (2, 768, 768, torch.bfloat16, torch.bfloat16),
    # bf16 weights of a shape the products work on unpadded: the last product writes the update
    (2, 768, 3072, torch.bfloat16, torch.bfloat16),
    (2, 3072, 768, torch.bfloat16, torch.float32),
    (70, 256, 512, torch.bfloat16, torch.bfloat16),    # its apply products run the 256 x 256 tile
]


@pytest.mark.parametrize("cnt,m,n,pd,gd", CASES)
@pytest.mark.parametrize("nesterov", [True, False])
def test_inner_step_matches_oracle(cnt, m, n, pd, gd, nesterov):
    hp = mlc.MuonHParams(eta=6.25e-2, weight_decay=1.25e-3, beta=0.95, nesterov=nesterov)
    lr_scale = math.sqrt(n / m)
    W0, g, mom0 = _make_group(cnt, m, n, pd, gd, seed=m + n)
    W, gg, mom = W0.to(DEV), g.to(DEV), mom0.to(DEV)
    grp = mlc.InnerGroup(W, gg, mom, lr_scale)
    ws = torch.empty(mlc.muloco_inner_workspace_bytes([grp]), dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step([grp], hp, ws)
    torch.cuda.synchronize()
    assert torch.equal(gg.cpu().view(torch.int16 if gd == torch.bfloat16 else torch.int32),
                       g.view(torch.int16 if gd == torch.bfloat16 else torch.int32)), "gradient was modified"
    _check_group(W0, g, mom0, W.cpu(), mom.cpu(), hp, lr_scale, f"{cnt}x{m}x{n} {dtype_name(W0)}")


# rows that end in a part of a vector: shorter than one, one element over or short of a multiple
# of 8, wide and tall (stored transposed), each combination of stored types
TAIL_CASES = [
    (2, 130, 5, torch.bfloat16, torch.bfloat16),
    (1, 5, 1, torch.float32, torch.float32),
    (2, 257, 129, torch.float32, torch.bfloat16),
    (2, 140, 641, torch.bfloat16, torch.float32),
    (1, 647, 263, torch.bfloat16, torch.bfloat16),
]


@pytest.mark.parametrize("cnt,m,n,pd,gd", TAIL_CASES)
def test_ragged_row_tails_match_oracle(cnt, m, n, pd, gd):
    test_inner_step_matches_oracle(cnt, m, n, pd, gd, True)



def test_several_groups_one_call_and_small_work_space():
    hp = mlc.MuonHParams(eta=0.05, weight_decay=0.01, beta=0.9)
    shapes = [(4, 128, 128), (2, 128, 512), (2, 512, 128)]
    host, dev = [], []
    for i, (c, m, n) in enumerate(shapes):
        W0, g, m0 = _make_group(c, m, n, torch.bfloat16, torch.bfloat16, seed=10 + i)
        host.append((W0, g, m0))
        dev.append(mlc.InnerGroup(W0.to(DEV), g.to(DEV), m0.to(DEV), math.sqrt(n / m)))
    ws = torch.empty(mlc.muloco_inner_workspace_min_bytes(dev), dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step(dev, hp, ws)
    torch.cuda.synchronize()
    for (W0, g, m0), grp, (c, m, n) in zip(host, dev, shapes):
        _check_group(W0, g, m0, grp.param.cpu(), grp.momentum.cpu(), hp, math.sqrt(n / m), f"group {m}x{n}")


def test_zero_gradient_decays_bf16_weights_through_the_last_product():
    hp = mlc.MuonHParams(eta=0.1, weight_decay=0.05, beta=0.9)
    W0 = S.normal((2, 256, 640), S.PARAM_STD, 0, 8, dtype=torch.bfloat16)
    W = W0.to(DEV)
    g = torch.zeros_like(W)
    mom = torch.zeros((2, 256, 640), dtype=torch.float32, device=DEV)
    grp = mlc.InnerGroup(W, g, mom, 1.0)
    ws = torch.empty(mlc.muloco_inner_workspace_bytes([grp]), dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step([grp], hp, ws)
    torch.cuda.synchronize()
    ref = storage.round_to_storage(to_f64(W0) * np.float64(np.float32(1) - np.float32(0.1) * np.float32(0.05)), "bf16")
    got = to_f64(W.cpu())
    # one bf16 rounding of decay * W: equal up to the fp32 product's own rounding before it
    assert np.max(np.abs(got - ref) / np.maximum(np.abs(ref), 1e-30)) <= 2.0 ** -7
    assert np.mean(got != ref) < 1e-3


def test_zero_gradient_and_momentum_only_decays():
    hp = mlc.MuonHParams(eta=0.1, weight_decay=0.05, beta=0.9)
    W0 = S.normal((1, 128, 256), S.PARAM_STD, 0, 7, dtype=torch.float32)
    W = W0.to(DEV)
    g = torch.zeros_like(W)
    mom = torch.zeros_like(W)
    grp = mlc.InnerGroup(W, g, mom, 1.0)
    ws = torch.empty(mlc.muloco_inner_workspace_bytes([grp]), dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step([grp], hp, ws)
    torch.cuda.synchronize()
    ref = to_f64(W0) * (1 - 0.1 * 0.05)
    assert_fp32_close(W.cpu(), ref, "decay only")
    assert torch.count_nonzero(mom) == 0


def test_zero_iterations_uses_normalised_direction():
    hp = mlc.MuonHParams(eta=0.1, weight_decay=0.0, beta=0.5, ns_iters=0)
    W0, g, m0 = _make_group(1, 128, 128, torch.float32, torch.float32, seed=77)
    grp = mlc.InnerGroup(W0.to(DEV), g.to(DEV), m0.to(DEV), 1.0)
    ws = torch.empty(mlc.muloco_inner_workspace_bytes([grp]), dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step([grp], hp, ws)
    torch.cuda.synchronize()
    Wr, mr, _ = _oracle_group(W0, g, m0, hp, 1.0)
    upd = to_f64(grp.param.cpu()) - to_f64(W0)
    assert rel_fro(upd, Wr - to_f64(W0)) <= 4e-3      # bf16 rounding of the direction only


# (groups of one call, their tiles for the Gram, polynomial and apply products when side by side)
SIDE_BY_SIDE = [
    # 150M-like proportions, scaled down: the Gram products of the wide and the tall group share a
    # launch (depth 1024; the tall one is held transposed), all three polynomial products share one,
    # and the three apply products (depth 256) share one
    ([(230, 256, 256), (130, 256, 1024), (130, 1024, 256)], [(256, 128, 256), (128, 128, 256), (128, 128, 256)]),
    # two groups of one shape and a group whose width 256 does not divide: only some products can share
    ([(50, 512, 512), (50, 512, 512), (3, 384, 640)], [(128, 128, 256), (128, 128, 256), (64, 64, 64)]),
    # a group that takes the one-workgroup chain beside two that do not
    ([(9, 128, 512), (140, 256, 512), (140, 512, 256)], [None, (128, 128, 256), (128, 128, 256)]),
    # large tiles throughout
    ([(40, 768, 768), (30, 768, 768)], [(256, 256, 256)] * 2),
]


@pytest.mark.parametrize("shapes,tiles", SIDE_BY_SIDE)
def test_groups_side_by_side_give_the_bits_of_one_group_after_the_other(shapes, tiles):
    """With a work space that holds all groups at once, products of several groups share launches;
    with the smaller one each group runs alone.  Both must give the same bits, and one group
    of each call is checked against the oracle."""
    assert ns_tiles(shapes) == tiles
    hp = mlc.MuonHParams(eta=0.05, weight_decay=0.01, beta=0.9)

    def build():
        out = []
        for i, (c, m, n) in enumerate(shapes):
            W0, g, m0 = _make_group(c, m, n, torch.bfloat16, torch.bfloat16, seed=40 + i)
            out.append((W0, g, m0, mlc.InnerGroup(W0.to(DEV), g.to(DEV), m0.to(DEV), math.sqrt(n / m))))
        return out

    both, alone = build(), build()
    groups = [t[3] for t in both]
    full = mlc.muloco_inner_workspace_bytes(groups)
    one = max(mlc.newton_schulz_workspace_bytes(c, m, n) for (c, m, n) in shapes)
    assert full > one
    ws = torch.empty(full, dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step(groups, hp, ws)
    mlc.muloco_inner_step([t[3] for t in alone], hp, ws[:one])
    torch.cuda.synchronize()
    for a, b in zip(both, alone):
        assert torch.equal(a[3].param.view(torch.int16), b[3].param.view(torch.int16))
        assert torch.equal(a[3].momentum.view(torch.int32), b[3].momentum.view(torch.int32))
    for (W0, g, m0, grp), (c, m, n) in zip(both, shapes):
        sl = slice(c - 1, c)        # the last matrix of every group
        _check_group(W0[sl], g[sl], m0[sl], grp.param[sl].cpu(), grp.momentum[sl].cpu(), hp, math.sqrt(n / m),
                     f"group {m}x{n}")


# bf16 weights of few, unpadded matrices: the last product writes the update from 64 x 64 tiles,
# transposed for the tall ones
SMALL_TILE_UPDATES = [
    ([(1, 384, 256)], [(64, 64, 64)]),
    ([(4, 256, 256), (1, 256, 1024), (1, 1024, 256)], [(64, 64, 64)] * 3),
    ([(1, 640, 384), (1, 384, 640)], [(64, 64, 64)] * 2),
]


@pytest.mark.parametrize("shapes,tiles", SMALL_TILE_UPDATES)
def test_update_from_small_tiles(shapes, tiles):
    assert ns_tiles(shapes) == tiles
    hp = mlc.MuonHParams(eta=6.25e-2, weight_decay=1.25e-3, beta=0.9)
    host = [_make_group(c, m, n, torch.bfloat16, torch.bfloat16, seed=90 + i) for i, (c, m, n) in enumerate(shapes)]
    grps = [mlc.InnerGroup(*[t.to(DEV) for t in h], math.sqrt(n / m)) for h, (_, m, n) in zip(host, shapes)]
    ws = torch.empty(mlc.muloco_inner_workspace_bytes(grps), dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step(grps, hp, ws)
    torch.cuda.synchronize()
    for (W0, g, m0), grp, (c, m, n) in zip(host, grps, shapes):
        _check_group(W0, g, m0, grp.param.cpu(), grp.momentum.cpu(), hp, math.sqrt(n / m), f"group {c}x{m}x{n}")


def test_groups_of_different_kinds_side_by_side():
    """One call over groups that take different routes: bf16 weights of an unpadded shape (the
    last product writes the update), fp32 weights (separate update pass), a ragged bf16 shape
    (padded work space, separate pass) and small matrices (one-launch chain).  Same bits as one
    group per call with the small work space, and every group against the oracle."""
    hp = mlc.MuonHParams(eta=0.05, weight_decay=0.01, beta=0.9)
    kinds = [(40, 256, 512, torch.bfloat16), (40, 512, 256, torch.float32), (3, 200, 520, torch.bfloat16),
             (5, 128, 256, torch.bfloat16)]

    def build():
        out = []
        for i, (c, m, n, pd) in enumerate(kinds):
            W0, g, m0 = _make_group(c, m, n, pd, torch.bfloat16, seed=70 + i)
            out.append((W0, g, m0, mlc.InnerGroup(W0.to(DEV), g.to(DEV), m0.to(DEV), math.sqrt(n / m))))
        return out

    both, alone = build(), build()
    groups = [t[3] for t in both]
    ws = torch.empty(mlc.muloco_inner_workspace_bytes(groups), dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step(groups, hp, ws)
    for t in alone:
        small = torch.empty(mlc.muloco_inner_workspace_min_bytes([t[3]]), dtype=torch.uint8, device=DEV)
        mlc.muloco_inner_step([t[3]], hp, small)
    torch.cuda.synchronize()
    for a, b, (c, m, n, pd) in zip(both, alone, kinds):
        bits = torch.int16 if pd == torch.bfloat16 else torch.int32
        assert torch.equal(a[3].param.view(bits), b[3].param.view(bits)), f"{m}x{n}: weights differ"
        assert torch.equal(a[3].momentum.view(torch.int32), b[3].momentum.view(torch.int32))
    for (W0, g, m0, grp), (c, m, n, pd) in zip(both, kinds):
        sl = slice(c - 2, c)
        _check_group(W0[sl], g[sl], m0[sl], grp.param[sl].cpu(), grp.momentum[sl].cpu(), hp, math.sqrt(n / m),
                     f"group {m}x{n} {dtype_name(W0)}")


@pytest.mark.parametrize("counts", [(3, 1, 2, 5), (200, 40, 10, 6), (250, 30, 1, 1)])
def test_small_batches_side_by_side_equal_one_call_each(counts):
    """Shapes of the one-workgroup chain in one call: their batches share a launch while all matrices
    fit the chip at once (256), and go one after the other beyond."""
    shapes = [(128, 128), (100, 250), (512, 128), (128, 384)]
    hp = mlc.MuonHParams(eta=6.25e-2, weight_decay=1.25e-3)

    def groups():
        return [mlc.InnerGroup(*[t.to(DEV) for t in _make_group(c, m, n, torch.float32, torch.float32, 31 + i)], 1.0)
                for i, (c, (m, n)) in enumerate(zip(counts, shapes))]

    def step(gs):
        ws = torch.empty(mlc.muloco_inner_workspace_bytes(gs), dtype=torch.uint8, device=DEV)
        mlc.muloco_inner_step(gs, hp, ws)
        torch.cuda.synchronize()
    one, many = groups(), groups()
    for g in one:
        step([g])
    step(many)
    for a, b in zip(one, many):
        assert torch.equal(a.param, b.param) and torch.equal(a.momentum, b.momentum)


def test_more_groups_than_one_momentum_launch_holds():
    """Seven groups of one kind (a launch holds four) between groups of other kinds: transposed,
    ragged, another gradient type."""
    shapes = [(128, 128)] * 3 + [(640, 256), (130, 77)] + [(128, 256)] * 4 + [(256, 384)]
    hp = mlc.MuonHParams(eta=6.25e-2, weight_decay=1.25e-3)

    def groups():
        return [mlc.InnerGroup(*[t.to(DEV) for t in _make_group(
                    2, m, n, torch.float32, torch.bfloat16 if i == 9 else torch.float32, 51 + i)], 1.0)
                for i, (m, n) in enumerate(shapes)]

    def step(gs):
        ws = torch.empty(mlc.muloco_inner_workspace_bytes(gs), dtype=torch.uint8, device=DEV)
        mlc.muloco_inner_step(gs, hp, ws)
        torch.cuda.synchronize()
    one, many = groups(), groups()
    for g in one:
        step([g])
    step(many)
    for i, (a, b) in enumerate(zip(one, many)):
        assert torch.equal(a.momentum, b.momentum), f"group {i}"
        assert torch.equal(a.param, b.param), f"group {i}"


@pytest.mark.parametrize("shapes", [[(5, 128, 128)] * 5 + [(1, 77, 333), (2, 333, 77)],       # more than share a launch; ragged apart
                                    [(1, 300, 200), (3, 200, 300)]])
@pytest.mark.parametrize("shared", [False, True])
def test_updates_that_share_a_launch(shapes, shared):
    """fp32 weights of several groups: the bits of one call per group, also where two groups name the
    same weights (which are then updated twice, in order)."""
    hp = mlc.MuonHParams(eta=0.05, weight_decay=1e-3, beta=0.9)
    if shared:
        shapes = shapes + shapes[:1]

    def groups():
        out = []
        for i, s in enumerate(shapes):
            W = S.normal(s, S.PARAM_STD, 31, i).to(DEV)
            if shared and i == len(shapes) - 1:
                W = out[0].param
            out.append(mlc.InnerGroup(W, S.normal(s, S.GRAD_STD, 32, i).to(DEV), S.normal(s, S.GRAD_STD, 33, i).to(DEV), 0.5 + i))
        return out

    def run(gs):
        ws = torch.empty(mlc.muloco_inner_workspace_bytes(gs), dtype=torch.uint8, device=DEV)
        mlc.muloco_inner_step(gs, hp, ws)
        torch.cuda.synchronize()
    together, apart = groups(), groups()
    run(together)
    for g in apart:
        run([g])
    for a, b in zip(together, apart):
        assert torch.equal(a.param, b.param) and torch.equal(a.momentum, b.momentum)


# Groups whose bf16 weights the last product updates, two of which name the same memory: in tiles of 64; in
# tiles of 256, where a launch would hold products of one depth, and of two
@pytest.mark.parametrize("shapes,tile", [([(2, 256, 384), (1, 384, 256), (2, 256, 384)], 64),
                                         ([(40, 768, 768), (40, 768, 768)], 256),
                                         ([(64, 512, 1024), (32, 1024, 1024)], 256)])
@pytest.mark.parametrize("what", ["param", "momentum"])
def test_groups_that_write_the_same_memory_go_one_after_the_other(shapes, tile, what):
    """The bits and the launches of one call per group."""
    assert all(ns_tiles([s])[0][2] == tile for s in shapes)          # the last product's
    hp = mlc.MuonHParams(eta=0.05, weight_decay=1e-3, beta=0.9)

    def groups():
        out = []
        for i, s in enumerate(shapes):
            g = mlc.InnerGroup(S.normal(s, S.PARAM_STD, 34, i, dtype=torch.bfloat16).to(DEV),
                               S.normal(s, S.GRAD_STD, 35, i, dtype=torch.bfloat16).to(DEV),
                               S.normal(s, S.GRAD_STD, 36, i).to(DEV), 0.5 + i)
            if i == len(shapes) - 1:
                setattr(g, what, getattr(out[0], what).view(s))
            out.append(g)
        return out

    def run(gs):
        ws = torch.empty(mlc.muloco_inner_workspace_bytes(gs), dtype=torch.uint8, device=DEV)
        mlc.muloco_timing_enable(True)
        mlc.muloco_timing_read()
        mlc.muloco_inner_step(gs, hp, ws)
        torch.cuda.synchronize()
        n = mlc.muloco_timing_read()["ns_gemm"]["launches"]
        mlc.muloco_timing_enable(False)
        return n
    together, apart = groups(), groups()
    launches = run(together)
    assert launches == sum(run([g]) for g in apart)
    for a, b in zip(together, apart):
        assert torch.equal(a.param.view(torch.int16), b.param.view(torch.int16)) and torch.equal(a.momentum, b.momentum)


# A group whose gradients are another's momentum, before or after it: rows of several kinds, which share a momentum pass
@pytest.mark.parametrize("reader,writer", [(0, 1), (1, 0), (2, 1)])
def test_groups_that_read_another_s_momentum_go_one_after_the_other(reader, writer):
    """The bits and the momentum passes of one call per group."""
    hp = mlc.MuonHParams(eta=0.05, weight_decay=1e-3, beta=0.9)
    shapes = [(2, 256, 384), (2, 384, 256), (4, 128, 384)]

    def groups():
        out = [mlc.InnerGroup(*[S.normal(s, std, 37, 10 * i + j).to(DEV) for j, std in enumerate((S.PARAM_STD, S.GRAD_STD, S.GRAD_STD))],
                              0.5) for i, s in enumerate(shapes)]
        out[reader].grad = out[writer].momentum.view(shapes[reader])
        return out

    def run(gs):
        ws = torch.empty(mlc.muloco_inner_workspace_bytes(gs), dtype=torch.uint8, device=DEV)
        mlc.muloco_timing_enable(True)
        mlc.muloco_timing_read()
        mlc.muloco_inner_step(gs, hp, ws)
        torch.cuda.synchronize()
        n = mlc.muloco_timing_read()["momentum"]["launches"]
        mlc.muloco_timing_enable(False)
        return n
    together, apart = groups(), groups()
    assert run(together) == sum(run([g]) for g in apart) == len(shapes)
    for a, b in zip(together, apart):
        assert torch.equal(a.param, b.param) and torch.equal(a.momentum, b.momentum)


# Gram products of two depths, both in 256 x 256 tiles: workgroups that are a tile short in the deeper one
# take several of the shallower one's; few and many tiles of either, and more products than share a launch
DEPTHS = [([(16, 1024, 2816), (32, 1024, 1024)], 15), ([(30, 512, 3072), (30, 3072, 512), (140, 512, 512)], 15),
          ([(27, 768, 3072), (60, 768, 768)], 15), ([(40, 768, 3072), (60, 768, 768)], 15),
          ([(16, 1024, 2816), (9, 2816, 1024), (16, 2048, 1024), (32, 1024, 1024)], 30),     # three and one
          # last products of three depths: the workgroups that are a tile short take the middle one whole
          ([(2, 2560, 2048), (24, 2560, 256), (4, 1280, 2048)], 30), ([(17, 256, 2816), (2, 2048, 2816), (3, 768, 4096)], 30)]


@pytest.mark.parametrize("shapes,launches", DEPTHS)
def test_products_of_two_depths_side_by_side(shapes, launches):
    """The bits of one group after the other (a work space with no room for all)."""
    hp = mlc.MuonHParams(eta=0.05, weight_decay=1e-3, beta=0.9)
    gen = torch.Generator(device=DEV).manual_seed(7)

    def groups():
        gen.manual_seed(7)
        out = []
        for s in shapes:
            few = torch.randn((3, *s[1:]), generator=gen, device=DEV) * S.GRAD_STD
            grad = few.repeat(-(-s[0] // 3), 1, 1)[:s[0]].bfloat16()
            out.append(mlc.InnerGroup(torch.zeros(s, dtype=torch.bfloat16, device=DEV), grad, torch.zeros(s, device=DEV), 1.0))
        return out
    a, b = groups(), groups()
    room = mlc.muloco_inner_workspace_bytes(a)
    ws = torch.empty(room, dtype=torch.uint8, device=DEV)
    mlc.muloco_timing_enable(True)
    mlc.muloco_timing_read()
    mlc.muloco_inner_step(a, hp, ws)
    n = mlc.muloco_timing_read()["ns_gemm"]["launches"]
    mlc.muloco_timing_enable(False)
    assert launches == n
    for g in b:
        mlc.muloco_inner_step([g], hp, ws)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x.param.view(torch.int16), y.param.view(torch.int16))
        assert all(torch.equal(x.param[i], x.param[i % 3]) for i in range(x.param.shape[0]))


# Triangles in a launch that mixes depths: products with and without operand A's transfers one behind the other in a
# workgroup, and shares that end in a triangle
@pytest.mark.parametrize("shapes", [
    [(30, 768, 3328), (40, 2560, 768), (60, 768, 768)], [(16, 1024, 2816), (32, 1024, 1024)],
    [(20, 1280, 2816), (30, 1280, 1280), (10, 2560, 1280)],
])
def test_triangles_of_several_depths_in_one_launch(shapes):
    """The bits of the matrices one by one, in smaller tiles."""
    hp = mlc.MuonHParams(eta=0.05, weight_decay=1e-3, beta=0.9)
    gen = torch.Generator(device=DEV).manual_seed(8)
    few = [(torch.randn((3, *s[1:]), generator=gen, device=DEV) * S.GRAD_STD).bfloat16() for s in shapes]
    zeros = lambda c, s, dt: torch.zeros((c, *s[1:]), dtype=dt, device=DEV)  # noqa: E731
    together = [mlc.InnerGroup(zeros(s[0], s, torch.bfloat16), f.repeat(-(-s[0] // 3), 1, 1)[:s[0]].contiguous(),
                               zeros(s[0], s, torch.float32), 1.0) for s, f in zip(shapes, few)]
    assert all(t[0] == 256 for t in ns_tiles(shapes))
    ws = torch.empty(mlc.muloco_inner_workspace_bytes(together), dtype=torch.uint8, device=DEV)
    mlc.muloco_timing_enable(True)
    mlc.muloco_timing_read()
    mlc.muloco_inner_step(together, hp, ws)
    launches = mlc.muloco_timing_read()["ns_gemm"]["launches"]
    mlc.muloco_timing_enable(False)
    assert launches == 15                    # the Gram products of all groups share one
    for g, s, f in zip(together, shapes, few):
        for i in range(3):
            assert 256 not in ns_tiles([(1, *s[1:])])[0]
            one = mlc.InnerGroup(zeros(1, s, torch.bfloat16), f[i:i + 1].clone(), zeros(1, s, torch.float32), 1.0)
            mlc.muloco_inner_step([one], hp, ws)
            for j in range(i, s[0], 3):
                assert torch.equal(g.param[j].view(torch.int16), one.param[0].view(torch.int16)), (s, j)


# Sides that the 256 x 256 tile does not divide: its last tile row (column) begins half a tile early, and what the
# neighbours compute too must not be stored twice (the last product updates the weights in place).  Rows, columns and both;
# tall and wide; a padded result and one without
@pytest.mark.parametrize("shapes,tiles", [
    ([(24, 1408, 1408)], [(256, 256, 256)]), ([(24, 1024, 1152)], [(256, 256, 256)]), ([(24, 1152, 1024)], [(256, 256, 256)]),
    ([(20, 896, 1664), (20, 1664, 896)], [(256, 128, 256)] * 2), ([(40, 1150, 901)], [(256, 256, 256)]),
])
def test_half_tiles_at_the_edge(shapes, tiles):
    """The bits of the matrices one by one, in tiles that divide every side; nothing beside the weights is written."""
    assert ns_tiles(shapes) == tiles
    hp = mlc.MuonHParams(eta=0.05, weight_decay=1e-2, beta=0.9)
    gen = torch.Generator(device=DEV).manual_seed(9)
    few = [[(torch.randn((3, *s[1:]), generator=gen, device=DEV) * d).bfloat16() for d in (S.GRAD_STD, S.PARAM_STD)] for s in shapes]
    guard, groups, held = 4096, [], []
    for s, (g, w) in zip(shapes, few):
        many = lambda t: t.repeat(-(-s[0] // 3), 1, 1)[:s[0]].contiguous()  # noqa: E731
        flat = torch.full((w[0].numel() * s[0] + 2 * guard,), 7.0, dtype=torch.bfloat16, device=DEV)
        held.append(flat)
        param = flat[guard:-guard].view(s)
        param.copy_(many(w))
        groups.append(mlc.InnerGroup(param, many(g), torch.zeros(s, device=DEV), 0.7))
    ws = torch.empty(mlc.muloco_inner_workspace_bytes(groups), dtype=torch.uint8, device=DEV)
    mlc.muloco_inner_step(groups, hp, ws)
    for s, (g, w), grp, flat in zip(shapes, few, groups, held):
        assert bool((flat[:guard] == 7).all()) and bool((flat[-guard:] == 7).all())
        assert 256 not in ns_tiles([(1, *s[1:])])[0]
        for i in range(3):
            one = mlc.InnerGroup(w[i:i + 1].clone(), g[i:i + 1].clone(), torch.zeros((1, *s[1:]), device=DEV), 0.7)
            mlc.muloco_inner_step([one], hp, ws)
            for j in range(i, s[0], 3):
                assert torch.equal(grp.param[j].view(torch.int16), one.param[0].view(torch.int16)), (s, j)
    (g, w), s = few[0], shapes[0]
    _check_group(w[:1].cpu(), g[:1].cpu(), torch.zeros((1, *s[1:])), groups[0].param[:1].cpu(), groups[0].momentum[:1].cpu(), hp,
                 0.7, f"{s}")


# Products of several depths that share launches in small tiles: in one round, in more, sets that run different small tiles
# and take one, a depth of two K tiles; momentum, norm and update launches of rows that are a multiple of 8 and others,
# plain and transposed, and of more groups than share one
JOINED = [([(4, 512, 512), (1, 512, 1536), (1, 1536, 512)], 15), ([(8, 303, 303), (2, 303, 640), (2, 640, 303)], 15),
          ([(16, 256, 256), (4, 256, 1000), (4, 1000, 256)], 15), ([(16, 768, 768), (4, 768, 2449), (4, 2449, 768)], 15),
          ([(8, 640, 640), (2, 640, 1192), (2, 1192, 640)], 15), ([(2, 384, 384), (3, 128, 640), (1, 512, 901)], 15),
          ([(2, 200, 136), (1, 300, 77), (1, 77, 901), (2, 333, 512), (1, 1001, 384)], None)]


@pytest.mark.parametrize("shapes,launches", JOINED)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_small_products_of_several_depths_share_launches(shapes, launches, dtype):
    """The bits of one group after the other."""
    hp = mlc.MuonHParams(eta=0.05, weight_decay=1e-2, beta=0.9)

    def build():
        host = [_make_group(c, m, n, dtype, torch.bfloat16, seed=60 + i) for i, (c, m, n) in enumerate(shapes)]
        return host, [mlc.InnerGroup(*[t.to(DEV) for t in h], 0.5) for h in host]
    (host, together), (_, apart) = build(), build()
    ws = torch.empty(mlc.muloco_inner_workspace_bytes(together), dtype=torch.uint8, device=DEV)
    mlc.muloco_timing_enable(True)
    mlc.muloco_timing_read()
    mlc.muloco_inner_step(together, hp, ws)
    n = mlc.muloco_timing_read()["ns_gemm"]["launches"]
    mlc.muloco_timing_enable(False)
    assert launches in (n, None)
    for g in apart:
        mlc.muloco_inner_step([g], hp, ws)
    torch.cuda.synchronize()
    for a, b in zip(together, apart):
        assert torch.equal(a.param, b.param) and torch.equal(a.momentum, b.momentum)
    for (W0, g, m0), grp, s in zip(host, together, shapes):
        _check_group(W0[-1:], g[-1:], m0[-1:], grp.param[-1:].cpu(), grp.momentum[-1:].cpu(), hp, 0.5, f"group {s}")
