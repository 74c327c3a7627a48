"""GPU parity: newton_schulz (C-ABI) against the fp64 oracle, element by element, on seeded
inputs whose shapes span several 128/256 tiles and ragged tails."""
import numpy as np
import pytest
import torch

import paper_2505_23725_amd as mlc
import synth_inputs as S
from oracle import muon
from helpers import NS_TOL, assert_ns_close, ns_executed_flops, ns_tiles, to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(x_cpu: torch.Tensor, iters=5, ws_bytes=None, coeffs=muon.NS_COEFFS, inplace=False):
    cnt, m, n = (1, *x_cpu.shape) if x_cpu.dim() == 2 else x_cpu.shape
    x = x_cpu.to(DEV)
    out = x if inplace else torch.empty_like(x)
    need = mlc.newton_schulz_workspace_bytes(cnt, m, n) if ws_bytes is None else ws_bytes
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    mlc.newton_schulz(x, out, ws, iters=iters, a=coeffs[0], b=coeffs[1], c=coeffs[2])
    torch.cuda.synchronize()
    return out.cpu()


def _check(x_cpu, out_cpu, iters=5, coeffs=muon.NS_COEFFS, tol=NS_TOL):
    xs = x_cpu if x_cpu.dim() == 3 else x_cpu[None]
    os_ = out_cpu if out_cpu.dim() == 3 else out_cpu[None]
    worst = 0.0
    for i in range(xs.shape[0]):
        ref = muon.newton_schulz(to_f64(xs[i]), iters, coeffs)
        st = assert_ns_close(to_f64(os_[i]), ref, f"matrix {i} of shape {tuple(xs[i].shape)}", tol)
        worst = max(worst, st["fro"])
    return worst


SHAPES = [
    (1, 128, 128),      # one tile
    (3, 128, 512),      # tiny-config wide
    (2, 512, 128),      # tiny-config tall
    (3, 100, 380),      # ragged wide that pads to 128 x 384: one-workgroup chain, L = 384
    (2, 128, 640),      # short side 128 but too long for the one-workgroup chain
    (2, 200, 136),      # ragged in both dimensions (pads to 256 x 256)
    (1, 72, 1000),      # ragged wide, row length not a multiple of 8? (1000 is) -> padded columns
    (1, 333, 77),       # ragged tall, odd row length: scalar load path; chain held transposed
    (300, 128, 256),    # more matrices than compute units on the one-workgroup chain
    (5, 384, 640),      # several tiles, wide
    (2, 640, 384),      # several tiles, tall
    (4, 768, 768),      # 150M-scale attention shape
]


@pytest.mark.parametrize("cnt,m,n", SHAPES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_newton_schulz_matches_oracle(cnt, m, n, dtype):
    x = S.normal((cnt, m, n), S.GRAD_STD, seed=0, stream=m * 131 + n, dtype=dtype)
    out = _run(x)
    worst = _check(x, out)
    print(f"NS {cnt}x{m}x{n} {dtype}: worst rel. Frobenius error {worst:.3e}")


@pytest.mark.parametrize("iters", [0, 1, 2, 7])
def test_iteration_counts(iters):
    x = S.normal((2, 256, 384), 1.0, seed=1, stream=iters, dtype=torch.bfloat16)
    out = _run(x, iters=iters)
    # iters = 0 is a pure scaling: only bf16 rounding separates it from the oracle
    _check(x, out, iters=iters, tol=4e-3 if iters == 0 else NS_TOL)


def test_cubic_coefficients_and_in_place():
    x = S.normal((2, 256, 256), 0.02, seed=2, stream=0, dtype=torch.float32)
    out = _run(x, iters=6, coeffs=(1.5, -0.5, 0.0), inplace=True)
    _check(x, out, iters=6, coeffs=(1.5, -0.5, 0.0))


def test_chunked_work_space_gives_same_result():
    x = S.normal((5, 256, 384), S.GRAD_STD, seed=3, stream=0, dtype=torch.bfloat16)
    full = _run(x)
    two = _run(x, ws_bytes=2 * mlc.newton_schulz_workspace_min_bytes(256, 384))
    one = _run(x, ws_bytes=mlc.newton_schulz_workspace_min_bytes(256, 384))
    assert torch.equal(full.view(torch.int16), two.view(torch.int16))
    assert torch.equal(full.view(torch.int16), one.view(torch.int16))


def test_zero_matrix_and_determinism():
    x = S.normal((3, 128, 256), S.GRAD_STD, seed=4, stream=0, dtype=torch.bfloat16)
    x[1].zero_()
    a = _run(x)
    b = _run(x)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert torch.count_nonzero(a[1]) == 0
    assert torch.isfinite(a.float()).all()
    _check(x, a)


def test_zero_matrix_with_eps_zero_stays_zero():
    # 1 / (norm + eps) must not turn into inf * 0 when both the matrix and eps are zero
    for shape in [(2, 128, 256), (2, 256, 384)]:      # one-workgroup chain, batched products
        x = S.normal(shape, S.GRAD_STD, seed=6, stream=shape[2], dtype=torch.bfloat16)
        x[0].zero_()
        xd = x.to(DEV)
        out = torch.empty_like(xd)
        ws = torch.empty(mlc.newton_schulz_workspace_bytes(*shape), dtype=torch.uint8, device=DEV)
        for iters in (0, 5):
            mlc.newton_schulz(xd, out, ws, iters=iters, eps=0.0)
            torch.cuda.synchronize()
            o = out.cpu()
            assert torch.count_nonzero(o[0]) == 0
            assert torch.isfinite(o.float()).all()
            ref = muon.newton_schulz(to_f64(x[1]), iters, eps=0.0)
            assert_ns_close(to_f64(o[1]), ref, f"{shape} eps=0 iters={iters}", 4e-3 if iters == 0 else NS_TOL)


# (count, m, n, tile widths of the Gram, polynomial and apply products): more output tiles than
# compute units at every width, tall and wide
MANY_TILES = [
    (100, 256, 256, (64, 64, 128)),       # 1000 tiles of 64, 400 of 128
    (230, 256, 256, (256, 128, 256)),
    (70, 384, 384, (128, 128, 128)),      # 420 and 630
    (45, 256, 512, (128, 128, 128)),
    (45, 512, 256, (128, 128, 128)),      # 360 whose result is stored transposed
    (130, 512, 1024, (256, 256, 256)),    # 390 and 1040
    (130, 1024, 512, (256, 256, 256)),
]
# the ring of operand tiles: products of few K tiles, and a workgroup's second output tile
RING = [
    (70, 128, 640, (64, 128, 128)), (70, 640, 128, (64, 128, 128)),      # K = 128: two K tiles; tall: transposed result
    (40, 256, 640, (128, 128, 128)), (40, 640, 250, (128, 128, 128)),    # K = 256: the short ring; ragged tall
    (90, 512, 768, (128, 128, 256)), (90, 768, 512, (128, 128, 256)),    # the long ring, several tiles a workgroup
    (1, 384, 1152, (64, 64, 64)), (1, 1152, 384, (64, 64, 64)),          # fewer tiles than compute units
    (1, 256, 1024, (64, 64, 64)), (1, 1024, 256, (64, 64, 64)),          # ... with as many K tiles as the ring holds ahead
    (9, 256, 1300, (64, 64, 128)), (9, 1300, 256, (64, 64, 128)),
    (1, 128, 1000, (64, 128, 128)),                                      # K = 128 again: too short for the 64 tile's ring
    (24, 640, 640, (128, 128, 128)), (60, 640, 640, (128, 128, 128)),    # K = 640: the short ring up to two rounds, and the long one
]


def _run_recorded(x, shape):
    """The result, after checking that the call executed the FLOP of the tiles it is said to use."""
    mlc.muloco_timing_enable(True)
    mlc.muloco_timing_read()
    out = _run(x)
    t = mlc.muloco_timing_read()["ns_gemm"]
    mlc.muloco_timing_enable(False)
    assert t["launches"] == 15
    assert abs(t["flops"] / ns_executed_flops([shape]) - 1) < 1e-9
    return out


@pytest.mark.parametrize("cnt,m,n,tiles", MANY_TILES)
def test_more_small_tiles_than_compute_units(cnt, m, n, tiles):
    """Batches with more output tiles than compute units (an earlier kernel put two workgroups on a CU
    then, and the second one's tiles came out as garbage): every matrix finite, two runs
    bit-identical, and matrices from the end of the batch, where the workgroups' later tiles are,
    match the oracle."""
    assert ns_tiles([(cnt, m, n)]) == [tiles]
    x = S.normal((cnt, m, n), S.GRAD_STD, seed=8, stream=cnt + n, dtype=torch.bfloat16)
    a = _run_recorded(x, (cnt, m, n))
    b = _run(x)
    assert torch.isfinite(a.float()).all()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    for i in (cnt // 8 - 1, cnt // 8, cnt - 1):       # around the end of the first XCD's range, and the last
        assert_ns_close(to_f64(a[i]), muon.newton_schulz(to_f64(x[i]), 5), f"matrix {i} of {cnt} x {m} x {n}")


@pytest.mark.parametrize("cnt,m,n,tiles", RING)
def test_ring_across_output_tiles(cnt, m, n, tiles):
    assert ns_tiles([(cnt, m, n)]) == [tiles]
    x = S.normal((cnt, m, n), S.GRAD_STD, seed=9, stream=cnt + m, dtype=torch.bfloat16)
    a = _run_recorded(x, (cnt, m, n))
    assert torch.equal(a.view(torch.int16), _run(x).view(torch.int16))
    for i in (0, cnt // 2, cnt - 1):
        assert_ns_close(to_f64(a[i]), muon.newton_schulz(to_f64(x[i]), 5), f"matrix {i} of {cnt} x {m} x {n}")


# (m, n, counts that take different tiles for one product or another)
SAME_BITS = [
    (512, 512, {1: (64, 64, 64), 9: (128, 128, 128), 64: (256, 128, 256)}),
    (1024, 256, {1: (64, 64, 64), 8: (64, 64, 128), 48: (128, 128, 256)}),
    (256, 1024, {1: (64, 64, 64), 8: (64, 64, 128), 48: (128, 128, 256)}),
    (768, 768, {1: (64, 64, 64), 8: (128, 128, 128), 64: (256, 256, 256)}),
]


@pytest.mark.parametrize("m,n,counts", SAME_BITS)
def test_every_tile_gives_the_same_bits(m, n, counts):
    """What lets a call with a small work space give the bits of one with a large one: the first
    matrix of the batch, orthogonalised in batches that run different tiles."""
    x = S.normal((max(counts), m, n), S.GRAD_STD, seed=13, stream=m + n, dtype=torch.bfloat16)
    first = None
    for c, tiles in counts.items():
        assert ns_tiles([(c, m, n)]) == [tiles], f"batch of {c}"
        out = _run_recorded(x[:c].contiguous(), (c, m, n))[0].view(torch.int16)
        assert first is None or torch.equal(out, first), f"batch of {c}"
        first = out


# more 256 x 256 tiles than compute units, whose stores a workgroup has left over go out during the next
# tile's K tiles: products of 4 and 6 K tiles (fewer than the stores take), 8 and 10 (exactly as many,
# and more), and many; tall ones store transposed
LEFT_OVER = [
    (600, 256, 256, (256, 128, 256)), (900, 256, 384, (256, 128, 128)), (300, 512, 512, (256, 256, 256)),
    (300, 512, 640, (256, 256, 128)), (700, 256, 512, (256, 128, 256)), (700, 512, 256, (256, 128, 256)),
    (100, 1024, 768, (256, 256, 256)),
]


@pytest.mark.parametrize("cnt,m,n,tiles", LEFT_OVER)
def test_stores_left_for_the_next_tile(cnt, m, n, tiles):
    """Every matrix has the bits that it gets alone or nearly so (in smaller tiles, where nothing is left
    over), also where the last product updates bf16 weights."""
    assert ns_tiles([(cnt, m, n)]) == [tiles]
    some = S.normal((6, m, n), S.GRAD_STD, seed=21, stream=m + n, dtype=torch.bfloat16).to(DEV)
    few = torch.stack([o for x in some for o in _run(x[None])])
    x = some.repeat((cnt + 5) // 6, 1, 1)[:cnt]
    out = _run(x)
    for i in range(cnt):
        assert torch.equal(out[i].view(torch.int16), few[i % 6].view(torch.int16)), i
    hp = mlc.MuonHParams(eta=0.05, weight_decay=1e-3, beta=0.9)

    def step(grad):
        W = torch.full_like(grad, 0.02)
        g = mlc.InnerGroup(W, grad.contiguous(), torch.zeros(grad.shape, device=DEV), 0.7)
        ws = torch.empty(mlc.muloco_inner_workspace_bytes([g]), dtype=torch.uint8, device=DEV)
        mlc.muloco_inner_step([g], hp, ws)
        torch.cuda.synchronize()
        return W.cpu().view(torch.int16)
    few = [step(v[None])[0] for v in some]
    W = step(x)
    for i in range(cnt):
        assert torch.equal(W[i], few[i % 6]), i


# 256 x 256 tiles on the diagonal, of which a triangle is computed: as many K tiles as go without operand A's
# transfers, and more; whole tiles before and behind them (several depths in a launch: test_gpu_inner_step.py)
@pytest.mark.parametrize("cnt,m,n,tiles", [
    (40, 768, 2560, (256, 256, 256)), (40, 768, 3328, (256, 256, 256)), (40, 3328, 768, (256, 256, 256)),
    (20, 1280, 1280, (256, 128, 256)), (300, 512, 512, (256, 256, 256)),
])
def test_triangles_give_the_bits_of_whole_tiles(cnt, m, n, tiles):
    assert ns_tiles([(cnt, m, n)]) == [tiles]
    some = S.normal((3, m, n), S.GRAD_STD, seed=22, stream=m + n, dtype=torch.bfloat16).to(DEV)
    few = torch.stack([o for x in some for o in _run(x[None])])         # in smaller tiles, without triangles
    assert all(256 not in t for t in ns_tiles([(1, m, n)]))
    out = _run(some.repeat((cnt + 2) // 3, 1, 1)[:cnt])
    for i in range(cnt):
        assert torch.equal(out[i].view(torch.int16), few[i % 3].view(torch.int16)), i


# The recorder counts executed FLOP: of a triangle its 144 of 256 MFMAs, also where the shape is padded and where
# only one of the two symmetric products takes large tiles.
@pytest.mark.parametrize("cnt,m,n,tiles", [
    (100, 1001, 1001, (256, 256, 256)), (20, 1280, 1280, (256, 128, 256)), (40, 3328, 768, (256, 256, 256)),
])
def test_recorder_counts_executed_flop(cnt, m, n, tiles):
    assert ns_tiles([(cnt, m, n)]) == [tiles]
    _run_recorded(S.normal((cnt, m, n), S.GRAD_STD, seed=23, stream=n, dtype=torch.bfloat16), (cnt, m, n))
    s, l = sorted(-(-x // 256) * 256 for x in (m, n))
    t = s // 256                              # tiles a side
    gram, poly = ((t * (t + 1) / 2 - t * 7 / 16) / t ** 2 if w == 256 else (2 * t + 1) / (4 * t) for w in tiles[:2])
    assert abs(ns_executed_flops([(cnt, m, n)]) / (5 * cnt * 2.0 * s * s * (gram * l + poly * s + l)) - 1) < 1e-12


@pytest.mark.parametrize("cnt,m,n", [(1, 384, 256), (2, 1000, 333), (6, 1536, 512), (48, 1024, 256), (12, 2048, 1024)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_tall_is_the_wide_result_transposed(cnt, m, n, dtype):
    """A tall matrix is held transposed while it is iterated on, so its result is the transposed result of
    its transpose, bit for bit, wherever the norm is the same: elements of one magnitude have an exact
    sum of squares in any order.  (Other values may differ in the sum's last bit, and through it in
    roundings of the iteration.)"""
    x = torch.sign(S.normal((cnt, m, n), 1.0, seed=14, stream=m + n)) * 2.0 ** -10
    x = x.to(dtype)
    tall, wide = _run(x), _run(x.transpose(1, 2).contiguous())
    assert torch.equal(tall, wide.transpose(1, 2))


def test_products_beside_lds_kernels_of_another_stream():
    """Newton-Schulz of small tiles (which leave most of the LDS unused) on one stream while kernels
    that hold LDS (top-k selection, small chains) keep the compute units busy on another: the bits of
    a run alone."""
    x = S.normal((60, 256, 640), S.GRAD_STD, seed=12, stream=0, dtype=torch.bfloat16).to(DEV)
    y = S.normal((900, 128, 128), S.GRAD_STD, seed=12, stream=1, dtype=torch.bfloat16).to(DEV)
    out, yout = torch.empty_like(x), torch.empty_like(y)
    ws = torch.empty(mlc.newton_schulz_workspace_bytes(*x.shape), dtype=torch.uint8, device=DEV)
    ws2 = torch.empty(mlc.newton_schulz_workspace_bytes(*y.shape), dtype=torch.uint8, device=DEV)
    mlc.newton_schulz(x, out, ws)
    torch.cuda.synchronize()
    alone = out.clone()
    theta = S.normal((8, 1024, 1024), S.PARAM_STD, seed=12, stream=2).to(DEV)
    grp = mlc.OuterGroup([theta + 0.01], theta, torch.zeros_like(theta))
    hp = mlc.OuterHParams(K=1, eta_out=0.0, mu=0.0, write_back=False)
    wsp = torch.empty(mlc.muloco_topk_workspace_bytes([grp], 1), dtype=torch.uint8, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for _ in range(5):
        with torch.cuda.stream(side):
            for _ in range(4):
                mlc.muloco_topk_outer_step([grp], hp, 0.05, wsp)
                mlc.newton_schulz(y, yout, ws2)
        for _ in range(4):
            mlc.newton_schulz(x, out, ws)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), alone.view(torch.int16))


def test_singular_values_land_in_the_band():
    x = S.normal((1, 256, 512), S.GRAD_STD, seed=5, stream=0, dtype=torch.bfloat16)
    out = _run(x)
    sv = np.linalg.svd(to_f64(out[0]), compute_uv=False)
    # band of the tuned quintic, widened by the bf16 error budget
    assert sv.max() <= 1.2024 * (1 + 2 * NS_TOL)
    assert np.median(sv) >= 0.6818 * (1 - 2 * NS_TOL)


def test_work_space_too_small_is_an_error():
    x = torch.zeros(1, 128, 128, dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(4096, dtype=torch.uint8, device=DEV)
    with pytest.raises(mlc.MulocoError) as e:
        mlc.newton_schulz(x, x, ws)
    assert e.value.code == -4


@pytest.mark.parametrize("cnt,m,n", [(3, 128, 128), (2, 128, 384), (2, 512, 128), (3, 256, 640), (3, 640, 256), (5, 768, 512), (70, 512, 512)])
@pytest.mark.parametrize("how", ["apart", "in place", "chunks"])
def test_bf16_results_without_padding_need_no_last_pass(cnt, m, n, how):
    """They have the values of fp32 results of the same input, which go through the work space."""
    x = S.normal((cnt, m, n), S.GRAD_STD, seed=23, stream=m + n, dtype=torch.bfloat16)
    ws = 2 * mlc.newton_schulz_workspace_bytes(1, m, n) if how == "chunks" else None
    mlc.muloco_timing_enable(True)
    mlc.muloco_timing_read()
    out = _run(x, ws_bytes=ws, inplace=how == "in place")
    passes = mlc.muloco_timing_read()["convert"]["launches"]
    mlc.muloco_timing_enable(False)
    assert passes == (1 if ws is None else -(-cnt // 2))          # the input's alone
    assert torch.equal(out.float(), _run(S.normal((cnt, m, n), S.GRAD_STD, seed=23, stream=m + n, dtype=torch.bfloat16).float()))
