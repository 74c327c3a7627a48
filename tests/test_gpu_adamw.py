"""GPU parity: muloco_adamw_step (C-ABI) against the fp64 oracle over several steps."""
import numpy as np
import pytest
import torch

import paper_2505_23725_amd as mlc
import synth_inputs as S
from oracle import adamw
from helpers import assert_fp32_close, assert_stored_close, to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # elements, param dtype, grad dtype, bias correction
    (4096, torch.float32, torch.float32, False),
    (50257 * 3, torch.bfloat16, torch.bfloat16, True),      # not a multiple of 8: scalar path
    (768 * 1024, torch.bfloat16, torch.float32, True),
    (1000, torch.float32, torch.bfloat16, False),
    (7, torch.float32, torch.float32, True),
]


@pytest.mark.parametrize("n,pd,gd,bc", CASES)
def test_adamw_steps_match_oracle(n, pd, gd, bc):
    th0 = S.normal((n,), S.PARAM_STD, n, 0, dtype=pd)
    th = th0.to(DEV)
    m = torch.zeros(n, dtype=torch.float32, device=DEV)
    v = torch.zeros(n, dtype=torch.float32, device=DEV)
    rth, rm, rv = to_f64(th0), np.zeros(n), np.zeros(n)
    kw = dict(lr=3e-3, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)
    for t in range(1, 5):
        g0 = S.normal((n,), S.GRAD_STD, n, 10 + t, dtype=gd)
        start = to_f64(th.cpu())          # both sides start each step from the stored parameters
        mlc.muloco_adamw_step([(th, g0.to(DEV), m, v)], mlc.AdamWHParams(bias_correction=bc, step=t, **kw))
        torch.cuda.synchronize()
        rth, rm, rv = adamw.adamw_step(start, rm, rv, to_f64(g0), step=t, bias_correction=bc, **kw)
        assert_fp32_close(m.cpu(), rm, f"first moment, step {t}")
        assert_fp32_close(v.cpu(), rv, f"second moment, step {t}")
        assert_stored_close(th.cpu(), rth, f"parameters, step {t}")


def test_adamw_several_tensors_in_one_call_and_zero_gradient():
    sizes = [1024, 24, 4104]
    ps = [S.normal((n,), 1.0, 5, i).to(DEV) for i, n in enumerate(sizes)]
    p0 = [p.cpu().clone() for p in ps]
    zs = [torch.zeros(n, device=DEV) for n in sizes]
    ms = [torch.zeros(n, device=DEV) for n in sizes]
    vs = [torch.zeros(n, device=DEV) for n in sizes]
    mlc.muloco_adamw_step(list(zip(ps, zs, ms, vs)), mlc.AdamWHParams(lr=0.1, weight_decay=0.5))
    torch.cuda.synchronize()
    for p, q in zip(ps, p0):          # zero gradient: pure decoupled decay
        assert_fp32_close(p.cpu(), to_f64(q) * (1 - 0.05), "decay only")
    assert all(torch.count_nonzero(x) == 0 for x in ms + vs)


@pytest.mark.parametrize("pd,gd", [(torch.bfloat16, torch.bfloat16), (torch.float32, torch.bfloat16)])
def test_adamw_many_tensors_share_launches(pd, gd):
    """More tensors than one launch holds, sizes around the chunk of a workgroup (8192) and off the
    8-element vector, a change of dtype in between, and in the last launch's run a tensor that
    appears twice and two overlapping slices of one: the same bits as one call per tensor."""
    sizes = [8192, 8191, 8193, 1, 7, 8, 16384 + 5] + [40 + i for i in range(70)]
    hp = mlc.AdamWHParams(lr=3e-3, weight_decay=0.1, bias_correction=True, step=3)
    other = torch.bfloat16 if pd == torch.float32 else torch.float32

    def state():
        out = []
        for i, n in enumerate(sizes):
            d = other if i == 30 else pd
            out.append((S.normal((n,), 1.0, 7, i, dtype=d).to(DEV), S.normal((n,), 1.0, 8, i, dtype=gd).to(DEV),
                        S.normal((n,), 1.0, 9, i).to(DEV), S.normal((n,), 1.0, 10, i).abs().to(DEV)))
        return out + [out[70], out[0], tuple(t[:48] for t in out[75]), tuple(t[16:] for t in out[75])]
    one, many = state(), state()
    for t in one:
        mlc.muloco_adamw_step([t], hp)
    mlc.muloco_adamw_step(many, hp)
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(one, many)):
        for x, y in zip(a, b):
            assert torch.equal(x, y), f"tensor {i} of {len(one)}"


@pytest.mark.parametrize("count", [2, 3, 4, 5, 9, 64])
def test_adamw_launches(count):
    """Tensors of one dtype pair go out in one launch; one that shares memory with a later one goes
    out before it, alone."""
    ts = [tuple(torch.ones(24 + 8 * i, device=DEV) for _ in range(4)) for i in range(count)]
    hp = mlc.AdamWHParams(lr=1e-3)

    def launches(tensors):
        mlc.muloco_timing_enable(True)
        mlc.muloco_timing_read()
        mlc.muloco_adamw_step(tensors, hp)
        torch.cuda.synchronize()
        n = mlc.muloco_timing_read()["adamw"]["launches"]
        mlc.muloco_timing_enable(False)
        return n
    assert launches(ts) == 1
    twice = ts[:-1] + [ts[0]]
    assert launches(twice) == 2
    part = ts[:-1] + [tuple(t[8:] for t in ts[0])]
    assert launches(part) == 2
