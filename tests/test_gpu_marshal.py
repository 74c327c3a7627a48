"""What the binding's native part answers for, and what it leaves to the checks in Python."""
import pytest
import torch

import paper_2505_23725_amd as mlc
from paper_2505_23725_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class Odd(torch.Tensor):
    pass


def test_addresses_and_refusals():
    from paper_2505_23725_amd import _marshal
    t = torch.zeros(4, 6, device=DEV)
    assert _marshal.pointer(t) == t.data_ptr() == binding._dev_ptr(t, "t")
    assert _marshal.pointer(t[1:]) == t.data_ptr() + 24
    assert _marshal.pointer(torch.nn.Parameter(t)) == t.data_ptr()
    for other in (t.T, t.cpu(), t[:, :3], t.to_sparse(), 7, None, t.as_subclass(Odd)):
        assert _marshal.pointer(other) is None
    assert binding._dev_ptr(t.as_subclass(Odd), "t") == t.data_ptr()
    with pytest.raises(ValueError, match="contiguous"):
        binding._dev_ptr(t.T, "t")
    with pytest.raises(ValueError, match="on the GPU"):
        binding._dev_ptr(t.cpu(), "t")


def _four(n, pd=torch.float32, gd=torch.float32):
    gen = torch.Generator(device=DEV).manual_seed(n)
    r = lambda: torch.randn(n, generator=gen, device=DEV)  # noqa: E731
    return r().to(pd), r().to(gd), r(), r().square()


@pytest.mark.parametrize("wrong,error", [((None, None, None, "half"), TypeError), ((None, None, "short", None), ValueError),
                                         (("cpu", None, None, None), ValueError), ((None, "int", None, None), TypeError)])
def test_adamw_refuses_what_it_refused(wrong, error):
    change = {None: lambda t: t, "half": lambda t: t.bfloat16(), "short": lambda t: t[:-1], "cpu": lambda t: t.cpu(),
              "int": lambda t: t.int()}
    bad = tuple(change[w](t) for w, t in zip(wrong, _four(64)))
    with pytest.raises(error):
        mlc.muloco_adamw_step([_four(32), bad], mlc.AdamWHParams(lr=0.1))


@pytest.mark.parametrize("wrap", [list, tuple, lambda ts: [list(t) for t in ts],
                                  lambda ts: [tuple(x.as_subclass(Odd) for x in t) for t in ts]])
def test_adamw_takes_the_sequences_it_took(wrap):
    """Lists of tuples go through the native part, other sequences through Python: the same step."""
    hp = mlc.AdamWHParams(lr=0.1, weight_decay=0.1)
    kinds = [(1, torch.bfloat16, torch.float32), (77, torch.float32, torch.bfloat16), (4096, torch.float32, torch.float32)]
    a, b = [_four(*k) for k in kinds], [_four(*k) for k in kinds]
    mlc.muloco_adamw_step(a, hp)
    mlc.muloco_adamw_step(wrap(b), hp)
    assert all(torch.equal(x, y) for s, t in zip(a, b) for x, y in zip(s, t))
    mlc.muloco_adamw_step([], hp)


def test_calls_are_the_same_without_the_native_part(monkeypatch):
    hp = mlc.AdamWHParams(lr=0.1, weight_decay=0.1)
    x = torch.randn(3, 40, 72, generator=torch.Generator(device=DEV).manual_seed(1), device=DEV)

    def both():
        four, out = [_four(77), _four(4096)], torch.empty_like(x)
        mlc.muloco_adamw_step(four, hp)
        mlc.newton_schulz_static_scratch(x, out)
        return [t for f in four for t in f] + [out]
    assert binding._marshal() is not None
    with_native = both()
    monkeypatch.setattr(binding, "_native", False)
    monkeypatch.setattr(binding, "_pointer", lambda t: None)
    assert all(torch.equal(a, b) for a, b in zip(with_native, both()))
