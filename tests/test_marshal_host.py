"""What the binding does around its native part (csrc/marshal.cpp), without a GPU."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2505_23725_amd as mlc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

def test_adamw_takes_an_array_of_tensors():
    """A NumPy object array is a sequence of tuples like any other: the tensors are looked at, not the array's truth value."""
    tensors = np.empty((2, 4), dtype=object)
    for i in range(8):
        tensors[i // 4, i % 4] = torch.zeros(8)
    with pytest.raises(ValueError, match="param must live on the GPU"):
        mlc.muloco_adamw_step(tensors, mlc.AdamWHParams(lr=0.1))


# Entry points without the native part: their own checks.
WITHOUT = """
import sys, types, warnings
import torch
import paper_2505_23725_amd as mlc
name = "paper_2505_23725_amd._marshal"
{plant}
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    for call in (lambda: mlc.newton_schulz_static_scratch(torch.zeros(8, 8), torch.zeros(8, 8)),
                 lambda: mlc.muloco_adamw_step([(torch.zeros(8),) * 4], mlc.AdamWHParams(lr=0.1))):
        try:
            call()
        except ValueError as e:
            assert "must live on the GPU" in str(e), e
        else:
            raise AssertionError("not refused")
told = [str(w.message) for w in seen if "_marshal.so" in str(w.message)]
assert len(told) == 1 and "python -m paper_2505_23725_amd.build" in told[0] and {reason!r} in told[0], told
print("done")
"""


@pytest.mark.parametrize("plant,reason", [
    ("sys.modules[name] = None", "_marshal"),
    ("other = types.ModuleType(name); other.torch_version = '0.1'; other.pointer = lambda t: 1 / 0; "
     "sys.modules[name] = other; mlc._marshal = other", "built for torch 0.1"),
])
def test_calls_without_the_native_part(plant, reason):
    """Not built, or built for another torch: tensors are checked in Python, and one warning says what is missing."""
    done = subprocess.run([sys.executable, "-c", WITHOUT.format(plant=plant, reason=reason)], cwd=ROOT,
                          capture_output=True, text=True)
    assert done.returncode == 0 and "done" in done.stdout, done.stderr


def test_native_part_is_built_for_this_torch():
    from paper_2505_23725_amd import _marshal, binding
    assert _marshal.torch_version == torch.__version__
    assert binding._marshal() is _marshal


def test_tables_of_another_layout_are_refused(monkeypatch):
    """A table whose entries are longer than the binding's is from another header: none of it reaches the library."""
    from paper_2505_23725_amd import binding
    size = binding.C.sizeof(binding._AdamWGroup)
    monkeypatch.setattr(binding, "_native", type("Longer", (), {"adamw_groups": staticmethod(lambda t: bytes(len(t) * (size + 8)))}))
    with pytest.raises(RuntimeError, match="another muloco.h"):
        mlc.muloco_adamw_step([(torch.zeros(8),) * 4] * 2, mlc.AdamWHParams(lr=0.1))


def test_native_part_fills_the_header_s_structure():
    """The entry is the header's own type, which the binding's is checked against (test_c_header.py), and no copy of it."""
    source = open(os.path.join(ROOT, "paper_2505_23725_amd", "csrc", "marshal.cpp")).read()
    assert '#include "muloco.h"' in source and "struct " not in source
    for field in ("count", "param", "param_dtype", "grad", "grad_dtype", "exp_avg", "exp_avg_sq"):
        assert f"g.{field} = " in source
