"""Which rows the quantised outer update gives a workgroup of their own size: csrc/quant_rule.h compiled for the host (no
GPU needed), held to measured points."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "quant_rule.h"
int main() {
  long n;
  int K, bits, f32, gbf, ef, second;
  while (std::scanf("%ld %d %d %d %d %d %d", &n, &K, &bits, &f32, &gbf, &ef, &second) == 7)
    std::printf("%d\n", mlc::quant_whole_row(mlc::QuantRow{n, K, bits, f32 != 0, gbf != 0, ef != 0, second != 0}));
}
"""

# row length, replicas, bits, fp32 replicas, bf16 global copy, error feedback, second quantisation; time of a workgroup
# of the row's size over that of 256 threads (26 M elements * 4 / (K + 3))
MEASURED = [
    (2056, 4, 4, 0, 0, 0, 0, 0.91), (2056, 8, 8, 0, 1, 0, 0, 0.87), (2560, 16, 8, 0, 0, 0, 0, 0.90),
    (2056, 4, 8, 1, 0, 0, 0, 1.04), (2056, 16, 8, 1, 0, 0, 0, 1.10), (2056, 32, 8, 0, 0, 1, 0, 1.05),
    (2808, 5, 4, 0, 0, 1, 0, 1.05), (3072, 32, 8, 0, 1, 0, 0, 1.03), (3001, 16, 8, 0, 0, 0, 0, 1.11),
    (2402, 4, 8, 0, 1, 0, 0, 0.95), (2523, 3, 8, 0, 0, 1, 0, 0.96), (2601, 12, 8, 0, 0, 0, 0, 1.06),
    (2901, 6, 8, 0, 0, 1, 0, 1.03), (2901, 5, 8, 0, 0, 0, 0, 0.96), (2049, 16, 8, 1, 0, 0, 0, 1.07),
    (3073, 4, 8, 0, 0, 0, 0, 1.05), (3073, 32, 8, 0, 0, 0, 0, 1.12), (4096, 16, 4, 0, 0, 1, 0, 1.06),
    (4104, 1, 4, 0, 0, 0, 0, 0.80), (4104, 4, 8, 0, 1, 0, 0, 0.83), (4104, 16, 8, 0, 1, 0, 0, 1.13),
    (4601, 8, 8, 1, 0, 0, 0, 0.64), (4601, 4, 8, 0, 1, 0, 0, 0.72), (5001, 1, 8, 0, 0, 0, 0, 0.90),
    (5001, 4, 8, 0, 0, 0, 0, 1.06), (5001, 4, 8, 0, 0, 1, 0, 1.07), (5001, 32, 8, 1, 0, 1, 0, 0.70),
    (5120, 4, 4, 0, 0, 0, 0, 0.93), (5120, 16, 4, 0, 0, 0, 0, 1.05), (5120, 6, 4, 0, 0, 0, 1, 1.03),
    (6144, 1, 4, 0, 0, 0, 0, 0.86), (6144, 2, 8, 0, 0, 1, 0, 0.95), (6144, 2, 4, 0, 0, 0, 1, 1.03),
    (6152, 5, 4, 0, 0, 0, 0, 1.04), (6152, 8, 2, 0, 0, 0, 0, 1.09), (6152, 4, 8, 0, 0, 1, 0, 0.90),
    (6600, 4, 8, 0, 0, 0, 0, 1.03), (7001, 8, 8, 0, 0, 1, 0, 0.92), (7168, 4, 4, 0, 0, 0, 1, 1.04),
    (8001, 2, 8, 0, 0, 0, 0, 0.82), (8001, 16, 8, 0, 0, 0, 0, 1.03), (8001, 32, 8, 1, 0, 0, 0, 0.70),
    (8192, 2, 8, 0, 0, 1, 0, 0.93), (8192, 4, 4, 0, 0, 0, 0, 0.95), (8192, 8, 4, 0, 0, 0, 0, 1.04),
    (8192, 32, 4, 0, 0, 0, 0, 1.16), (12296, 1, 4, 0, 0, 0, 0, 0.80), (12289, 8, 8, 0, 1, 0, 0, 0.62),
    (16384, 32, 8, 0, 0, 1, 0, 0.71), (24576, 4, 4, 0, 0, 0, 0, 0.79),
]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("quant_rule")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run([gxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2505_23725_amd", "csrc"),
                    str(d / "main.cpp"), "-o", str(d / "rule")], check=True)

    def ask(rows):
        text = "\n".join(" ".join(str(int(x)) for x in r) for r in rows)
        out = subprocess.run([str(d / "rule")], input=text, capture_output=True, text=True, check=True)
        return [int(x) for x in out.stdout.split()]
    return ask


def test_no_row_takes_the_slower_workgroup(rule):
    for row, vectors in zip(MEASURED, rule([r[:7] for r in MEASURED])):
        assert (vectors > 0) == (row[7] < 1), row


def test_a_row_fits_its_workgroup(rule):
    rows = [(n, K, 8, f32, gbf, ef, 0) for n in range(1, 24577, 7) for K in (1, 3, 8, 32)
            for f32, gbf, ef in ((0, 0, 0), (1, 0, 0), (0, 1, 1))]
    for row, vectors in zip(rows, rule(rows)):
        assert vectors in (0, 2, 3)
        if vectors:
            assert -(-row[0] // (vectors * 512)) * 64 <= 1024, row
        else:
            assert row[0] <= 12288, row          # 256 threads hold at most six vectors each
