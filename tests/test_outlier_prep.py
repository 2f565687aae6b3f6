"""The launch that prepares a prefill-size linear's outlier columns has a wave for every group of 1024 columns, whatever the
shape of the linear: the list of more than 64 outlier columns is written by the wave of the group's number."""
import os
import shutil
import subprocess

import pytest

from paper_2209_01188_amd import build

PROGRAM = r"""
#include <cstdio>
#include "outlier_prep.h"
int main() {
    int bad = 0, count = 0;
    for (int N = 64; N <= 65536; N += N < 2048 ? 64 : 4096)          // the linears of every span there can be
        for (int K = 64; K <= 65536; K += 64)
            for (int M : {65, 66, 128, 513, 2048}) {
                OutlierPrep p{};
                p.w.N = N;
                p.w.K = K;
                p.count = &count;
                const int items = outlier_prep_items(p, M);
                if (items * 1024 < K || items < N / 16 + (M + 15) / 16) { if (!bad++) printf("N %d K %d M %d: %d waves\n", N, K, M, items); }
                p.count = nullptr;
                if (outlier_prep_items(p, M) != 0) bad++;
            }
    printf("bad %d\n", bad);
}
"""


def test_every_group_of_columns_has_a_wave(tmp_path):
    if not shutil.which(build.HIPCC):
        pytest.skip("needs hipcc")
    src = tmp_path / "t.hip"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "-O1", "--cuda-host-only", "-std=c++17", "-I", build.CSRC, "-o", str(tmp_path / "t"), str(src)], check=True)
    out = subprocess.run([str(tmp_path / "t")], check=True, capture_output=True, text=True).stdout
    assert out.strip() == "bad 0", out
