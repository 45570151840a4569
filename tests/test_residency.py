"""The residency table of the decode grids (host code): the answers of the
runtime for every size, and few questions however many sizes are asked for."""
from __future__ import annotations

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_15652_amd", "csrc")

MAIN = r"""
#include "residency.h"
#include <stdio.h>
#include <stdlib.h>

static mq_host::ResidencyTable table;
static int asked = 0;

static int answer(int kernel, size_t lds) {          // falls with the LDS size, in granules
    const size_t a = ((kernel + 1) * 8240 + lds + 1279) / 1280 * 1280, n = 163840 / a;
    return n > 4 ? 4 : (int)n;
}

int main() {
    static const char kernels[40] = {};
    srand(7);
    for (int i = 0; i < 20000; ++i) {
        const int k = rand() % 3;
        const size_t lds = (size_t)96 * (1 + rand() % 680);
        const int want = answer(k, lds);
        if (table.get(&kernels[k], lds, [&] { ++asked; return want; }) != want) return printf("wrong at %d\n", i), 1;
    }
    const int settled = asked;
    if (settled > 200) return printf("asked %d times\n", settled), 1;
    // a failed query gives one and is not remembered
    if (table.get(&kernels[3], 96, [] { return 0; }) != 1) return printf("failure\n"), 1;
    if (table.get(&kernels[3], 96, [] { return 3; }) != 3) return printf("failure remembered\n"), 1;
    // more kernels than rows: the answers stay right
    for (int k = 4; k < 40; ++k)
        for (int r = 0; r < 2; ++r)
            if (table.get(&kernels[k], 960, [&] { return 1 + k % 4; }) != 1 + k % 4) return printf("full\n"), 1;
    printf("ok %d\n", settled);
    return 0;
}
"""


def test_residency_table(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
