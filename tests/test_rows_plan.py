"""The row-wise decoder's launch plan (rows per block, LDS layout) on the CPU:
every row in a block, no more rows than waves, regions that do not overlap and
fit a CU's 160 KB, over the sizes a session can have."""
import itertools
import subprocess

import pytest

from .conftest import ROOT

MAIN = r"""
#include <cstdio>
#include "rows_plan.hpp"
using namespace mnmt;
int main() {
  RowsSizes g;
  while (std::scanf("%d %d %d %d %d %d %d", &g.R, &g.d, &g.h, &g.F, &g.T, &g.S, &g.t) == 7) {
    const RowsPlan p = rows_plan(g);
    std::printf("%d %d %d %d %d %d %d %d %d %d %d\n", p.rows, p.blocks, p.lds.ln, p.lds.a, p.lds.hist, p.lds.act,
                p.lds.p, p.lds.np, p.lds.total, rows_waves(g.d), kVtBytes);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", f"{ROOT}/paper_2306_04235_amd/csrc", str(d / "main.cpp"), "-o",
                    str(d / "plan")], check=True)

    def run(cases):
        text = "\n".join(" ".join(map(str, c)) for c in cases) + "\n"
        out = subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, ln.split())) for ln in out.splitlines()]

    return run


def test_rows_and_lds_over_the_range(plan):
    cases = []
    for d, ratio, dh in itertools.product((64, 128, 256, 384, 512), (2, 4), (16, 32, 48, 64)):
        if d % dh:
            continue
        for T, S in ((1, 1), (64, 9), (65, 64), (130, 256), (200, 9), (256, 256)):
            for t in {-1, 0, 62, 63, 64, 127, 191, 192, T - 1}:
                if t < T:
                    cases += [(R, d, d // dh, ratio * d, T, S, t)
                              for R in (1, 3, 16, 255, 256, 257, 600, 1025, 2050, 3073, 4090, 4096, 4097, 9001)]
    got = plan(cases)
    assert len(got) == len(cases)
    for (R, d, h, F, T, S, t), (rows, blocks, ln, a, hist, act, p, np_, total, waves, vt) in zip(cases, got):
        where = f"R={R} d={d} h={h} F={F} T={T} S={S} t={t}"
        assert 1 <= rows <= waves and (blocks - 1) * rows < R <= blocks * rows, where
        keys = max(T if t < 0 else t + 1, S)
        assert np_ >= keys and np_ % 64 == 0, where
        # xs (fp32 rows, padded), LayerNorm constants, int8 rows, histories, q|k|v rows, attention scratch
        assert ln >= rows * (d + 4) * 4 and a >= ln + 6 * d * 4 and hist >= a + rows * (d + 16), where
        assert act >= hist + rows * ((T + 63) // 64 * 64) and p >= act + rows * (3 * d + 16), where
        assert total >= p + min(waves, rows * h) * (np_ * 4 + vt) and total >= act + rows * (F + 16), where
        assert all(x % 16 == 0 for x in (ln, a, hist, act, p)) and total <= 160 * 1024, where


def test_rows_per_block(plan):
    """As few rows as keep one block per CU; two rounds of blocks where one
    would need more rows than a block has waves or LDS for (d 512, from 128
    positions on: 15 rows at most)."""
    sizes = lambda R, t=0, d=256, F=1024, T=64: (R, d, d // 64, F, T, 9, t)  # noqa: E731
    rows = [p[:2] for p in plan([sizes(4), sizes(256), sizes(512), sizes(4090), sizes(4097),
                                 sizes(4090, 127, 512, 2048, 200), sizes(4090, 128, 512, 2048, 200),
                                 sizes(4090, -1, 512, 2048, 200)])]
    assert rows == [(1, 4), (1, 256), (2, 256), (16, 256), (9, 456), (16, 256), (8, 512), (8, 512)]
