"""workload.FitWorkspace, by which the benchmark and the tests read a workspace that fit+score has used, against the library's own structures:
a host program compiled from its headers prints them."""
import os
import subprocess

import pytest

from paper_2605_26660_amd import build, workload

SHAPES = [(512, 512, 64, 0, 20), (1000, 1056, 96, 0, 10), (11008, 4096, 128, 0, 20), (256, 24, 8, 128, 1), (4200, 8192, 256, 0, 64), (1024, 1024, 512, 128, 16)]

PROGRAM = """
#include "windq_fit.hpp"
#include <cstddef>
#include <cstdio>
using namespace windq;
int main() {
    const int64_t shapes[][5] = {%s};
    for (const auto& s : shapes) {
        Geometry g;
        g.rows = s[0]; g.cols = g.ld = s[1]; g.chunk_w = (int32_t)s[2]; g.R_u = s[3] ? s[3] : s[0];
        g.n_chunks = g.cols / g.chunk_w; g.n_rb = g.rows / g.R_u; g.U = g.n_rb * g.n_chunks;
        g.tiles_per_unit = (g.R_u + TILE_ROWS - 1) / TILE_ROWS; g.n_tiles = g.U * g.tiles_per_unit;
        const int32_t K = (int32_t)s[4];
        const FitScoreLayout L = fit_score_layout(g, K);
        std::printf("%%zu %%d %%d %%zu %%zu %%zu %%d %%d %%zu %%zu %%d", L.partial, fit_score_ncand(K), fit_score_noise_slot(K), L.redo_count, L.redo_list, L.colsel,
                    colsel_words(g.chunk_w), g.chunk_w + FS_HMAX, fit_score_noise_slot(K) * sizeof(double) + offsetof(FitPlan, low),
                    fit_score_noise_slot(K) * sizeof(double) + offsetof(FitPlan, high), PLAN_STEPS);
        for (int i = 0; i < PLAN_STEPS; ++i) std::printf(" %%d", plan_columns(g.chunk_w, i));
        std::printf("\\n");
    }
}
size_t windq::round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
"""


def test_layout_is_the_librarys(tmp_path):
    src = tmp_path / "layout.hip"
    src.write_text(PROGRAM % ", ".join("{%s}" % ", ".join(map(str, s)) for s in SHAPES))
    exe = tmp_path / "layout"
    try:
        hipcc = build.hipcc_path()
    except RuntimeError:
        pytest.skip("no hipcc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(lines) == len(SHAPES)
    for (rows, cols, G, unit_rows, K), line in zip(SHAPES, lines):
        L = workload.FitWorkspace(rows, cols, G, unit_rows, K)
        mine = [L.partial, L.n_sums, L.noise_slot, L.redo_count, L.redo_list, L.colsel, L.record_words, L.count_word, L.plan_low, L.plan_high, L.plan_steps]
        assert mine + workload.plan_columns(G) == [int(v) for v in line.split()]
