"""The banded lists and the position-major table by arithmetic (rf_band.h), as the kernels that split the keys of 64-row blocks
have them, against the lists and the table that build_plan makes: every entry of every block of 64 rows (and of 128 and 256, at
which no kernel works them out: the arithmetic does not depend on it) and every row, over layouts with and without text, in front and behind, frames and positions that tiles divide and that they do
not, one frame, one position, and bands from nothing to everything."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def test_bands_and_rows_are_those_of_the_plan(tmp_path):
    exe, csrc = str(tmp_path / "band_driver"), os.path.join(ROOT, "paper_2505_21036_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-static-libubsan",
                           "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(ROOT, "tests", "band_driver.cpp"),
                           os.path.join(csrc, "rf_plan.cpp"), "-o", exe])
    layouts = [(1, 1, 1), (1, 7, 9), (2, 1, 1), (300, 1, 2), (4, 8, 8), (7, 10, 13), (9, 16, 28), (3, 45, 80), (33, 5, 7), (13, 30, 45), (517, 3, 1), (16, 32, 32)]
    cases = [(*l, text, bw, first) for l in layouts for text in (0, 1, 50, 63, 64, 77, 226) for bw in (0.0, 0.1, 0.25, 0.5, 1.0) for first in ((0, 1) if text else (0,))]
    run = subprocess.run([exe], input="\n".join("%d %d %d %d %f %d" % c for c in cases), capture_output=True, text=True)
    lines = run.stdout.split()
    assert run.returncode == 0, (run.stdout[-200:], run.stderr[-200:], cases[len(lines)] if len(lines) < len(cases) else None)
    assert len(lines) == len(cases) and all(int(n) > 0 for n in lines)


def test_rows_of_the_longest_sequences(tmp_path):
    """2^24 tokens: the quotient's error is largest where rows are many and positions few frames long."""
    src = tmp_path / "rows.cpp"
    src.write_text("""#include "rf_band.h"
#include <cstdio>
int main() {
    const int N = 1 << 24;
    for (int T : {1, 2, 3, 7, 33, 127, 4095, 65537, 8388607, 16777216}) {
        const int HW = N / T, Nv = HW * T;
        for (int n = 0; n < Nv; n += n < 70000 || n > Nv - 70000 ? 1 : 61)
            if (rf::position_major_row(n, T, HW, Nv, 0, 0) != static_cast<long long>(n % T) * HW + n / T) return std::printf("%d %d", T, n), 2;
    }
    return 0;
}
""")
    exe = str(tmp_path / "rows")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2505_21036_amd", "csrc"), str(src), "-o", exe])
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_plans_without_banded_lists(tmp_path):
    """As blocks of 64 rows have them on the device: the banded lists are empty, the rest is the whole plan's."""
    src = tmp_path / "parts.cpp"
    src.write_text("""#include <cstdio>
#include "rf_internal.h"
int main() {
    for (const rf_layout layout : {rf_layout{13, 30, 45, 226}, rf_layout{4, 8, 8, 0}, rf_layout{3, 7, 9, 40}, rf_layout{1, 1, 1, 1}}) {
        rf::Geometry g;
        if (rf::resolve_geometry(&layout, nullptr, &g) != RF_OK) return 1;
        rf::TokenTables tables;
        rf::build_tables(g, &tables);
        rf::HostPlan whole, some;
        rf::build_plan(g, tables, 64, false, &whole);
        rf::build_plan(g, tables, 64, false, &some, false);
        if (some.row_ptr[RF_TEXTURAL] != whole.row_ptr[RF_TEXTURAL] || some.cols[RF_TEXTURAL] != whole.cols[RF_TEXTURAL]) return 2;
        if (some.nQB != whole.nQB || some.nKT != whole.nKT || some.nCT != whole.nCT || some.first_text_qb != whole.first_text_qb) return 3;
        for (int c = 0; c < rf::kLists; ++c)
            if (c != RF_TEXTURAL && (!some.cols[c].empty() || some.row_ptr[c] != std::vector<int32_t>(some.nQB + 1, 0))) return 4;
    }
    return 0;
}
""")
    exe, csrc = str(tmp_path / "parts"), os.path.join(ROOT, "paper_2505_21036_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", csrc, str(src), os.path.join(csrc, "rf_plan.cpp"), "-o", exe])
    subprocess.check_call([exe])


@pytest.mark.gpu
def test_device_memory_of_a_long_layouts_plans():
    """119056 tokens: 14.3 MB; with the banded lists of 64-row blocks, which no kernel reads, it would be 26.7."""
    import torch

    import paper_2505_21036_amd as rf
    lay = rf.rf_layout(33, 45, 80, 256)
    Q = torch.randn(1, 1, 119056, 64, device="cuda").bfloat16()
    classes, out = torch.zeros(1, 1, dtype=torch.int32, device="cuda"), torch.empty_like(Q)
    ws = torch.empty(rf.RF_ATTENTION_MIN_WORKSPACE, dtype=torch.uint8, device="cuda")
    rf.rf_sparse_attention(Q, Q, Q, classes, lay, rf.rf_params(0.5, 0.5, 2, 0, 0), 128, out=out, workspace=ws)  # code and plans of another
    rf.rf_plan_clear()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    rf.rf_sparse_attention(Q, Q, Q, classes, lay, None, 128, out=out, workspace=ws)
    torch.cuda.synchronize()
    assert 10e6 < before - torch.cuda.mem_get_info()[0] < 20e6
