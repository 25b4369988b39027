"""What a call of rf_sparse_attention asks of the runtime and which kernel it launches with what, seen on the host side
alone (calls_driver.cpp counts the allocations and records the launches).  Contracts of include/rainfusion.h: after one
warm-up call for a (layout, params) no call allocates, whatever its heads, head_dim, block, workspace and dense flag."""
import os
import shutil
import subprocess

import pytest
import torch

import paper_2505_21036_amd as rf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP = "/opt/rocm/include"
needs_gxx = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(os.path.join(HIP, "hip", "hip_runtime.h")), reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe, csrc = str(tmp_path_factory.mktemp("calls") / "calls_driver"), os.path.join(ROOT, "paper_2505_21036_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-Wno-unused-result", "-I", HIP, "-I", os.path.join(ROOT, "include"), "-I", csrc,
                           os.path.join(ROOT, "tests", "calls_driver.cpp"), os.path.join(csrc, "rf_api.cpp"), os.path.join(csrc, "rf_plan.cpp"), "-o", exe])

    def run(calls):
        """calls: (layout 4-tuple, bandwidth, stride, flags, block, B, nH, D, full workspace) -> rows of the driver's output"""
        text = "\n".join(" ".join(str(v) for v in c[0] + tuple(int(x) if isinstance(x, bool) else x for x in c[1:])) for c in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        return [tuple(v if i == 7 else int(v) for i, v in enumerate(l.split())) for l in out]
    return run


LAYOUTS = [(4, 8, 8, 0), (7, 10, 13, 50), (9, 16, 28, 77), (13, 30, 45, 226), (33, 45, 80, 256), (3, 400, 500, 5)]


def every_call(layout, flags=0):
    return [(layout, 0.25, 2, flags | dense, block, B, nH, D, full) for dense in (0, rf.RF_FLAG_FORCE_DENSE) for block in (64, 384)
            for B, nH in ((1, 1), (1, 6), (2, 24), (4, 60)) for D in (64, 96, 128) for full in (False, True)]


@needs_gxx
@pytest.mark.parametrize("layout", LAYOUTS)
def test_one_warm_up_call_covers_every_later_call_of_the_layout(driver, layout):
    warm = (layout, 0.25, 2, 0, 128, 1, 1, 64, False)
    calls = every_call(layout) + every_call(layout, rf.RF_FLAG_FIXED_ORDER)
    out = driver([warm] + calls)
    assert all(r[0] == 0 and r[1] == 1 for r in out), sorted({r[:2] for r in out})
    assert len({r[2] for r in out}) > 1 or layout == LAYOUTS[-1]  # the calls do differ in their row counts


@pytest.mark.gpu
def test_a_capture_takes_other_forms_than_its_warm_up():
    """One head without a workspace warms up; the captured call has 60 heads and a full workspace."""
    print("case capture of another form", flush=True)
    layout = rf.rf_layout(5, 32, 33, 37)
    N = 5 * 32 * 33 + 37
    for D in (64, 128):
        g = torch.Generator(device="cuda")
        g.manual_seed(D)
        Q, K, V = (torch.randn(1, 60, N, D, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
        hc = (torch.arange(60, dtype=torch.int32) % 4).reshape(1, 60).cuda()
        O, ws = torch.empty_like(Q), torch.empty(rf.rf_attention_workspace_bytes(1, 60, D, layout), dtype=torch.uint8, device="cuda")
        rf.rf_plan_clear()
        rf.rf_sparse_attention(Q[:, :1].contiguous(), K[:, :1].contiguous(), V[:, :1].contiguous(), hc[:, :1].contiguous(), layout)
        torch.cuda.synchronize()
        params = rf.rf_params(0.25, 0.25, 2, 0, rf.RF_FLAG_FIXED_ORDER)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            rf.rf_sparse_attention(Q, K, V, hc, layout, None, 128, out=O, workspace=ws)
            fixed = rf.rf_sparse_attention(Q, K, V, hc, layout, params, 128, workspace=ws)
        for _ in range(3):
            O.zero_()
            fixed.zero_()
            graph.replay()
            torch.cuda.synchronize()
            want = rf.rf_sparse_attention(Q, K, V, hc, layout, params, 128, workspace=ws)
            assert torch.equal(fixed, want)
            assert (O.double() - want.double()).norm() <= 1e-2 * want.double().norm()  # bf16 weights at another reference
