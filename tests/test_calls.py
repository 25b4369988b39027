"""What a call of rf_sparse_attention asks of the runtime and which kernel it launches with what, seen on the host side
alone (calls_driver.cpp counts the allocations and records the launches).  Contracts of include/rainfusion.h: after one
warm-up call for a (layout, params) no call allocates, whatever its heads, head_dim, block, workspace and dense flag;
RF_FLAG_FIXED_ORDER gives a head the same bits in any call of the layout."""
import os
import resource
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

    def run(calls, memory=None):
        """memory: limit on the process's address space, bytes; calls: (layout 4-tuple, bandwidth, stride, flags, block, B, nH, D, full workspace) -> rows of the driver's output"""
        text = "\n".join(" ".join(str(v) for v in c[0] + tuple(int(x) if isinstance(x, bool) else x for x in c[1:])) for c in calls)
        limit = (lambda: resource.setrlimit(resource.RLIMIT_AS, (memory, memory))) if memory else None
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, preexec_fn=limit).stdout.splitlines()
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


@needs_gxx
def test_lists_that_do_not_fit_in_host_memory_are_an_error_and_leave_the_library_usable(driver):
    long, short = (33, 200, 300, 0), LAYOUTS[1]
    out = driver([(long, 0.25, 2, 0, 128, 1, 1, 64, False), (short, 0.25, 2, 0, 128, 1, 1, 64, False)], memory=256 << 20)
    assert out[0][:2] == (-7, 0) and out[1][:2] == (0, 1), out  # RF_ERR_HIP, then as ever


@needs_gxx
@pytest.mark.parametrize("layout", LAYOUTS)
def test_fixed_order_takes_one_form_per_layout_and_head_dim(driver, layout):
    calls = every_call(layout, rf.RF_FLAG_FIXED_ORDER)
    out = driver(calls)
    for D in (64, 96, 128):
        assert len({(r[2], r[3], r[4], r[6], r[7]) for r, c in zip(out, calls) if c[7] == D}) == 1, D


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("T,H,W,tl", [(4, 8, 8, 0), (7, 10, 13, 50), (5, 32, 33, 37), (6, 64, 65, 11)])
def test_fixed_order_bits_do_not_depend_on_the_other_heads(D, T, H, W, tl):
    """Bitwise: a head alone, in a batch, with and without a workspace; all heads dense by class and by flag."""
    print("case fixed order", D, (T, H, W, tl), flush=True)
    layout, N, nH = rf.rf_layout(T, H, W, tl), T * H * W + tl, 30
    params = rf.rf_params(0.25, 0.25, 2, 0, rf.RF_FLAG_FIXED_ORDER)
    flagged = rf.rf_params(0.25, 0.25, 2, 0, rf.RF_FLAG_FIXED_ORDER | rf.RF_FLAG_FORCE_DENSE)
    g = torch.Generator(device="cuda")
    g.manual_seed(D + N)
    Q, K, V = (torch.randn(2, nH // 2, N, D, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    hc = (torch.arange(nH, dtype=torch.int32) % 4).reshape(2, nH // 2).cuda()
    ws = torch.empty(rf.rf_attention_workspace_bytes(2, nH // 2, D, layout), dtype=torch.uint8, device="cuda")
    want = rf.rf_sparse_attention(Q, K, V, hc, layout, params, 128)
    assert torch.equal(want, rf.rf_sparse_attention(Q, K, V, hc, layout, params, 256, workspace=ws))
    for b, h0, n in ((0, 0, 1), (0, 1, 1), (1, 2, 1), (1, 3, 4), (0, 0, nH // 2)):
        part = [t[b:b + 1, h0:h0 + n].contiguous() for t in (Q, K, V, hc)]
        for workspace in (None, ws):
            got = rf.rf_sparse_attention(*part, layout, params, 64, workspace=workspace)
            assert torch.equal(got[0], want[b, h0:h0 + n]), (b, h0, n)
    dense = rf.rf_sparse_attention(Q, K, V, torch.full_like(hc, rf.RF_DENSE), layout, params, workspace=ws)
    assert torch.equal(dense, rf.rf_sparse_attention(Q, K, V, None, layout, flagged))
    assert torch.equal(dense[0, 3], want[0, 3])


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
