"""The words at the start of the workspace (eight work-queue counters, 64 sweep words) are reset by every call from
queues, whatever an earlier call or the allocator left there.  Under RF_FLAG_FIXED_ORDER no workgroup publishes its
walk, so after the call the sweep words read as they were reset.  RF_FLAG_WIDE_ROWS: always from queues."""
import pytest
import torch

import paper_2505_21036_amd as rf
import rf_inputs as inp

pytestmark = pytest.mark.gpu


def test_every_queue_word_is_reset():
    w = inp.WORKLOADS["ragged128"]
    print("case queue reset", flush=True)
    Q, K, V = inp.full_qkv(w, "cuda:0")
    rl = rf.rf_layout(w.T, w.H, w.W, w.text_len)
    ws = torch.empty(rf.RF_ATTENTION_MIN_WORKSPACE, dtype=torch.uint8, device="cuda")
    hc = torch.zeros(w.B, w.nH, dtype=torch.int32, device="cuda")
    params = rf.rf_params(0.25, 0.25, 2, 0, rf.RF_FLAG_FIXED_ORDER | rf.RF_FLAG_WIDE_ROWS)
    for poison in (0x7fffffff, 0, 5 << 18):
        words = ws.view(torch.int32)
        words.fill_(poison)
        rf.rf_sparse_attention(Q, K, V, hc, rl, params, 256, workspace=ws)
        got = words.cpu().tolist()
        assert min(got[:8]) >= 0 and sum(got[:8]) >= w.B * w.nH * 4 and max(got[:8]) < 10000, got[:8]  # 4 blocks per head
        assert got[8:72] == [-1] * 64, got[8:72]
