"""256-row blocks at head_dim 64 without copies of K and V: Temporal heads gathered in position-major order, Textural
heads through the compacted index, by wavefronts of 64 rows."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2505_21036_amd as rf
import rf_inputs as inp
from paper_2505_21036_amd.binding import attention_form

D = 64
# (layout, heads): no text; a ragged last block; text whose blocks walk every tile, in both places
CASES = [((8, 32, 33, 0), 14, False), ((12, 30, 31, 0), 11, False), ((5, 48, 49, 19), 29, False), ((5, 48, 49, 19), 29, True)]


@pytest.mark.gpu
@pytest.mark.parametrize("lay,nH,text_first", CASES)
def test_wide_rows_gather_against_the_oracle(lay, nH, text_first):
    T, H, W, tl = lay
    print("case", lay, nH, text_first, flush=True)
    w = inp.Workload("wide_gather", 1, nH, D, T, H, W, tl, 64, 9100 + tl)
    rl, ol = rf.rf_layout(T, H, W, tl), orc.Layout(T, H, W, tl)
    rp, op = rf.rf_params(0.25, 0.25, 2, 0, rf.RF_FLAG_TEXT_FIRST if text_first else 0), orc.Params(text_first=text_first)
    assert attention_form(1, nH, D, rl, rp) == (256, 1, True, False)
    shift, scale = (tl if text_first else 0), 5.0
    Q, K, V = (torch.roll(t, shift, dims=2).contiguous() for t in inp.full_qkv(w, "cuda:0", scale))
    classes = [i % 4 for i in range(nH)]
    hc = torch.as_tensor(classes, dtype=torch.int32).reshape(1, nH).cuda()
    O = rf.rf_sparse_attention(Q, K, V, hc, rl, rp, 128, out=torch.full_like(Q, float("nan")))
    torch.cuda.synchronize()
    assert torch.isfinite(O).all()  # every row of every head is written
    for i in (0, 1, 2, 3, nH - 1):
        q, k, v = (np.roll(t.float().numpy(), shift, axis=0) for t in inp.head_qkv(w, 0, i, scale))
        ref = orc.attention(q, k, v, classes[i], ol, op)
        err = O[0, i].double().cpu().numpy() - ref
        rel = np.linalg.norm(err) / np.linalg.norm(ref)
        assert np.abs(err).max() <= 2e-2 and np.abs(err).mean() <= 2e-3 and rel <= 5.2e-3, (i, rel)  # the suite's bounds
