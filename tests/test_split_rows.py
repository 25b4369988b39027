"""Keys split four ways: while every workgroup has a CU to itself a block of 64 rows is two workgroups' work, whose
wavefronts have tiles of their own; otherwise one's.  On both sides of that line a head's output is the same bits, and the
oracle's within the suite's bounds, where the last block has rows in its second half and where it has none, with and
without text, with the masks of all patterns, with more groups than tiles and with a tile left over."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2505_21036_amd as rf
import rf_inputs as inp
from attn_forms import attention_as

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("lay,text_first", [((2, 3, 5, 0), False), ((3, 7, 9, 5), False), ((2, 8, 10, 0), False), ((4, 9, 13, 45), False),
                                            ((4, 9, 13, 45), True), ((5, 11, 8, 0), False), ((7, 10, 13, 50), False)])
def test_both_ways_of_a_block(D, lay, text_first):
    T, H, W, tl = lay
    print("case", D, lay, text_first, flush=True)
    nH = 4
    rl, ol = rf.rf_layout(T, H, W, tl), orc.Layout(T, H, W, tl)
    rp = rf.rf_params(0.25, 0.25, 2, 0, rf.RF_FLAG_TEXT_FIRST if text_first else 0)
    w = inp.Workload("split_rows", 1, nH, D, T, H, W, tl, 64, 9300 + D + T)
    shift, scale = (tl if text_first else 0), 5.0
    Q, K, V = (torch.roll(t, shift, dims=2).contiguous() for t in inp.full_qkv(w, "cuda:0", scale))
    classes = torch.arange(nH, dtype=torch.int32, device="cuda").reshape(1, nH) % 4
    blocks = (w.N + 63) // 64
    assert nH * blocks <= 8 * 15  # 16 on an XCD at most: a CU for each half
    O = attention_as((64, 4, 0), Q, K, V, classes, rl, rp, out=torch.full_like(Q, float("nan")))
    # the same heads among so many that there are more workgroups than CUs
    times = 8 * 17 // (nH * blocks) + 1
    many = attention_as((64, 4, 0), *(t.repeat(1, times, 1, 1) for t in (Q, K, V)), classes.repeat(1, times), rl, rp)
    torch.cuda.synchronize()
    for i in range(times):
        assert torch.equal(many[:, i * nH:(i + 1) * nH], O), i
    for h in range(nH):
        q, k, v = (t.float().numpy() for t in inp.head_qkv(w, 0, h, scale))
        ref = orc.attention(q, k, v, h % 4, ol)  # text behind; the shift is the test's
        err = torch.roll(O[0, h], -shift, dims=0).double().cpu().numpy() - ref
        rel = np.linalg.norm(err) / np.linalg.norm(ref)
        assert np.abs(err).max() <= 2e-2 and np.abs(err).mean() <= 2e-3 and rel <= 5.2e-3, (h, rel)
