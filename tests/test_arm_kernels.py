"""The two forms of the ARM's recall kernel (keys split over four groups of wavefronts for small launches, one
group otherwise) on either side of the rule between them, at ragged sample counts, with one and with several
candidate bandwidths, against the oracle on some heads.  Bound 1e-5: the weights are exponentials of scores of up
to ~20 in base 2 formed in 32 bits (relative error ~20 * 2^-24 each), summed in 32 bits."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_2505_21036_amd as rf
import rf_inputs as inp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("nH", [1, 150])  # 150 heads of 130 samples: 300 workgroups with both passes, 600 apart
@pytest.mark.parametrize("T,H,W,omega", [(7, 10, 13, 0), (3, 9, 17, 2), (5, 11, 6, 1)])
def test_recalls_of_both_forms(D, nH, T, H, W, omega):
    print("case arm forms", D, nH, T, H, W, omega, flush=True)
    w = inp.Workload("arm", 1, nH, D, T, H, W, 21, 64, 8000 + D + nH + T)
    rl, ol = rf.rf_layout(T, H, W, 21), orc.Layout(T, H, W, 21)
    rp, op = rf.rf_params(0.25, 0.2, 2, omega, 0), orc.Params(0.25, 0.2, 2, omega)
    Q, K, _ = inp.full_qkv(w, "cuda:0", 4.0)
    bws = [0.5, 0.125, 0.3, 0.0]
    for mode in (rf.RF_SAMPLE_FIRST_FRAME, rf.RF_SAMPLE_EQUAL_INTERVAL):
        _, rec = rf.rf_arm_classify(Q, K, rl, rp, mode, 0.9)
        _, _, recp = rf.rf_arm_classify_plus(Q, K, rl, rp, mode, 0.9, bws)
        rec, recp = rec.cpu().numpy()[0], recp.cpu().numpy()[0]
        for h in sorted({0, nH // 2, nH - 1}):
            q, k, _ = (t.float().numpy() for t in inp.head_qkv(w, 0, h, 4.0))
            want = orc.arm_classify(q, k, ol, op, mode, 0.9)[1]
            assert np.abs(rec[h] - np.array(want)).max() <= 1e-5, (h, rec[h], want)
            wantp = orc.arm_classify_plus(q, k, ol, op, mode, 0.9, bws)[2]
            assert np.abs(recp[h] - wantp).max() <= 1e-5, (h, recp[h], wantp)


# Frames and positions are carried from tile to tile: positions up to 67599 and frames up to 516, strides that cross
# many frames between samples or none, samples that end inside a tile, one sample alone and two at the far ends, a stride
# beyond every token; 40 heads of 858 samples are in one group of wavefronts, the others split their keys over four.
@pytest.mark.parametrize("D,nH,T,H,W,omega", [(64, 1, 2, 260, 260, 997), (128, 2, 2, 260, 260, 4001), (96, 3, 300, 4, 5, 7),
                                              (64, 40, 300, 4, 5, 7), (128, 5, 300, 4, 5, 33), (96, 2, 6, 9, 11, 1 << 30),
                                              (128, 2, 6, 9, 11, 593), (64, 2, 1, 31, 33, 1), (96, 2, 517, 1, 2, 1)])
def test_attributes_of_any_size(D, nH, T, H, W, omega):
    print("case arm attributes", D, nH, T, H, W, omega, flush=True)
    w = inp.Workload("arm_digits", 1, nH, D, T, H, W, 3, 64, 8500 + D + nH + T)
    rl, ol = rf.rf_layout(T, H, W, 3), orc.Layout(T, H, W, 3)
    Q, K, _ = inp.full_qkv(w, "cuda:0", 4.0)
    mode, bws = rf.RF_SAMPLE_EQUAL_INTERVAL, [0.5, 0.125, 0.003, 0.0]
    for bs, bt in ((0.25, 0.2), (0.01, 0.0)):
        rp, op = rf.rf_params(bs, bt, 2, omega, 0), orc.Params(bs, bt, 2, omega)
        _, rec = rf.rf_arm_classify(Q, K, rl, rp, mode, 0.9)
        _, _, recp = rf.rf_arm_classify_plus(Q, K, rl, rp, mode, 0.9, bws)
        rec, recp = rec.cpu().numpy()[0], recp.cpu().numpy()[0]
        for h in sorted({0, nH - 1}):
            q, k, _ = (t.float().numpy() for t in inp.head_qkv(w, 0, h, 4.0))
            want = orc.arm_classify(q, k, ol, op, mode, 0.9)[1]
            assert np.abs(rec[h] - np.array(want)).max() <= 1e-5, (h, rec[h], want)
            wantp = orc.arm_classify_plus(q, k, ol, op, mode, 0.9, bws)[2]
            assert np.abs(recp[h] - wantp).max() <= 1e-5, (h, recp[h], wantp)
