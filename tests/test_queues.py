"""The division of an attention launch's items over the eight XCDs (rf_queues.h, host arithmetic asked through a small
driver): every (head, block) exactly once, equal counts, text-holding blocks first, and, in the order of the launches
whose XCDs cannot help each other, equal work however the heads' classes lie."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EIGHTHS, HEADS, DEALT = 0, 1, 2
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def queues(tmp_path, cases):
    """[[(head, ordinal), ...] per XCD] for each (heads, video blocks, text blocks, order)."""
    exe = str(tmp_path / "queues_driver")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-static-libubsan", "-I", os.path.join(ROOT, "paper_2505_21036_amd", "csrc"),
                           os.path.join(ROOT, "tests", "queues_driver.cpp"), "-o", exe])
    out = subprocess.run([exe], input="\n".join("%d %d %d %d" % c for c in cases), capture_output=True, text=True, check=True).stdout.split("\n")
    line = lambda l: [tuple(int(v) for v in item.split(",")) for item in l.split()]  # noqa: E731
    return [[line(l) for l in out[8 * i:8 * i + 8]] for i in range(len(cases))]


def test_every_item_once_and_text_blocks_first(tmp_path):
    cases = [(bh, video, text, order) for bh in (1, 2, 7, 8, 9, 23, 24, 25, 31, 48, 60) for video in (0, 1, 4, 15, 64, 139)
             for text in (0, 1, 3) if video + text for order in (EIGHTHS, HEADS, DEALT)]
    for (bh, video, text, order), qs in zip(cases, queues(tmp_path, cases)):
        items = [i for q in qs for i in q]
        assert sorted(items) == [(h, o) for h in range(bh) for o in range(video + text)], (bh, video, text, order)
        for q in qs:  # ordinals below `text` are the blocks that hold text rows
            longs = [o < text for _, o in q]
            assert longs == sorted(longs, reverse=True)
        counts = [len(q) for q in qs]
        assert max(counts) == counts[0]  # what the launcher sizes the grid by
        if order == DEALT:
            assert max(counts) - min(counts) <= 4 + 1, (bh, video, text, counts)  # a run of blocks, a text block


# class of head i -> its blocks' work: Dense twice a sparse one's, as with bandwidths of a quarter
MIXES = {"one dense": lambda i, n: 2 if i == 0 else 1, "one dense in the middle": lambda i, n: 2 if i == n // 2 else 1,
         "first half dense": lambda i, n: 2 if 2 * i < n else 1, "every other dense": lambda i, n: 2 - i % 2,
         "every fourth dense": lambda i, n: 2 if i % 4 == 0 else 1, "every eighth dense": lambda i, n: 2 if i % 8 == 0 else 1,
         "first third dense": lambda i, n: 2 if 3 * i < n else 1, "classes in turn": lambda i, n: 2 if i % 3 == 0 else 1}


def test_no_xcd_waits_long_for_another_whatever_the_classes(tmp_path):
    cases = [(bh, video, 0, DEALT) for bh in (4, 6, 8, 12, 16, 20, 24, 25, 30, 32, 40, 48, 60) for video in (32, 60, 64, 139)]
    for (bh, video, _, order), qs in zip(cases, queues(tmp_path, cases)):
        for name, work in MIXES.items():
            load = [sum(work(h, bh) for h, _ in q) for q in qs]
            mean = sum(load) / 8
            # whole heads: at most one heavier head than the mean, of three or more (four eighths in a row: 24 heads)
            assert max(load) <= (1.34 if bh >= 24 else 1.15) * mean, (bh, video, name, load)
            if bh in (24, 48) and name == "classes in turn":
                assert max(load) == min(load), (bh, video, load)
