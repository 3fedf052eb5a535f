"""The launch rules of the chunk kernel (csrc/chunk_rules.h) against what was measured on the two sides of each, for 256 compute
units: with one unit per workgroup a call takes 128 rows per workgroup while 256-row ones leave compute units idle."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SHAPES = {"256": (8, 2), "128": (8, 4), "192": (16, 1), "64": (1, 8)}   # head width: KV heads, query heads per KV head


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "chunk_rules_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe, os.path.join(HERE, "host_c", "chunk_rules_check.cpp")], check=True)

    def ask(calls):
        args = []
        for width, layers, agents, q_len, max_seq_len, windows in calls:
            heads, rep = SHAPES[width]
            args += [layers * agents * heads, q_len * rep, rep, max_seq_len, "%d:%s" % (q_len, ",".join(map(str, windows)))]
        out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True).stdout.split()
        assert len(out) == len(calls)
        return [int(x) for x in out]
    return ask


# (head width, layers, agents, new tokens, bound of the lengths, windows), us with 128 rows, us with 256
ALONE = [
    (("256", 1, 1, 512, 8512, (0,)), 315.8, 584.2),
    (("256", 1, 4, 512, 8512, (0,)), 380.1, 587.2),
    (("256", 1, 1, 2048, 10048, (0,)), 403.0, 684.1),
    (("256", 1, 1, 512, 16512, (1024,)), 57.6, 100.3),      # the window, not the bound, is what a workgroup sees
    (("256", 1, 10, 512, 8512, (1024,)), 185.0, 217.7),
    (("256", 2, 4, 512, 6512, (0,)), 563.5, 545.2),
    (("256", 3, 4, 512, 6512, (0,)), 824.9, 940.6),
    (("256", 6, 4, 512, 6512, (0,)), 1626.9, 1523.8),
    (("256", 6, 4, 512, 8512, (1024,) * 5 + (0,)), 666.8, 801.1),
    (("256", 12, 4, 512, 6512, ((1024,) * 5 + (0,)) * 2), 1152.5, 1213.7),
    (("256", 12, 10, 512, 6512, ((1024,) * 5 + (0,)) * 2), 2931.1, 2886.0),
    (("128", 1, 1, 512, 8512, (0,)), 182.9, 320.4),
    (("128", 1, 1, 512, 16512, (1024,)), 36.2, 53.6),
    (("128", 1, 4, 512, 8512, (0,)), 391.8, 374.9),
    (("128", 6, 10, 512, 4512, (0,)), 3033.0, 2769.5),
    (("128", 8, 1, 512, 8512, (1024,) * 5 + (0,) + (1024,) * 2), 256.6, 375.0),
    (("128", 12, 4, 512, 6512, ((1024,) * 5 + (0,)) * 2), 1343.8, 1121.7),
    (("192", 1, 1, 512, 8512, (0,)), 209.9, 371.8),
    (("192", 1, 1, 2048, 10048, (0,)), 266.5, 438.2),
    (("192", 2, 4, 512, 6512, (0,)), 388.3, 362.5),
    (("64", 1, 1, 512, 8512, (0,)), 134.1, 239.1),
    (("64", 1, 10, 512, 8512, (1024,)), 55.8, 45.2),        # ten units on eight dies: two dies hold two each
    (("64", 2, 4, 1024, 7024, (0,)), 225.9, 215.9),
]


def test_rows_without_shares_take_the_faster_side(rules):
    got = rules([call for call, _, _ in ALONE])
    assert got == [128 if narrow < wide else 256 for _, narrow, wide in ALONE]


def test_rows_without_shares_at_the_ends_of_the_range(rules):
    # no cached token at all, one token, the largest bound, 2^31 - 1 tokens of window
    assert rules([("256", 1, 1, 2, 0, (0,)), ("128", 1, 1, 2, 1, (0,)), ("256", 1, 1, 512, 2 ** 31 - 1, (0,)),
                  ("256", 1, 1, 512, 8512, (2 ** 31 - 1,)), ("64", 48, 256, 700, 32768, (0,))]) == [128, 128, 128, 128, 256]
