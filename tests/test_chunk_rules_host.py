"""The launch rules of the chunk kernel (csrc/chunk_rules.h) against what was measured on the two sides of each, for 256 compute
units: with one unit per workgroup a call takes 128 rows per workgroup while 256-row ones leave compute units idle, and tiles
are shared out evenly only where that is done first."""
import os
import subprocess

import pytest

from tests.test_gpu_chunk import ONE_TILE, WIDE_ALONE, WIDE_EDGES, WIDE_SHARED

HERE = os.path.dirname(os.path.abspath(__file__))
SHAPES = {"256": (8, 2), "128": (8, 4), "192": (16, 1), "64": (1, 8)}   # head width: KV heads, query heads per KV head


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "chunk_rules_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe, os.path.join(HERE, "host_c", "chunk_rules_check.cpp")], check=True)

    def ask(calls):
        args = []
        for width, layers, agents, q_len, max_seq_len, windows in calls:
            heads, rep = SHAPES[width] if isinstance(width, str) else width[1:]
            width = width if isinstance(width, str) else width[0]
            args += [width, agents, layers * agents * heads, q_len * rep, rep, max_seq_len, "%d:%s" % (q_len, ",".join(map(str, windows)))]
        out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(calls)
        return [tuple(int(x) for x in line.split()) for line in out]
    return ask


# (head width, layers, agents, new tokens, bound of the lengths, windows), us with 128 rows, us with 256
ALONE = [
    (("256", 1, 1, 512, 8512, (0,)), 315.4, 517.0),
    (("256", 1, 4, 512, 8512, (0,)), 348.1, 524.0),
    (("256", 1, 1, 2048, 10048, (0,)), 392.4, 611.5),
    (("256", 1, 1, 512, 16512, (1024,)), 55.6, 93.8),      # the window, not the bound, is what a workgroup sees
    (("256", 1, 10, 512, 8512, (1024,)), 171.7, 194.2),
    (("256", 2, 4, 512, 6512, (0,)), 525.5, 470.3),
    (("256", 3, 4, 512, 6512, (0,)), 798.7, 873.9),
    (("256", 6, 4, 512, 6512, (0,)), 1601.6, 1428.4),
    (("256", 6, 4, 512, 8512, (1024,) * 5 + (0,)), 640.3, 736.0),
    (("256", 12, 4, 512, 6512, ((1024,) * 5 + (0,)) * 2), 1135.6, 1134.7),
    (("256", 12, 10, 512, 6512, ((1024,) * 5 + (0,)) * 2), 2919.0, 2703.3),
    (("128", 1, 1, 512, 8512, (0,)), 166.9, 290.6),
    (("128", 1, 1, 512, 16512, (1024,)), 32.3, 48.6),
    (("128", 1, 4, 512, 8512, (0,)), 358.5, 327.1),
    (("128", 6, 10, 512, 4512, (0,)), 2961.7, 2680.1),
    (("128", 8, 1, 512, 8512, (1024,) * 5 + (0,) + (1024,) * 2), 233.0, 351.8),
    (("128", 12, 4, 512, 6512, ((1024,) * 5 + (0,)) * 2), 1236.1, 1062.8),
    (("192", 1, 1, 512, 8512, (0,)), 196.6, 333.4),
    (("192", 1, 1, 2048, 10048, (0,)), 250.3, 393.3),
    (("192", 2, 4, 512, 6512, (0,)), 332.0, 300.8),
    (("64", 1, 1, 512, 8512, (0,)), 129.4, 220.1),
    (("64", 1, 10, 512, 8512, (1024,)), 46.9, 37.7),        # ten units on eight dies: two dies hold two each
    (("64", 2, 4, 1024, 7024, (0,)), 205.7, 190.3),
]


def test_rows_without_shares_take_the_faster_side(rules):
    got = [r[0] for r in rules([call for call, _, _ in ALONE])]
    for rows, (call, narrow, wide) in zip(got, ALONE):   # sides within 0.2 % of each other are one: two runs of a side differ by more
        assert rows == (128 if narrow < wide else 256) or abs(narrow - wide) < 0.002 * narrow, call


def test_rows_without_shares_at_the_ends_of_the_range(rules):
    # no cached token at all, one token, the largest bound, 2^31 - 1 tokens of window
    got = rules([("256", 1, 1, 2, 0, (0,)), ("128", 1, 1, 2, 1, (0,)), ("256", 1, 1, 512, 2 ** 31 - 1, (0,)),
                  ("256", 1, 1, 512, 8512, (2 ** 31 - 1,)), ("64", 48, 256, 700, 32768, (0,))])
    assert [r[0] for r in got] == [128, 128, 128, 128, 256]
    assert [r[2:] for r in got] == [(0, 0), (0, 0), (1, 0), (1, 1), (0, 0)]   # the third has too many tiles to number


# ..., us with one unit per workgroup (the better row count), us with equal shares (the row count of the rule)
SHARES = [
    (("256", 1, 1, 512, 8512, (0,)), 315.4, 120.2),
    (("256", 1, 1, 512, 2512, (0,)), 107.4, 60.7),
    (("256", 1, 10, 512, 33280, (0,)), 2454.8, 2088.4),
    (("256", 1, 1, 512, 16512, (1024,)), 55.6, 49.1),
    (("256", 1, 10, 2, 282, (0,)), 16.8, 29.7),
    (("256", 1, 10, 70, 350, (0,)), 28.9, 41.1),
    (("256", 1, 3, 512, 792, (0,)), 47.1, 59.5),
    (("256", 1, 3, 512, 1212, (0,)), 62.0, 69.2),
    (("256", 1, 1, 70, 350, (0,)), 27.6, 22.1),
    (("128", 1, 1, 512, 792, (0,)), 26.8, 37.1),
    (("128", 1, 1, 512, 1212, (0,)), 34.1, 42.6),
    (("128", 1, 1, 512, 2512, (0,)), 58.0, 53.1),
    (("128", 1, 1, 512, 8512, (0,)), 166.9, 108.8),
    (("128", 1, 3, 200, 480, (0,)), 19.7, 34.4),
    (("128", 1, 10, 16, 296, (0,)), 13.1, 21.7),
    (("128", 1, 10, 16, 1516, (0,)), 29.9, 26.9),
    (("128", 1, 1, 512, 16512, (1024,)), 32.3, 43.7),
    (("192", 1, 10, 70, 350, (0,)), 17.9, 34.4),
    (("192", 1, 1, 512, 2012, (0,)), 57.0, 42.4),
    (("192", 1, 3, 2, 702, (0,)), 17.8, 17.3),
    (("192", 1, 10, 512, 792, (0,)), 92.0, 83.6),
    (("64", 2, 70, 3, 703, (0,)), 12.7, 21.7),
    (("64", 1, 1, 512, 8512, (0,)), 129.4, 38.3),
]


def test_shares_are_taken_where_they_are_done_first(rules):
    got = rules([call for call, _, _ in SHARES])
    assert [r[2] for r in got] == [1 if shared < alone else 0 for _, alone, shared in SHARES]
    assert all(r[3] == 1 for r in got)                  # all of them come with a workspace


def test_shares_never_need_more_rows_than_the_workspace_was_sized_for(rules):
    """The size is asked for without a window; the call then goes by what its window lets it see."""
    calls = [(width, 1, agents, q_len, top, (window,)) for width in SHAPES for agents in (1, 3, 10) for q_len in (2, 70, 300, 512)
             for top in (600, 5000, 40000, 131072) for window in (0, 1, 300, 1024, 8192)]
    got = rules(calls)
    sized = {c[:5]: r[1] for c, r in zip(calls, got) if c[5] == (0,)}
    assert all(r[1] <= sized[c[:5]] for c, r in zip(calls, got))


def test_the_gpu_tests_of_256_rows_take_256_rows(rules):
    def call(case, max_seq_len):
        Hq, Hkv, D, lens, q_len = case
        return ((D[0] if isinstance(D, tuple) else D, Hkv, Hq // Hkv), 1, len(lens), q_len, max_seq_len or max(lens) + q_len, (0,))

    got = rules([call(c, 131072) for c in WIDE_SHARED])
    assert [r[1:] for r in got] == [(256, 1, 1)] * len(WIDE_SHARED)
    got = rules([call(c, 131072)[:5] + ((300,),) for c in WIDE_SHARED])   # with a window they may take either
    assert all(r[3] == 1 for r in got)
    got = rules([call(c, 0) for c in WIDE_ALONE + WIDE_EDGES])
    assert [r[0] for r in got] == [256] * len(WIDE_ALONE + WIDE_EDGES)
    got = rules([call(c, 0) for c in ONE_TILE] + [call((*c[:3], c[3][:1], c[4]), max(c[3]) + c[4]) for c in ONE_TILE])
    assert [r[0] for r in got] == [256, 256, 128, 128]


def test_the_library_is_built_from_these_sources():
    """Else the next test reads the kernels of another state of the sources, and so does every GPU test."""
    from paper_2603_04428_amd import binding, build

    binding.lib()                           # raises and says how to build where there is no library
    with open(build.LIB, "rb") as f:
        assert f"q4kv sources {build.sources_hash()}".encode() in f.read(), "sources changed since the library was built: build it again"


def test_a_build_with_a_spilling_chunk_kernel_is_refused():
    from paper_2603_04428_amd import build

    line = "/a/chunk_attention.hip:289:1: remark: %s [-Rpass-analysis=kernel-resource-usage]\n"
    names = ("    AGPRs: %d", "    ScratchSize [bytes/lane]: %d", "    SGPRs Spill: 7", "    VGPRs Spill: %d")

    def remarks(kernel, agprs, scratch, spilled):
        return "".join(line % t for t in ("Function Name: " + kernel, "    VGPRs: 256", names[0] % agprs, names[1] % scratch, names[2], names[3] % spilled))

    assert build.spills(remarks("_Z1a", 0, 0, 0) + remarks("_Z1b", 0, 0, 0)) == []
    assert build.spills(remarks("_Z1a", 0, 0, 0) + remarks("_Z1b", 0, 8, 1)) == ["_Z1b: ScratchSize [bytes/lane] 8", "_Z1b: VGPRs Spill 1"]
    assert build.spills(remarks("_Z1a", 12, 0, 0) + remarks("_Z1b", 0, 0, 0)) == ["_Z1a: AGPRs 12"]
    assert "chunk_attention.hip" in build.NO_SPILLS


def test_chunk_kernels_need_no_scratch_memory():
    """The kernel metadata of the built library: every chunk attention kernel keeps all it has in registers (the header of
    csrc/chunk_attention.hip tells what a spill did)."""
    import struct

    import msgpack

    from paper_2603_04428_amd import build

    data = open(build.LIB, "rb").read()
    scratch, at = {}, data.find(b"AMDGPU\0\0")
    while at >= 0:
        name_size, size, kind = struct.unpack_from("<III", data, at - 12)
        if name_size == 7 and kind == 32:   # an ELF note of kernel metadata
            for kernel in msgpack.unpackb(data[at + 8:at + 8 + size])["amdhsa.kernels"]:
                scratch[kernel[".name"]] = [kernel[k] for k in (".private_segment_fixed_size", ".vgpr_spill_count", ".agpr_count")]
        at = data.find(b"AMDGPU\0\0", at + 1)
    chunk = {k: v for k, v in scratch.items() if "chunk_attention_kernel" in k}
    assert len(chunk) == 128                # 4 widths, 4 head groupings, 2 row counts, with and without shares, 2 formats
    assert not {k: v for k, v in chunk.items() if any(v)}
