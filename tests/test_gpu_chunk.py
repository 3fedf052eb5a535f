"""GPU parity of chunked-append attention (q4kv_append, then q4kv_batched_attention with q_len > 1) with the
CPU oracle.  Tolerance: |gpu - oracle| <= 2e-3 + 2e-3*|oracle| on the binary16 outputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_04428_amd import binding as b
from paper_2603_04428_amd import synth
from tests.gpu_util import DEV, bits, gpu_cache, host_cache, oracle_unit
from tests.util import within_tol

pytestmark = pytest.mark.gpu


def assert_close(got, want, what=""):
    ok, over, worst = within_tol(got, want)
    assert ok, f"{what}: exceeds 2e-3 abs/rel by {over:.3e} (max abs err {worst:.3e})"
    assert not np.isnan(got.astype(np.float32)).any()


def append_chunk_and_attend(w, window=0, param_format=0):
    """Cache of seq_lens tokens, then the library appends the chunk and attends; returns (gpu out, pools, table)."""
    spec, kpool, vpool, table, table_d = gpu_cache(w, tokens=w.seq_lens, param_format=param_format)   # blocks for cache + chunk are reserved
    C = w.q_len
    before = torch.tensor(w.seq_lens, dtype=torch.int32, device=DEV)
    for l in range(w.num_layers):
        k_new = torch.stack([w.k_rows(l, a, n, n + C, DEV) for a, n in enumerate(w.seq_lens)])[None].contiguous()
        v_new = torch.stack([w.v_rows(l, a, n, n + C, DEV) for a, n in enumerate(w.seq_lens)])[None].contiguous()
        b.q4kv_append(spec, kpool, vpool, k_new, v_new, table_d, before, l, l + 1)
    after = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV)
    out = b.q4kv_batched_attention(spec, kpool, vpool, w.q_all(DEV), table_d, after, max(w.final_lens()), w.sm_scale,
                                   window)
    torch.cuda.synchronize()
    return out.cpu().numpy(), (spec, kpool, vpool, table_d)


SHAPES = [
    # layers, Hq, Hkv, D, cached tokens per agent, chunk length
    (1, 4, 2, 64, (20, 3), 6),
    (2, 4, 2, 128, (300, 0, 70), 70),        # an agent with an empty cache; chunk spans two query tiles
    (1, 8, 2, 128, (250,), 130),             # n_rep 4: 32 positions per query tile
    (1, 2, 2, 256, (513, 64), 129),          # n_rep 1: 128 positions per tile, ragged last tile
    (1, 16, 8, 256, (100,), 64),
    (1, 8, 1, 64, (1000, 40), 33),           # n_rep 8
    # decompressed per-head MLA cache (Sec. 3.6): keys 192, values 128, one KV head per query head; the K rows of a
    # tile do not divide evenly among the threads of a workgroup
    (1, 4, 4, (192, 128), (300, 0), 130),
    (2, 16, 16, (192, 128), (70, 513), 40),
    (1, 8, 4, (192, 128), (257,), 64),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_chunk_matches_oracle_small(shape):
    L, Hq, Hkv, D, lens, C = shape
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    w = synth.small(41, L, Hq, Hkv, Dk, Dv, False, lens, q_len=C)
    got, _ = append_chunk_and_attend(w)
    ospec, okp, ovp, otable = host_cache(w)                  # cache + chunk, quantized by the oracle
    want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale)
    assert_close(got, want, f"{shape}")


@pytest.mark.parametrize("shape", [(4, 2, 256), (4, 4, (192, 128)), (8, 2, 128), (8, 1, 64)])
def test_chunk_around_the_edges_of_its_tiles(shape):
    """Units of one, two and a few tiles of 64 and 128 tokens (128 rows per workgroup), and one token more or less: the product
    runs a tile behind the scores, so the first, the second and the last tile of a unit each take a turn of their own."""
    Hq, Hkv, D = shape
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    for C in (2, 40):                                        # tokens seen by the last row: 2 or 40 more than these
        lens = (0, 29, 30, 31, 61, 62, 63, 125, 126, 127, 191, 254) if C == 2 else (0, 24, 88, 89, 216, 473)
        w = synth.small(52, 1, Hq, Hkv, Dk, Dv, False, lens, q_len=C)
        got, _ = append_chunk_and_attend(w)
        ospec, okp, ovp, otable = host_cache(w)
        want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale)
        assert_close(got, want, f"{shape} {C}")


@pytest.mark.parametrize("seed", [44, 45, 46, 47, 48, 49])
def test_chunk_tolerance_does_not_depend_on_the_draw(seed):
    """Short contexts with the generator's large key channels make a softmax that a few keys dominate: the case in
    which a score error reaches the output undamped.  (Key rows rounded to binary16 before the product fail this for
    about every second seed, by up to twice the tolerance.)"""
    for shape in ((2, 4, 2, 128, (300, 0, 70), 70), (1, 8, 1, 64, (1000, 40), 33), (1, 2, 2, 256, (90, 5), 40)):
        L, Hq, Hkv, D, lens, C = shape
        w = synth.small(seed, L, Hq, Hkv, D, D, False, lens, q_len=C)
        got, _ = append_chunk_and_attend(w)
        ospec, okp, ovp, otable = host_cache(w)
        want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale)
        assert_close(got, want, f"seed {seed} {shape}")


def test_chunk_rows_equal_decode_steps_and_window():
    w = synth.small(42, 1, 4, 2, 128, 128, False, (200, 31), q_len=40)
    got, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    ospec, okp, ovp, otable = host_cache(w)
    q = w.q_all(DEV)
    # row r of the chunk call == a decode call that sees before + r + 1 tokens (same Q4 cache, other kernel)
    for r in (0, 17, 39):
        lens = [n + r + 1 for n in w.seq_lens]
        sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
        one = b.q4kv_batched_attention(spec, kpool, vpool, q[:, :, r:r + 1].contiguous(), table_d, sl, max(lens),
                                       w.sm_scale)
        torch.cuda.synchronize()
        assert_close(got[:, :, r], one.cpu().numpy()[:, :, 0].astype(np.float64), f"row {r} vs decode")
    # sliding windows, also shorter than the chunk
    for win in (1, 16, 100, 1000):
        sl = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV)
        g = b.q4kv_batched_attention(spec, kpool, vpool, q, table_d, sl, max(w.final_lens()), w.sm_scale, win)
        torch.cuda.synchronize()
        want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale, window=win)
        assert_close(g.cpu().numpy(), want, f"window {win}")
    # deterministic
    sl = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV)
    again = b.q4kv_batched_attention(spec, kpool, vpool, q, table_d, sl, max(w.final_lens()), w.sm_scale)
    torch.cuda.synchronize()
    assert np.array_equal(again.cpu().numpy().view(np.uint16), got.view(np.uint16))


def test_chunk_per_layer_windows_match_oracle():
    w = synth.small(45, 3, 4, 2, 128, 128, False, (300, 40), q_len=70)
    got, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    ospec, okp, ovp, otable = host_cache(w)
    sl = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV)
    for windows in ([0, 16, 200], [1000, 1, 64]):
        g = b.q4kv_batched_attention(spec, kpool, vpool, w.q_all(DEV), table_d, sl, max(w.final_lens()), w.sm_scale,
                                     windows)
        torch.cuda.synchronize()
        want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale,
                                window_per_layer=windows)
        assert_close(g.cpu().numpy(), want, f"windows {windows}")


def test_poisoned_slots_past_the_chunk_are_never_used():
    # the last block of every agent is only partly filled; everything else in the pool decodes to NaN
    w = synth.small(43, 1, 4, 2, 64, 64, False, (130, 255), q_len=10)
    got, _ = append_chunk_and_attend(w)
    assert not np.isnan(got.astype(np.float32)).any()


def test_config4_one_layer_sampled_rows():
    """Gemma-3-12B-shaped chunked append at the benchmark's shape (10 agents, ragged 4,096..32,768 cached tokens,
    512-token chunk), one layer in the test to bound the set-up time; the oracle recomputes chunk rows 0, 255 and
    511 of a seeded sample of (agent, kv head) units from the generator alone."""
    full = synth.config(4)
    w = synth.Workload(full.name + "_layer0", full.seed, 1, full.num_q_heads, full.num_kv_heads, full.k_dim,
                       full.v_dim, False, full.seq_lens, q_len=full.q_len)
    got, _ = append_chunk_and_attend(w)
    assert not np.isnan(got.astype(np.float32)).any()
    shortest, longest = int(np.argmin(w.seq_lens)), int(np.argmax(w.seq_lens))
    R = w.n_rep
    for (a, h) in [(shortest, 0), (longest, 7), (3, 4)]:
        n = w.final_lens()[a]
        for r in (0, 255, 511):
            vis = n - (w.q_len - 1 - r)
            q = w.q_rows(0, a).numpy()[r:r + 1]
            want = oracle_unit(w, 0, a, h, vis, q=q)
            assert_close(got[0, a, r, h * R:(h + 1) * R], want[0], f"agent {a} kv head {h} chunk row {r}")


def test_config4_full_size_sampled_rows():
    """The same at full size with the benchmark's launches: one q4kv_append and one attention call for all 48 layers
    (21 GB of Q4 cache, 1 GB of new K and of new V, 2 GB of output).  Sampled appended rows are compared bit for bit
    and sampled (layer, agent, kv head, chunk row) outputs within the tolerance with the oracle, which rebuilds each
    of them from the generator alone."""
    w = synth.config(4)
    spec, kpool, vpool, table, table_d = gpu_cache(w, tokens=w.seq_lens)
    C = w.q_len
    before = torch.tensor(w.seq_lens, dtype=torch.int32, device=DEV)
    k_new = torch.empty((w.num_layers, w.num_agents, C, w.num_kv_heads, w.k_dim), dtype=torch.float16, device=DEV)
    v_new = torch.empty((w.num_layers, w.num_agents, C, w.num_kv_heads, w.v_dim), dtype=torch.float16, device=DEV)
    for l in range(w.num_layers):
        for a, n in enumerate(w.seq_lens):
            k_new[l, a] = w.k_rows(l, a, n, n + C, DEV)
            v_new[l, a] = w.v_rows(l, a, n, n + C, DEV)
    b.q4kv_append(spec, kpool, vpool, k_new, v_new, table_d, before, 0, w.num_layers)
    after = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV)
    got = b.q4kv_batched_attention(spec, kpool, vpool, w.q_all(DEV), table_d, after, max(w.final_lens()), w.sm_scale, 0)
    torch.cuda.synchronize()
    assert not torch.isnan(got).any()
    shortest, longest = int(np.argmin(w.seq_lens)), int(np.argmax(w.seq_lens))
    R = w.n_rep
    for (l, a, h) in [(0, shortest, 0), (w.num_layers - 1, longest, 7), (20, 3, 4)]:
        n0, n = w.seq_lens[a], w.final_lens()[a]
        for c in (0, 255, 511):          # appended rows, bit for bit
            t = n0 + c
            blk, slot = int(table[a, t // 256]), t % 256
            for pool, rows in ((kpool, w.k_rows(l, a, t, t + 1, h0=h, h1=h + 1)), (vpool, w.v_rows(l, a, t, t + 1, h0=h, h1=h + 1))):
                codes, scale, bias = oracle.quantize(rows.numpy().reshape(1, -1))
                assert np.array_equal(bits(pool.codes[l, blk, h, slot]), codes[0]), f"codes of layer {l} agent {a} token {t}"
                assert np.array_equal(bits(pool.scale[l, blk, h, slot]), scale[0])
                assert np.array_equal(bits(pool.bias[l, blk, h, slot]), bias[0])
        for r in (0, 255, 511):
            vis = n - (w.q_len - 1 - r)
            q = w.q_rows(l, a).numpy()[r:r + 1]
            want = oracle_unit(w, l, a, h, vis, q=q)
            assert_close(got[l, a, r, h * R:(h + 1) * R].cpu().numpy(), want[0],
                         f"layer {l} agent {a} kv head {h} chunk row {r}")


def test_append_and_chunk_attention_replay_from_a_graph():
    """One step of a prefill loop (append a chunk, attend over cache + chunk) recorded into a graph once and replayed
    for the following chunks: lengths, the new rows and the queries live in device buffers that the host refills
    between replays.  Every replay must equal the same step issued eagerly on a second copy of the cache."""
    C = 64
    w = synth.small(52, 2, 8, 4, 128, 128, False, (300, 10, 700), q_len=4 * C)   # blocks for four chunks are reserved
    spec, kpool, vpool, table, table_d = gpu_cache(w, tokens=w.seq_lens)
    spec2, kpool2, vpool2, _, table2_d = gpu_cache(w, tokens=w.seq_lens)
    A, L = w.num_agents, w.num_layers
    before = torch.tensor(w.seq_lens, dtype=torch.int32, device=DEV)
    after = before + C
    k_new = torch.empty((L, A, C, w.num_kv_heads, w.k_dim), dtype=torch.float16, device=DEV)
    v_new = torch.empty_like(k_new)
    q = torch.empty((L, A, C, w.num_q_heads, w.k_dim), dtype=torch.float16, device=DEV)
    out = torch.empty((L, A, C, w.num_q_heads, w.v_dim), dtype=torch.float16, device=DEV)
    msl = max(w.seq_lens) + 4 * C

    def fill(step):
        for l in range(L):
            for a, n in enumerate(w.seq_lens):
                k_new[l, a] = w.k_rows(l, a, n + step * C, n + (step + 1) * C, DEV)
                v_new[l, a] = w.v_rows(l, a, n + step * C, n + (step + 1) * C, DEV)
        q.copy_(torch.randn(q.shape, generator=torch.Generator().manual_seed(100 + step)).to(torch.float16))
        before.copy_(torch.tensor([n + step * C for n in w.seq_lens], dtype=torch.int32))
        after.copy_(before + C)

    def step_on(kp, vp, tab, dst):
        b.q4kv_append(spec, kp, vp, k_new, v_new, tab, before, 0, L)
        b.q4kv_batched_attention(spec, kp, vp, q, tab, after, msl, w.sm_scale, 0, 0, 0, None, dst)

    fill(0)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step_on(kpool, vpool, table_d, out)            # warm-up on the capture stream (writes chunk 0, rewritten below)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step_on(kpool, vpool, table_d, out)
    for step in range(4):
        fill(step)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = torch.empty_like(out)
        step_on(kpool2, vpool2, table2_d, want)
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {step}"
    assert torch.equal(kpool.codes, kpool2.codes) and torch.equal(vpool.scale, vpool2.scale)


# (query heads, KV heads, D, cached tokens, chunk): row counts around the 128 and 256 rows of a workgroup and the 32 of a
# wave, lengths around the tiles of 32 and 64 tokens, agents without a token, one unit shared by every workgroup
SHARED = [
    (4, 2, 256, (1300, 0, 700), 64),          # 128 rows: a workgroup's waves share the tokens of a tile
    (4, 2, 256, (641, 990), 65),              # one row pair more
    (2, 2, 256, (2049,), 256),                # 256 rows, 32-token tiles, lengths one past a tile
    (2, 2, 256, (480, 1000), 33),
    (8, 2, 128, (1999, 64, 513), 70),         # 280 rows: three tiles of 128, the last nearly empty
    (4, 4, (192, 128), (1500, 300), 130),
    (8, 1, 64, (5000,), 2),                   # one unit of 79 tiles: every workgroup takes one
    (8, 1, 64, (700,) * 70, 3),               # more agents than lanes
]


@pytest.mark.parametrize("param_format", [0, 1])
@pytest.mark.parametrize("case", SHARED)
def test_chunk_shared_by_workgroups_matches_oracle(case, param_format):
    """With a workspace the tiles of all units are dealt out over the compute units and shared units are merged; without
    one a workgroup takes a unit.  Both against the oracle, with and without a window, with the lengths' own bound and with a
    bound of 131,072 tokens (the work a call might hold decides how many rows a workgroup takes, and whether sharing pays); the workspace is not
    left, the result does not change from run to run."""
    Hq, Hkv, D, lens, C = case
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    w = synth.small(61, 2, Hq, Hkv, Dk, Dv, False, lens, q_len=C)
    got, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w, param_format=param_format)
    ospec, okp, ovp, otable = host_cache(w, param_format=param_format)
    sl = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV)
    q, wide = w.q_all(DEV), torch.nn.functional.pad(table_d, (0, 512 - table_d.shape[1])).contiguous()
    for window in (0, 300):
        want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale, window=window)
        for table, msl in ((table_d, max(w.final_lens())), (wide, 512 * 256)):
            need = b.q4kv_attention_workspace_bytes(spec, w.num_agents, C, msl, 0, w.num_layers)
            assert need > 0
            ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device=DEV)
            outs = [b.q4kv_batched_attention(spec, kpool, vpool, q, table, sl, msl, w.sm_scale, window, workspace=ws[:size])
                    for size in (need, need, need - 1)]
            torch.cuda.synchronize()
            assert bool((ws[need:] == 0x5A).all())
            assert torch.equal(outs[0], outs[1])
            assert_close(outs[0].cpu().numpy(), want, f"{case} window {window} bound {msl}, shared")
            assert_close(outs[2].cpu().numpy(), want, f"{case} window {window} bound {msl}, one unit per workgroup")


# 20 to 72 rows of a workgroup's 128: one, two and three of its four row groups have rows of the chunk
FEW_ROWS = [
    (2, 2, 256, (1501, 300), 20),
    (4, 2, 256, (900,), 20),
    (4, 4, (192, 128), (1500, 300), 70),
    (8, 2, 128, (1200,), 9),
    (8, 1, 64, (3000, 200), 9),
]


@pytest.mark.parametrize("case", FEW_ROWS)
def test_chunk_of_few_rows_matches_oracle(case):
    """Waves without rows of the chunk only stage, and the others are placed differently over the SIMDs."""
    test_chunk_shared_by_workgroups_matches_oracle(case, 0)


@pytest.mark.parametrize("shape", [(4, 2, 256, (700, 40), 60), (4, 4, (192, 128), (500,), 130), (8, 2, 128, (900,), 70), (8, 1, 64, (300, 65), 33)])
def test_a_row_does_not_depend_on_the_other_rows_of_its_chunk(shape):
    """Queries of other positions eight times larger: the rows that keep theirs give the same bits, with and without shares."""
    Hq, Hkv, D, lens, C = shape
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    w = synth.small(69, 1, Hq, Hkv, Dk, Dv, False, lens, q_len=C)
    _, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    sl, msl, q = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV), 512 * 256, w.q_all(DEV)
    wide = torch.nn.functional.pad(table_d, (0, 512 - table_d.shape[1])).contiguous()
    kept = torch.zeros(C, dtype=torch.bool, device=DEV)
    kept[::5] = True
    q2 = torch.where(kept[None, None, :, None, None], q, 8 * q)
    ws = torch.empty(b.q4kv_attention_workspace_bytes(spec, len(lens), C, msl, 0, 1), dtype=torch.uint8, device=DEV)
    for workspace in (ws, None):
        one, two = (b.q4kv_batched_attention(spec, kpool, vpool, x, wide, sl, msl, w.sm_scale, workspace=workspace) for x in (q, q2))
        torch.cuda.synchronize()
        assert torch.equal(one[:, :, kept], two[:, :, kept]), f"{shape} shares {workspace is not None}"
        assert not torch.equal(one, two)


@pytest.mark.parametrize("bits_down", [16.0, 20.3, 25.2, 26.4])
@pytest.mark.parametrize("shape", [(2, 2, 256), (2, 2, 64), (4, 2, 128), (2, 2, (192, 128))])
def test_chunk_with_a_long_light_tail(shape, bits_down):
    """One token of weight 1 in front of 131,071 of weight 2^-bits_down, values +1 and -1 in turn: the output is 1 over the
    denominator, in which each weight of the tail is less than binary16 resolves and all of them together are not.  Tolerance: the
    output's rounding (2^-12 below 1) and that of a binary32 sum of 1 and a lane's at most 2,048 parts of the tail (2^-24 each)."""
    Hq, Hkv, D = shape
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    C, n = 2, 131072
    spec = b.make_spec(1, Hq, Hkv, Dk, Dv, False)
    kpool, vpool = b.Pool(spec, Dk, n // 256), b.Pool(spec, Dv, n // 256)     # codes and scales 0: a row is its bias
    kpool.bias[0, 0, :, 0] = 0x3C00
    vpool.bias[:, :, :, 0::2] = 0x3C00
    vpool.bias[:, :, :, 1::2] = 0xBC00 - 0x10000
    ospec = oracle.make_spec(1, Hq, Hkv, Dk, Dv, False)
    okp, ovp = oracle.Pool(ospec, Dk, n // 256), oracle.Pool(ospec, Dv, n // 256)
    okp.bias[...], ovp.bias[...] = bits(kpool.bias), bits(vpool.bias)
    table = np.arange(n // 256, dtype=np.int32)[None]
    q = np.ones((1, 1, C, Hq, Dk), np.float16)
    sm_scale = bits_down * np.log(2.0) / Dk
    _, exact = oracle.attention(ospec, okp, ovp, q, table, [n], sm_scale, return_f64=True)
    got = b.q4kv_batched_attention(spec, kpool, vpool, torch.from_numpy(q).to(DEV), torch.from_numpy(table).to(DEV),
                                   torch.tensor([n], dtype=torch.int32, device=DEV), n, sm_scale)
    torch.cuda.synchronize()
    err = np.abs(got.cpu().numpy().astype(np.float64) - exact).max()
    assert err < 2.0 ** -12 + 2048 * 2.0 ** -24, f"{shape} 2^-{bits_down}: {err:.3e}"


def test_chunk_call_leaves_a_workspace_of_another_size_alone():
    """A chunk call uses a workspace of exactly the size it was told; any other (a decode call's, which may hold the plan
    of the step in progress) keeps its bytes, and the planned calls that follow find their plan."""
    w = synth.small(62, 2, 4, 2, 256, 256, False, (1300, 0, 700), q_len=64)
    _, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    lens, A, L = w.final_lens(), w.num_agents, w.num_layers
    sl, msl, q = torch.tensor(lens, dtype=torch.int32, device=DEV), max(lens), w.q_all(DEV)
    need = b.q4kv_attention_workspace_bytes(spec, A, w.q_len, msl, 0, L)
    decode_need = b.q4kv_attention_workspace_bytes(spec, A, 1, msl, 0, L)
    assert need > decode_need > 0 and need % 8 == 4 and decode_need % 8 == 0
    want = b.q4kv_batched_attention(spec, kpool, vpool, q, table_d, sl, msl, w.sm_scale, workspace=torch.empty(16, dtype=torch.uint8, device=DEV))
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device=DEV)
    for size in (need + 4096, need + 1, need - 1, need - 4, decode_need, 16):
        got = b.q4kv_batched_attention(spec, kpool, vpool, q, table_d, sl, msl, w.sm_scale, workspace=ws[:size])
        torch.cuda.synchronize()
        assert bool((ws == 0x5A).all()), size
        assert torch.equal(got, want), size
    # a decode step's plan survives a chunk call that is handed the same workspace
    q1 = q[:, :, -1:].contiguous()
    decode = b.q4kv_batched_attention(spec, kpool, vpool, q1, table_d, sl, msl, w.sm_scale)
    b.q4kv_decode_plan(spec, sl, msl, ws, layers_in_call=L)
    b.q4kv_batched_attention(spec, kpool, vpool, q, table_d, sl, msl, w.sm_scale, workspace=ws)
    out = torch.full_like(decode, float("nan"))
    b.q4kv_batched_attention_planned(spec, kpool, vpool, q1, out, table_d, msl, w.sm_scale, ws)
    torch.cuda.synchronize()
    assert torch.equal(out, decode)


# Calls that take 256 rows per workgroup: (query heads, KV heads, D, agents' cached tokens, chunk), one for each head width and
# each number of query heads per KV head, 150 to 248 rows of 256, so that the last waves' rows are ragged or absent.  With
# the bound of 131,072 tokens they take them with shares; WIDE_ALONE without, having enough units that twice the workgroups
# would be two rounds (tests/test_chunk_rules_host.py asks the rules for both).
WIDE_SHARED = [
    (2, 2, 64, (900, 0), 200), (4, 2, 64, (900, 37), 101), (4, 1, 64, (700,), 61), (8, 1, 64, (3000,), 31),
    (2, 2, 128, (700, 65), 150), (4, 2, 128, (700,), 97), (8, 2, 128, (1999, 0, 513), 50), (8, 1, 128, (700,), 29),
    (4, 4, (192, 128), (600, 33), 161), (8, 4, (192, 128), (700, 40), 100), (4, 1, (192, 128), (600,), 50), (8, 1, (192, 128), (900,), 30),
    (2, 2, 256, (700, 64), 201), (4, 2, 256, (900,), 77), (8, 2, 256, (900, 0), 52), (8, 1, 256, (800,), 31),
]
WIDE_ALONE = [(rep * kvh, kvh, D, (150, 0, 37, 64, 3, 101, 33, 70, 5, 128, 1, 90, 31, 12, 55, 200, 17), q_len)
              for D in (64, 128, (192, 128), 256) for rep, kvh, q_len in ((1, 8, 130), (2, 8, 65), (4, 8, 33), (8, 8, 17))]


@pytest.mark.parametrize("case", WIDE_SHARED)
def test_chunk_of_256_rows_with_shares_matches_oracle(case):
    Hq, Hkv, D, lens, C = case
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    w = synth.small(63, 1, Hq, Hkv, Dk, Dv, False, lens, q_len=C)
    _, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    ospec, okp, ovp, otable = host_cache(w)
    sl, msl = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV), 512 * 256
    q, wide = w.q_all(DEV), torch.nn.functional.pad(table_d, (0, 512 - table_d.shape[1])).contiguous()
    need = b.q4kv_attention_workspace_bytes(spec, len(lens), C, msl, 0, 1)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    assert need == units * (2 * 256 * (Dv + 2) * 4 + 24) + 4         # two records of 256 rows for each compute unit
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    for window in (0, 300):
        got = b.q4kv_batched_attention(spec, kpool, vpool, q, wide, sl, msl, w.sm_scale, window, workspace=ws)
        torch.cuda.synchronize()
        want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale, window=window)
        assert_close(got.cpu().numpy(), want, f"{case} window {window}")


@pytest.mark.parametrize("case", WIDE_ALONE)
def test_chunk_of_256_rows_without_shares_matches_oracle(case):
    Hq, Hkv, D, lens, C = case
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    w = synth.small(64, 1, Hq, Hkv, Dk, Dv, False, lens, q_len=C)
    got, _ = append_chunk_and_attend(w)
    ospec, okp, ovp, otable = host_cache(w)
    want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale)
    assert_close(got, want, f"{case}")


# Calls that take 256 rows per workgroup without shares, tiles of 32 (256-wide), else 64 tokens: the last row sees one tile, two, three
# and one token more or less
WIDE_EDGES = [(64, 8, D, tuple(n + d - 17 for n in (tile, 2 * tile, 3 * tile) for d in (-1, 0, 1)) * 2, 17)
              for D, tile in ((256, 32), ((192, 128), 64), (128, 64), (64, 64))]


@pytest.mark.parametrize("case", WIDE_EDGES)
def test_chunk_of_256_rows_around_the_edges_of_its_tiles(case):
    test_chunk_of_256_rows_without_shares_matches_oracle(case)


ONE_TILE = [(64, 8, D, (0, 1, 15, 2, 14, 3, 13, 4, 12, 5, 11, 6, 10, 7, 9, 8, 0), 17) for D in (256, (192, 128))]


@pytest.mark.parametrize("case", ONE_TILE)
def test_keys_unpacked_when_staged_give_the_bits_of_packed_ones(case):
    """Seventeen agents of at most 32 tokens take 256 rows per workgroup (keys unpacked when staged), each of them alone 128 (by
    every wave): one tile is summed in the same order by both."""
    Hq, Hkv, D, lens, C = case
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    w = synth.small(70, 1, Hq, Hkv, Dk, Dv, False, lens, q_len=C)
    got, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    sl, q = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV), w.q_all(DEV)
    for a in range(len(lens)):
        one = b.q4kv_batched_attention(spec, kpool, vpool, q[:, a:a + 1].contiguous(), table_d[a:a + 1].contiguous(), sl[a:a + 1].contiguous(),
                                       max(w.final_lens()), w.sm_scale)
        torch.cuda.synchronize()
        assert torch.equal(one.cpu()[:, 0], torch.from_numpy(got[:, a])), f"{D} agent {a}"


@pytest.mark.parametrize("scale", [-0.11, 0.0])
@pytest.mark.parametrize("D", [64, 256])
def test_shared_chunk_with_a_scale_that_is_not_positive(scale, D):
    """A scale <= 0 takes the path that assumes nothing about the order of scores; here with shares and without."""
    w = synth.small(65, 1, 4, 2, D, D, False, (700, 130), q_len=65)
    _, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    ospec, okp, ovp, otable = host_cache(w)
    sl, msl = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV), 512 * 256
    q, wide = w.q_all(DEV), torch.nn.functional.pad(table_d, (0, 512 - table_d.shape[1])).contiguous()
    ws = torch.empty(b.q4kv_attention_workspace_bytes(spec, 2, w.q_len, msl, 0, 1), dtype=torch.uint8, device=DEV)
    want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), scale)
    for workspace in (ws, None):
        got = b.q4kv_batched_attention(spec, kpool, vpool, q, wide, sl, msl, scale, workspace=workspace)
        torch.cuda.synchronize()
        assert_close(got.cpu().numpy(), want, f"scale {scale} width {D} shares {workspace is not None}")


@pytest.mark.parametrize("shape", [(32, 8, 128), (16, 16, (192, 128)), (8, 4, 256)])
def test_shared_chunk_with_agents_that_see_nothing(shape):
    """Agents without tokens, or with fewer than the chunk has positions, between long ones: a workgroup's range then has parts of no
    tokens, before parts whose row groups lie on other waves (a chunk's last 128-row tile is partly empty, its first are not)."""
    Hq, Hkv, D = shape
    Dk, Dv = D if isinstance(D, tuple) else (D, D)
    C = 70 if Hq // Hkv > 1 else 150
    w = synth.small(71, 1, Hq, Hkv, Dk, Dv, False, (600, 2500, 300, 300, 1900, 300, 300, 1100), q_len=C)
    _, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    ospec, okp, ovp, otable = host_cache(w)
    lens = [0, w.final_lens()[1], 0, 0, w.final_lens()[4], 30, 0, w.final_lens()[7]]
    sl, msl, q = torch.tensor(lens, dtype=torch.int32, device=DEV), 512 * 256, w.q_all(DEV)
    wide = torch.nn.functional.pad(table_d, (0, 512 - table_d.shape[1])).contiguous()
    for bound, table in ((max(lens), table_d), (msl, wide)):
        need = b.q4kv_attention_workspace_bytes(spec, len(lens), C, bound, 0, 1)
        ws = torch.empty(need, dtype=torch.uint8, device=DEV)
        for window in (0, 300):
            want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, lens, w.sm_scale, window=window)
            for workspace in (ws, None):
                got = b.q4kv_batched_attention(spec, kpool, vpool, q, table, sl, bound, w.sm_scale, window, workspace=workspace)
                torch.cuda.synchronize()
                assert_close(got.cpu().numpy(), want, f"{shape} bound {bound} window {window} shares {workspace is not None}")


def test_chunk_of_more_agents_than_shares_are_numbered_for():
    """Shares are dealt out to 256 agents at most: one more and the call asks for no workspace and runs without."""
    lens = [(37 * i) % 90 for i in range(257)]
    w = synth.small(66, 1, 8, 1, 64, 64, False, lens, q_len=3)
    got, (spec, _, _, _) = append_chunk_and_attend(w)
    assert b.q4kv_attention_workspace_bytes(spec, 256, 3, 131072, 0, 1) > 0
    assert b.q4kv_attention_workspace_bytes(spec, 257, 3, 131072, 0, 1) == 0
    ospec, okp, ovp, otable = host_cache(w)
    want = oracle.attention(ospec, okp, ovp, w.q_all().numpy(), otable, w.final_lens(), w.sm_scale)
    assert_close(got, want)


def test_shared_chunk_replays_from_a_graph():
    """The two kernels of a call with shares, recorded once and replayed with other lengths and queries, the program's own work
    between the replays; every replay equals the eager call."""
    w = synth.small(67, 1, 4, 2, 256, 256, False, (1300, 700), q_len=64)
    _, (spec, kpool, vpool, table_d) = append_chunk_and_attend(w)
    msl, q = max(w.final_lens()), w.q_all(DEV).clone()
    sl = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV)
    ws, ws2 = (torch.empty(b.q4kv_attention_workspace_bytes(spec, 2, w.q_len, msl, 0, 1), dtype=torch.uint8, device=DEV) for _ in range(2))

    def call(out, workspace):
        return b.q4kv_batched_attention(spec, kpool, vpool, q, table_d, sl, msl, w.sm_scale, out=out, workspace=workspace)

    want = call(None, ws2)
    out = torch.empty_like(want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(out, ws)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out, ws)
    alone = call(None, None)
    torch.cuda.synchronize()
    assert not torch.equal(alone, want)                 # the call recorded is the one with shares
    for step, lens in enumerate((w.final_lens(), (64, 700), (1000, 0), w.final_lens())):
        sl.copy_(torch.tensor(lens, dtype=torch.int32))
        q.copy_(torch.randn(q.shape, generator=torch.Generator().manual_seed(step)).to(torch.float16))
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = call(None, ws2)
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {step}"


def test_shared_chunk_with_an_infinite_value():
    """A cached infinity (bias of group 0, scale zero) that every row sees makes that group's outputs infinite, whatever the number
    of records that are merged; here 28 or 29 a unit, and the merge takes them four at a time."""
    w = synth.small(68, 1, 16, 8, 256, 256, False, (7000,), q_len=64)
    spec, kpool, vpool, table, table_d = gpu_cache(w)
    for t in range(6000, 7000, 10):
        vpool.scale[:, int(table[0, t // 256]), :, t % 256, 0] = 0
        vpool.bias[:, int(table[0, t // 256]), :, t % 256, 0] = 0x7C00
    sl, q, msl = torch.tensor(w.final_lens(), dtype=torch.int32, device=DEV), w.q_all(DEV), max(w.final_lens())
    ws = torch.empty(b.q4kv_attention_workspace_bytes(spec, 1, w.q_len, msl, 0, 1), dtype=torch.uint8, device=DEV)
    alone = b.q4kv_batched_attention(spec, kpool, vpool, q, table_d, sl, msl, w.sm_scale)
    shared = b.q4kv_batched_attention(spec, kpool, vpool, q, table_d, sl, msl, w.sm_scale, workspace=ws)
    torch.cuda.synchronize()
    assert not torch.equal(alone[..., 64:], shared[..., 64:])        # the call with shares is another sum
    for out in (alone, shared):
        assert bool((out[..., :64] == float("inf")).all())
    assert_close(shared[..., 64:].cpu().numpy(), alone[..., 64:].cpu().numpy())
