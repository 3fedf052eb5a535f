"""GPU parity of q4kv_quantize / q4kv_dequantize / q4kv_append with the CPU oracle: bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_04428_amd import binding as b
from paper_2603_04428_amd import synth
from tests.gpu_util import DEV, bits, gpu_cache
from tests.util import tie_adjacent_rows

pytestmark = pytest.mark.gpu
F16 = np.float16


def check_quantize(x_np):
    x = torch.from_numpy(x_np).to(DEV)
    codes, scale, bias = b.q4kv_quantize(x)
    oc, os_, ob = oracle.quantize(x_np)
    assert np.array_equal(bits(scale), os_), "scale bits"
    assert np.array_equal(bits(bias), ob), "bias bits"
    assert np.array_equal(bits(codes), oc), "codes"
    # and back
    xh = b.q4kv_dequantize(codes, scale, bias)
    assert np.array_equal(bits(xh), oracle.dequantize(oc, os_, ob).view(np.uint16)), "dequantized"


@pytest.mark.parametrize("dim", [64, 128, 256, 576])
def test_quantize_random_rows_bit_exact(dim):
    rng = np.random.default_rng(dim)
    # several workgroups (32 groups each) and a ragged tail
    check_quantize(rng.standard_normal((1000 + 7, dim)).astype(F16))
    x = rng.standard_normal((333, dim))
    x[:, ::11] *= 8
    check_quantize(x.astype(F16))


@pytest.mark.parametrize("rows,dim", [(1, 64), (3, 64), (131, 64), (77, 192), (1001, 576)])
def test_quantize_parameter_arrays_at_odd_offsets(rows, dim):
    """The kernel stores scales and biases two at a time where it can: arrays that start on an odd 2-byte offset,
    and an odd number of groups, must come out the same, and nothing outside the arrays may be touched."""
    rng = np.random.default_rng(rows * 1000 + dim)
    x_np = rng.standard_normal((rows, dim)).astype(F16)
    x = torch.from_numpy(x_np).to(DEV)
    groups = rows * dim // 64
    guard = 0x5A5A                 # int16 pattern around the arrays
    scale_buf = torch.full((groups + 3,), guard, dtype=torch.int16, device=DEV)
    bias_buf = torch.full((groups + 3,), guard, dtype=torch.int16, device=DEV)
    codes = torch.empty((rows, dim // 8), dtype=torch.int32, device=DEV)
    scale = scale_buf[1:1 + groups].view(rows, dim // 64)
    bias = bias_buf[1:1 + groups].view(rows, dim // 64)
    assert scale.data_ptr() % 4 == 2 and bias.data_ptr() % 4 == 2
    b.q4kv_quantize(x, codes, scale, bias)
    oc, os_, ob = oracle.quantize(x_np)
    assert np.array_equal(bits(codes), oc)
    assert np.array_equal(bits(scale), os_) and np.array_equal(bits(bias), ob)
    for buf in (scale_buf, bias_buf):
        edge = buf.cpu().numpy()
        assert edge[0] == guard and (edge[1 + groups:] == guard).all()
    # one array aligned, the other not
    bias2 = torch.empty((rows, dim // 64), dtype=torch.int16, device=DEV)
    b.q4kv_quantize(x, codes, scale, bias2)
    assert np.array_equal(bits(scale), os_) and np.array_equal(bits(bias2), ob)


def test_quantize_special_groups_bit_exact():
    rng = np.random.default_rng(0)
    rows = []
    ramp = np.tile(np.arange(16), 4).astype(np.float64)
    rows.append(ramp)                                             # scale 1, codes = values
    rows.append(np.full(64, 3.25))                                # constant group
    z = np.zeros(64); z[3] = 7 * 2.0 ** -24; rows.append(z)       # scale rounds to zero
    z = np.zeros(64); z[3] = 8 * 2.0 ** -24; rows.append(z)       # smallest non-zero stored scale
    t = np.zeros(64); t[1] = 15; t[2:10] = [0.5, 1.5, 2.5, 3.5, 13.5, 14.5, 7.5, 8.5]; rows.append(t)   # ties
    nz = np.zeros(64); nz[0] = -0.0; nz[1] = 1.0; rows.append(nz)  # -0 is the first minimum
    pz = np.zeros(64); pz[5] = -0.0; pz[9] = 2.0; rows.append(pz)  # +0 first, -0 later
    x = np.stack(rows).astype(F16)
    check_quantize(x)
    check_quantize((rng.standard_normal((200, 64)) * 3e-6).astype(F16))          # subnormal inputs
    check_quantize((rng.standard_normal((200, 128)) * 1e-3).astype(F16))
    check_quantize(rng.uniform(-60000, 60000, (200, 64)).astype(F16))            # near the binary16 limit
    k = rng.integers(0, 15, (300, 64)) + 0.5                                     # values on code boundaries
    k[:, 0], k[:, 1] = 0, 15
    check_quantize(k.astype(F16))
    check_quantize((k * 0.37 - 2.0).astype(F16))
    # every binary16 magnitude pattern appears somewhere (finite only)
    allbits = np.arange(0, 0x7C00, dtype=np.uint16)
    allbits = np.concatenate([allbits, allbits | 0x8000])
    rng.shuffle(allbits)
    check_quantize(allbits[: (len(allbits) // 64) * 64].view(F16).reshape(-1, 64))


def test_quantize_quotients_next_to_rounding_ties_bit_exact():
    """Groups whose quotients (x - min) / scale sit on, just below and just above k + 0.5 for every code k and many
    scales (normal and subnormal binary16): a quotient approximated in any cheaper way than the correctly rounded
    binary32 division flips some of these codes."""
    x = tie_adjacent_rows(7)
    check_quantize(x)
    # the same rows tiled into wide rows (several groups per row, ragged row count)
    check_quantize(np.ascontiguousarray(x[: (len(x) // 4) * 4].reshape(-1, 256)))


def test_empty_input():
    x = torch.empty((0, 128), dtype=torch.float16, device=DEV)
    codes, scale, bias = b.q4kv_quantize(x)
    assert codes.shape == (0, 16) and scale.shape == (0, 2)
    assert b.q4kv_dequantize(codes, scale, bias).shape == (0, 128)


def test_dequantize_arbitrary_codes_bit_exact():
    rng = np.random.default_rng(5)
    codes = rng.integers(0, 2 ** 32, (777, 32), dtype=np.uint64).astype(np.uint32)
    scale = (rng.standard_normal((777, 4)) * 0.3).astype(F16)
    bias = (rng.standard_normal((777, 4)) * 2).astype(F16)
    scale[5] = 0
    scale[6] = np.array(2.0 ** -24, F16)
    bias[7] = 60000
    got = b.q4kv_dequantize(torch.from_numpy(codes.view(np.int32)).to(DEV),
                            torch.from_numpy(scale.view(np.int16)).to(DEV),
                            torch.from_numpy(bias.view(np.int16)).to(DEV))
    assert np.array_equal(bits(got), oracle.dequantize(codes, scale, bias).view(np.uint16))


@pytest.mark.parametrize("alias", [False, True])
def test_append_bit_exact_and_touches_nothing_else(alias):
    if alias:
        w = synth.small(21, 2, 4, 1, 576, 512, True, (250, 7, 600), 1)
    else:
        w = synth.small(21, 3, 4, 2, 128, 64, False, (250, 7, 600), 1)
    A, Cn = 3, 300                                                 # chunks cross block boundaries
    lens = np.array(w.seq_lens, np.int32)
    need = (lens + Cn + 255) // 256
    mb = int(need.max())
    rng = np.random.default_rng(3)
    nb = int(need.sum()) + 2
    perm = rng.permutation(nb - 2)
    table = np.zeros((A, mb), np.int32)
    pos = 0
    for a in range(A):
        table[a, :need[a]] = perm[pos:pos + need[a]]
        pos += need[a]
    gspec = b.make_spec(w.num_layers, w.num_q_heads, w.num_kv_heads, w.k_dim, w.v_dim, alias)
    ospec = oracle.make_spec(w.num_layers, w.num_q_heads, w.num_kv_heads, w.k_dim, w.v_dim, alias)
    gk = b.Pool(gspec, w.k_dim, nb, DEV, poison=True)
    gv = None if alias else b.Pool(gspec, w.v_dim, nb, DEV, poison=True)
    ok = oracle.Pool(ospec, w.k_dim, nb, fill=0x7E00)
    ov = None if alias else oracle.Pool(ospec, w.v_dim, nb, fill=0x7E00)
    L0, L1 = (0, 2) if alias else (1, 3)
    k_new = torch.stack([torch.stack([w.k_rows(l, a, 1000, 1000 + Cn) for a in range(A)]) for l in range(L0, L1)])
    v_new = None if alias else torch.stack([torch.stack([w.v_rows(l, a, 1000, 1000 + Cn) for a in range(A)])
                                            for l in range(L0, L1)])
    oracle.append(ospec, ok, ov, k_new.numpy(), None if alias else v_new.numpy(), table, lens, L0, L1)
    b.q4kv_append(gspec, gk, gv, k_new.to(DEV), None if alias else v_new.to(DEV), torch.from_numpy(table).to(DEV),
                  torch.from_numpy(lens).to(DEV), L0, L1)
    for gp, op in ((gk, ok), (gv, ov)):
        if gp is None:
            continue
        assert np.array_equal(bits(gp.codes), op.codes)
        assert np.array_equal(bits(gp.scale), op.scale)
        assert np.array_equal(bits(gp.bias), op.bias)


def test_append_of_the_longest_chunk_the_library_admits():
    """chunk_len = 2^20 tokens (Q4KV_MAX_CHUNK_LEN) behind an odd number of cached tokens: the kernel places rows
    with quotients that are exact up to there, and the block index runs over 4,097 blocks.  One layer, one narrow
    head: 128 MB of rows.  Random values drawn on the device; the oracle appends the same rows on the host."""
    Cn, n0 = 1 << 20, 37
    spec = b.make_spec(1, 1, 1, 64)
    ospec = oracle.make_spec(1, 1, 1, 64)
    nb = (n0 + Cn + 255) // 256 + 1
    rng = np.random.default_rng(5)
    table = rng.permutation(nb)[None, :nb - 1].astype(np.int32)
    g = torch.Generator(device="cpu").manual_seed(5)
    rows = torch.randn((1, 1, Cn, 1, 64), generator=g, dtype=torch.float32).to(torch.float16)
    rows[0, 0, ::4097, 0, ::7] *= 8
    gk, gv = b.Pool(spec, 64, nb, DEV, poison=True), b.Pool(spec, 64, nb, DEV, poison=True)
    ok, ov = oracle.Pool(ospec, 64, nb, fill=0x7E00), oracle.Pool(ospec, 64, nb, fill=0x7E00)
    lens = np.array([n0], np.int32)
    oracle.append(ospec, ok, ov, rows.numpy(), rows.numpy(), table, lens, 0, 1)
    d = rows.to(DEV)
    b.q4kv_append(spec, gk, gv, d, d, torch.from_numpy(table).to(DEV), torch.from_numpy(lens).to(DEV), 0, 1)
    for gp, op in ((gk, ok), (gv, ov)):
        assert np.array_equal(bits(gp.codes), op.codes)
        assert np.array_equal(bits(gp.scale), op.scale)
        assert np.array_equal(bits(gp.bias), op.bias)
    with pytest.raises(Exception):          # one token more is refused before anything is launched
        b.q4kv_append(spec, gk, gv, torch.empty((1, 1, Cn + 1, 1, 64), dtype=torch.float16, device=DEV), d,
                      torch.from_numpy(table).to(DEV), torch.from_numpy(lens).to(DEV), 0, 1)


def test_append_skips_tokens_outside_the_table_or_pool():
    w = synth.small(22, 1, 2, 2, 64, 64, False, (250,), 1)
    spec = b.make_spec(1, 2, 2, 64)
    k = b.Pool(spec, 64, 2, DEV, poison=True)
    v = b.Pool(spec, 64, 2, DEV, poison=True)
    before = bits(k.codes).copy()
    k_new = w.k_rows(0, 0, 0, 20, DEV)[None, None].contiguous()
    table = torch.tensor([[0, 7]], dtype=torch.int32, device=DEV)       # second block id is outside the pool
    b.q4kv_append(spec, k, v, k_new, k_new, table, torch.tensor([250], dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    after = bits(k.codes)
    assert not np.array_equal(after[0, 0, :, 250:256], before[0, 0, :, 250:256])    # slots 250..255 written
    assert np.array_equal(after[0, 1], before[0, 1])                                 # nothing else


def test_full_size_cache_quantize_sampled_rows():
    """One fresh 4,096-token Gemma-shaped agent cache (the size the benchmark times): K and V of 48 layers,
    8 heads, 256 wide.  Quantized layer by layer on the GPU; seeded sample rows are regenerated on the host
    and checked bit-exact against the oracle, then the round trip through q4kv_dequantize likewise."""
    w = synth.Workload("gemma_one_agent_4k", 2, 48, 16, 8, 256, 256, False, [4096])
    rng = np.random.default_rng(7)
    for l in (0, 17, 47):
        for tensor, rows_fn in (("k", w.k_rows), ("v", w.v_rows)):
            x = rows_fn(l, 0, 0, 4096, DEV)                      # [4096][8][256]
            codes, scale, bias = b.q4kv_quantize(x)
            xh = b.q4kv_dequantize(codes, scale, bias)
            toks = sorted(set([0, 4095] + rng.integers(0, 4096, 24).tolist()))
            for t in toks:
                ref = rows_fn(l, 0, t, t + 1).numpy()            # regenerated on the host
                oc, os_, ob = oracle.quantize(ref)
                assert np.array_equal(bits(codes[t:t + 1]), oc)
                assert np.array_equal(bits(scale[t:t + 1]), os_)
                assert np.array_equal(bits(bias[t:t + 1]), ob)
                assert np.array_equal(bits(xh[t:t + 1]), oracle.dequantize(oc, os_, ob).view(np.uint16))
            # property that holds at any size: every reconstruction within scale/2 of its input
            s = torch.from_numpy(bits(scale).view(F16).astype(np.float32)).to(DEV).repeat_interleave(64, dim=-1)
            err = (xh.float() - x.float()).abs()
            ulp = torch.ldexp(torch.ones_like(err), torch.frexp(xh.float().abs().clamp_min(2.0 ** -14))[1] - 12)
            assert bool((err <= s / 2 * 1.001 + ulp).all())


def test_read_probe_reads_only():
    """The measurement helper touches nothing but (possibly) its sink word, for sizes below, at and off its 16 KiB step."""
    g = torch.Generator(device="cpu").manual_seed(7)
    for nbytes in (0, 100, 16384, 16384 * 5 + 48, 16384 * 2049):
        host = torch.randint(0, 2 ** 31 - 1, (nbytes // 4 + 4,), dtype=torch.int32, generator=g)
        buf = host.to(DEV)
        sink = torch.zeros(1, dtype=torch.int32, device=DEV)
        b.q4kv_read_probe(buf[: nbytes // 4], sink)
        torch.cuda.synchronize()
        assert torch.equal(buf.cpu(), host)
    with pytest.raises(b.Q4KVError):
        b.q4kv_read_probe(buf.view(torch.uint8)[4:4 + 32768], sink)   # not 16-byte aligned


@pytest.mark.parametrize("dims", [(256, 256), (192, 128), (64, 64)])
@pytest.mark.parametrize("chunk", [1, 5, 21, 70])
def test_small_append_matches_oracle(dims, chunk):
    """Appends that do not fill the chip (rounds of 16 groups per wave): group counts around a wave's round and a
    workgroup's four, a chunk that crosses a block boundary, a table entry outside the pool, bit for bit."""
    w = synth.small(81, 2, 6, 3, dims[0], dims[1], False, (254, 0, 300), q_len=chunk if chunk > 1 else 2)
    spec, kpool, vpool, table, table_d = gpu_cache(w, tokens=w.seq_lens)
    bad = table_d.clone()
    bad[2, 1] = -7                                      # agent 2's tokens from 256 on fall into a block outside the pool
    k_new = torch.stack([torch.stack([w.k_rows(l, a, n, n + chunk, DEV) for a, n in enumerate(w.seq_lens)]) for l in range(2)])
    v_new = torch.stack([torch.stack([w.v_rows(l, a, n, n + chunk, DEV) for a, n in enumerate(w.seq_lens)]) for l in range(2)])
    before = torch.tensor(w.seq_lens, dtype=torch.int32, device=DEV)
    b.q4kv_append(spec, kpool, vpool, k_new.contiguous(), v_new.contiguous(), bad, before)
    torch.cuda.synchronize()
    for l in range(2):
        for pool, new, dim in ((kpool, k_new, dims[0]), (vpool, v_new, dims[1])):
            for a, n in enumerate(w.seq_lens):
                for c in range(chunk):
                    if a == 2:
                        continue
                    blk, slot = int(table[a, (n + c) // 256]), (n + c) % 256
                    codes, scale, bias = oracle.quantize(new[l, a, c].cpu().numpy())
                    assert np.array_equal(bits(pool.codes[l, blk, :, slot]), codes)
                    assert np.array_equal(bits(pool.scale[l, blk, :, slot]), scale)
                    assert np.array_equal(bits(pool.bias[l, blk, :, slot]), bias)
            # the skipped agent's own block keeps its poison
            assert bool((pool.scale[l, int(table[2, 1]), :, 300 - 256:] == 0x7E00).all())


@pytest.mark.parametrize("param_format", [0, 1])
@pytest.mark.parametrize("dims", [(192, 128), (128, 64)])
def test_long_append_matches_oracle(dims, param_format):
    """Appends of more groups than the chip holds at once (rounds of 64 groups per wave): K and V rows of unequal width, group
    counts that end inside a round, blocks crossed, a table entry outside the pool and one past the table; the whole pools."""
    heads, chunk = (6, 701) if dims[0] == 192 else (12, 533)
    w = synth.small(82, 2, heads, heads, dims[0], dims[1], False, (254, 0, 300), q_len=2)
    A, L, groups = 3, 2, chunk * heads * (dims[0] // 64)
    assert 2 * L * A * ((groups + 63) // 64) > 8 * torch.cuda.get_device_properties(0).multi_processor_count and groups % 64
    lens = np.array(w.seq_lens, np.int32)
    need = (lens + chunk + 255) // 256
    nb, mb = int(need.sum()) + 1, int(need.max()) - 1               # the longest agent's last block is past the table
    perm = np.random.default_rng(5).permutation(nb - 1)
    table, at = np.zeros((A, mb), np.int32), 0
    for a in range(A):
        k = min(int(need[a]), mb)
        table[a, :k] = perm[at:at + k]
        at += k
    table[0, 2] = nb                                                # one id past the pool
    whole = np.concatenate([table, np.full((A, 1), nb + 1, np.int32)], axis=1)   # the oracle has blocks for the skipped tokens
    gspec = b.make_spec(L, heads, heads, dims[0], dims[1], param_format=param_format)
    ospec = oracle.make_spec(L, heads, heads, dims[0], dims[1], False, param_format=param_format)
    fill = 0x7FC0 if param_format else 0x7E00
    gk, gv = b.Pool(gspec, dims[0], nb, DEV, poison=True), b.Pool(gspec, dims[1], nb, DEV, poison=True)
    ok, ov = oracle.Pool(ospec, dims[0], nb + 2, fill=fill), oracle.Pool(ospec, dims[1], nb + 2, fill=fill)
    k_new = torch.stack([torch.stack([w.k_rows(l, a, 0, chunk) for a in range(A)]) for l in range(L)])
    v_new = torch.stack([torch.stack([w.v_rows(l, a, 0, chunk) for a in range(A)]) for l in range(L)])
    oracle.append(ospec, ok, ov, k_new.numpy(), v_new.numpy(), whole, lens)
    b.q4kv_append(gspec, gk, gv, k_new.to(DEV), v_new.to(DEV), torch.from_numpy(table).to(DEV), torch.from_numpy(lens).to(DEV))
    for gp, op in ((gk, ok), (gv, ov)):
        assert np.array_equal(bits(gp.codes), op.codes[:, :nb])
        assert np.array_equal(bits(gp.scale), op.scale[:, :nb])
        assert np.array_equal(bits(gp.bias), op.bias[:, :nb])


@pytest.mark.parametrize("param_format", [0, 1])
def test_append_in_one_piece_and_in_pieces(param_format):
    """The kernel of long appends (above 96 groups per workgroup slot: 64 groups per wave and round) writes what the kernel
    of short ones writes piece by piece: rows of unequal width, group counts that end inside a round, blocks crossed."""
    heads, dims, A, L, chunk = 6, (192, 128), 3, 2, 1001
    slots = 8 * torch.cuda.get_device_properties(0).multi_processor_count
    groups = chunk * heads * (dims[0] // 64)
    assert 2 * L * A * groups > 96 * slots and 2 * L * A * (groups // 4) <= 96 * slots and groups % 64
    spec = b.make_spec(L, heads, heads, dims[0], dims[1], param_format=param_format)
    lens = torch.tensor([254, 0, 300], dtype=torch.int32, device=DEV)
    table = torch.randperm(18, generator=torch.Generator().manual_seed(3)).view(A, 6).to(torch.int32).to(DEV)
    table[0, 2] = 18                                                # one id past the pool
    g = torch.Generator(device=DEV).manual_seed(9)
    k_new, v_new = (torch.randn((L, A, chunk, heads, d), device=DEV, generator=g).half() for d in dims)
    pools = [[b.Pool(spec, d, 18, DEV, poison=True) for d in dims] for _ in range(2)]
    b.q4kv_append(spec, *pools[0], k_new, v_new, table, lens)
    for c in range(0, chunk, 250):
        b.q4kv_append(spec, *pools[1], k_new[:, :, c:c + 250].contiguous(), v_new[:, :, c:c + 250].contiguous(), table, lens + c)
    for one, other in zip(*pools):
        assert torch.equal(one.codes, other.codes) and torch.equal(one.scale, other.scale) and torch.equal(one.bias, other.bias)
