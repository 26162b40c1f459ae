"""GPU parity at the sizes where the kernels' tiles and dispatch rules change: remainders, the smallest and
the largest of a range, against the CPU oracle on the same seeded inputs."""
import numpy as np
import pytest

from oracle import bitdecode_oracle as O
from paper_2503_18773_amd import binding as B
from paper_2503_18773_amd import workloads as W
from tests.test_gpu_parity import BITS, GROUP, _int_cache_pair
from tests.util import assert_attn_close, attn_errors, out_to_f64, to_dev

pytestmark = pytest.mark.gpu


def _attend_f32(gc, w, q, num_splits):
    import torch
    gc.desc.out_type = B.BD_OUT_F32
    out = torch.full((w.batch, w.n_q_heads, 128), 7.0, dtype=torch.float32, device="cuda:0")
    gc.decode_attn(to_dev(q, w.in_dtype), W.softmax_scale(w), out, num_splits=num_splits)
    torch.cuda.synchronize()
    return out_to_f64(out)


def _partials(ws, ns, batch, hq):
    """The workspace's partial rows [ns, batch, hq, 128] and their (maximum, sum) [ns, batch, hq, 2]."""
    import torch
    f = ws.view(torch.float32)
    n = ns * batch * hq
    return f[:n * 128].view(ns, batch, hq, 128), f[n * 128:n * 130].view(ns, batch, hq, 2)


@pytest.mark.parametrize("fmt,gq", [("int4", 4), ("int4", 16), ("int2_kt", 7), ("int4_g32", 3), ("int2_kt_g64", 8)])
def test_residual_slices_of_every_remainder(fmt, gq):
    """Nothing but residual tokens, 1 .. 127 of them, in one slice and in several, some empty: the slice ends on and beside
    the steps of the second product (4 tokens a load, 32 a k-step).  Scores and weights are fp32 (weights enter
    the product whole), so the bar is fp32's: a score is a sum of 128 products whose magnitudes add up to
    about 1e2, which the matrix unit rounds (truncating) at 2^-23 of its size, i.e. 1e-5 in the exponent; the
    result's relative L2 error is at most that."""
    for L in (1, 3, 4, 5, 31, 32, 33, 64, 97, 127):
        w = W.scaled(W.CONFIGS["cfg1"], batch=2, n_q_heads=2 * gq, n_kv_heads=2, context=L, fmt=fmt, seed=300 + L)
        K, V, oc, gc = _int_cache_pair(w, 128)
        q = W.make_q(w)
        ref = O.decode_attn(oc, q, W.softmax_scale(w))
        for ns in (1, 3, 9):   # (9: empty slices among them at L < 9)
            ma, rl = attn_errors(_attend_f32(gc, w, q, ns), ref)
            assert rl <= 1e-5, f"{fmt} gq={gq} L={L} splits={ns}: rel-L2 {rl:.2e} max-abs {ma:.2e}"


@pytest.mark.parametrize("L", [1, 2, 7, 8, 31, 32, 33, 63, 65, 96, 126, 127, 129])
def test_mx_prompt_ends_inside_a_block(L):
    """The block at the end of an MXFP4 prompt: the tokens' codes and scales bit for bit, and the bytes past them
    left as they were (pre-set to a pattern; an odd last token's byte gets a zero high nibble)."""
    import torch
    w = W.scaled(W.CONFIGS["cfg4"], batch=2, n_q_heads=4, n_kv_heads=2, context=L, seed=500 + L)
    K, V = W.make_kv(w)
    oc = O.MxCache(2, 2, 256); oc.quant_pack_kv(K, V)
    gc = B.KVCache(2, 4, 2, "mxfp4", 256)
    for buf in gc.buffers[:4]:
        buf.fill_(0xA5)
    gc.quant_pack_kv(to_dev(K, "bf16"), to_dev(V, "bf16"))
    torch.cuda.synchronize()
    assert gc.packed_len == L
    for i, name in enumerate(["k_codes", "v_codes", "k_scales", "v_scales"]):
        ref = getattr(oc, name).copy()
        if name == "v_codes":   # [.., block, channel, byte of two tokens]
            tok = 128 * np.arange(2)[:, None, None] + 2 * np.arange(64)[None, None, :] + np.zeros((2, 128, 64), int)
            ref[:, :, tok >= L] = 0xA5
        else:
            ref[:, :, L:] = 0xA5
        assert np.array_equal(gc.host_buffer(i).reshape(ref.shape), ref), name


@pytest.mark.parametrize("fmt", ["int4", "int2_kt", "int4_g32"])
@pytest.mark.parametrize("L", [1, 15, 63, 64, 65, 127, 128, 129, 255])
def test_prompt_tails_go_to_the_residual(fmt, L):
    """One launch quantizes a prompt's whole blocks and copies its L mod 128 last tokens (four rounds of 64
    rows' pieces): contiguous against the oracle, rows past the tail untouched, and a paged sequence the same
    bytes."""
    import torch
    from tests.test_gpu_parity import _assert_int_cache_equal
    w = W.scaled(W.CONFIGS["cfg1"], batch=2, n_q_heads=6, n_kv_heads=3, context=L, fmt=fmt, seed=600 + L)
    K, V = W.make_kv(w)
    oc = O.IntCache(2, 3, BITS[fmt], 256, k_per_token="_kt" in fmt, group=GROUP.get(fmt, 128))
    oc.quant_pack_kv(K, V)
    gc = B.KVCache(2, 6, 3, fmt, 256)
    pc = B.PagedKVCache(2, 6, 3, fmt, 4, np.array([[2, 0], [3, 1]], np.int32))
    for c in (gc, pc):
        for buf in c.buffers[4:]:
            buf.fill_(0x3C)
    k, v = to_dev(K, "fp16"), to_dev(V, "fp16")
    gc.quant_pack_kv(k, v)
    for s in range(2):
        pc.quant_pack_kv(s, k[s], v[s])
    _assert_int_cache_equal(oc, gc)
    assert pc.seq_lens.tolist() == [L, L] and pc.status.item() == 0
    for i in (4, 5):
        res = gc.host_buffer(i).view(np.uint16).reshape(2, 3, 128, 128)
        assert np.all(res[:, :, L % 128:] == 0x3C3C)
        assert np.array_equal(pc.host_buffer(i), gc.host_buffer(i))
    for i in range(4):
        pages = pc.host_buffer(i).reshape(4, 3, -1)[[[2, 0], [3, 1]]]   # [sequence][block][head]
        blocks = gc.host_buffer(i).reshape(2, 3, 2, -1).transpose(0, 2, 1, 3)
        assert np.array_equal(pages[:, :L // 128], blocks[:, :L // 128])


@pytest.mark.parametrize("fmt", ["int4", "int2", "int4_kt", "int2_kt"])
@pytest.mark.parametrize("gq", [1, 2, 3, 4])
def test_small_query_groups_hold_the_precision_of_their_pieces(fmt, gq):
    """Query groups of up to 4 heads run both products on 8-bit matrix operands, queries as integers in four bytes and
    weights as sums of e4m3 pieces, whose products add up exactly: one block, fewer blocks than waves, several rounds of
    blocks, and enough rounds (17 a wave) to fold the centre sum.  Weights hold 19 bits, a relative error of 2^-20 each, and
    queries all that shows here (2^-30 of a block's largest product, which is of the scores' size); the scores' fp32
    roundings (about eight of 2^-23) are of a sum of magnitudes of at most some tens in log2 units, up to 1e-5 in the
    exponent."""
    bar = 2.0 ** -20 + 1e-5
    for L, ns in [(128, 1), (128 * 3 + 1, 1), (128 * 5, 2), (128 * 4 * 17 + 130, 1)]:
        w = W.scaled(W.CONFIGS["cfg1"], batch=1, n_q_heads=2 * gq, n_kv_heads=2, context=L, fmt=fmt, seed=700 + L + gq)
        K, V, oc, gc = _int_cache_pair(w, (L // 128 + 1) * 128)
        q = W.make_q(w)
        ma, rl = attn_errors(_attend_f32(gc, w, q, ns), O.decode_attn(oc, q, W.softmax_scale(w)))
        assert rl <= bar, f"{fmt} gq={gq} L={L}: rel-L2 {rl:.2e} max-abs {ma:.2e}"


@pytest.mark.parametrize("fmt,hq", [("int4", 8), ("int2_kt", 16), ("int4_g32", 8), ("mxfp4", 8), ("mxfp4", 20)])
@pytest.mark.parametrize("batch", [2, 33, 64, 65])
def test_ragged_batches_attend_their_own_lengths_in_any_order(fmt, hq, batch):
    """A paged launch whose last round of workgroups is short (257 .. 384, 513 .. 640, ..) takes up to 64 sequences
    longest first: equal, empty and one-token lengths among them, every row is bit for bit that of the batch in
    reverse order and that of a batch of one."""
    import torch
    mx = fmt == "mxfp4"
    rng = np.random.default_rng(batch)
    lens = rng.integers(0, 500, batch)
    lens[:2] = 300, 300
    if batch > 8:
        lens[3:8] = 0, 1, 499, 499, 128
    maxp = 4
    dt = torch.bfloat16 if mx else torch.float16
    table = torch.randperm(batch * maxp).view(batch, maxp).to(torch.int32)
    gen = torch.Generator(device="cuda:0").manual_seed(batch)
    pc, back = (B.PagedKVCache(batch, hq, 2, fmt, batch * maxp, table) for _ in range(2))   # back: in reverse order
    q = torch.randn((batch, hq, 128), device="cuda:0", generator=gen).to(dt)
    kv = []
    for s in range(batch):
        k, v = (torch.randn((2, int(lens[s]), 128), device="cuda:0", generator=gen).to(dt) for _ in range(2))
        pc.quant_pack_kv(s, k, v)
        back.quant_pack_kv(batch - 1 - s, k, v)
        kv.append((k, v))
    wgs = 2 * batch
    for ns in (2, 3, 256 // wgs + 1, 512 // wgs + 1):   # the last two: just above one and two rounds
        out, rev = (torch.full((batch, hq, 128), x, dtype=dt, device="cuda:0") for x in (7.0, 5.0))
        pc.decode_attn(q, 0.088, out, num_splits=ns)
        back.decode_attn(q.flip(0).contiguous(), 0.088, rev, num_splits=ns)
        torch.cuda.synchronize()
        assert torch.equal(out, rev.flip(0)), f"{fmt} batch {batch} splits {ns}"
        for s in range(0, batch, 1 + batch // 8):
            one = B.PagedKVCache(1, hq, 2, fmt, maxp, torch.arange(maxp, dtype=torch.int32).view(1, maxp))
            one.quant_pack_kv(0, *kv[s])
            ref = torch.full((1, hq, 128), 9.0, dtype=dt, device="cuda:0")
            one.decode_attn(q[s:s + 1].contiguous(), 0.088, ref, num_splits=ns)
            torch.cuda.synchronize()
            assert torch.equal(out[s], ref[0]), f"{fmt} batch {batch} splits {ns}: sequence {s} of {lens[s]}"
    assert pc.status.item() == 0


@pytest.mark.parametrize("fmt,batch,ns", [("int4", 64, 4), ("int2_kt", 49, 4), ("mxfp4", 29, 8), ("int4_g32", 3, 80),
                                          ("int4_kt_g64", 2, 128), ("int4", 33, 4)])
def test_second_layers_of_workgroups_attend_their_own_sequences(fmt, batch, ns):
    """Up to 512 workgroups with tables of eight blocks a split: the shortest sequences share a compute unit with the
    next shortest (512 = all of them, odd batches, a second layer of more than half of the sequences).  Every row is bit
    for bit that of a batch of one."""
    import torch
    dt = torch.bfloat16 if fmt == "mxfp4" else torch.float16
    rng = np.random.default_rng(batch)
    lens = rng.integers(0, 500, batch)
    lens[:2] = 1, 300
    table = torch.full((batch, 8 * ns), -1, dtype=torch.int32)
    table[:, :4] = torch.randperm(batch * 4).view(batch, 4).to(torch.int32)
    gen = torch.Generator(device="cuda:0").manual_seed(batch)
    pc = B.PagedKVCache(batch, 8, 2, fmt, batch * 4, table)
    q = torch.randn((batch, 8, 128), device="cuda:0", generator=gen).to(dt)
    kv = [tuple(torch.randn((2, int(n), 128), device="cuda:0", generator=gen).to(dt) for _ in range(2)) for n in lens]
    for s, (k, v) in enumerate(kv):
        pc.quant_pack_kv(s, k, v)
    out = torch.full((batch, 8, 128), 7.0, dtype=dt, device="cuda:0")
    pc.decode_attn(q, 0.088, out, num_splits=ns)
    for s, (k, v) in enumerate(kv):
        one = B.PagedKVCache(1, 8, 2, fmt, 4, torch.arange(4, dtype=torch.int32).view(1, 4))
        one.quant_pack_kv(0, k, v)
        ref = torch.full((1, 8, 128), 9.0, dtype=dt, device="cuda:0")
        one.decode_attn(q[s:s + 1].contiguous(), 0.088, ref, num_splits=ns)
        torch.cuda.synchronize()
        assert torch.equal(out[s], ref[0]), f"{fmt} batch {batch} splits {ns}: sequence {s} of {lens[s]}"
    assert pc.status.item() == 0


@pytest.mark.parametrize("hq", [8, 16, 32])
@pytest.mark.parametrize("batch,ns,pages,L", [(40, 4, 3, 300), (40, 4, 3, 0), (64, 4, 32, 129), (33, 4, 17, 128 * 17), (3, 43, 1, 128)])
def test_mx_batches_of_equal_lengths_in_launches_that_sort(hq, batch, ns, pages, L):
    """Equal lengths keep the order as given, for which a wave asks for its first page's number before it knows: tables
    narrower and wider than the waves of a sequence, every row bit for bit that of a batch of one."""
    import torch
    gen = torch.Generator(device="cuda:0").manual_seed(L)
    rows = lambda *shape: torch.randn(shape, device="cuda:0", generator=gen).to(torch.bfloat16)
    table = torch.randperm(batch * pages).view(batch, pages).to(torch.int32)
    pc = B.PagedKVCache(batch, hq, 2, "mxfp4", batch * pages, table)
    q, kv = rows(batch, hq, 128), [(rows(2, L, 128), rows(2, L, 128)) for _ in range(batch)]
    for s, (k, v) in enumerate(kv):
        pc.quant_pack_kv(s, k, v)
    out, ref = (torch.full((batch, hq, 128), x, dtype=torch.bfloat16, device="cuda:0") for x in (7.0, 9.0))
    pc.decode_attn(q, 0.088, out, num_splits=ns)
    for s, (k, v) in enumerate(kv):
        one = B.PagedKVCache(1, hq, 2, "mxfp4", pages, torch.arange(pages - 1, -1, -1, dtype=torch.int32).view(1, pages))
        one.quant_pack_kv(0, k, v)
        one.decode_attn(q[s:s + 1].contiguous(), 0.088, ref[s:s + 1], num_splits=ns)
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and pc.status.item() == 0


@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("fmt,hq,batch,ns", [("int4", 8, 48, 4), ("int4", 8, 40, 7), ("int2_kt", 16, 60, 4), ("int4_g32", 8, 44, 4),
                                             ("int4_g32", 16, 64, 3), ("mxfp4", 8, 40, 4), ("mxfp4", 32, 50, 4)])
def test_steps_of_batches_dealt_by_length(fmt, hq, batch, ns, lazy):
    """Two fused steps in launches that deal the sequences by length (2 KV heads: 320 to 560 workgroups, tables of eight blocks
    a split): each sequence's token goes to its own residual or page, a block that it fills to the sequence's own page, one that
    needs a page it does not have is dropped.  Eager, against append + attention on a twin; lazy, each sequence against a
    lazy step of a batch of one: outputs, residual rows, pages and lengths bit for bit."""
    import torch
    mx, H, P = fmt == "mxfp4", 2, 5
    dt = torch.bfloat16 if mx else torch.float16
    rng = np.random.default_rng(batch + ns)
    lens = rng.integers(0, 500, batch)
    lens[:8] = 127, 128 * 3 + 127, 0, 128 * 2 + 127, 128 * 3 + 127, 126, 128, 300
    lens[-3:] = 128 + 127, 1, 128 * 2 + 126
    table = torch.full((batch, 8 * ns), -1, dtype=torch.int32)
    table[:, :P] = torch.as_tensor(rng.permutation(batch * P).reshape(batch, P).astype(np.int32))
    table[4, 3 if not mx else 4] = -1   # (128 * 3 + 127 tokens: no page for the block that is filled, or begun, next)
    if mx:
        lens[4] = 128 * 4
    gen = torch.Generator(device="cuda:0").manual_seed(batch)
    rows = lambda *shape: torch.randn(shape, device="cuda:0", generator=gen).to(dt)
    kv = [(rows(H, int(n), 128), rows(H, int(n), 128)) for n in lens]

    def paged(seqs, t):
        c = B.PagedKVCache(len(seqs), hq, H, fmt, batch * P, t)
        for i, s in enumerate(seqs):
            c.quant_pack_kv(i, *kv[s])
        return c

    a = paged(range(batch), table)
    twin = None if lazy else paged(range(batch), table)
    ones = [paged([s], table[s:s + 1]) for s in range(batch)] if lazy else []
    for step in range(2):
        kn, vn, q = rows(batch, H, 128), rows(batch, H, 128), rows(batch, hq, 128)
        out, ref = (torch.full((batch, hq, 128), x, dtype=dt, device="cuda:0") for x in (7.0, 9.0))
        a.decode_step(kn, vn, q, 0.088, out, ns, lazy=lazy)
        if lazy:
            for s, one in enumerate(ones):
                one.decode_step(*(x[s:s + 1].contiguous() for x in (kn, vn, q)), 0.088, ref[s:s + 1], ns, lazy=True)
        else:
            twin.append_kv(kn, vn)
            twin.decode_attn(q, 0.088, ref, ns)
        torch.cuda.synchronize()
        for s in range(batch):
            assert torch.equal(out[s], ref[s]), f"{fmt} step {step}: sequence {s} of {lens[s]}"
        assert a.status.item() == 2
    want = [int(n) + 2 for n in lens]
    want[4] = int(lens[4])
    assert a.seq_lens.tolist() == want
    per_page = [n // (batch * P) for n in a.sizes[:4]]
    per_seq = [n // batch for n in a.sizes[4:6]]
    if lazy:
        for s, one in enumerate(ones):
            assert one.seq_lens.item() == want[s]
            for i in range(0 if mx else 2):
                assert torch.equal(a.buffers[4 + i][s * per_seq[i]:(s + 1) * per_seq[i]], one.buffers[4 + i][:per_seq[i]]), (s, i)
            for page in table[s, :P].tolist():
                for i in range(4):
                    at = slice(page * per_page[i], (page + 1) * per_page[i])
                    assert page < 0 or torch.equal(a.buffers[i][at], one.buffers[i][at]), (s, page, i)
    else:
        for i in range(4 if mx else 6):
            assert torch.equal(a.buffers[i], twin.buffers[i]), i


@pytest.mark.parametrize("fmt,gq", [("int4", 4), ("int2_kt", 8), ("int4_g32", 8), ("mxfp4", 4), ("mxfp4", 12)])
@pytest.mark.parametrize("L,asked", [(600, 2), (600, 5), (128 * 9 + 40, 14), (0, 3), (128 * 9 + 40, None)])
def test_a_call_that_merges_is_its_partials_and_a_merge(fmt, gq, L, asked):
    """Whatever count is asked for (None: the one bd_choose_splits names) is run: the workspace holds that many
    partials, whatever was in it before (NaNs here), which merge to the rows of the call that writes `out`, bit for
    bit, by bd_splitk_combine and, to fp32 rounding, by the formula that the interface states."""
    import torch
    mx = fmt == "mxfp4"
    dt = torch.bfloat16 if mx else torch.float16
    gen = torch.Generator(device="cuda:0").manual_seed(L + (asked or 0))
    gc = B.KVCache(3, 2 * gq, 2, fmt, 1280)
    k, v = (torch.randn((3, 2, L, 128), device="cuda:0", generator=gen).to(dt) for _ in range(2))
    gc.quant_pack_kv(k, v)
    gc.desc.out_type = B.BD_OUT_F32
    asked = asked or gc.choose_splits()
    q = torch.randn((3, 2 * gq, 128), device="cuda:0", generator=gen).to(dt)
    out, merged, split = (torch.full((3, 2 * gq, 128), x, device="cuda:0") for x in (3.0, 5.0, 7.0))
    ws = gc.workspace(asked)
    ws.fill_(0xFF)
    B.bd_decode_attn(gc.desc, q, gc.packed_len, gc.res_len, 0.088, asked, ws, out)
    B.bd_splitk_combine(gc.desc, ws, asked, merged)
    rows, ml = (x.double() for x in _partials(ws, asked, 3, 2 * gq))
    gc.decode_attn(q, 0.088, split, num_splits=asked, fused=False)
    torch.cuda.synchronize()
    assert torch.equal(merged, out) and torch.equal(split, out)
    blocks = (gc.packed_len + 127) // 128
    assert ((ml[..., 1] > 0).all(-1).all(-1).sum().item() >= min(asked, (blocks + 3) // 4))
    if L:
        f = torch.exp2(ml[..., 0] - ml[..., 0].amax(0))
        formula = (rows * f[..., None]).sum(0) / (ml[..., 1] * f).sum(0)[..., None]
        assert torch.allclose(formula.float(), out, rtol=1e-5, atol=1e-6)
    else:
        assert not rows.any() and not out.any()


@pytest.mark.parametrize("fmt,gq", [("int4", 4), ("int2_kt", 8), ("int4_g32", 8), ("mxfp4", 4)])
def test_the_count_of_a_step_left_to_the_library(fmt, gq):
    """No count given: the call runs bd_step_splits, and its rows are those of that count given."""
    import torch
    dt = torch.bfloat16 if fmt == "mxfp4" else torch.float16
    for L in (0, 100, 900, 5000, 40000):
        gen = torch.Generator(device="cuda:0").manual_seed(L)
        gc = B.KVCache(1, 2 * gq, 2, fmt, L // 128 * 128 + 128)
        k, v = (torch.randn((1, 2, L, 128), device="cuda:0", generator=gen).to(dt) for _ in range(2))
        gc.quant_pack_kv(k, v)
        q = torch.randn((1, 2 * gq, 128), device="cuda:0", generator=gen).to(dt)
        a, b = (torch.full((1, 2 * gq, 128), x, device="cuda:0", dtype=dt) for x in (3.0, 5.0))
        gc.decode_attn(q, 0.088, a)
        gc.decode_attn(q, 0.088, b, num_splits=B.bd_step_splits(gc.desc, gc.packed_len))
        torch.cuda.synchronize()
        assert torch.equal(a, b), (fmt, L)


@pytest.mark.parametrize("fmt", ["int4", "int2_kt", "int4_g32"])
def test_the_count_of_a_lazy_step_that_fills_the_residual(fmt):
    """It has a quantizing workgroup per KV head beside the attending ones and runs bd_choose_splits of them; the step
    after it, and the same step in the other order, bd_step_splits."""
    import torch
    L = 128 * 200 + 127
    gen = torch.Generator(device="cuda:0").manual_seed(7)
    k, v = (torch.randn((1, 8, L, 128), device="cuda:0", generator=gen).half() for _ in range(2))
    kn, vn = (torch.randn((2, 1, 8, 128), device="cuda:0", generator=gen).half() for _ in range(2))
    q = torch.randn((1, 32, 128), device="cuda:0", generator=gen).half()
    for lazy in (True, False):
        a, b = (B.KVCache(1, 32, 8, fmt, L + 1 + 128) for _ in range(2))
        for step in range(2):
            outs = [torch.full((1, 32, 128), x, device="cuda:0", dtype=torch.float16) for x in (3.0, 5.0)]
            if step == 0:
                a.quant_pack_kv(k, v)
                b.quant_pack_kv(k, v)
            counts = B.bd_choose_splits(b.desc, b.packed_len), B.bd_step_splits(b.desc, b.packed_len)
            assert counts[0] > counts[1] or "_g" in fmt
            a.decode_step(kn[step], vn[step], q, 0.088, outs[0], lazy=lazy)
            b.decode_step(kn[step], vn[step], q, 0.088, outs[1], lazy=lazy, num_splits=counts[0 if lazy and step == 0 else 1])
            torch.cuda.synchronize()
            assert a.res_len == step and torch.equal(*outs), (fmt, lazy, step, counts)
            assert all(np.array_equal(a.host_buffer(i), b.host_buffer(i)) for i in range(6))


def _caches_of(K, V, fmt, gq):
    """Oracle cache and GPU cache of one sequence, K and V [1, H, L, 128] fp16."""
    H, cap = K.shape[1], (K.shape[2] // 128 + 1) * 128
    oc = O.IntCache(1, H, BITS[fmt], cap, k_per_token="_kt" in fmt, group=GROUP.get(fmt, 128))
    oc.quant_pack_kv(K, V)
    gc = B.KVCache(1, gq * H, H, fmt, cap)
    gc.quant_pack_kv(to_dev(K, "fp16"), to_dev(V, "fp16"))
    return oc, gc


@pytest.mark.parametrize("fmt", ["int4", "int2", "int4_kt", "int2_kt"])
@pytest.mark.parametrize("factor", [30, 100, 1000])
def test_outlier_queries_keep_their_bits(fmt, factor):
    """Query groups of up to 4 heads, an outlier channel in q that is not K's: every Q' = q * scale then lies far below
    max|q| * max scale, and all of it still has to be there.  The bar: a score goes through about eight fp32 roundings
    (up to 2^-23 each where the matrix unit truncates) of at most M, the largest sum of magnitudes in log2 units,
    i.e. 8 * 2^-23 * M in the exponent, ln 2 times that in a weight and twice that in numerator and denominator
    together (12 * 2^-23 * M); and a weight is held to 2^-20 of itself."""
    scale = W.softmax_scale(W.CONFIGS["cfg1"])
    for gq in (1, 4):
        for seed in range(3):
            rng = np.random.default_rng(800 + seed)
            q = rng.standard_normal((1, 2 * gq, 128))
            K, V = (rng.standard_normal((1, 2, 4096, 128)) for _ in range(2))
            q[..., 7 + seed] *= factor
            K[..., 70 + seed] *= factor
            q[..., 70 + seed] /= factor   # (both at once would leave one token with all the weight)
            q, K, V = (x.astype(np.float16) for x in (q, K, V))
            oc, gc = _caches_of(K, V, fmt, gq)
            w = W.scaled(W.CONFIGS["cfg1"], batch=1, n_q_heads=2 * gq, n_kv_heads=2, context=4096, fmt=fmt)
            qa, ka = np.abs(q.astype(np.float64)).reshape(2, gq, 128), np.abs(K.astype(np.float64))[0]
            M = scale * 1.4427 * max((qa[h] @ ka[h].T).max() for h in range(2))
            bar = 12 * 2.0 ** -23 * M + 2.0 ** -20
            ma, rl = attn_errors(_attend_f32(gc, w, q, 1), O.decode_attn(oc, q, scale))
            assert rl <= bar, f"{fmt} gq={gq} seed {seed}: rel-L2 {rl:.2e} against {bar:.2e} (M {M:.3g})"


@pytest.mark.parametrize("fmt", ["int4", "int2", "int4_kt", "int2_kt"])
@pytest.mark.parametrize("gq", [1, 4])
@pytest.mark.parametrize("nb,ns", [(3, 1), (6, 1), (9, 1), (9, 2)])
def test_a_large_product_takes_no_bits_from_the_others(fmt, gq, nb, ns):
    """Query groups of up to 4 heads, Q' relative to its largest in the block.  K by channel: every third block has one token
    of 10^4 and more in a channel of zeros, where the query is negative: the token weighs nothing and the others' codes there
    are 0, but the channel's scale is the block's largest.  Per-token K: keys of one sign, so that the zero terms are 0, and a
    query of 6 * 10^4 where every key is 0.  The bar is that of test_outlier_queries_keep_their_bits, M that of the tokens
    that weigh something."""
    import torch
    kt, L = "_kt" in fmt, 128 * nb
    for big, factor in [(1e4, 30), (1e4, 1000), (6e4, 30), (6e4, 1000)][:1 if kt else 4]:
        rng = np.random.default_rng(nb + gq)
        q = rng.standard_normal((1, 2 * gq, 128))
        K, V = (rng.standard_normal((1, 2, L, 128)) for _ in range(2))
        K[..., 9] = 0
        scale = W.softmax_scale(W.CONFIGS["cfg1"])
        if kt:
            K, q, scale = np.abs(K), 0.02 * q, 50 * scale
            q[..., 9] = 6e4
        else:
            q[..., 9] = -factor
        ka = np.abs(K.astype(np.float16).astype(np.float64))[0]
        if not kt:
            K[:, :, 5::384, 9] = big
        q, K, V = (x.astype(np.float16) for x in (q, K, V))
        M = scale * 1.4427 * max((np.abs(q.astype(np.float64)).reshape(2, gq, 128)[h] @ ka[h].T).max() for h in range(2))
        bar = 12 * 2.0 ** -23 * M + 2.0 ** -20
        oc, gc = _caches_of(K, V, fmt, gq)
        gc.desc.out_type = B.BD_OUT_F32
        out = torch.full((1, 2 * gq, 128), 7.0, dtype=torch.float32, device="cuda:0")
        gc.decode_attn(to_dev(q, "fp16"), scale, out, num_splits=ns)
        torch.cuda.synchronize()
        ma, rl = attn_errors(out_to_f64(out), O.decode_attn(oc, q, scale))
        assert rl <= bar, f"{fmt} gq={gq} {nb} blocks, {big:g} x {factor}: rel-L2 {rl:.2e} against {bar:.2e} (M {M:.3g})"


@pytest.mark.parametrize("fmt", ["int4", "int2", "int4_kt", "int2_kt"])
@pytest.mark.parametrize("gq", [1, 4, 5])
@pytest.mark.parametrize("ns", [1, 2])
def test_infinities_show(fmt, gq, ns):
    """A packed key of plus or minus infinity (its scale is a NaN then) gives every head of its KV head a row of zeros, as a
    sum of weights that is no number does, an infinite query that head's; whatever arithmetic the size of the group takes, and
    no other row is touched."""
    import torch
    rng = np.random.default_rng(gq)
    K, V = (rng.standard_normal((1, 3, 640, 128)).astype(np.float16) for _ in range(2))
    q = rng.standard_normal((1, 3 * gq, 128)).astype(np.float16)
    q[:, :, 9] = np.arange(3 * gq) % 2   # (0: the channel's product is 0 x its scale)
    scale = W.softmax_scale(W.CONFIGS["cfg1"])
    ref = O.decode_attn(_caches_of(K, V, fmt, gq)[0], q, scale)
    K[0, 0, 133, 9], K[0, 1, 7, 9] = np.inf, -np.inf
    q[0, 2 * gq, 50] = -np.inf
    gc = B.KVCache(1, 3 * gq, 3, fmt, 768)
    gc.quant_pack_kv(to_dev(K, "fp16"), to_dev(V, "fp16"))
    gc.desc.out_type = B.BD_OUT_F32
    out = torch.full((1, 3 * gq, 128), 7.0, dtype=torch.float32, device="cuda:0")
    gc.decode_attn(to_dev(q, "fp16"), scale, out, num_splits=ns)
    torch.cuda.synchronize()
    got = out_to_f64(out)
    assert np.all(got[0, :2 * gq + 1] == 0.0)
    if gq > 1:
        assert attn_errors(got[0, 2 * gq + 1:], ref[0, 2 * gq + 1:])[1] <= (1e-5 if gq <= 4 else 1e-3)


@pytest.mark.parametrize("fmt", ["int4", "int2", "int4_kt", "int2_kt"])
@pytest.mark.parametrize("x", [8, 13, 18, 23.5])
def test_a_long_tail_behind_one_dominating_token_is_kept(fmt, x):
    """6144 tokens that weigh about 2^-x of one other, their values alike: what rounding takes from each weight adds up.
    Up to 4 heads per KV head hold 19 bits of a weight, or 2^-25 of the largest where that is more: at most
    2^-20 + 6144 * 2^-26 * 2^-x' of the result, x' = 0 where the step is the limit (no more than the tail itself, 6144 *
    2^-x); and the scores' fp32 roundings (about eight, 2^-23 of up to x + 1 in log2 units, as above)."""
    scale = W.softmax_scale(W.CONFIGS["cfg1"])
    rng = np.random.default_rng(900)
    L, gq = 6144, 4
    d = rng.standard_normal(128)
    d /= np.linalg.norm(d)
    q = np.broadcast_to(16 * d, (1, 2 * gq, 128)).astype(np.float16)
    K = 0.02 * rng.standard_normal((1, 2, L, 128))
    K[:, :, 0] += d * (x * np.log(2) / (16 * scale))
    V = 0.3 * rng.standard_normal((1, 2, L, 128)) + np.where(np.arange(128) % 2, 1.5, -1.5)
    V[:, :, 0] = rng.standard_normal((2, 128))
    oc, gc = _caches_of(K.astype(np.float16), V.astype(np.float16), fmt, gq)
    w = W.scaled(W.CONFIGS["cfg1"], batch=1, n_q_heads=2 * gq, n_kv_heads=2, context=L, fmt=fmt)
    ma, rl = attn_errors(_attend_f32(gc, w, q, 1), O.decode_attn(oc, q, scale))
    bar = 12 * 2.0 ** -23 * (x + 1) + 2.0 ** -20 + min(L * 2.0 ** -26, 2.0 ** -3 * L * 2.0 ** -x)
    assert rl <= bar, f"{fmt} 2^-{x}: rel-L2 {rl:.2e} against {bar:.2e}"


@pytest.mark.parametrize("fmt,gq", [("int4", 4), ("int2", 16), ("int4_g32", 8)])
@pytest.mark.parametrize("L", [2, 33, 127])
def test_residual_weights_enter_the_product_whole(fmt, gq, L):
    """Token t's value row is one in channel t only, so the unnormalised output row holds the weights as the product
    takes them: all 24 bits of the fp32 exp2(s_t - m), for scores that fp32 gives exactly (one channel in q)."""
    import torch
    rng = np.random.default_rng(L)
    q = np.zeros((1, 2 * gq, 128), np.float16)
    q[..., 5] = 1.0
    K, V = np.zeros((1, 2, L, 128), np.float16), np.zeros((1, 2, L, 128), np.float16)
    K[..., 5] = rng.uniform(-40, 40, (1, 2, L)).astype(np.float16)
    K[:, :, 0, 5] = 41   # (the largest in the first round: no running maximum is raised, which would round what is summed)
    V[:, :, np.arange(L), np.arange(L)] = 1.0
    _, gc = _caches_of(K, V, fmt, gq)
    ws = gc.workspace(1)
    scale = np.float32(0.088)
    B.bd_decode_attn(gc.desc, to_dev(q, "fp16"), 0, L, float(scale), 1, ws, None)
    torch.cuda.synchronize()
    rows = ws[:2 * gq * 128 * 4].view(torch.float32).view(2, gq, 128)
    s = torch.from_numpy(K[0, :, :, 5].astype(np.float32) * (scale * np.float32(1.4426950408889634))).cuda()
    p = torch.exp2(s - s.amax(-1, keepdim=True))
    whole = p > 2.0 ** -13
    assert whole.sum() > 2
    for h in range(2):
        for i in range(gq):
            got = rows[h, i, :L]
            assert torch.equal(got[whole[h]], p[h][whole[h]]), (fmt, gq, L, (got - p[h]).abs().max().item())
            assert (got - p[h]).abs().max() <= 2.0 ** -38


@pytest.mark.parametrize("fmt", ["int4", "int2_kt", "int4_g32", "mxfp4"])
@pytest.mark.parametrize("hq,asked", [(8, 16), (16, 7)])
def test_a_paged_batch_runs_the_splits_asked_for(fmt, hq, asked):
    """One long sequence among 49 short ones (100 (sequence, KV head) units: asked * units is more than two rounds of
    workgroups): the long one's partials are all there, each over its share of the blocks, and the rows are those of
    the long sequence alone, bit for bit."""
    import torch
    mx = fmt == "mxfp4"
    dt = torch.bfloat16 if mx else torch.float16
    L, batch, H = 128 * 4 * asked + 77, 50, 2
    maxp = L // 128 + 1
    lens = [L] + [1 + 5 * i for i in range(1, batch)]
    table = torch.full((batch, maxp), -1, dtype=torch.int32)
    table[:, 0] = torch.arange(batch)
    table[:, 1] = torch.arange(batch, 2 * batch)
    table[0] = torch.arange(2 * batch, 2 * batch + maxp)
    pc = B.PagedKVCache(batch, hq, H, fmt, 2 * batch + maxp, table)
    one = B.PagedKVCache(1, hq, H, fmt, maxp, torch.arange(maxp, dtype=torch.int32).view(1, maxp))
    gen = torch.Generator(device="cuda:0").manual_seed(asked)
    for s, n in enumerate(lens):
        k, v = (torch.randn((H, n, 128), device="cuda:0", generator=gen).to(dt) for _ in range(2))
        pc.quant_pack_kv(s, k, v)
        if s == 0:
            one.quant_pack_kv(0, k, v)
    q = torch.randn((batch, hq, 128), device="cuda:0", generator=gen).to(dt)
    out, ref = torch.zeros((batch, hq, 128), dtype=dt, device="cuda:0"), torch.zeros((1, hq, 128), dtype=dt, device="cuda:0")
    ws, ws1 = pc.workspace(asked), one.workspace(asked)
    ws.fill_(0xFF)
    pc.decode_attn(q, 0.088, out, num_splits=asked)
    one.decode_attn(q[:1].contiguous(), 0.088, ref, num_splits=asked)
    torch.cuda.synchronize()
    rows, ml = _partials(ws, asked, batch, hq)
    rows1, ml1 = _partials(ws1, asked, 1, hq)
    assert (ml[:, 0, :, 1] > 0).all()
    assert torch.equal(ml[:, :1], ml1) and torch.equal(rows[:, :1], rows1) and torch.equal(out[:1], ref)
    assert pc.status.item() == 0


@pytest.mark.parametrize("fmt,gq", [("int4", 4), ("int2_kt", 8), ("int4", 16), ("int4_g32", 8)])
@pytest.mark.parametrize("r", [29, 30, 31, 32, 48, 63, 64, 95, 96, 126])
def test_a_step_with_a_residual_slice_of_one_round_or_more(fmt, gq, r):
    """r residual tokens and the step's own, in one, two and three slices: on either side of the 32 tokens that one round
    takes, of the 16 of a tile and of the 32 of a wave, the new token first or last of one, beside one block per wave
    and beside two, contiguous and in pages.  fp32 rows, so the bar is that of the blocks' weights: 1e-5 where they are held
    whole (up to 4 heads), else half an fp16 step, 2^-12."""
    bar = 1e-5 if gq <= 4 else 2.0 ** -12
    import torch
    H, hq = 2, 2 * gq
    for nb in (3, 7):
        L = 128 * nb + r
        w = W.scaled(W.CONFIGS["cfg1"], batch=1, n_q_heads=hq, n_kv_heads=H, context=L, fmt=fmt)
        K, V = W.make_kv(w)
        kn, vn = W.make_new_kv(w, 0)
        q = W.make_q(w)
        oc, _ = _caches_of(K, V, fmt, gq)
        oc.append_kv(kn, vn)
        ref = O.decode_attn(oc, q, W.softmax_scale(w))
        k, v, kd, vd, qd = (to_dev(x, "fp16") for x in (K, V, kn, vn, q))
        for ns in (1, 2, 3):
            _, gc = _caches_of(K, V, fmt, gq)
            pc = B.PagedKVCache(1, hq, H, fmt, nb + 2, torch.arange(nb + 1, -1, -1, dtype=torch.int32)[None])
            pc.quant_pack_kv(0, k[0], v[0])
            rows = []
            for c in (gc, pc):
                c.desc.out_type = B.BD_OUT_F32
                out = torch.full((1, hq, 128), 7.0, dtype=torch.float32, device="cuda:0")
                c.decode_step(kd, vd, qd, W.softmax_scale(w), out, ns)
                rows.append(out_to_f64(out))
            torch.cuda.synchronize()
            for got in rows:
                ma, rl = attn_errors(got, ref)
                assert rl <= bar, f"{fmt} {L} tokens, {ns} splits: rel-L2 {rl:.2e}"
            assert np.array_equal(gc.host_buffer(4), pc.host_buffer(4)) and np.array_equal(gc.host_buffer(5), pc.host_buffer(5))


@pytest.mark.parametrize("fmt,gq", [("int4", 4), ("int2", 8), ("int2_kt", 3), ("int4_kt", 8), ("int4", 16)])
@pytest.mark.parametrize("r,lazy", [(29, False), (30, False), (31, False), (33, False), (63, False), (64, False), (95, False),
                                    (96, False), (126, False), (127, True)])
def test_long_residual_slices_of_many_workgroups(fmt, gq, r, lazy):
    """257 and more workgroups of one block a wave: a residual slice of more than 32 tokens is attended ahead of the block.
    Steps with 1 to 4 blocks (and none) a unit, in one split and in two, against a batch of one, whose workgroups are few:
    residual and packed block bit for bit; the fp32 rows come from another form of the kernel, whose sums and products are
    fused as its compilation has it, so that a score differs by an fp32 step or two of its size (scores up to 2^6 in log2
    units: 2^-17 in a weight, 1e-5), and where weights are rounded to fp16 (5 and more heads) some round the other way: not
    more than 2^-11 of each, half of that in the row."""
    import torch
    bar = 1e-5 if gq <= 4 else 2.0 ** -12
    H, hq, batch = 2, 2 * gq, 129
    gen = torch.Generator(device="cuda:0").manual_seed(r)
    rows = lambda *shape: torch.randn(shape, device="cuda:0", generator=gen).to(torch.float16)
    for nb, ns in ((0, 1), (1, 1), (3, 1), (4, 1), (5, 2), (8, 2)):
        L = 128 * nb + r
        k, v, kn, vn, q = rows(batch, H, L, 128), rows(batch, H, L, 128), rows(batch, H, 128), rows(batch, H, 128), rows(batch, hq, 128)

        def step(s):
            c = B.KVCache(k[s].shape[0], hq, H, fmt, 128 * (nb + 1))
            c.desc.out_type = B.BD_OUT_F32
            out = torch.full((k[s].shape[0], hq, 128), 7.0, dtype=torch.float32, device="cuda:0")
            c.quant_pack_kv(k[s].contiguous(), v[s].contiguous())
            c.decode_step(kn[s].contiguous(), vn[s].contiguous(), q[s].contiguous(), 0.088, out, ns, lazy=lazy)
            return c, out

        many, got = step(slice(0, batch))
        for s in (0, 1, 63, 127, 128):
            one, ref = step(slice(s, s + 1))
            torch.cuda.synchronize()
            off = ((got[s] - ref[0]).double().norm() / ref[0].double().norm()).item()
            assert off <= bar, f"{fmt} gq {gq}, {L} tokens, {ns} splits: sequence {s}: {off:.2e}"
            for i in range(6):
                n = one.sizes[i]
                assert torch.equal(many.buffers[i][s * n:(s + 1) * n], one.buffers[i][:n]), (s, i)
        assert (many.packed_len, many.res_len) == (one.packed_len, one.res_len)


@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("fmt", ["int4", "int2_kt_g32", "mxfp4"])
def test_the_step_wrappers_are_the_caches_step(fmt, lazy):
    """bd_decode_step / bd_decode_step_lazy of the binding, which KVCache.decode_step does not go through: the lengths they
    return, the row and the cache bit for bit those of the method, over the step that fills the residual; the same error."""
    import torch
    dt = torch.bfloat16 if fmt == "mxfp4" else torch.float16
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    rows = lambda *shape: torch.randn(shape, device="cuda:0", generator=gen).to(dt)
    a, b = (B.KVCache(2, 8, 2, fmt, 512) for _ in range(2))
    k, v = rows(2, 2, 382, 128), rows(2, 2, 382, 128)
    for c in (a, b):
        c.quant_pack_kv(k, v)
    wrapper = B.bd_decode_step_lazy if lazy else B.bd_decode_step
    for ns in (1, 3, 2):
        kn, vn, q = rows(2, 2, 128), rows(2, 2, 128), rows(2, 8, 128)
        got, ref = (torch.full((2, 8, 128), x, dtype=dt, device="cuda:0") for x in (7.0, 9.0))
        a.decode_step(kn, vn, q, 0.088, ref, ns, lazy=lazy)
        b.packed_len, b.res_len = wrapper(b.desc, kn, vn, q, b.packed_len, b.res_len, 0.088, ns, b.workspace(ns), got)
        torch.cuda.synchronize()
        assert torch.equal(got, ref) and (a.packed_len, a.res_len) == (b.packed_len, b.res_len)
        assert all(torch.equal(x, y) for x, y in zip(a.buffers, b.buffers))
    for call in (lambda: a.decode_step(kn, vn, None, 0.088, ref, 1, lazy=lazy),
                 lambda: wrapper(b.desc, kn, vn, None, b.packed_len, b.res_len, 0.088, 1, b.workspace(1), got)):
        with pytest.raises(B.BitDecodeError, match=wrapper.__name__ + ": invalid argument"):
            call()


@pytest.mark.parametrize("fmt,hq,batch,lazy", [
    ("int4", 2, 1, False), ("int4", 8, 5, True), ("int2_kt", 16, 40, False), ("int4", 34, 17, True), ("int4_g32", 8, 16, True),
    ("int2_g64", 34, 33, False), ("mxfp4", 8, 70, False), ("mxfp4", 16, 150, False), ("mxfp4", 40, 15, False)])
def test_a_step_in_one_split_raises_the_lengths_in_any_workspace(fmt, hq, batch, lazy):
    """Paged steps in one split, whose launch counts its workgroups in the workspace (2 KV heads; 1 to 16 counters, 300
    workgroups and more that are dealt by length among them): in a workspace of random bytes, of zeros, of another call's
    partials, as the step before left it, and replayed from a graph, every step raises every length by one, but not that of a
    sequence without a page for its token and of a negative one, and attends as append and attention do."""
    import torch
    mx, H, P = fmt == "mxfp4", 2, 4
    dt = torch.bfloat16 if mx else torch.float16
    rng = np.random.default_rng(batch + hq)
    lens = rng.integers(1, 380, batch)
    lens[-1] = 127
    table = torch.as_tensor(rng.permutation(batch * P).reshape(batch, P).astype(np.int32))
    gen = torch.Generator(device="cuda:0").manual_seed(batch)
    rows = lambda *shape: torch.randn(shape, device="cuda:0", generator=gen).to(dt)
    kv = [(rows(H, int(n), 128), rows(H, int(n), 128)) for n in lens]
    a, twin = (B.PagedKVCache(batch, hq, H, fmt, batch * P, table) for _ in range(2))
    for c in (a, twin):
        for s, (k, v) in enumerate(kv):
            c.quant_pack_kv(s, k, v)
        if batch > 2:
            c.seq_lens[1] = -3
            if mx:
                c.seq_lens[0] = 128 * P   # no page for the next token
    want = np.array([int(n) for n in a.seq_lens.tolist()])
    still = (want < 0) | (want == 128 * P)
    kn, vn, q = rows(batch, H, 128), rows(batch, H, 128), rows(batch, hq, 128)
    out, ref = (torch.full((batch, hq, 128), x, dtype=dt, device="cuda:0") for x in (7.0, 9.0))
    ws = a.workspace(4)

    def step():
        a.decode_step(kn, vn, q, 0.088, out, 1, lazy=lazy)

    graph = None
    for i in range(8):
        if i == 0:
            ws.copy_(torch.randint(0, 256, ws.shape, device="cuda:0", generator=gen, dtype=torch.uint8))
        elif i == 1:
            ws.zero_()
        elif i == 3:
            a.decode_attn(q, 0.088, out, 4)   # its partials
        elif i == 5:
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                step()
        if graph is not None:
            graph.replay()
        else:
            step()
        twin.append_kv(kn, vn)
        twin.decode_attn(q, 0.088, ref, 1)
        torch.cuda.synchronize()
        want += ~still
        assert a.seq_lens.tolist() == want.tolist() == twin.seq_lens.tolist(), i
        full = torch.as_tensor(lazy & (want % 128 == 0) & ~still, device="cuda:0")   # (a lazy step attends those in fp16)
        assert torch.equal(out[~full], ref[~full]), i
    for i in range(4 if mx else 6):
        assert torch.equal(a.buffers[i], twin.buffers[i]), i


@pytest.mark.parametrize("fmt,hq,batch", [("int4", 8, 3), ("int2_kt", 16, 40), ("int4", 34, 17), ("int4_g32", 8, 16), ("mxfp4", 8, 70), ("mxfp4", 40, 5)])
@pytest.mark.parametrize("lazy", [False, True])
def test_a_step_in_one_split_leaves_the_workspace_alone(fmt, hq, batch, lazy):
    """The library's paged steps (the cache class counts in memory of its own): caches whose steps overlap may share a workspace
    while they run one split.  Step by step the rows, the lengths and the cache of the class's steps, whose counters are zeros
    after each."""
    import torch
    mx, H, P = fmt == "mxfp4", 2, 2
    dt = torch.bfloat16 if mx else torch.float16
    rng = np.random.default_rng(batch)
    lens = rng.integers(1, 250, batch)
    lens[-1] = 126
    table = torch.as_tensor(rng.permutation(batch * P).reshape(batch, P).astype(np.int32))
    gen = torch.Generator(device="cuda:0").manual_seed(batch)
    rows = lambda *shape: torch.randn(shape, device="cuda:0", generator=gen).to(dt)
    a, twin = (B.PagedKVCache(batch, hq, H, fmt, batch * P, table) for _ in range(2))
    for s in range(batch):
        k, v = rows(H, int(lens[s]), 128), rows(H, int(lens[s]), 128)
        a.quant_pack_kv(s, k, v)
        twin.quant_pack_kv(s, k, v)
    out, ref = (torch.full((batch, hq, 128), x, dtype=dt, device="cuda:0") for x in (7.0, 9.0))
    ws = torch.randint(0, 256, (B.bd_paged_workspace_bytes(a.desc, 1),), device="cuda:0", generator=gen, dtype=torch.uint8)
    before = ws.clone()
    for i in range(3):
        kn, vn, q = rows(batch, H, 128), rows(batch, H, 128), rows(batch, hq, 128)
        (B.bd_paged_decode_step_lazy if lazy else B.bd_paged_decode_step)(a.desc, kn, vn, q, 0.088, 1, ws, out)
        twin.decode_step(kn, vn, q, 0.088, ref, 1, lazy=lazy)
        torch.cuda.synchronize()
        assert torch.equal(ws, before), i
        assert a.seq_lens.tolist() == twin.seq_lens.tolist() == [int(n) + i + 1 for n in lens]
        assert torch.equal(out, ref) and not twin.counters.any()
    for i in range(4 if mx else 6):
        assert torch.equal(a.buffers[i], twin.buffers[i]), i


@pytest.mark.parametrize("fmt,gq", [("int4", 1), ("int4", 4), ("int2", 3), ("int4_kt", 4)])
@pytest.mark.parametrize("nb,ns", [(4, 1), (5, 1), (8, 1), (9, 1), (9, 2), (16, 2), (33, 8), (64, 8)])
def test_workgroups_of_eight_waves(fmt, gq, nb, ns):
    """On either side of one block and two for each of a workgroup's four waves (where eight take one each), with no residual,
    slices of one token, of one round and more, and the step that packs a block.  fp32 rows against the oracle; 1e-5, as weights
    are held whole."""
    import torch
    H, hq = 2, 2 * gq
    for r in (0, 40 * ns, 127):
        if r > 127:
            continue
        w = W.scaled(W.CONFIGS["cfg1"], batch=1, n_q_heads=hq, n_kv_heads=H, context=128 * nb + r, fmt=fmt, seed=nb)
        K, V = W.make_kv(w)
        kn, vn = W.make_new_kv(w, 0)
        q = W.make_q(w)
        oc, gc = _caches_of(K, V, fmt, gq)
        oc.append_kv(kn, vn)
        ref = O.decode_attn(oc, q, W.softmax_scale(w))
        gc.desc.out_type = B.BD_OUT_F32
        out = torch.full((1, hq, 128), 7.0, dtype=torch.float32, device="cuda:0")
        gc.decode_step(*(to_dev(x, "fp16") for x in (kn, vn, q)), W.softmax_scale(w), out, ns)
        torch.cuda.synchronize()
        _, rl = attn_errors(out_to_f64(out), ref)
        assert rl <= 1e-5, f"{fmt} {nb} blocks and {r} tokens, {ns} splits: rel-L2 {rl:.2e}"


@pytest.mark.parametrize("fmt", ["int4", "int2"])
@pytest.mark.parametrize("gq,nb,ns", [(1, 5, 1), (4, 8, 1), (3, 11, 2), (4, 12, 2)])
def test_lazy_steps_in_workgroups_of_eight_waves(fmt, gq, nb, ns):
    """The lazy step that fills the residual, its packing workgroup of eight waves too: the oracle's lazy mode, and the cache
    that the eager step leaves, whose attending workgroup packs."""
    import torch
    from tests.test_gpu_parity import _assert_int_cache_equal
    w = W.scaled(W.CONFIGS["cfg1"], batch=1, n_q_heads=2 * gq, n_kv_heads=2, context=128 * nb + 126, fmt=fmt, seed=nb)
    K, V, oc, lazy = _int_cache_pair(w, 128 * (nb + 2))
    eager = B.KVCache(1, 2 * gq, 2, fmt, 128 * (nb + 2))
    eager.quant_pack_kv(to_dev(K, "fp16"), to_dev(V, "fp16"))
    for c in (lazy, eager):
        c.desc.out_type = B.BD_OUT_F32
    for step in range(3):
        kn, vn, q = *W.make_new_kv(w, step), W.make_q(w, step)
        outs = [torch.full((1, 2 * gq, 128), x, dtype=torch.float32, device="cuda:0") for x in (7.0, 5.0)]
        for c, out in zip((lazy, eager), outs):
            c.decode_step(*(to_dev(x, "fp16") for x in (kn, vn, q)), W.softmax_scale(w), out, ns, lazy=c is lazy)
        torch.cuda.synchronize()
        oc.append_kv(kn, vn, flush=False)
        ref = O.decode_attn(oc, q, W.softmax_scale(w))
        fills = oc.res_len == 128
        oc.flush_if_full()
        assert attn_errors(out_to_f64(outs[0]), ref)[1] <= 1e-5
        assert fills or torch.equal(*outs)
        assert lazy.packed_len == eager.packed_len == oc.packed_len
        assert all(np.array_equal(lazy.host_buffer(i), eager.host_buffer(i)) for i in range(6))
        _assert_int_cache_equal(oc, lazy)
