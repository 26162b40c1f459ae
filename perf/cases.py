"""The work that programs give this framework, as cases that can be timed and compared.

A case is one of four things a serving program does with the packed KV cache:

  step           one decode step: every layer's KVCache.decode_step (append the new token, attend, and
                 pack the residual block on the step that fills it), one call per layer
  paged_step     the same over PagedKVCache, a batch of sequences of different lengths; the program owns
                 the lengths and writes them before the step, once for all layers
  prefill        KVCache.quant_pack_kv of a prompt (all sequences of the batch at once)
  paged_prefill  PagedKVCache.quant_pack_kv, one call per sequence of a ragged batch

"context" is the number of tokens resident before a step, or the prompt's length; of a ragged batch it
is the longest sequence's.  "layers" is how many layers' caches (independent buffers) one pass goes
through.  Head dimension is 128 throughout.  Inputs are standard normal, in one percent of the
(KV head, channel) pairs ten times that (the integer formats' workloads), rounded to the format's type.
"""
import math

import torch

from paper_2503_18773_amd import binding as B

D = BLOCK = 128
DEVICE = "cuda:0"
FORMATS = ["int4", "int2", "mxfp4", "int4_kt", "int2_kt", "int4_g64", "int4_g32", "int2_g64", "int2_g32",
           "int4_kt_g64", "int4_kt_g32", "int2_kt_g64", "int2_kt_g32"]


def _case(name, kind, fmt, batch, q_heads, kv_heads, context, layers=1, lazy=False, out="half"):
    return {"name": name, "kind": kind, "fmt": fmt, "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads,
            "context": context, "layers": layers, "lazy": lazy, "out": out}


def listed():
    return [
        # a short chat, no grouped heads: sixteen layers of a few hundred kilobytes each, all latency
        _case("step_1k", "step", "int4", 1, 8, 8, 1024, layers=16),
        # a chat of ordinary length on the LLaMA-3.1-8B shape
        _case("step_6k", "step", "int4", 1, 32, 8, 6001, layers=8),
        # one user at 32K and at 128K tokens: the benchmark's two headline lengths
        _case("step_32k", "step", "int4", 1, 32, 8, 32768 + 20, layers=8),
        _case("step_128k", "step", "int4", 1, 32, 8, 131072 + 64, layers=4),
        # 2-bit codes, eight users at 32K
        _case("step_int2_8x32k", "step", "int2", 8, 32, 8, 32768, layers=2),
        # MXFP4, sixteen users at 16K
        _case("step_mxfp4_16x16k", "step", "mxfp4", 16, 32, 8, 16384, layers=3),
        # finer quantization groups, four users; the paper's flush order, on the step that fills the residual
        _case("step_g32_4x8k_fills", "step", "int4_g32", 4, 32, 8, 8192 + 127, layers=4, lazy=True),
        # serving: a ragged batch in pages
        _case("paged_24x5k", "paged_step", "int4", 24, 32, 8, 5000, layers=4),
        # the same with 8 query heads per KV head, keys quantized per token, 2-bit codes, wide enough for one split
        _case("paged_kt_gq8_40x3k", "paged_step", "int2_kt", 40, 64, 8, 3100, layers=4),
        # prompts: one long one, a batch of short ones of odd length in MXFP4, a ragged batch into pages
        _case("prefill_128k", "prefill", "int4", 1, 32, 8, 131072),
        _case("prefill_mxfp4_4x2k", "prefill", "mxfp4", 4, 32, 8, 2079),
        _case("prefill_paged_8x1k", "paged_prefill", "int4", 8, 32, 8, 1333),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["paged_step"] * 2 + ["prefill"] * 2 + ["paged_prefill"])
    fmt = rng.choice(["int4"] * 5 + ["int2"] * 4 + ["mxfp4"] * 4 + FORMATS[3:])
    kv_heads = rng.choice([1, 2, 4, 8, 8, 8])
    q_heads = kv_heads * rng.choice([1, 3, 4, 4, 4, 5, 8, 8, 16])
    # tokens times (sequence, KV head) units of one pass: up to the largest listed of the kind
    most = {"step": 1 << 21, "paged_step": 1 << 20, "prefill": 1 << 20, "paged_prefill": 1 << 17}[kind]
    context = _log(rng, 16, {"step": 131072, "paged_step": 16384, "prefill": 131072, "paged_prefill": 4096}[kind])
    batch = min(_log(rng, 1, 64 if kind != "paged_prefill" else 16), max(1, most // (context * kv_heads)))
    if kind in ("step", "paged_step"):
        layers = max(1, min(8, 2 * most // (batch * kv_heads * context)))
        lazy = rng.random() < 0.3
        if kind == "step" and rng.random() < 0.15:   # the step that fills the residual block
            context = context // BLOCK * BLOCK + BLOCK - 1
    else:
        layers, lazy = 1, False
    c = _case("", kind, fmt, batch, q_heads, kv_heads, context, layers, lazy, rng.choice(["half", "half", "f32"]))
    del c["name"]
    return c


# ---- sizes -------------------------------------------------------------------------------------------

def _is_mx(case):
    return case["fmt"] == "mxfp4"


def _bits(case):
    return 2 if case["fmt"].startswith("int2") else 4


def _group(case):
    return 64 if case["fmt"].endswith("_g64") else 32 if case["fmt"].endswith("_g32") else BLOCK


def _per_token(case):
    return "_kt" in case["fmt"]


def _lengths(case):
    """Tokens of every sequence: equal, or, paged, from a third of the longest up to it.  The second sequence
    of a long enough ragged batch is one token short of a whole block: the step fills its residual."""
    n, L = case["batch"], case["context"]
    if not case["kind"].startswith("paged"):
        return [L] * n
    lens = [max(1, int(L * (1 - (2 / 3) * ((0.618034 * i) % 1)))) for i in range(n)]
    if n > 1 and lens[1] >= BLOCK:
        lens[1] = lens[1] // BLOCK * BLOCK - 1
    return lens


def _packed_bytes(case, tokens):
    """Codes and parameters of K and V of `tokens` packed tokens of one KV head."""
    return tokens * (2 * 64 + 2 * 4) if _is_mx(case) else tokens * 2 * (D * _bits(case) // 8 + 4 * (BLOCK // _group(case)))


def work(case):
    """Prefill: the source rows read, the packed rows and the residual written.  Step: the packed rows and the
    residual tokens read (and, on a filling step, a block written), the new token and the query read, the new
    token and the output written; two products of 2 * 128 flops per token and query head."""
    H, Hq = case["kv_heads"], case["q_heads"]
    nbytes = flops = 0
    for L in _lengths(case):
        if case["kind"] in ("prefill", "paged_prefill"):
            packed = L if _is_mx(case) else L // BLOCK * BLOCK
            nbytes += H * (L * 2 * D * 2 + _packed_bytes(case, packed) + (L - packed) * 2 * D * 2)
            flops += H * L * 2 * D * 3   # subtract, divide, round
        else:
            L += 1
            packed = L if _is_mx(case) else L // BLOCK * BLOCK
            nbytes += H * (_packed_bytes(case, packed) + (L - packed) * 2 * D * 2 + 2 * 2 * D * 2)
            nbytes += Hq * D * (2 + (4 if case["out"] == "f32" else 2))
            flops += Hq * L * 4 * D
    return {"bytes": case["layers"] * nbytes, "flops": case["layers"] * flops}


def tolerance(case):
    """Packed bytes are exact.  Attention, four times what was measured against 64 bits: fp16 outputs are 1.8e-4 to
    2.7e-4 off (their rounding alone is 2.1e-4), bf16 ones 1.7e-3; fp32 ones show the rounding of the
    probabilities to fp16, 0.7e-4 to 0.8e-4 (MXFP4, whose values are coarser: 1.9e-4)."""
    if case["kind"] in ("prefill", "paged_prefill"):
        return "exact"
    if _is_mx(case):
        return {"rel": 8e-4 if case["out"] == "f32" else 7e-3}
    return {"rel": 3.2e-4 if case["out"] == "f32" else 1.1e-3}


# ---- inputs ------------------------------------------------------------------------------------------

def _dtype(case):
    return torch.bfloat16 if _is_mx(case) else torch.float16


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _outliers(case, gen):
    """[H, 1, D] factors: 10 in one percent of the (KV head, channel) pairs."""
    n = case["kv_heads"] * D
    f = torch.ones(n, device=DEVICE)
    if not _is_mx(case):
        f[torch.randperm(n, device=DEVICE, generator=gen)[:round(0.01 * n)]] = 10.0
    return f.view(case["kv_heads"], 1, D)


def _draw_layer(case, seed, layer):
    """One layer's (prompt k, v per sequence, new token k, v, query)."""
    gen = _generator(1000003 * seed + layer)
    fk, fv = _outliers(case, gen), _outliers(case, gen)
    H, dt = case["kv_heads"], _dtype(case)

    def rows(shape, f):
        return (torch.randn(shape, device=DEVICE, generator=gen) * f).to(dt)

    lens = _lengths(case)
    if case["kind"].startswith("paged"):
        k = [rows((H, L, D), fk) for L in lens]
        v = [rows((H, L, D), fv) for L in lens]
    else:
        k = rows((len(lens), H, lens[0], D), fk)
        v = rows((len(lens), H, lens[0], D), fv)
    kn, vn = (rows((len(lens), H, 1, D), f).squeeze(2) for f in (fk, fv))
    q = torch.randn((len(lens), case["q_heads"], D), device=DEVICE, generator=gen).to(dt)
    return k, v, kn, vn, q


def _new_cache(case, seed):
    lens = _lengths(case)
    shape = (case["batch"], case["q_heads"], case["kv_heads"], case["fmt"])
    need = (max(lens) + 1 + BLOCK - 1) // BLOCK
    if case["kind"].startswith("paged"):
        gen = torch.Generator().manual_seed(seed)
        pages = torch.randperm(need * len(lens), generator=gen).to(torch.int32)   # scattered over the pool
        cache = B.PagedKVCache(*shape, num_pages=need * len(lens), block_table=pages.view(len(lens), need), device=DEVICE)
    else:
        cache = B.KVCache(*shape, capacity=need * BLOCK, device=DEVICE)
    cache.desc.out_type = B.BD_OUT_F32 if case["out"] == "f32" else B.BD_OUT_HALF
    return cache


def prepare(case, seed):
    torch.cuda.set_device(0)
    state = {"case": case, "layers": []}
    if case["kind"] in ("prefill", "paged_prefill"):
        k, v, _, _, _ = _draw_layer(case, seed, 0)
        state["cache"], state["k"], state["v"] = _new_cache(case, seed), k, v
        return state
    lens = _lengths(case)
    out_dtype = torch.float32 if case["out"] == "f32" else _dtype(case)
    state["out"] = torch.zeros((case["layers"], case["batch"], case["q_heads"], D), dtype=out_dtype, device=DEVICE)
    if case["kind"] == "paged_step":
        state["lens"] = torch.tensor(lens, dtype=torch.int32, device=DEVICE).repeat(case["layers"], 1)
        state["all_lens"] = torch.zeros_like(state["lens"])
    for i in range(case["layers"]):
        cache = _new_cache(case, seed + i)
        k, v, kn, vn, q = _draw_layer(case, seed, i)
        if case["kind"] == "paged_step":
            cache.seq_lens = state["all_lens"][i]   # all layers' lengths are one tensor of the program's
            cache.desc.seq_lens = cache.seq_lens.data_ptr()
            for s in range(len(lens)):
                cache.quant_pack_kv(s, k[s], v[s])
            # as the interface advises: from a contiguous cache of the same shape and the longest sequence
            shape = B.bd_cache(case["batch"], case["q_heads"], case["kv_heads"], D, B.FORMATS[case["fmt"]],
                               (max(lens) + BLOCK) // BLOCK * BLOCK)
            state["splits"] = B.bd_choose_splits(shape, max(lens) + 1)
        else:
            cache.quant_pack_kv(k, v)
        state["layers"].append((cache, kn, vn, q, getattr(cache, "packed_len", 0), getattr(cache, "res_len", 0)))
    state["written"] = [_written(case, layer[0], lens) for layer in state["layers"][:4]]
    return state


# ---- one pass ----------------------------------------------------------------------------------------

SCALE = 1.0 / math.sqrt(D)


def _written(case, cache, lens):
    """The cache bytes a step writes: the residual rows; the block that the new token completes (integer
    formats, filling step) or goes to (MXFP4).  Views of the cache's own buffers."""
    H, n = case["kv_heads"], case["batch"]
    views = []
    if not _is_mx(case):
        views += [cache.buffers[i].view(torch.int16) for i in (4, 5)]
    paged = case["kind"] == "paged_step"
    table = cache.block_table.cpu() if paged else None
    for s in (range(min(n, 2)) if paged else [0]):
        blk = lens[s] // BLOCK
        if not _is_mx(case) and (lens[s] + 1) % BLOCK:
            continue
        for i in range(4):
            if paged:
                pool = cache.buffers[i][:cache.sizes[i]].view(cache.desc.num_pages, -1)
                views.append(pool[int(table[s, blk])])
            else:
                views.append(cache.buffers[i][:cache.sizes[i]].view(n * H, cache.desc.capacity // BLOCK, -1)[:, blk])
    return views


def run(state):
    case = state["case"]
    if case["kind"] == "prefill":
        cache = state["cache"]
        cache.quant_pack_kv(state["k"], state["v"])
        return [buf[:size] for buf, size in zip(cache.buffers, cache.sizes) if size]
    if case["kind"] == "paged_prefill":
        cache = state["cache"]
        for s, (k, v) in enumerate(zip(state["k"], state["v"])):
            cache.quant_pack_kv(s, k, v)
        return [buf[:size] for buf, size in zip(cache.buffers, cache.sizes) if size] + [cache.seq_lens]
    out = state["out"]
    if case["kind"] == "paged_step":
        state["all_lens"].copy_(state["lens"])
        for i, (cache, kn, vn, q, _, _) in enumerate(state["layers"]):
            cache.decode_step(kn, vn, q, SCALE, out[i], state["splits"], lazy=case["lazy"])
    else:
        for i, (cache, kn, vn, q, packed, res) in enumerate(state["layers"]):
            cache.packed_len, cache.res_len = packed, res   # this step, again
            cache.decode_step(kn, vn, q, SCALE, out[i], lazy=case["lazy"])
    return {"out": out, "written": state["written"], "lens": state.get("all_lens", 0)}


# ---- the same in 64 bits -----------------------------------------------------------------------------

def _groups(x, mode, group):
    """x [.., 128 tokens, 128 channels] as [.., groups, members] with the statistics' members last, and the
    way back.  mode "channel": over `group` tokens of a channel; "token": over `group` channels of a token."""
    lead = x.shape[:-2]
    if mode == "channel":
        y = x.reshape(*lead, BLOCK // group, group, D).transpose(-1, -2)
        return y, lambda z: z.transpose(-1, -2).reshape(*lead, BLOCK, D)
    return x.reshape(*lead, BLOCK, D // group, group), lambda z: z.reshape(*lead, BLOCK, D)


def _quantize_int(x, bits, mode, group):
    """Codes, parameters (as int32 words: scale below, zero above) and values of whole blocks
    x [.., 128, 128] fp16.  The format is defined on fp32 steps: one subtraction and one division
    (the quotient in 64 bits, rounded to fp32, is the fp32 quotient), the scale then rounded to fp16."""
    y, back = _groups(x, mode, group)
    y32 = y.float()
    lo, hi = y32.amin(-1, keepdim=True) + 0.0, y32.amax(-1, keepdim=True)
    top = 2 ** bits - 1
    scale = ((hi - lo).double() / top).float().half()
    s64 = scale.double()
    safe = torch.where(s64 == 0, torch.ones_like(s64), s64)
    codes = ((y32 - lo).double() / safe).float().round().clamp_(0, top)
    codes = torch.where(s64 == 0, torch.zeros_like(codes), codes).double()
    value = codes * s64 + lo.double()
    word = (scale.view(torch.int16).int() & 0xFFFF) | (lo.half().view(torch.int16).int() << 16)
    return back(codes), word.squeeze(-1), back(value)


def _quantize_mx(x):
    """e2m1 codes (with sign, 0..15), scale bytes and values of rows x [.., 128] bf16, 32 channels a block."""
    y = x.double().reshape(*x.shape[:-1], D // 32, 32)
    amax = y.abs().amax(-1, keepdim=True)
    e = (torch.frexp(amax)[1] - 3).clamp(-127, 127)
    e = torch.where(amax == 0, torch.zeros_like(e), e)
    power = torch.exp2(e.double())
    a = y.abs() / power
    # nearest of 0, .5, 1, 1.5, 2, 3, 4, 6; ties to the even code
    code = ((a > 0.25).int() + (a >= 0.75) + (a > 1.25) + (a >= 1.75) + (a > 2.5) + (a >= 3.5) + (a > 5.0))
    grid = torch.tensor([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0], dtype=torch.float64, device=x.device)
    value = grid[code.long()] * power * torch.where(y < 0, -1.0, 1.0)
    code = code + 8 * ((y < 0) & (code > 0)).int()
    return code.reshape(x.shape), (e + 127).to(torch.uint8).squeeze(-1), value.reshape(x.shape)


def _pack(codes, bits):
    """Codes [.., n] -> bytes [.., n * bits / 8], the first code in the low bits."""
    per = 8 // bits
    c = codes.to(torch.int32).reshape(*codes.shape[:-1], -1, per)
    return sum(c[..., i] << (bits * i) for i in range(per)).to(torch.uint8)


def _attend(case, q, k, v, out):
    """Attention of one sequence: q [Hq, D], k and v [H, L, D] float64, into out [Hq, D]."""
    g = case["q_heads"] // case["kv_heads"]
    for h in range(case["kv_heads"]):
        s = (q[g * h:g * (h + 1)].double() @ k[h].T) * SCALE
        out[g * h:g * (h + 1)] = torch.softmax(s, -1) @ v[h]


def _stored(case, k, v, lazy_fill):
    """What a cache that holds tokens k, v [H, L, D] gives back, in 64 bits."""
    if _is_mx(case):
        return _quantize_mx(k)[2], _quantize_mx(v)[2]
    H, L, _ = k.shape
    nb = L // BLOCK - (1 if lazy_fill else 0)
    kd, vd = k.double(), v.double()
    step = max(1, (1 << 24) // (BLOCK * D))   # blocks at a time
    for h in range(H):
        for b in range(0, nb, step):
            t = slice(b * BLOCK, min(nb, b + step) * BLOCK)
            modes = ((k, kd, "token" if _per_token(case) else "channel"), (v, vd, "token"))
            for src, dst, mode in modes:
                dst[h, t] = _quantize_int(src[h, t].reshape(-1, BLOCK, D), _bits(case), mode, _group(case))[2].reshape(-1, D)
    return kd, vd


def _exact_prefill(case, seed):
    k, v, _, _, _ = _draw_layer(case, seed, 0)
    cap = (case["context"] + 1 + BLOCK - 1) // BLOCK * BLOCK
    n, H, L, _ = k.shape
    pad = torch.zeros((n, H, cap - L, D), dtype=k.dtype, device=k.device)
    kc, vc = torch.cat([k, pad], 2), torch.cat([v, pad], 2)
    if _is_mx(case):
        (kcode, kscale, _), (vcode, vscale, _) = _quantize_mx(kc), _quantize_mx(vc)
        kscale[:, :, L:] = 0   # nothing is stored past the end
        vscale[:, :, L:] = 0
        vcode = vcode.reshape(n, H, cap // BLOCK, BLOCK, D).transpose(-1, -2)
        parts = [_pack(kcode, 4), _pack(vcode, 4), kscale, vscale]
        return [p.contiguous().view(-1) for p in parts]
    nb, bits, group = L // BLOCK, _bits(case), _group(case)
    blocks = [x[:, :, :nb * BLOCK].reshape(n, H, nb, BLOCK, D) for x in (kc, vc)]
    sizes = [D * BLOCK * bits // 8] * 2 + [4 * BLOCK * (BLOCK // group)] * 2
    whole = [torch.zeros((n, H, cap // BLOCK, s), dtype=torch.uint8, device=k.device) for s in sizes]
    for i in range(n):
        for h in range(H):
            kcode, kword, _ = _quantize_int(blocks[0][i, h], bits, "token" if _per_token(case) else "channel", group)
            vcode, vword, _ = _quantize_int(blocks[1][i, h], bits, "token", group)
            parts = [_pack(kcode, bits), _pack(vcode.transpose(-1, -2), bits), kword, vword]
            for w, p in zip(whole, parts):
                w[i, h, :nb] = p.contiguous().view(torch.uint8).reshape(nb, -1)
    res = [torch.zeros((n, H, BLOCK, D), dtype=k.dtype, device=k.device) for _ in range(2)]
    for r, x in zip(res, (k, v)):
        r[:, :, :L - nb * BLOCK] = x[:, :, nb * BLOCK:]
    return [w.view(-1) for w in whole] + [r.view(torch.uint8).view(-1) for r in res]


def exact(case, seed):
    """Attention outputs in 64 bits over the values that the format stores; the packed bytes of a prefill as its
    definition gives them.  The cache bytes a step writes are whole numbers, compared as they are."""
    if case["kind"] == "prefill":
        return _exact_prefill(case, seed)
    if case["kind"] == "paged_prefill":
        return None
    lens = _lengths(case)
    out = torch.zeros((case["layers"], case["batch"], case["q_heads"], D), dtype=torch.float64, device=DEVICE)
    for i in range(case["layers"]):
        k, v, kn, vn, q = _draw_layer(case, seed, i)
        for s, L in enumerate(lens):
            ks, vs = torch.cat([k[s], kn[s][:, None]], 1), torch.cat([v[s], vn[s][:, None]], 1)
            _attend(case, q[s], *_stored(case, ks, vs, case["lazy"] and (L + 1) % BLOCK == 0), out[i, s])
    return {"out": out, "written": None, "lens": None}
