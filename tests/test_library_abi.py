"""CPU-side checks of the C-ABI library: it loads, exports every declared symbol, and
validates arguments before touching the GPU (no kernel is launched here)."""
import ctypes
import os
import re
import shutil
import subprocess
import sysconfig

import pytest

from paper_2503_18773_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
needs_lib = pytest.mark.skipif(not os.path.exists(B._LIB_PATH), reason="libbitdecode.so not built")


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "bitdecode.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(bd_[a-z_0-9]+)\s*\(", text)))


@needs_lib
def test_every_declared_symbol_is_exported():
    names = _declared_symbols()
    assert sorted(B.EXPORTS) == names
    for n in names:
        assert hasattr(B.lib(), n), n


def _desc(**kw):
    d = dict(batch=1, n_q_heads=32, n_kv_heads=8, head_dim=128, format=B.BD_FMT_INT4, capacity=32768)
    d.update(kw)
    return B.bd_cache(d["batch"], d["n_q_heads"], d["n_kv_heads"], d["head_dim"], d["format"], d["capacity"],
                      None, None, None, None, None, None)


@needs_lib
def test_cache_bytes_match_the_format():
    c = _desc()
    units, cap = 8, 32768
    assert [B.bd_cache_bytes(c, i) for i in range(6)] == [
        units * cap * 64, units * cap * 64, units * (cap // 128) * 128 * 4, units * cap * 4,
        units * 128 * 128 * 2, units * 128 * 128 * 2]
    c2 = _desc(format=B.BD_FMT_INT2)
    assert B.bd_cache_bytes(c2, 0) == units * cap * 32 and B.bd_cache_bytes(c2, 3) == units * cap * 4
    c4 = _desc(format=B.BD_FMT_MXFP4, batch=16, capacity=16384)
    assert [B.bd_cache_bytes(c4, i) for i in range(6)] == [128 * 16384 * 64, 128 * 16384 * 64, 128 * 16384 * 4,
                                                          128 * 16384 * 4, 0, 0]
    # 136 / 72 / 136 bytes per token per KV head
    for c_, per in [(c, 136), (c2, 72)]:
        assert sum(B.bd_cache_bytes(c_, i) for i in range(4)) == per * units * cap
    assert B.bd_cache_bytes(_desc(head_dim=64), 0) == 0
    assert B.bd_cache_bytes(c, 6) == 0
    # quantization groups of 64 / 32: the codes stay, the parameter arrays grow by 128 / group
    for fmt, per in [(B.BD_FMT_INT4_G64, 144), (B.BD_FMT_INT4_G32, 160), (B.BD_FMT_INT2_G64, 80), (B.BD_FMT_INT2_G32, 96),
                     (B.BD_FMT_INT4_KT_G64, 144), (B.BD_FMT_INT4_KT_G32, 160), (B.BD_FMT_INT2_KT_G64, 80),
                     (B.BD_FMT_INT2_KT_G32, 96)]:
        cg = _desc(format=fmt)
        assert sum(B.bd_cache_bytes(cg, i) for i in range(4)) == per * units * cap
        assert B.bd_cache_bytes(cg, 4) == units * 128 * 128 * 2
    assert B.bd_cache_bytes(_desc(format=13), 0) == 0


@needs_lib
def test_split_heuristic_and_workspace():
    c = _desc()
    for L in (0, 128, 1024, 32768, 131072):
        s = B.bd_choose_splits(c, L)
        assert 1 <= s <= max(1, L // 128)
    assert B.bd_workspace_bytes(c, 64) == 64 * 32 * 130 * 4
    assert B.bd_workspace_bytes(c, 0) == 0


@needs_lib
def test_argument_validation_happens_before_any_launch():
    L = B.lib()
    c = _desc()
    pl, rl = ctypes.c_int32(0), ctypes.c_int32(0)
    # NULL cache buffers
    assert L.bd_quant_pack_kv(ctypes.byref(c), None, None, 128, ctypes.byref(pl), ctypes.byref(rl), None) == -1
    c.k_codes = c.v_codes = c.k_params = c.v_params = c.k_res = c.v_res = 4096
    assert L.bd_quant_pack_kv(ctypes.byref(c), None, None, 128, ctypes.byref(pl), ctypes.byref(rl), None) == -1
    assert L.bd_quant_pack_kv(ctypes.byref(c), 4096, 4096, -1, ctypes.byref(pl), ctypes.byref(rl), None) == -1
    assert L.bd_quant_pack_kv(ctypes.byref(c), 4096, 4100, 128, ctypes.byref(pl), ctypes.byref(rl), None) == -3
    assert L.bd_quant_pack_kv(ctypes.byref(c), 4096, 4096, 32768 + 128, ctypes.byref(pl), ctypes.byref(rl),
                              None) == -4
    # append that would overflow the packed buffers leaves the lengths alone
    pl, rl = ctypes.c_int32(32768), ctypes.c_int32(127)
    assert L.bd_append_kv(ctypes.byref(c), 4096, 4096, ctypes.byref(pl), ctypes.byref(rl), None) == -4
    assert (pl.value, rl.value) == (32768, 127)
    pl, rl = ctypes.c_int32(100), ctypes.c_int32(0)
    assert L.bd_append_kv(ctypes.byref(c), 4096, 4096, ctypes.byref(pl), ctypes.byref(rl), None) == -1
    # decode: bad split count, bad lengths, misaligned workspace
    assert L.bd_decode_attn(ctypes.byref(c), 4096, 1024, 0, 0.1, 0, 4096, 4096, None) == -1
    assert L.bd_decode_attn(ctypes.byref(c), 4096, 1000, 0, 0.1, 4, 4096, 4096, None) == -1
    assert L.bd_decode_attn(ctypes.byref(c), 4096, 1024, 128, 0.1, 4, 4096, 4096, None) == -1
    assert L.bd_decode_attn(ctypes.byref(c), 4096, 1024, 0, 0.1, 4, 4100, 4096, None) == -3
    assert L.bd_splitk_combine(ctypes.byref(c), None, 4, 4096, None) == -1
    # allocation-free variant: `out` is required; partials beyond the static array are refused
    assert L.bd_decode_attn_static(ctypes.byref(c), 4096, 1024, 0, 0.1, 4, None, None) == -1
    too_many = B.BD_STATIC_SCRATCH_BYTES // (c.batch * c.n_q_heads * 130 * 4) + 1
    assert L.bd_decode_attn_static(ctypes.byref(c), 4096, 1024, 0, 0.1, too_many, 4096, None) == -4
    # the streaming-read probe: whole blocks inside the capacity, an aligned sink
    assert L.bd_probe_stream_read(ctypes.byref(c), 1000, None, None) == -1
    assert L.bd_probe_stream_read(ctypes.byref(c), c.capacity + 128, None, None) == -1
    assert L.bd_probe_stream_read(ctypes.byref(c), 1024, 4098, None) == -3
    pl, rl = ctypes.c_int32(1024), ctypes.c_int32(5)
    assert L.bd_decode_step(ctypes.byref(c), 4096, 4096, 4096, ctypes.byref(pl), ctypes.byref(rl), 0.1, 4, 4096,
                            None, None) == -1                       # out is required
    assert L.bd_decode_step(ctypes.byref(c), 4096, 4100, 4096, ctypes.byref(pl), ctypes.byref(rl), 0.1, 4, 4096,
                            4096, None) == -3
    assert (pl.value, rl.value) == (1024, 5)
    # shapes this build has no kernel for
    assert B.bd_cache_bytes(_desc(n_q_heads=64), 0) > 0                # 8 per KV head
    assert B.bd_cache_bytes(_desc(n_q_heads=8 * 40), 0) > 0            # 40 per KV head: 16 at a time
    bad = _desc(n_kv_heads=40000, n_q_heads=40000 * 17)                # 2 x 40000 workgroups per split
    assert L.bd_decode_attn(ctypes.byref(bad), 4096, 1024, 0, 0.1, 4, 4096, 4096, None) == -2
    bad = _desc(batch=65536)                                           # beyond the launch grid
    assert L.bd_decode_attn(ctypes.byref(bad), 4096, 1024, 0, 0.1, 4, 4096, 4096, None) == -2
    assert B.bd_cache_bytes(bad, 0) == 0
    bad = _desc(batch=8192, n_kv_heads=8, n_q_heads=32)                # 65536 (sequence, KV head) units
    assert L.bd_quant_pack_kv(ctypes.byref(bad), 4096, 4096, 128, ctypes.byref(pl), ctypes.byref(rl), None) == -2
    assert B.bd_cache_bytes(_desc(batch=8191, n_kv_heads=8, n_q_heads=32), 0) > 0
    assert L.bd_strerror(-4) == b"cache capacity exceeded"


def test_missing_library_fails_loudly(monkeypatch):
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_LIB_PATH", "/nonexistent/libbitdecode.so")
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        B.lib()


def _paged(**kw):
    d = dict(batch=4, n_q_heads=32, n_kv_heads=8, head_dim=128, format=B.BD_FMT_INT4, num_pages=100, max_pages=10)
    d.update(kw)
    return B.bd_paged_cache(d["batch"], d["n_q_heads"], d["n_kv_heads"], d["head_dim"], d["format"], d["num_pages"],
                            d["max_pages"])


@needs_lib
def test_paged_sizes_and_argument_validation():
    c = _paged()
    pool = 100 * 8
    assert [B.bd_paged_cache_bytes(c, i) for i in range(8)] == [
        pool * 128 * 64, pool * 128 * 64, pool * 128 * 4, pool * 128 * 4, 4 * 8 * 128 * 128 * 2, 4 * 8 * 128 * 128 * 2,
        4 * 10 * 4, 4 * 4]
    assert B.bd_paged_cache_bytes(_paged(format=B.BD_FMT_INT2), 0) == pool * 128 * 32
    mx = _paged(format=B.BD_FMT_MXFP4)                    # no residual: every token is quantized on arrival
    assert [B.bd_paged_cache_bytes(mx, i) for i in range(8)] == [
        pool * 128 * 64, pool * 128 * 64, pool * 128 * 4, pool * 128 * 4, 0, 0, 4 * 10 * 4, 4 * 4]
    assert B.bd_paged_cache_bytes(_paged(num_pages=0), 0) == 0
    g32 = _paged(format=B.BD_FMT_INT4_G32)               # smaller groups: the parameter arrays grow by 128 / group
    assert [B.bd_paged_cache_bytes(g32, i) for i in range(4)] == [pool * 128 * 64, pool * 128 * 64, pool * 4 * 128 * 4,
                                                                 pool * 128 * 4 * 4]
    assert B.bd_paged_workspace_bytes(c, 16) == 16 * 4 * 32 * 130 * 4
    L = B.lib()
    # NULL buffers are refused before anything is launched
    assert L.bd_paged_append_kv(ctypes.byref(c), 16, 16, None) == -1
    for name in ("k_codes", "v_codes", "k_params", "v_params", "k_res", "v_res", "block_table", "seq_lens"):
        setattr(c, name, 4096)
    assert L.bd_paged_append_kv(ctypes.byref(c), None, 16, None) == -1
    assert L.bd_paged_append_kv(ctypes.byref(c), 8, 16, None) == -3
    assert L.bd_paged_quant_pack_kv(ctypes.byref(c), 4, 16, 16, 10, None) == -1     # sequence out of range
    assert L.bd_paged_quant_pack_kv(ctypes.byref(c), 0, 16, 16, 128 * 11, None) == -4   # more blocks than table columns
    assert L.bd_paged_decode_attn(ctypes.byref(c), 16, ctypes.c_float(0.1), 0, 16, 16, None) == -1
    assert L.bd_paged_decode_attn(ctypes.byref(c), 16, ctypes.c_float(0.1), 4, 16, None, None) == -1
    c.seq_lens = 4098
    assert L.bd_paged_append_kv(ctypes.byref(c), 16, 16, None) == -3
    for name in ("k_codes", "v_codes", "k_params", "v_params", "block_table", "seq_lens"):
        setattr(mx, name, 4096)
    # MXFP4 keeps partly filled blocks in pages: 128 * 10 + 1 tokens need an eleventh table column
    assert L.bd_paged_quant_pack_kv(ctypes.byref(mx), 0, 16, 16, 128 * 10 + 1, None) == -4
    assert L.bd_paged_quant_pack_kv(ctypes.byref(mx), 0, 16, 20, 128, None) == -3


@needs_lib
def test_split_heuristic_properties():
    """One resident round of workgroups: splits x units stays near 512, never exceeds the number of
    4-block quanta, and short contexts get one block per wave at most."""
    for batch, hkv in [(1, 8), (8, 8), (16, 8), (1, 1), (64, 2)]:
        c = _desc(batch=batch, n_q_heads=4 * hkv, n_kv_heads=hkv, capacity=1 << 20)
        prev = 0
        for L in (128, 512, 4096, 32768, 131072, 1 << 20):
            s = B.bd_choose_splits(c, L)
            quanta = (L // 128 + 3) // 4
            assert 1 <= s <= quanta
            assert s * batch * hkv <= max(768, batch * hkv)
            assert s >= prev or s * batch * hkv >= 256        # grows with the context until the chip is full
            prev = s
    assert B.bd_choose_splits(_desc(), 32768) == 64 and B.bd_choose_splits(_desc(), 131072) == 64
    assert B.bd_choose_splits(_desc(batch=8), 32768) == 8
    # a chip already full of units takes one split (no merge kernel) unless the call is long
    assert B.bd_choose_splits(_desc(batch=48), 4096) == 1 and B.bd_choose_splits(_desc(batch=32), 4096) == 1
    assert B.bd_choose_splits(_desc(batch=32), 16384) == 2
    # one block per wave is kept up to three workgroups per compute unit (integer formats, groups <= 8)
    assert B.bd_choose_splits(_desc(), 40960) == 80 and B.bd_choose_splits(_desc(), 49152) == 96
    assert B.bd_choose_splits(_desc(), 57344) == 64                     # beyond that: one round of 512 workgroups
    assert B.bd_choose_splits(_desc(format=B.BD_FMT_MXFP4), 49152) == 64
    assert B.bd_choose_splits(_desc(format=B.BD_FMT_MXFP4), 32768 + 1) == 64   # quanta need not divide evenly
    # one instance of the kernel for smaller quantization groups runs one workgroup per compute unit
    assert B.bd_choose_splits(_desc(format=B.BD_FMT_INT4_G32), 32768) == 64
    assert B.bd_choose_splits(_desc(format=B.BD_FMT_INT4_G32, n_q_heads=64), 32768) == 32
    assert B.bd_choose_splits(_desc(format=B.BD_FMT_INT2_G64, n_q_heads=128), 32768) == 32   # two workgroups per KV head


@needs_lib
def test_the_count_of_a_step():
    for fmt in range(13):
        for batch, hkv, gq in [(1, 8, 4), (1, 1, 1), (3, 2, 8), (24, 8, 4), (40, 8, 8), (16, 4, 16), (64, 8, 4)]:
            c = _desc(format=fmt, batch=batch, n_kv_heads=hkv, n_q_heads=hkv * gq)
            for L in (1, 100, 128, 600, 1024, 3100, 8192, 32768, 131072):
                assert 1 <= B.bd_step_splits(c, L) <= B.bd_choose_splits(c, L), (fmt, batch, hkv, gq, L)
    # two rounds of blocks in one workgroup, one round of workgroups for few units, two where the blocks are long
    assert [B.bd_step_splits(_desc(), L) for L in (1024, 1025, 6016, 32768, 131072)] == [1, 3, 12, 32, 32]
    assert [B.bd_step_splits(_desc(format=B.BD_FMT_INT2), L) for L in (1024, 32768, 131072)] == [1, 32, 64]
    assert [B.bd_step_splits(_desc(format=B.BD_FMT_INT4_G32), L) for L in (1024, 32768)] == [2, 64]
    # bad arguments and an empty cache: one
    assert B.bd_step_splits(_desc(), 0) == B.bd_step_splits(_desc(), -5) == B.bd_step_splits(_desc(head_dim=64), 999) == 1


@needs_lib
def test_counters_of_a_paged_step():
    """Where the C structure has them (behind a bd_paged_cache that other calls take as it is), room for the counters of any
    batch, and what a step without them says."""
    assert B.bd_paged_counted.counters.offset == ctypes.sizeof(B.bd_paged_cache) == 14 * 8
    assert B.BD_STEP_COUNTER_BYTES == 64 * 17
    assert f"#define BD_STEP_COUNTER_BYTES {B.BD_STEP_COUNTER_BYTES}\n" in open(os.path.join(ROOT, "include", "bitdecode.h")).read()
    dummy = 4096   # (never read: every call is refused before a launch)
    c = B.bd_paged_counted(1, 8, 2, 128, B.BD_FMT_INT4, 4, 4, *[dummy] * 9)
    L = B.lib()
    for step in (L.bd_paged_counted_step, L.bd_paged_counted_step_lazy):
        call = lambda: step(ctypes.byref(c), dummy, dummy, dummy, 0.1, 0, dummy, dummy, None)   # 0 splits
        c.counters = None
        assert call() == -1
        c.counters = dummy + 8
        assert call() == -3
        c.counters = dummy
        assert call() == -1
        assert step(None, dummy, dummy, dummy, 0.1, 1, dummy, dummy, None) == -1


@pytest.mark.parametrize("lazy", [False, True])
def test_a_description_without_counters_takes_the_step_without_them(lazy, monkeypatch):
    """One that a caller has put in the place of the cache class's own ends where the counters would be."""
    cache, taken = object.__new__(B.PagedKVCache), []
    monkeypatch.setattr(B, "_address", lambda name: name)
    monkeypatch.setattr(B, "_stream", lambda stream: 0)
    monkeypatch.setattr(B, "_call", type("", (), {"paged_step": staticmethod(lambda entry, desc, *rest: taken.append(entry) or 0)}))
    monkeypatch.setattr(cache, "workspace", lambda num_splits: None, raising=False)
    for cache.desc in (B.bd_paged_counted(), B.bd_paged_cache()):
        cache.decode_step(None, None, None, 0.1, None, 1, lazy=lazy)
    assert taken == ["bd_paged_counted_step" + "_lazy" * lazy, "bd_paged_decode_step" + "_lazy" * lazy]


ECHO = """
#include <stdint.h>
#include <string.h>
int64_t seen[16];
static int64_t bits(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
#define P(x) (int64_t)(uintptr_t)(x)
int splits(const int32_t* c, int32_t n) { seen[0] = c[0]; seen[1] = n; return 7; }
int step(const int32_t* c, void* k, void* v, void* q, int32_t* p, int32_t* r, float s, int32_t n, void* w, void* o, void* st) {
  int64_t x[] = {c[0], P(k), P(v), P(q), *p, *r, bits(s), n, P(w), P(o), P(st)}; memcpy(seen, x, sizeof x); *p += 128; *r = -1; return -3; }
int paged_step(const int32_t* c, void* k, void* v, void* q, float s, int32_t n, void* w, void* o, void* st) {
  int64_t x[] = {c[0], P(k), P(v), P(q), bits(s), n, P(w), P(o), P(st)}; memcpy(seen, x, sizeof x); return -4; }
int paged_quant(const int32_t* c, int32_t b, void* k, void* v, int32_t n, void* st) {
  int64_t x[] = {c[0], b, P(k), P(v), n, P(st)}; memcpy(seen, x, sizeof x); return 0; }
int quant(const int32_t* c, void* k, void* v, int32_t n, int32_t* p, int32_t* r, void* st) {
  int64_t x[] = {c[0], P(k), P(v), n, P(st)}; memcpy(seen, x, sizeof x); *p = n - 5; *r = 5; return 2; }
"""


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
@pytest.mark.parametrize("call", ["ctypes", "module"])
def test_calls_pass_every_argument_and_give_back_what_comes(call, tmp_path):
    """Both ways that the cache classes call the library, against functions that record what they are given: tensors, None,
    addresses beyond 32 bits, negative integers."""
    if call == "module":
        if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
            pytest.skip("the calling module needs Python's headers")
        from paper_2503_18773_amd import _bdcall
        assert B._call is _bdcall
    call = B._call if call == "module" else B._CtypesCall
    (tmp_path / "echo.c").write_text(ECHO)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(tmp_path / "echo.c"), "-o", str(tmp_path / "echo.so")], check=True)
    L = ctypes.CDLL(str(tmp_path / "echo.so"))
    at = lambda name: ctypes.cast(getattr(L, name), ctypes.c_void_p).value
    seen = lambda n: list((ctypes.c_int64 * 16).in_dll(L, "seen"))[:n]

    class Tensor:
        def __init__(self, at):
            self.data_ptr = lambda: at

    k, v, q, w, o = (Tensor(x) for x in (0x7F0012345670, 16, 2 ** 40, 48, 64))
    c, half = B.bd_cache(batch=11), 0x3F000000
    assert call.splits(at("splits"), c, -5) == 7 and seen(2) == [11, -5]
    assert call.step(at("step"), c, k, v, q, 256, 127, 0.5, 3, w, o, 2 ** 41) == (-3, 384, -1)
    assert seen(11) == [11, 0x7F0012345670, 16, 2 ** 40, 256, 127, half, 3, 48, 64, 2 ** 41]
    assert call.step(at("step"), c, k, v, q, -1, 0, 1, -7, w, None, 0)[0] == -3
    assert seen(11)[4:] == [-1, 0, 0x3F800000, -7, 48, 0, 0]
    p = B.bd_paged_cache(batch=12)
    assert call.paged_step(at("paged_step"), p, k, None, q, 0.5, 9, w, o, 0) == -4
    assert seen(9) == [12, 0x7F0012345670, 0, 2 ** 40, half, 9, 48, 64, 0]
    assert call.paged_quant(at("paged_quant"), p, 6, k, v, 1333, 80) == 0 and seen(6) == [12, 6, 0x7F0012345670, 16, 1333, 80]
    assert call.quant(at("quant"), c, k, v, 133, 0) == (2, 128, 5) and seen(5) == [11, 0x7F0012345670, 16, 133, 0]


@pytest.mark.parametrize("compiler", ["/bin/false", "/no/such/compiler", "cp"])
def test_a_calling_module_that_does_not_build_is_gone(compiler, tmp_path, monkeypatch, capsys):
    """One of an earlier build would be imported, with the library's calls of then."""
    from paper_2503_18773_amd import build
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setenv("CC", compiler)
    (tmp_path / ("_bdcall" + sysconfig.get_config_var("EXT_SUFFIX"))).write_bytes(b"old")
    build._build_call()
    assert list(tmp_path.iterdir()) == [] and "not built" in capsys.readouterr().err
