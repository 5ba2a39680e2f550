"""The C ABI on the CPU: the library loads, exports every declared symbol, its
host helpers are right, and invalid arguments are rejected before any HIP call
(so these run without a GPU; no kernel is launched)."""
import ctypes
import os
import re

import pytest

import oracle
from paper_2607_06827_amd import speechkv as skv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "speechkv.h")
lib = skv._lib

FAKE = 0x10000000  # 16-byte aligned, never dereferenced on these paths


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(speechkv_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = declared_functions()
    assert set(names) == {"speechkv_pool_kv", "speechkv_decode_attn", "speechkv_prefill_attn",
                          "speechkv_decode_attn_noalloc",
                          "speechkv_pool_hidden", "speechkv_pool_prefill_attn",
                          "speechkv_pool_kv_segments", "speechkv_prefill_attn_segments",
                          "speechkv_compressed_len_segments", "speechkv_prefill_attn_bwd_segments",
                          "speechkv_pool_kv_bwd_segments",
                          "speechkv_prefill_attn_bwd",
                          "speechkv_prefill_attn_bwd_workspace_bytes", "speechkv_pool_kv_bwd",
                          "speechkv_pool_kv_bwd_workspace_bytes",
                          "speechkv_compressed_len", "speechkv_decode_num_splits",
                          "speechkv_decode_workspace_bytes", "speechkv_status_string",
                          "speechkv_version"}
    for n in names:
        assert hasattr(lib, n), n


def test_status_strings_and_version():
    for code in (0, -1, -2, -3, -4, -5, -6):
        assert skv.speechkv_status_string(code) and skv.speechkv_status_string(code) != "unknown status"
    assert skv.speechkv_status_string(17) == "unknown status"
    assert re.fullmatch(r"\d+\.\d+\.\d+", skv.speechkv_version())


def test_compressed_len_agrees_with_oracle():
    for P in (0, 3, 32):
        for T in (0, 1, 3, 4, 5, 60, 375, 750, 7500):
            for N in (0, 7):
                for w in (1, 2, 3, 4, 8):
                    for layer, l0 in ((0, 0), (3, 5), (14, 14), (27, 14)):
                        assert skv.speechkv_compressed_len(P, T, N, w, layer, l0) == \
                            oracle.compressed_len(P, T, N, w, layer, l0)
    assert skv.speechkv_compressed_len(32, 375, 0, 4, 0, 0) == 32 + 94
    assert skv.speechkv_compressed_len(32, 1500, 64, 4, 0, 0) == 471
    assert skv.speechkv_compressed_len(-1, 3, 0, 4, 0, 0) == -1
    assert skv.speechkv_compressed_len(1, 3, 0, 0, 0, 0) == -1


def test_split_choice_and_workspace():
    s = skv.speechkv_decode_num_splits(64, 8, 348)
    assert 1 <= s <= 64
    assert skv.speechkv_decode_num_splits(1, 2, 39) == 1
    assert skv.speechkv_decode_num_splits(0, 8, 10) == -1
    assert skv.speechkv_decode_workspace_bytes(1, 4, 2, 64, 39, 1) == 0
    n = skv.speechkv_decode_workspace_bytes(16, 16, 8, 128, 7788, 8)
    assert n >= 16 * 16 * 8 * (128 + 2) * 4
    assert skv.speechkv_decode_workspace_bytes(16, 16, 8, 128, 7788, 0) == \
        skv.speechkv_decode_workspace_bytes(16, 16, 8, 128, 7788,
                                            skv.speechkv_decode_num_splits(16, 8, 7788))


def test_split_heuristic_properties():
    """The split count minimises a launch-time estimate: no split where the
    merge launch would cost more than the parallelism saves (short caches,
    or enough (sequence, KV head) pairs to reach the bandwidth bound), more
    splits for long caches of few sequences; always a power of two in
    1..32 with at least 16 groups of 4 keys per split."""
    split = skv.speechkv_decode_num_splits
    for B, H in ((2, 8), (8, 8), (32, 8), (64, 8), (128, 8)):
        for L in range(0, 260, 7):
            assert split(B, H, L) == 1
    for L in range(0, 128):
        assert split(1, 1, L) == 1                     # too short for two splits of 16 groups
    for B in (64, 128, 512):
        for L in (1, 300, 910, 4000, 7788):
            assert split(B, 8, L) == 1                 # 512+ pairs: bandwidth-bound as one split
    assert split(1, 8, 7788) > split(4, 8, 7788) > split(16, 8, 7788) > 1  # fewer sequences, more splits
    for B in (1, 2, 3, 8, 16, 33):
        for L in (0, 63, 64, 65, 500, 2000, 7788, 65536):
            s = split(B, 8, L)
            assert 1 <= s <= 32 and s & (s - 1) == 0
            assert s == 1 or (L + 3) // 4 >= 16 * s


def cache(**kw):
    c = dict(k_pages=FAKE, v_pages=FAKE + (1 << 24), block_table=FAKE + (2 << 24), num_pages=64,
             page_size=16, max_pages_per_seq=8, num_kv_heads=2, head_dim=64,
             dtype=skv.DTYPE_BF16)
    c.update(kw)
    return skv._PagedKV(**c)


def spans(**kw):
    s = dict(prefix_len=FAKE + (3 << 24), speech_len=FAKE + (3 << 24) + 64,
             suffix_len=FAKE + (3 << 24) + 128, max_speech_len=40, max_total_len=60)
    s.update(kw)
    return skv._Spans(**s)


RAW = FAKE + (8 << 24)


def pool(c=None, s=None, **kw):
    a = dict(k=RAW, v=RAW + (1 << 22), sb=60 * 2 * 64, ss=2 * 64, sh=64, batch=2, raw_len=60, w=4,
             gate=None, layer=1, l0=0, clen=None)
    a.update(kw)
    c = c or cache()
    s = s or spans()
    return lib.speechkv_pool_kv(a["k"], a["v"], a["sb"], a["ss"], a["sh"], a["batch"], a["raw_len"],
                                ctypes.byref(s), a["w"], a["gate"], a["layer"], a["l0"],
                                ctypes.byref(c), a["clen"], None)


def decode(c=None, **kw):
    a = dict(q=FAKE + (9 << 24), batch=2, hq=4, clen=FAKE + (10 << 24), max_len=100, kn=None,
             vn=None, scale=0.125, splits=0, out=FAKE + (11 << 24), ws=None, ws_bytes=0)
    a.update(kw)
    c = c or cache()
    return lib.speechkv_decode_attn(a["q"], a["batch"], a["hq"], ctypes.byref(c), a["clen"],
                                    a["max_len"], a["kn"], a["vn"], a["scale"], a["splits"],
                                    a["out"], a["ws"], a["ws_bytes"], None)


def prefill(c=None, s=None, **kw):
    a = dict(q=FAKE + (12 << 24), batch=2, hq=4, q_len=60, w=4, layer=1, l0=0, mode=0,
             scale=0.125, out=FAKE + (13 << 24), lse=None)
    a.update(kw)
    c = c or cache()
    s = s or spans()
    return lib.speechkv_prefill_attn(a["q"], a["batch"], a["hq"], a["q_len"], ctypes.byref(c),
                                     ctypes.byref(s), a["w"], a["layer"], a["l0"], a["mode"],
                                     a["scale"], a["out"], a["lse"], None)


E_ARG, E_UNS, E_WS, E_ALIAS = skv.ERR_INVALID_ARG, skv.ERR_UNSUPPORTED, skv.ERR_WORKSPACE, skv.ERR_ALIAS

FQ, FOUT = FAKE + (23 << 24), FAKE + (24 << 24)


def fused(c=None, s=None, **kw):
    """speechkv_pool_prefill_attn with the pooling arguments of pool() and
    the attention arguments of prefill()."""
    a = dict(q=FQ, batch=2, hq=4, q_len=60, k=RAW, v=RAW + (1 << 22), sb=60 * 2 * 64, ss=2 * 64,
             sh=64, raw_len=60, w=4, gate=None, layer=1, l0=0, clen=None, mode=0, scale=0.125,
             out=FOUT, lse=None)
    a.update(kw)
    c = c or cache()
    s = s or spans()
    return lib.speechkv_pool_prefill_attn(a["q"], a["batch"], a["hq"], a["q_len"], a["k"], a["v"],
                                          a["sb"], a["ss"], a["sh"], a["raw_len"], ctypes.byref(s),
                                          a["w"], a["gate"], a["layer"], a["l0"], ctypes.byref(c),
                                          a["clen"], a["mode"], a["scale"], a["out"], a["lse"], None)


@pytest.mark.parametrize("kw,code", [
    (dict(k=None), E_ARG), (dict(batch=0), E_ARG), (dict(raw_len=0), E_ARG), (dict(w=0), E_ARG),
    (dict(layer=-1), E_ARG), (dict(sb=-8), E_ARG), (dict(ss=3), E_ARG), (dict(k=RAW + 4), E_ARG),
    (dict(gate=FAKE + 4), E_ARG), (dict(raw_len=50), E_ARG),
    (dict(k=FAKE), E_ALIAS), (dict(v=FAKE + (1 << 24) + 256), E_ALIAS),
])
def test_pool_rejects(kw, code):
    assert pool(**kw) == code


def test_pool_rejects_an_oversized_grid():
    """One sequence's pooling launch has max_total_len * Hkv * D / 512 blocks;
    past 2^31 - 1 the call is UNSUPPORTED before any launch."""
    H, D = 65535, 128
    rows = (1 << 33) // H + 1  # rows * H * D / 512 > 2^31 - 1
    base = 1 << 44  # far-apart fake ranges: nothing overlaps
    c = cache(num_kv_heads=H, head_dim=D, k_pages=base, v_pages=2 * base, block_table=3 * base)
    s = spans(max_speech_len=rows, max_total_len=rows)
    assert pool(c=c, s=s, k=4 * base, v=6 * base, raw_len=rows, sb=rows * H * D, ss=H * D, sh=D) == E_UNS


@pytest.mark.parametrize("kw,ckw", [
    (dict(clen=FAKE + 256), {}), (dict(clen=FAKE + (3 << 24)), {}), (dict(clen=RAW + 64), {}),
    (dict(gate=FAKE + (1 << 24) + 1024), {}), ({}, dict(block_table=FAKE + 2048)),
    ({}, dict(v_pages=FAKE + 4096)), (dict(clen=FAKE + (2 << 24) + 16), {}),
])
def test_pool_rejects_overlaps(kw, ckw):
    """The pools and cache_len_out may not overlap the raw K/V, the gate, the
    block table, the span lengths or each other."""
    assert pool(c=cache(**ckw), **kw) == E_ALIAS


HID = FAKE + (14 << 24)


def pool_hidden(s=None, **kw):
    a = dict(h=HID, sb=60 * 2048, ss=2048, batch=2, raw_len=60, hidden=2048, dtype=skv.DTYPE_BF16,
             w=4, gate=None, out=HID + (4 << 20), ob=60 * 2048, os=2048, cap=60, olen=None)
    a.update(kw)
    s = s or spans()
    return lib.speechkv_pool_hidden(a["h"], a["sb"], a["ss"], a["batch"], a["raw_len"], a["hidden"],
                                    a["dtype"], ctypes.byref(s), a["w"], a["gate"], a["out"], a["ob"],
                                    a["os"], a["cap"], a["olen"], None)


@pytest.mark.parametrize("kw,code", [
    (dict(h=None), E_ARG), (dict(out=None), E_ARG), (dict(batch=0), E_ARG), (dict(raw_len=0), E_ARG),
    (dict(w=0), E_ARG), (dict(sb=-8), E_ARG), (dict(ss=3), E_ARG), (dict(os=5), E_ARG),
    (dict(h=HID + 4), E_ARG), (dict(gate=FAKE + 4), E_ARG), (dict(raw_len=50), E_ARG),
    (dict(cap=0), E_ARG), (dict(hidden=768), E_UNS), (dict(hidden=128), E_UNS), (dict(dtype=7), E_UNS),
    (dict(out=HID + 2048 * 2), E_ALIAS),
])
def test_pool_hidden_rejects(kw, code):
    assert pool_hidden(**kw) == code


def test_pool_hidden_rejects_bad_spans():
    assert pool_hidden(s=spans(prefix_len=None)) == E_ARG


@pytest.mark.parametrize("ckw,code", [
    (dict(dtype=7), E_UNS), (dict(head_dim=96), E_UNS), (dict(page_size=12), E_UNS),
    (dict(page_size=4), E_UNS), (dict(page_size=512), E_UNS), (dict(num_pages=0), E_ARG),
    (dict(k_pages=None), E_ARG), (dict(block_table=None), E_ARG), (dict(k_pages=FAKE + 2), E_ARG),
])
def test_cache_description_rejected_by_every_call(ckw, code):
    assert pool(c=cache(**ckw)) == code
    assert decode(c=cache(**ckw)) == code
    assert prefill(c=cache(**ckw)) == code
    assert fused(c=cache(**ckw)) == code


@pytest.mark.parametrize("skw", [dict(prefix_len=None), dict(max_total_len=-1),
                                 dict(max_speech_len=70)])
def test_bad_spans(skw):
    assert pool(s=spans(**skw)) == E_ARG
    assert prefill(s=spans(**skw)) == E_ARG
    assert fused(s=spans(**skw)) == E_ARG


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), E_ARG), (dict(out=None), E_ARG), (dict(clen=None), E_ARG), (dict(batch=0), E_ARG),
    (dict(hq=3), E_ARG), (dict(hq=6), E_UNS), (dict(hq=32), E_UNS), (dict(max_len=-1), E_ARG),
    (dict(max_len=129), E_ARG), (dict(kn=FAKE), E_ARG), (dict(splits=-1), E_ARG),
    (dict(scale=float("nan")), E_ARG), (dict(scale=0.0), E_ARG), (dict(scale=-0.1), E_ARG),
    (dict(scale=float("inf")), E_ARG), (dict(q=FAKE + 8), E_ARG),
    (dict(splits=4), E_WS), (dict(splits=4, ws=FAKE + (14 << 24), ws_bytes=64), E_WS),
])
def test_decode_rejects(kw, code):
    assert decode(**kw) == code
    # the no-alloc call takes no workspace: the WORKSPACE cases are valid
    # there (and would reach the device), so only the others are repeated
    if code != E_WS:
        assert decode_noalloc(**kw) == code


def decode_noalloc(c=None, **kw):
    a = dict(q=FAKE + (9 << 24), batch=2, hq=4, clen=FAKE + (10 << 24), max_len=100, kn=None,
             vn=None, scale=0.125, splits=0, out=FAKE + (11 << 24))
    a.update({k: v for k, v in kw.items() if k in a})
    c = c or cache()
    return lib.speechkv_decode_attn_noalloc(a["q"], a["batch"], a["hq"], ctypes.byref(c), a["clen"],
                                            a["max_len"], a["kn"], a["vn"], a["scale"], a["splits"],
                                            a["out"], None)


Q, CLEN, OUT, WS = FAKE + (9 << 24), FAKE + (10 << 24), FAKE + (11 << 24), FAKE + (14 << 24)
KN, VN = FAKE + (15 << 24), FAKE + (16 << 24)


@pytest.mark.parametrize("kw", [
    dict(out=Q + 256), dict(out=FAKE + 4096), dict(out=FAKE + (1 << 24)), dict(out=CLEN - 64),
    dict(out=FAKE + (2 << 24)), dict(out=KN, kn=KN - 256, vn=VN),
    dict(splits=4, ws=Q, ws_bytes=1 << 20), dict(splits=4, ws=OUT - 4096, ws_bytes=1 << 20),
    dict(splits=4, ws=FAKE + 8192, ws_bytes=1 << 20),
    dict(kn=FAKE + 1024, vn=VN), dict(kn=KN, vn=FAKE + (1 << 24) + 512),
    dict(kn=KN, vn=VN, q=FAKE + 2048), dict(kn=KN, vn=VN, clen=FAKE + (1 << 24)),
])
def test_decode_rejects_overlaps(kw):
    """out, the split partials and (with a new token to store) the page pools
    may not overlap anything the step reads or each other."""
    assert decode(**kw) == E_ALIAS
    if "ws" not in kw:
        assert decode_noalloc(**kw) == E_ALIAS


def test_decode_pools_written_only_with_a_new_token():
    # the block table inside a pool is only an error when the pool is written
    c = cache(block_table=FAKE + 4096)
    assert decode(c=c, kn=KN, vn=VN) == E_ALIAS
    assert decode_noalloc(c=c, kn=KN, vn=VN) == E_ALIAS
    assert decode(c=cache(v_pages=FAKE + 8192), kn=KN, vn=VN) == E_ALIAS


def test_noalloc_rejects_steps_beyond_its_scratch():
    """speechkv_decode_attn_noalloc rejects a step whose split partials need
    more than SPEECHKV_NOALLOC_SCRATCH_BYTES before any HIP call, and the
    automatic split count never needs that much."""
    need = skv.speechkv_decode_workspace_bytes(8, 4, 2, 64, 100, 4096)
    assert need > skv.NOALLOC_SCRATCH_BYTES
    assert decode_noalloc(batch=8, splits=4096) == skv.ERR_SCRATCH
    assert "scratch" in skv.speechkv_status_string(skv.ERR_SCRATCH)
    worst = 0
    for B in (1, 2, 3, 5, 8, 16, 33, 64, 127, 128, 129, 512, 2048):
        for H in (1, 2, 4, 8, 16):
            for L in (0, 64, 1000, 7788, 65536, 1 << 20):
                for D in (64, 128):
                    worst = max(worst, skv.speechkv_decode_workspace_bytes(B, 8 * H, H, D, L, 0))
    assert 0 < worst <= skv.NOALLOC_SCRATCH_BYTES


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), E_ARG), (dict(out=None), E_ARG), (dict(q_len=59), E_ARG), (dict(mode=2), E_ARG),
    (dict(w=0), E_ARG), (dict(hq=6), E_UNS), (dict(hq=5), E_ARG), (dict(lse=FAKE + 2), E_ARG),
    (dict(scale=float("nan")), E_ARG), (dict(scale=0.0), E_ARG), (dict(scale=-1.0), E_ARG),
    (dict(batch=0), E_ARG),
])
def test_prefill_rejects(kw, code):
    assert prefill(**kw) == code


@pytest.mark.parametrize("kw", [
    dict(out=FAKE + (12 << 24) + 512), dict(out=FAKE + 64), dict(out=FAKE + (1 << 24) + 64),
    dict(out=FAKE + (2 << 24)), dict(out=FAKE + (3 << 24) + 64), dict(lse=FAKE + (12 << 24)),
    dict(lse=FAKE + (13 << 24) + 128), dict(lse=FAKE + 1024), dict(lse=FAKE + (3 << 24)),
])
def test_prefill_rejects_overlaps(kw):
    """out and lse may not overlap the queries, the pools, the block table,
    the span lengths or each other."""
    assert prefill(**kw) == E_ALIAS
    assert prefill_seg(**{k: (v if v != FAKE + (3 << 24) + 64 and v != FAKE + (3 << 24) else SEG)
                          for k, v in kw.items()}) == E_ALIAS


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), E_ARG), (dict(out=None), E_ARG), (dict(k=None), E_ARG), (dict(v=None), E_ARG),
    (dict(batch=0), E_ARG), (dict(q_len=59), E_ARG), (dict(raw_len=59), E_ARG), (dict(w=0), E_ARG),
    (dict(layer=-1), E_ARG), (dict(l0=-1), E_ARG), (dict(mode=2), E_ARG), (dict(scale=0.0), E_ARG),
    (dict(scale=float("nan")), E_ARG), (dict(scale=float("inf")), E_ARG), (dict(hq=5), E_ARG),
    (dict(hq=6), E_UNS), (dict(sb=-8), E_ARG), (dict(ss=3), E_ARG), (dict(k=RAW + 4), E_ARG),
    (dict(gate=FAKE + 4), E_ARG), (dict(lse=FAKE + 2), E_ARG), (dict(q=FQ + 8), E_ARG),
    (dict(k=FAKE), E_ALIAS), (dict(v=FAKE + (1 << 24) + 256), E_ALIAS), (dict(out=FQ + 4096), E_ALIAS),
    (dict(out=RAW), E_ALIAS), (dict(lse=FOUT + 64), E_ALIAS), (dict(lse=FAKE + 1024), E_ALIAS),
    (dict(gate=FAKE + 512), E_ALIAS), (dict(q=FAKE + (1 << 24)), E_ALIAS),
])
def test_fused_rejects(kw, code):
    assert fused(**kw) == code


def test_fused_is_bf16_only():
    assert fused(c=cache(dtype=skv.DTYPE_F32)) == E_UNS


def test_window_and_row_count_bounds():
    """w beyond SPEECHKV_MAX_WINDOW and row counts whose window count could
    overflow 32-bit arithmetic are rejected by every pooling and attention call."""
    big_w = skv.MAX_WINDOW + 1
    assert pool(w=big_w) == E_ARG
    assert pool_hidden(w=big_w) == E_ARG
    assert prefill(w=big_w) == E_ARG
    assert fused(w=big_w) == E_ARG
    too_many = 2**31 - 1 - skv.MAX_WINDOW + 1
    assert pool(raw_len=too_many) == E_ARG
    assert pool_hidden(raw_len=too_many) == E_ARG
    assert prefill(q_len=too_many) == E_ARG
    assert fused(q_len=too_many, raw_len=too_many) == E_ARG


def test_binding_constants_match_header():
    import re
    defs = dict(re.findall(r"#define SPEECHKV_(\w+) \(?(-?\d+)\)?", open(HEADER).read()))
    for name in ("OK", "ERR_INVALID_ARG", "ERR_UNSUPPORTED", "ERR_WORKSPACE", "ERR_ALIAS", "ERR_HIP",
                 "ERR_SCRATCH", "DTYPE_F32", "DTYPE_BF16", "MASK_WINDOW_END", "MASK_WINDOW_START",
                 "MAX_WINDOW", "MAX_SEGMENTS", "NOALLOC_SCRATCH_BYTES"):
        assert int(defs[name]) == getattr(skv, name), name


# ---------------------------------------------------------------- backward

def prefill_bwd(c=None, s=None, **kw):
    a = dict(q=FAKE + (15 << 24), batch=2, hq=4, q_len=60, w=4, layer=1, l0=0, mode=0, scale=0.125,
             out=FAKE + (16 << 24), lse=FAKE + (17 << 24), dout=FAKE + (18 << 24),
             dq=FAKE + (19 << 24), dk=FAKE + (20 << 24), dv=FAKE + (21 << 24), cap=60,
             ws=FAKE + (22 << 24), ws_bytes=1 << 20)
    a.update(kw)
    c = c or cache()
    s = s or spans()
    return lib.speechkv_prefill_attn_bwd(a["q"], a["batch"], a["hq"], a["q_len"], ctypes.byref(c),
                                         ctypes.byref(s), a["w"], a["layer"], a["l0"], a["mode"],
                                         a["scale"], a["out"], a["lse"], a["dout"], a["dq"], a["dk"],
                                         a["dv"], a["cap"], a["ws"], a["ws_bytes"], None)


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), E_ARG), (dict(out=None), E_ARG), (dict(lse=None), E_ARG), (dict(dout=None), E_ARG),
    (dict(dq=None), E_ARG), (dict(dk=None), E_ARG), (dict(dv=None), E_ARG), (dict(cap=0), E_ARG),
    (dict(w=0), E_ARG), (dict(w=skv.MAX_WINDOW + 1), E_ARG), (dict(q_len=59), E_ARG),
    (dict(mode=2), E_ARG), (dict(scale=0.0), E_ARG), (dict(hq=5), E_ARG), (dict(hq=6), E_UNS),
    (dict(batch=0), E_ARG), (dict(dq=FAKE + (19 << 24) + 4), E_ARG), (dict(lse=FAKE + (17 << 24) + 2), E_ARG),
    (dict(ws=None), E_WS), (dict(ws_bytes=2 * 4 * 60 * 4 - 4), E_WS),
    (dict(dq=FAKE + (15 << 24)), E_ALIAS), (dict(dv=FAKE + (20 << 24) + 256), E_ALIAS),
    (dict(dk=FAKE + 4096), E_ALIAS), (dict(ws=FAKE + (18 << 24)), E_ALIAS),
])
def test_prefill_bwd_rejects(kw, code):
    assert prefill_bwd(**kw) == code


def test_prefill_bwd_rejects_bad_cache_and_spans():
    assert prefill_bwd(c=cache(head_dim=96)) == E_UNS
    assert prefill_bwd(c=cache(k_pages=None)) == E_ARG
    assert prefill_bwd(s=spans(prefix_len=None)) == E_ARG


def test_bwd_workspace_sizes():
    assert skv.speechkv_prefill_attn_bwd_workspace_bytes(8, 16, 1596) == 8 * 16 * 1596 * 4
    assert skv.speechkv_prefill_attn_bwd_workspace_bytes(0, 16, 1596) == 0
    # per-block partial gate gradients (head_dim floats per block), about
    # 4096 blocks in all: at head_dim 128 a 256-thread pass covers 16 slots of
    # one head; 64 x 8 (sequence, head) pairs of 782 slots (49 passes) take 8
    # blocks of 7 passes (112 slots) each -> 7 blocks cover them
    assert skv.speechkv_pool_kv_bwd_workspace_bytes(64, 782, 8, 128) == 64 * 7 * 8 * 128 * 4
    # 8 x 8 pairs of 1596 slots (100 passes): 64 blocks of 2 passes (32 slots) -> 50 blocks
    assert skv.speechkv_pool_kv_bwd_workspace_bytes(8, 1596, 8, 128) == 8 * 50 * 8 * 128 * 4
    assert skv.speechkv_pool_kv_bwd_workspace_bytes(2, 0, 8, 128) == 2 * 1 * 8 * 128 * 4
    # any head count: 60 slots take 4 one-pass blocks per pair
    assert skv.speechkv_pool_kv_bwd_workspace_bytes(2, 60, 3, 128) == 2 * 4 * 3 * 128 * 4
    # at head_dim 64 a pass covers 32 slots
    assert skv.speechkv_pool_kv_bwd_workspace_bytes(2, 60, 2, 64) == 2 * 2 * 2 * 64 * 4
    assert skv.speechkv_pool_kv_bwd_workspace_bytes(2, 60, 8, 96) == 0


def pool_bwd(s=None, **kw):
    a = dict(k=RAW, v=RAW + (1 << 22), sb=60 * 2 * 64, ss=2 * 64, sh=64, batch=2, raw_len=60, heads=2,
             hd=64, dtype=skv.DTYPE_BF16, w=4, gate=None, layer=1, l0=0, dk=FAKE + (23 << 24),
             dv=FAKE + (24 << 24), cap=60, dkr=FAKE + (25 << 24), dvr=FAKE + (26 << 24), du=None,
             ws=None, ws_bytes=0)
    a.update(kw)
    s = s or spans()
    return lib.speechkv_pool_kv_bwd(a["k"], a["v"], a["sb"], a["ss"], a["sh"], a["batch"], a["raw_len"],
                                    a["heads"], a["hd"], a["dtype"], ctypes.byref(s), a["w"], a["gate"],
                                    a["layer"], a["l0"], a["dk"], a["dv"], a["cap"], a["dkr"], a["dvr"],
                                    a["du"], a["ws"], a["ws_bytes"], None)


@pytest.mark.parametrize("kw,code", [
    (dict(k=None), E_ARG), (dict(dk=None), E_ARG), (dict(dkr=None), E_ARG), (dict(dvr=None), E_ARG),
    (dict(dtype=7), E_UNS), (dict(hd=96), E_UNS), (dict(heads=65536), E_UNS),
    (dict(heads=0), E_ARG), (dict(batch=0), E_ARG), (dict(raw_len=50), E_ARG), (dict(w=0), E_ARG),
    (dict(w=skv.MAX_WINDOW + 1), E_ARG), (dict(cap=0), E_ARG), (dict(layer=-1), E_ARG),
    (dict(sb=-8), E_ARG), (dict(ss=3), E_ARG), (dict(dkr=FAKE + (25 << 24) + 4), E_ARG),
    (dict(gate=FAKE + 4), E_ARG), (dict(du=FAKE + (27 << 24)), E_WS),
    (dict(du=FAKE + (27 << 24), ws=FAKE + (28 << 24), ws_bytes=64), E_WS),
    (dict(dkr=RAW), E_ALIAS), (dict(dvr=FAKE + (25 << 24) + 1024), E_ALIAS),
    (dict(dkr=FAKE + (23 << 24) + 2048), E_ALIAS),
])
def test_pool_bwd_rejects(kw, code):
    assert pool_bwd(**kw) == code


# ----------------------------------------------------------- segment tables

def test_compressed_len_segments_agrees_with_oracle():
    from oracle import segments as seg
    cases = [[], [(0, 0)], [(32, 375), (24, 250), (16, 500), (64, 0)], [(3, 1), (0, 7), (5, 0)],
             [(0, 9)] * 5]
    for segs in cases:
        for w in (1, 2, 3, 4, 8):
            for layer, l0 in ((0, 0), (3, 5), (14, 14)):
                assert skv.speechkv_compressed_len_segments(segs, w, layer, l0) == \
                    seg.compressed_len(segs, w, layer, l0)
    assert skv.speechkv_compressed_len_segments([(1, -1)], 4, 0, 0) == -1
    assert skv.speechkv_compressed_len_segments([(1, 1)], 0, 0, 0) == -1


SEG = FAKE + (25 << 24)


def segments(**kw):
    g = dict(seg_start=SEG, text_len=SEG + 256, speech_len=SEG + 512, num_segments=6,
             max_segments=3, max_total_len=60)
    g.update(kw)
    return skv._Segments(**g)


def pool_seg(c=None, g=None, **kw):
    a = dict(k=RAW, v=RAW + (1 << 22), sb=60 * 2 * 64, ss=2 * 64, sh=64, batch=2, raw_len=60, w=4,
             gate=None, layer=1, l0=0, clen=None)
    a.update(kw)
    c = c or cache()
    g = g or segments()
    return lib.speechkv_pool_kv_segments(a["k"], a["v"], a["sb"], a["ss"], a["sh"], a["batch"],
                                         a["raw_len"], ctypes.byref(g), a["w"], a["gate"], a["layer"],
                                         a["l0"], ctypes.byref(c), a["clen"], None)


def prefill_seg(c=None, g=None, **kw):
    a = dict(q=FAKE + (12 << 24), batch=2, hq=4, q_len=60, w=4, layer=1, l0=0, mode=0,
             scale=0.125, out=FAKE + (13 << 24), lse=None)
    a.update(kw)
    c = c or cache()
    g = g or segments()
    return lib.speechkv_prefill_attn_segments(a["q"], a["batch"], a["hq"], a["q_len"],
                                              ctypes.byref(c), ctypes.byref(g), a["w"], a["layer"],
                                              a["l0"], a["mode"], a["scale"], a["out"], a["lse"],
                                              None)


@pytest.mark.parametrize("gkw", [dict(seg_start=None), dict(text_len=None), dict(speech_len=None),
                                 dict(num_segments=-1), dict(max_segments=-1),
                                 dict(max_segments=skv.MAX_SEGMENTS + 1), dict(max_total_len=-1)])
def test_segment_tables_rejected(gkw):
    assert pool_seg(g=segments(**gkw)) == E_ARG
    assert prefill_seg(g=segments(**gkw)) == E_ARG


@pytest.mark.parametrize("kw,code", [
    (dict(k=None), E_ARG), (dict(batch=0), E_ARG), (dict(raw_len=59), E_ARG), (dict(w=0), E_ARG),
    (dict(w=skv.MAX_WINDOW + 1), E_ARG), (dict(layer=-1), E_ARG), (dict(ss=3), E_ARG),
    (dict(gate=FAKE + 4), E_ARG), (dict(k=FAKE), E_ALIAS),
])
def test_pool_segments_rejects(kw, code):
    assert pool_seg(**kw) == code


@pytest.mark.parametrize("kw,code", [
    (dict(q=None), E_ARG), (dict(out=None), E_ARG), (dict(q_len=59), E_ARG), (dict(mode=2), E_ARG),
    (dict(w=0), E_ARG), (dict(hq=6), E_UNS), (dict(hq=5), E_ARG), (dict(lse=FAKE + 2), E_ARG),
    (dict(scale=0.0), E_ARG), (dict(batch=0), E_ARG),
])
def test_prefill_segments_rejects(kw, code):
    assert prefill_seg(**kw) == code


def test_segment_calls_check_the_cache():
    assert pool_seg(c=cache(head_dim=96)) == E_UNS
    assert prefill_seg(c=cache(dtype=7)) == E_UNS
    assert pool_seg(c=cache(k_pages=None)) == E_ARG


def test_backward_segment_calls_check_their_tables():
    g = segments(seg_start=None)
    ws = FAKE + (22 << 24)
    st = lib.speechkv_prefill_attn_bwd_segments(FAKE + (15 << 24), 2, 4, 60, ctypes.byref(cache()),
                                                ctypes.byref(g), 4, 1, 0, 0, 0.125, FAKE + (16 << 24),
                                                FAKE + (17 << 24), FAKE + (18 << 24), FAKE + (19 << 24),
                                                FAKE + (20 << 24), FAKE + (21 << 24), 60, ws, 1 << 20,
                                                None)
    assert st == E_ARG
    st = lib.speechkv_pool_kv_bwd_segments(RAW, RAW + (1 << 22), 60 * 2 * 64, 2 * 64, 64, 2, 60, 2, 64,
                                           skv.DTYPE_BF16, ctypes.byref(segments(max_segments=-1)), 4,
                                           None, 1, 0, FAKE + (20 << 24), FAKE + (21 << 24), 60,
                                           FAKE + (26 << 24), FAKE + (27 << 24), None, None, 0, None)
    assert st == E_ARG
    # a valid table with a broken cache or window is still rejected
    st = lib.speechkv_prefill_attn_bwd_segments(FAKE + (15 << 24), 2, 4, 60,
                                                ctypes.byref(cache(head_dim=96)),
                                                ctypes.byref(segments()), 4, 1, 0, 0, 0.125,
                                                FAKE + (16 << 24), FAKE + (17 << 24), FAKE + (18 << 24),
                                                FAKE + (19 << 24), FAKE + (20 << 24), FAKE + (21 << 24),
                                                60, ws, 1 << 20, None)
    assert st == E_UNS
    st = lib.speechkv_pool_kv_bwd_segments(RAW, RAW + (1 << 22), 60 * 2 * 64, 2 * 64, 64, 2, 60, 2, 64,
                                           skv.DTYPE_BF16, ctypes.byref(segments()), 0, None, 1, 0,
                                           FAKE + (20 << 24), FAKE + (21 << 24), 60, FAKE + (26 << 24),
                                           FAKE + (27 << 24), None, None, 0, None)
    assert st == E_ARG


# ------------------------------------------------ valid calls pass validation

NO_GPU = pytest.mark.skipif(__import__("torch").cuda.device_count() > 0,
                            reason="valid calls would launch kernels on the fake pointers")


@NO_GPU
def test_valid_calls_pass_every_check():
    """Valid arguments (the fake, non-overlapping layout above) get past every
    host check, so on a machine without a GPU the call fails only at the
    device (HIP error).  This guards the overlap checks against flagging a
    legitimate call, e.g. decode reading and writing the same page pools when
    it stores the new token."""
    E_HIP = skv.ERR_HIP
    assert decode() == E_HIP
    assert decode(kn=KN, vn=VN) == E_HIP
    assert decode(kn=KN, vn=VN, splits=4, ws=WS, ws_bytes=1 << 20) == E_HIP
    assert decode_noalloc() == E_HIP
    assert decode_noalloc(kn=KN, vn=VN, splits=4) == E_HIP
    assert prefill() == E_HIP and prefill(lse=FAKE + (20 << 24)) == E_HIP
    assert prefill_seg() == E_HIP
    assert pool() == E_HIP and pool(clen=FAKE + (20 << 24), gate=FAKE + (21 << 24)) == E_HIP
    assert pool_seg() == E_HIP
    assert fused() == E_HIP
    assert prefill_bwd() == E_HIP
    assert pool_bwd() == E_HIP
    assert pool_hidden() == E_HIP


def descriptions():
    """A cache, one-run spans and a segment table on the host, for the
    binding's own checks (nothing is launched on these paths)."""
    import torch
    i32 = lambda *n: torch.zeros(*n, dtype=torch.int32)  # noqa: E731
    pages = torch.zeros(4, 2, 16, 64, dtype=torch.bfloat16)
    return dict(cache=skv.PagedKV(pages, pages.clone(), i32(1, 4)),
                spans=skv.Spans(i32(1), i32(1), i32(1), 0, 8),
                segs=skv.Segments(i32(2), i32(3), i32(3), 3, 8))


def binding_calls(d, where, cache):
    """Every call of the binding that takes a description, with the segment
    table's object in `where["segs"]` and the one-run spans' in `where["spans"]`."""
    import torch
    z = lambda *n, t=torch.bfloat16: torch.zeros(*n, dtype=t)  # noqa: E731
    raw, q, lse, hat = z(1, 8, 2, 64), z(1, 8, 4, 64), z(1, 4, 8, t=torch.float32), z(1, 8, 2, 64, t=torch.float32)
    ws, gate = z(4096, t=torch.uint8), None
    one, seg = where["spans"], where["segs"]
    bwd = lambda f, w: f(q, cache, w, 4, 1, 0, q.clone(), lse, q.clone(), q.clone(), hat, hat.clone(), ws, stream=0)  # noqa: E731,E501
    pbwd = lambda f, w: f(raw, raw.clone(), w, 4, gate, 1, 0, hat, hat.clone(), raw.clone(), raw.clone(), stream=0)  # noqa: E731,E501
    return {
        "pool_kv": lambda: skv.speechkv_pool_kv(raw, raw, one, 4, gate, 1, 0, cache, stream=0),
        "pool_kv_segments": lambda: skv.speechkv_pool_kv_segments(raw, raw, seg, 4, gate, 1, 0, cache, stream=0),
        "prefill_attn": lambda: skv.speechkv_prefill_attn(q, cache, one, 4, 1, 0, q.clone(), stream=0),
        "prefill_attn_segments": lambda: skv.speechkv_prefill_attn_segments(q, cache, seg, 4, 1, 0, q.clone(), stream=0),
        "pool_prefill_attn": lambda: skv.speechkv_pool_prefill_attn(q, raw, raw, one, 4, gate, 1, 0, cache, q.clone(), stream=0),
        "prefill_attn_bwd": lambda: bwd(skv.speechkv_prefill_attn_bwd, one),
        "prefill_attn_bwd_segments": lambda: bwd(skv.speechkv_prefill_attn_bwd_segments, seg),
        "pool_kv_bwd": lambda: pbwd(skv.speechkv_pool_kv_bwd, one),
        "pool_kv_bwd_segments": lambda: pbwd(skv.speechkv_pool_kv_bwd_segments, seg),
        "pool_hidden": lambda: skv.speechkv_pool_hidden(z(1, 8, 128), one, 4, gate, z(1, 8, 128), stream=0),
        "decode_attn": lambda: skv.speechkv_decode_attn(q[:, 0].contiguous(), cache, z(1, t=torch.int32), 8,
                                                        q[:, 1].contiguous(), stream=0),
        "decode_attn_noalloc": lambda: skv.speechkv_decode_attn_noalloc(
            q[:, 0].contiguous(), cache, z(1, t=torch.int32), 8, q[:, 1].contiguous(), stream=0),
    }


ONE_RUN_CALLS = ("pool_kv", "prefill_attn", "pool_prefill_attn", "prefill_attn_bwd", "pool_kv_bwd", "pool_hidden")
SEGMENT_CALLS = ("pool_kv_segments", "prefill_attn_segments", "prefill_attn_bwd_segments", "pool_kv_bwd_segments")
CACHE_CALLS = ("pool_kv", "pool_kv_segments", "prefill_attn", "prefill_attn_segments", "pool_prefill_attn",
               "prefill_attn_bwd", "prefill_attn_bwd_segments", "decode_attn", "decode_attn_noalloc")


@pytest.mark.parametrize("call,given", [(c, g) for c in ONE_RUN_CALLS for g in ("segs", "cache")] +
                         [(c, g) for c in SEGMENT_CALLS for g in ("spans", "cache")])
def test_binding_refuses_the_other_kind_of_span_description(call, given):
    """The descriptions have different layouts: one taken for another would
    have the library read lengths where it expects pointers."""
    d = descriptions()
    calls = binding_calls(d, dict(spans=d[given], segs=d[given]), d["cache"])
    with pytest.raises(TypeError):
        calls[call]()


@pytest.mark.parametrize("call", CACHE_CALLS)
@pytest.mark.parametrize("given", ["spans", "segs"])
def test_binding_refuses_spans_for_a_cache(call, given):
    d = descriptions()
    with pytest.raises(TypeError):
        binding_calls(d, d, d[given])[call]()


@pytest.mark.parametrize("name,pack,struct", [("cache", "_paged_kv", skv._PagedKV), ("spans", "_spans", skv._Spans),
                                              ("segs", "_segments", skv._Segments)])
def test_packed_descriptions_fill_their_c_structures(name, pack, struct):
    """The bytes the library is handed are as long as the structure it reads,
    and read back field by field as what the object holds."""
    x = descriptions()[name]
    packed = getattr(x, pack)()
    assert len(packed) == ctypes.sizeof(struct)
    c = struct.from_buffer_copy(packed)
    if name == "cache":
        want = dict(k_pages=x.k_pages.data_ptr(), v_pages=x.v_pages.data_ptr(),
                    block_table=x.block_table.data_ptr(), num_pages=4, page_size=16, max_pages_per_seq=4,
                    num_kv_heads=2, head_dim=64, dtype=skv.DTYPE_BF16)
    elif name == "spans":
        want = dict(prefix_len=x.prefix_len.data_ptr(), speech_len=x.speech_len.data_ptr(),
                    suffix_len=x.suffix_len.data_ptr(), max_speech_len=0, max_total_len=8)
    else:
        want = dict(seg_start=x.seg_start.data_ptr(), text_len=x.text_len.data_ptr(),
                    speech_len=x.speech_len.data_ptr(), num_segments=3, max_segments=3, max_total_len=8)
    assert {f: getattr(c, f) for f, _ in struct._fields_} == want


@pytest.mark.parametrize("bound", [2**31, 2**32 + 8, -1, -2**31 - 1, -2**32 + 8])
@pytest.mark.parametrize("call", ONE_RUN_CALLS + SEGMENT_CALLS)
def test_binding_refuses_bounds_the_library_cannot_hold(call, bound):
    """A row bound outside int32 is the library's invalid argument, whatever
    its low 32 bits are (8 here is a valid bound)."""
    d = descriptions()
    d["spans"].max_total_len = d["segs"].max_total_len = bound
    with pytest.raises(skv.SpeechKVError) as e:
        binding_calls(d, d, d["cache"])[call]()
    assert e.value.status == skv.ERR_INVALID_ARG


@pytest.mark.parametrize("call", ONE_RUN_CALLS + SEGMENT_CALLS)
def test_binding_takes_integers_only_as_bounds(call):
    d = descriptions()
    d["spans"].max_total_len = d["segs"].max_total_len = 8.0
    with pytest.raises(TypeError):
        binding_calls(d, d, d["cache"])[call]()
