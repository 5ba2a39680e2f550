"""GPU parity for sequences with several speech runs (segment tables): the
pooling into the paged cache and the prefill attention, through the C ABI,
against the fp64 multi-run oracle (oracle/segments.py), on adversarial
shapes (empty segments, runs shorter than w, ragged last windows, text-only
and speech-only sequences, many segments) and a multi-turn workload; then
the training backward of both (attention, then pooling down to the raw K/V
and the gate) against the oracle's backward.  A table holding one run per
sequence must give the bits of the one-run calls, forward and backward.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from oracle import segments as seg
from gpu_case import launches
from helpers import GRAD_TOL, TOL, f64, fwd_err, gather, grad_err
from paper_2607_06827_amd import inputs
from paper_2607_06827_amd import speechkv as skv

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def build(segs, Hq=4, Hkv=2, D=64, dtype="bf16", page_size=16, w=4, layer=1, l0=0, seed=0,
          zero_gate=False):
    B = len(segs)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rows = [seg.raw_len(s) for s in segs]
    S = max(max(rows), 1)
    s0 = 5000 + seed * 10
    x = dict(B=B, S=S, dt=dt, rows=rows)
    x["k"] = inputs.normal((B, S, Hkv, D), s0 + 1, dtype=dt)
    x["v"] = inputs.normal((B, S, Hkv, D), s0 + 2, dtype=dt)
    x["u"] = None if zero_gate else inputs.normal((Hkv, D), s0 + 3, scale=1 / math.sqrt(D))
    x["q"] = inputs.normal((B, S, Hq, D), s0 + 4, dtype=dt)
    x["clen"] = [seg.compressed_len(s, w, layer, l0) for s in segs]
    pages = max(1, -(-max(max(x["clen"]), 1) // page_size))
    table, total = inputs.block_table(B, pages, seed, shuffle=True, spare_pages=2)
    nan = lambda: torch.full((total, Hkv, page_size, D), float("nan"), dtype=dt, device="cuda")
    x["cache"] = skv.PagedKV(nan(), nan(), table.cuda())
    x["segs"] = skv.Segments.from_lists(segs)
    return x


def run_segments(x, segs, w, layer, l0, mode):
    dev = torch.device("cuda")
    B, S = x["B"], x["S"]
    Hq, D = x["q"].shape[2], x["q"].shape[3]
    clen = torch.full((B,), -7, dtype=torch.int32, device=dev)
    u = None if x["u"] is None else x["u"].cuda()
    skv.speechkv_pool_kv_segments(x["k"].cuda(), x["v"].cuda(), x["segs"], w, u, layer, l0,
                                  x["cache"], clen)
    out = torch.full((B, S, Hq, D), float("nan"), dtype=x["dt"], device=dev)
    lse = torch.full((B, Hq, S), float("nan"), dtype=torch.float32, device=dev)
    skv.speechkv_prefill_attn_segments(x["q"].cuda(), x["cache"], x["segs"], w, layer, l0, out,
                                       mask_mode=mode, scale=D ** -0.5, lse=lse)
    torch.cuda.synchronize()
    return clen.cpu().tolist(), out, lse


def check(segs, w=4, layer=1, l0=0, mode=0, **kw):
    x = build(segs, w=w, layer=layer, l0=l0, **kw)
    clen, out, lse = run_segments(x, segs, w, layer, l0, mode)
    assert clen == x["clen"]
    dts = "bf16" if x["dt"] == torch.bfloat16 else "f32"
    tol = TOL[dts]
    u64 = None if x["u"] is None else f64(x["u"])
    kh, vh, oclen = seg.pool(f64(x["k"]), f64(x["v"]), segs, w, layer, l0, u64)
    assert oclen.tolist() == x["clen"]
    D = x["q"].shape[3]
    ref, ref_lse = seg.attention(f64(x["q"]), kh, vh, segs, w, layer, l0, mode, D ** -0.5)
    errs = {}
    for b, s in enumerate(segs):
        L, R = x["clen"][b], x["rows"][b]
        if L:
            gk, gv = gather(x["cache"], b, L)
            errs[f"pool_k[{b}]"] = fwd_err(f64(gk), kh[b, :L], dts)
            errs[f"pool_v[{b}]"] = fwd_err(f64(gv), vh[b, :L], dts)
            # text rows are copies, bit for bit
            slots, _ = seg.layout(s, w if layer >= l0 else 1)
            for c, (first, n, _, _) in enumerate(slots):
                if n == 1:
                    assert torch.equal(gk[c].cpu(), x["k"][b, first])
        if R:
            go = f64(out[b, :R])
            assert np.all(np.isfinite(go))
            errs[f"prefill[{b}]"] = fwd_err(go, ref[b, :R], dts)
            gl, rl = f64(lse[b, :, :R]), ref_lse[b, :, :R]
            assert np.array_equal(np.isneginf(gl), np.isneginf(rl))
            fin = np.isfinite(rl)
            if fin.any():
                errs[f"lse[{b}]"] = float(np.max(np.abs(gl[fin] - rl[fin])))
        if R < x["S"]:
            assert torch.isnan(out[b, R:]).all()
    bad = {k: e for k, e in errs.items() if not e <= tol}
    assert not bad, f"{segs}: above {tol}: {bad}"
    return x, clen, out, lse


CASES = {
    "three-turns": dict(segs=[[(8, 60), (5, 33), (6, 0)]], D=128),
    "turns-varlen": dict(segs=[[(4, 17), (2, 9), (0, 30), (7, 0)], [(0, 41)], [(3, 0)],
                               [(1, 2), (1, 3), (1, 5), (1, 7), (2, 0)]]),
    "empty-and-zero-segments": dict(segs=[[], [(0, 0), (0, 0)], [(0, 0), (5, 12), (0, 0), (0, 3)]]),
    "runs-shorter-than-w": dict(segs=[[(2, 3), (1, 2), (4, 1), (2, 0)]], w=8),
    "speech-first-rows-see-nothing": dict(segs=[[(0, 30), (4, 25)], [(0, 7), (0, 9), (3, 0)]]),
    "window-start-mask": dict(segs=[[(3, 41), (2, 30), (7, 0)], [(9, 30), (1, 1)]], mode=1),
    "identity-below-l0": dict(segs=[[(6, 50), (3, 20), (4, 0)]], layer=2, l0=5),
    "w1": dict(segs=[[(6, 50), (3, 20), (4, 0)]], w=1),
    "w16": dict(segs=[[(3, 200), (5, 77), (2, 0)]], w=16, D=128),
    "many-segments": dict(segs=[[(2, 5)] * 40 + [(6, 0)], [(1, 11)] * 25]),
    "g8-d128": dict(segs=[[(4, 90), (3, 80), (3, 0)]], Hq=8, Hkv=1, D=128),
    "g1": dict(segs=[[(4, 90), (3, 80), (3, 0)]], Hq=2, Hkv=2, D=128),
    "fp32": dict(segs=[[(8, 60), (5, 33), (6, 0)], [(0, 17), (2, 0)]], dtype="f32"),
    "fp32-d128-g4": dict(segs=[[(8, 160), (5, 33), (6, 0)]], dtype="f32", D=128, Hq=8, Hkv=2),
    "page8": dict(segs=[[(5, 77), (2, 30), (1, 0)], [(2, 64), (6, 1)]], page_size=8),
    "zero-gate": dict(segs=[[(4, 70), (3, 21), (3, 0)]], zero_gate=True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_segments_match_oracle(name):
    print(f"case {name}", flush=True)
    kw = dict(CASES[name])
    check(kw.pop("segs"), **kw)


@pytest.mark.parametrize("dtype,D,mode", [("bf16", 128, 0), ("bf16", 64, 1), ("f32", 64, 0)])
def test_one_run_table_equals_one_run_calls(dtype, D, mode):
    """{(P, T), (N, 0)} per sequence gives the bits of the one-run calls."""
    P, T, N, w = [8, 0, 5], [60, 37, 0], [5, 3, 9], 4
    segs = [[(p, t), (n, 0)] for p, t, n in zip(P, T, N)]
    x = build(segs, D=D, dtype=dtype, Hq=8, Hkv=2, w=w)
    clen_s, out_s, lse_s = run_segments(x, segs, w, 1, 0, mode)
    B, S = x["B"], x["S"]
    cache = skv.PagedKV(torch.full_like(x["cache"].k_pages, float("nan")),
                        torch.full_like(x["cache"].v_pages, float("nan")), x["cache"].block_table)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    spans = skv.Spans(i32(P), i32(T), i32(N), max(T), max(p + t + n for p, t, n in zip(P, T, N)))
    clen = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    u = x["u"].cuda()
    skv.speechkv_pool_kv(x["k"].cuda(), x["v"].cuda(), spans, w, u, 1, 0, cache, clen)
    out = torch.full_like(out_s, float("nan"))
    lse = torch.full_like(lse_s, float("nan"))
    skv.speechkv_prefill_attn(x["q"].cuda(), cache, spans, w, 1, 0, out, mask_mode=mode,
                              scale=D ** -0.5, lse=lse)
    torch.cuda.synchronize()
    assert clen.cpu().tolist() == clen_s
    for b in range(B):
        L, R = clen_s[b], x["rows"][b]
        ka, va = gather(x["cache"], b, L)
        kb, vb = gather(cache, b, L)
        assert torch.equal(ka, kb) and torch.equal(va, vb)
        assert torch.equal(out_s[b, :R], out[b, :R])
        fin = torch.isfinite(lse_s[b, :, :R])
        assert torch.equal(fin, torch.isfinite(lse[b, :, :R]))
        assert torch.equal(lse_s[b, :, :R][fin], lse[b, :, :R][fin])


def test_decode_after_segment_pooling():
    """Decoding needs only the cache length: after the multi-run pooling a
    decode step attends over exactly the pooled rows and the new token."""
    segs = [[(8, 60), (5, 33), (6, 0)], [(0, 17), (2, 40)]]
    x, clen, _, _ = check(segs, D=128, Hq=8, Hkv=2)
    B, Hq, Hkv, D = 2, 8, 2, 128
    q = inputs.normal((B, Hq, D), 5101, dtype=x["dt"])
    kn = inputs.normal((B, Hkv, D), 5102, dtype=x["dt"])
    vn = inputs.normal((B, Hkv, D), 5103, dtype=x["dt"])
    lens = [c + 1 for c in clen]
    out = torch.empty(B, Hq, D, dtype=x["dt"], device="cuda")
    ws_bytes = skv.speechkv_decode_workspace_bytes(B, Hq, Hkv, D, max(lens), 0)
    ws = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda")
    skv.speechkv_decode_attn(q.cuda(), x["cache"], torch.tensor(lens, dtype=torch.int32).cuda(),
                             max(lens), out, k_new=kn.cuda(), v_new=vn.cuda(), scale=D ** -0.5,
                             workspace=ws)
    torch.cuda.synchronize()
    kh, vh, _ = seg.pool(f64(x["k"]), f64(x["v"]), segs, 4, 1, 0, f64(x["u"]))
    K = np.zeros((B, max(lens), Hkv, D))
    V = np.zeros((B, max(lens), Hkv, D))
    for b in range(B):
        K[b, :clen[b]] = kh[b, :clen[b]]
        V[b, :clen[b]] = vh[b, :clen[b]]
        K[b, clen[b]] = f64(kn[b])
        V[b, clen[b]] = f64(vn[b])
    ref, _ = oracle.decode(f64(q), K, V, lens, D ** -0.5)
    assert fwd_err(f64(out), ref, "bf16") <= TOL["bf16"]


def test_multi_turn_workload():
    """A multi-turn batch at full size: 16 sequences of three speech turns
    (30 s, 20 s and 40 s of 80 ms frames) between text, 16/8 heads, d=128,
    every pooled row and prefill output against the oracle."""
    turns = [(32, 375), (24, 250), (16, 500), (64, 0)]
    segs = [list(turns) for _ in range(16)]
    segs[3] = [(32, 375), (64, 0)]          # one turn only
    segs[7] = [(0, 500), (24, 250), (8, 0)]  # speech first
    check(segs, Hq=16, Hkv=8, D=128, seed=3)


# ------------------------------------------------------------------ backward

BWD_CASES = {
    "three-turns-d128": dict(segs=[[(8, 60), (5, 33), (6, 0)], [(0, 41), (2, 9)]], D=128),
    "turns-varlen-g4": dict(segs=[[(4, 17), (2, 9), (0, 30), (7, 0)], [(1, 2), (1, 3), (1, 5), (2, 0)]],
                            Hq=8, Hkv=2, D=128),
    "window-start-w5": dict(segs=[[(3, 41), (2, 30), (7, 0)]], mode=1, w=5, D=64),
    "w16": dict(segs=[[(3, 70), (5, 37), (2, 0)]], w=16, D=128),
    "fp32": dict(segs=[[(8, 60), (5, 33), (6, 0)], [(0, 17), (2, 0)]], dtype="f32"),
    "identity-below-l0": dict(segs=[[(6, 50), (3, 20), (4, 0)]], layer=2, l0=5, D=128),
}


def run_backward(segs, w=4, layer=1, l0=0, mode=0, **kw):
    x = build(segs, w=w, layer=layer, l0=l0, **kw)
    clen, out, lse = run_segments(x, segs, w, layer, l0, mode)
    B, S = x["B"], x["S"]
    Hq, D = x["q"].shape[2], x["q"].shape[3]
    Hkv = x["k"].shape[2]
    dev = torch.device("cuda")
    dout = inputs.normal((B, S, Hq, D), 5200, dtype=x["dt"]).to(dev)
    for b, R in enumerate(x["rows"]):
        dout[b, R:] = 0
    cap = max(clen) + 2
    dq = torch.full_like(out, float("nan"))
    dkh = torch.full((B, cap, Hkv, D), float("nan"), dtype=torch.float32, device=dev)
    dvh = torch.full_like(dkh, float("nan"))
    ws = torch.empty(skv.speechkv_prefill_attn_bwd_workspace_bytes(B, Hq, S), dtype=torch.uint8,
                     device=dev)
    skv.speechkv_prefill_attn_bwd_segments(x["q"].cuda(), x["cache"], x["segs"], w, layer, l0, out,
                                           lse, dout, dq, dkh, dvh, ws, mask_mode=mode,
                                           scale=D ** -0.5)
    k, v = x["k"].cuda(), x["v"].cuda()
    dkr = torch.full_like(k, float("nan"))
    dvr = torch.full_like(v, float("nan"))
    du = torch.full((Hkv, D), float("nan"), dtype=torch.float32, device=dev)
    nb = skv.speechkv_pool_kv_bwd_workspace_bytes(B, x["segs"].max_total_len, Hkv, D)
    pws = torch.empty(max(nb, 16), dtype=torch.uint8, device=dev)
    u = None if x["u"] is None else x["u"].cuda()
    # the pooling backward from the attention's key gradients (rows past the
    # compressed lengths are zero: they reach no raw row)
    dkh_in, dvh_in = torch.nan_to_num(dkh, nan=0.0), torch.nan_to_num(dvh, nan=0.0)
    skv.speechkv_pool_kv_bwd_segments(k, v, x["segs"], w, u, layer, l0, dkh_in, dvh_in, dkr, dvr,
                                      du, pws)
    torch.cuda.synchronize()
    return x, clen, dout, dict(dq=dq, dkh=dkh, dvh=dvh, dkr=dkr, dvr=dvr, du=du, dkh_in=dkh_in,
                               dvh_in=dvh_in)


@pytest.mark.parametrize("name", sorted(BWD_CASES))
def test_segments_backward_matches_oracle(name):
    print(f"case {name}", flush=True)
    kw = dict(BWD_CASES[name])
    check_backward(kw.pop("segs"), **kw)


def check_backward(segs, **kw):
    """Both backward calls on segment tables against the multi-run oracle."""
    w, layer, l0, mode = kw.get("w", 4), kw.get("layer", 1), kw.get("l0", 0), kw.get("mode", 0)
    x, clen, dout, g = run_backward(segs, **kw)
    D = x["q"].shape[3]
    tol = GRAD_TOL["bf16" if x["dt"] == torch.bfloat16 else "f32"]
    # attention backward: the oracle on the GPU's cache rows (what the kernel reads)
    Lmax = max(max(clen), 1)
    kh = np.zeros((x["B"], Lmax) + tuple(x["k"].shape[2:]))
    vh = np.zeros_like(kh)
    for b, L in enumerate(clen):
        if L:
            gk, gv = gather(x["cache"], b, L)
            kh[b, :L], vh[b, :L] = f64(gk), f64(gv)
    rq, rk, rv = seg.attention_bwd(f64(x["q"]), kh, vh, segs, w, layer, l0, f64(dout), mode,
                                   D ** -0.5)
    for b, (L, R) in enumerate(zip(clen, x["rows"])):
        if R:
            assert grad_err(f64(g["dq"][b, :R]), rq[b, :R]) <= tol["dq"]
        if L:
            assert grad_err(f64(g["dkh"][b, :L]), rk[b, :L]) <= tol["dkv_hat"]
            assert grad_err(f64(g["dvh"][b, :L]), rv[b, :L]) <= tol["dkv_hat"]
    # pooling backward: the oracle on the same raw K/V, gate and fp32 key gradients
    u64 = None if x["u"] is None else f64(x["u"])
    pk, pv, pu = seg.pool_bwd(f64(x["k"]), f64(x["v"]), segs, w, layer, l0, u64,
                              f64(g["dkh_in"]), f64(g["dvh_in"]))
    for b, R in enumerate(x["rows"]):
        if R:
            assert grad_err(f64(g["dkr"][b, :R]), pk[b, :R]) <= tol["dkv_raw"]
            assert grad_err(f64(g["dvr"][b, :R]), pv[b, :R]) <= tol["dkv_raw"]
        if R < x["S"]:
            assert torch.isnan(g["dkr"][b, R:]).all()
    assert grad_err(f64(g["du"]), pu) <= tol["du"]


def _turns(B, a, t, n, step=4):
    """B sequences of two turns each around text, shorter by `step` frames from
    one to the next, and an empty one."""
    return [[(a, t - step * b), (b % 3, a + b), (n, 0)] for b in range(B - 1)] + [[]]


# the bf16 dK/dV kernel's shapes by threads a block (see test_gpu_bwd.py), with a
# segment table: (threads, segments, arguments)
DKDV_SHAPES = [
    (512, _turns(5, 60, 200, 9), dict(D=128, Hq=8, Hkv=2, mode=1)),
    (1024, _turns(5, 60, 200, 9), dict(D=64, Hq=8, Hkv=2, w=3)),
    (768, _turns(9, 110, 180, 20), dict(D=128, Hq=64, Hkv=16, mode=1, w=2)),
    (768, _turns(9, 110, 180, 20), dict(D=64, Hq=64, Hkv=16, w=2)),
    (256, _turns(10, 100, 40, 130, step=2), dict(D=128, Hq=16, Hkv=16, w=5)),
    (256, _turns(10, 100, 40, 130, step=2), dict(D=64, Hq=16, Hkv=16, mode=1, w=5)),
]


@pytest.mark.parametrize("threads,segs,kw", DKDV_SHAPES, ids=lambda x: str(x.get("D", "")) if isinstance(x, dict)
                         else str(x) if isinstance(x, int) else "")
def test_segments_backward_block_shapes(threads, segs, kw):
    print(f"{threads} threads: {kw}", flush=True)
    check_backward(segs, **kw)
    x, clen, dout, g = run_backward(segs, **kw)
    Hq, S = x["q"].shape[2], x["S"]
    q, lse = x["q"].cuda(), torch.zeros(x["B"], Hq, S, device="cuda")
    ws = torch.empty(skv.speechkv_prefill_attn_bwd_workspace_bytes(x["B"], Hq, S), dtype=torch.uint8, device="cuda")
    run = launches(lambda: skv.speechkv_prefill_attn_bwd_segments(
        q, x["cache"], x["segs"], kw.get("w", 4), 1, 0, dout, lse, dout, g["dq"], g["dkh"], g["dvh"], ws,
        mask_mode=kw.get("mode", 0)))
    assert run[-1][1] == threads, run


# the fp32 forward of shared K/V tiles (more than 512 row tiles of 128 / G rows at
# 64-wide heads, 256 at 128-wide), with a segment table
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_segments_f32_shared_tiles(D, G):
    Hkv, rows = 8, {1: 128, 2: 64, 4: 32, 8: 32}[G]
    B = (513 if D == 64 else 257) // (2 * Hkv) + 2
    n = rows + 17  # two row tiles for most sequences
    segs = [[(3 + b % 4, n // 3 + b % 5), (b % 3, n // 3), (n // 4, 0)] for b in range(B - 1)] + [[(2, 9)]]
    kw = dict(w=1 + G % 5, mode=G % 3 == 2, D=D, Hq=G * Hkv, Hkv=Hkv, dtype="f32", page_size=8 if G == 4 else 16)
    x, _, out, lse = check(segs, **kw)
    q = x["q"].cuda()
    run = launches(lambda: skv.speechkv_prefill_attn_segments(q, x["cache"], x["segs"], kw["w"], 1, 0, out,
                                                              mask_mode=kw["mode"], lse=lse))
    tiles = B * Hkv * -(-max(x["rows"]) // rows)
    assert tiles > (512 if D == 64 else 256) and run == [(tiles, 512 if G == 8 else 256)], run


def test_one_run_table_backward_equals_one_run_calls():
    """{(P, T), (N, 0)} per sequence: the backward calls give the bits of the
    one-run backward calls."""
    P, T, N, w = [8, 0, 5], [60, 37, 0], [5, 3, 9], 4
    segs = [[(p, t), (n, 0)] for p, t, n in zip(P, T, N)]
    x, clen, dout, g = run_backward(segs, D=128, Hq=8, Hkv=2)
    B, S = x["B"], x["S"]
    Hq, D, Hkv = 8, 128, 2
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    spans = skv.Spans(i32(P), i32(T), i32(N), max(T), max(p + t + n for p, t, n in zip(P, T, N)))
    out = torch.empty(B, S, Hq, D, dtype=x["dt"], device="cuda")
    lse = torch.empty(B, Hq, S, dtype=torch.float32, device="cuda")
    skv.speechkv_prefill_attn(x["q"].cuda(), x["cache"], spans, w, 1, 0, out, scale=D ** -0.5, lse=lse)
    dq = torch.full_like(out, float("nan"))
    dkh = torch.full_like(g["dkh"], float("nan"))
    dvh = torch.full_like(dkh, float("nan"))
    ws = torch.empty(skv.speechkv_prefill_attn_bwd_workspace_bytes(B, Hq, S), dtype=torch.uint8,
                     device="cuda")
    skv.speechkv_prefill_attn_bwd(x["q"].cuda(), x["cache"], spans, w, 1, 0, out, lse, dout, dq,
                                  dkh, dvh, ws, scale=D ** -0.5)
    k, v = x["k"].cuda(), x["v"].cuda()
    dkr, dvr = torch.full_like(k, float("nan")), torch.full_like(v, float("nan"))
    du = torch.empty(Hkv, D, dtype=torch.float32, device="cuda")
    nb = skv.speechkv_pool_kv_bwd_workspace_bytes(B, spans.max_total_len, Hkv, D)
    pws = torch.empty(max(nb, 16), dtype=torch.uint8, device="cuda")
    skv.speechkv_pool_kv_bwd(k, v, spans, w, x["u"].cuda(), 1, 0, g["dkh_in"], g["dvh_in"], dkr,
                             dvr, du, pws)
    torch.cuda.synchronize()
    for b in range(B):
        R, L = x["rows"][b], clen[b]
        assert torch.equal(dq[b, :R], g["dq"][b, :R])
        assert torch.equal(dkh[b, :L], g["dkh"][b, :L]) and torch.equal(dvh[b, :L], g["dvh"][b, :L])
        assert torch.equal(dkr[b, :R], g["dkr"][b, :R]) and torch.equal(dvr[b, :R], g["dvr"][b, :R])
    assert torch.equal(du, g["du"])
