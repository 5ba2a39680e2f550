"""GPU parity on small and adversarial shapes, through the C ABI.

Each case runs pool -> prefill -> decode steps and is compared with the fp64
oracle element by element (tests/gpu_case.py): pooled K/V, prefill outputs and
LSE, every decode output, and the bit-exact text copies and new-token writes.
Sizes span several tiles and a ragged tail while the oracle stays fast.
"""
import pytest
import torch

from gpu_case import Case, build, launches, run_and_check
from paper_2607_06827_amd import speechkv as skv

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

CASES = {
    # name: Case
    "basic-bf16": Case(P=[8], T=[60], N=[5], D=128, Hq=4, Hkv=2),
    "basic-f32": Case(P=[8], T=[60], N=[5], dtype="f32", D=64),
    "prefix-empty": Case(P=[0, 0], T=[37, 9], N=[3, 0], w=4),          # rows that see nothing
    "speech-shorter-than-w": Case(P=[5], T=[3], N=[4], w=8),
    "no-speech": Case(P=[7], T=[0], N=[6]),
    "no-suffix": Case(P=[4], T=[45], N=[0], w=6),                       # ragged last window
    "window-start-mask": Case(P=[3, 9], T=[41, 30], N=[2, 7], mode=1),
    "identity-below-l0": Case(P=[6], T=[50], N=[4], layer=2, l0=5),
    "w1": Case(P=[6], T=[50], N=[4], w=1),
    "varlen-batch": Case(P=[0, 17, 3, 40], T=[150, 7, 91, 0], N=[9, 33, 0, 1], w=3, D=128,
                         Hq=8, Hkv=2),
    "page8": Case(P=[5, 2], T=[77, 64], N=[6, 1], page_size=8),
    "page64-w5": Case(P=[5, 2], T=[77, 64], N=[6, 1], page_size=64, w=5),
    "identity-pages": Case(P=[9], T=[70], N=[3], shuffle=False),
    "g1": Case(P=[4], T=[70], N=[3], Hq=2, Hkv=2, D=128),
    "g4": Case(P=[4], T=[70], N=[3], Hq=8, Hkv=2, D=128),
    "g8": Case(P=[4], T=[70], N=[3], Hq=8, Hkv=1, D=128),
    "g8-f32-d64": Case(P=[4], T=[70], N=[3], Hq=16, Hkv=2, D=64, dtype="f32"),
    # bf16, 64-wide heads, group 8: half the waves of a prefill block load no
    # tile rows and wait only for their query rows
    "g8-bf16-d64": Case(P=[4, 9], T=[170, 61], N=[3, 12], Hq=16, Hkv=2, D=64),
    "zero-gate": Case(P=[4], T=[70], N=[3], zero_gate=True),
    "sharp-gate-and-queries": Case(P=[4, 1], T=[70, 33], N=[3, 2], gate_scale=10.0, q_scale=3.0,
                                   D=128),
    "long-split": Case(P=[32, 0], T=[1100, 700], N=[10, 0], D=128, Hq=16, Hkv=8, decode_steps=2),
    "forced-splits": Case(P=[32, 5], T=[500, 130], N=[10, 2], D=128, num_splits=7),
    "f32-d128-split": Case(P=[3], T=[400], N=[2], D=128, dtype="f32", num_splits=3),
    # decode's host bound well above every cache length: the batches requested
    # from the bound before the lengths arrive must not be reduced
    "loose-decode-bound": Case(P=[8, 0, 30], T=[300, 45, 9], N=[5, 3, 0], D=128, Hq=8, Hkv=2,
                               bound_slack=200),
    "loose-decode-bound-split": Case(P=[8, 2], T=[300, 45], N=[5, 3], D=128, num_splits=3,
                                     bound_slack=150),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_case_matches_oracle(name):
    print(f"case {name}", flush=True)
    run_and_check(CASES[name])


# fp32 prefill: the kernel of 16-row blocks (few row tiles) at the edges of its
# row and key tiles, with fewer and more key tiles than waves, and the kernel of
# shared tiles (more row tiles than 512, or 256 at 128-wide heads).
F32_EDGES = [1, 2, 15, 16, 17, 33, 63, 64, 65, 130]
F32_CASES = {
    "rows-d64": Case(P=F32_EDGES, T=[0] * 10, N=[0] * 10, D=64, Hq=2, Hkv=2, dtype="f32"),
    "rows-d128-g8": Case(P=[0] * 10, T=F32_EDGES, N=[0] * 10, w=2, D=128, Hq=8, Hkv=1, dtype="f32"),
    "page8-start-mask": Case(P=[3, 0], T=[120, 37], N=[2, 9], mode=1, D=128, Hq=4, Hkv=2,
                             page_size=8, dtype="f32"),
    "shared-d64": Case(P=[i % 5 for i in range(65)], T=[17 + i for i in range(65)],
                       N=[i % 3 for i in range(65)], D=64, Hq=8, Hkv=8, dtype="f32"),
    "shared-d128-g4": Case(P=[i % 4 for i in range(65)], T=[9 + i for i in range(65)],
                           N=[i % 3 for i in range(65)], D=128, Hq=8, Hkv=2, dtype="f32"),
}


@pytest.mark.parametrize("name", sorted(F32_CASES))
def test_f32_prefill_kernels_match_oracle(name):
    print(f"case {name}", flush=True)
    run_and_check(F32_CASES[name])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_f32_prefill_shared_tiles(D, G):
    """The kernel of shared tiles, for every group and head size: two row tiles
    for most sequences, an empty one, both masks, pages of 8 and 16, copied
    (group 8) and pooled keys."""
    Hkv, rows = 8, {1: 128, 2: 64, 4: 32, 8: 32}[G]
    B = (513 if D == 64 else 257) // (2 * Hkv) + 2
    n = rows + 19
    case = Case(P=[b % 7 for b in range(B - 1)] + [0], T=[n - 12 - b % 5 for b in range(B - 1)] + [0],
                N=[b % 6 for b in range(B - 1)] + [0], w=1 + G % 5, mode=G % 3 == 2, D=D, Hq=G * Hkv, Hkv=Hkv,
                dtype="f32", page_size=8 if G == 4 else 16, l0=5 if G == 8 else 0, decode_steps=1)
    run_and_check(case)
    x = build(case)
    q = x["q"].to(x["dev"])
    out = torch.empty_like(q)
    run = launches(lambda: skv.speechkv_prefill_attn(q, x["cache"], x["spans"], case.w, case.layer, case.l0, out,
                                                     mask_mode=case.mode))
    tiles = B * Hkv * -(-x["S"] // rows)
    assert tiles > (512 if D == 64 else 256) and run == [(tiles, 512 if G == 8 else 256)], run


@pytest.mark.parametrize("Hkv,D", [(1, 64), (1, 128), (520, 64), (260, 128)])
def test_f32_prefill_keeps_an_infinite_value_infinite(Hkv, D):
    """Rows that see an infinite value with a positive weight are infinite,
    not NaN: the unused keys of a tile must not meet their zero weight as 0 *
    infinity.  Key 4 is the last visible one of rows 4..44 (the window closes
    at row 44); few KV heads take the kernel of 16-row blocks, many the one of
    shared tiles."""
    case = Case(P=[5], T=[41], N=[0], w=64, Hq=Hkv, Hkv=Hkv, D=D, dtype="f32", decode_steps=1)
    x = build(case)
    x["v_raw"][:, 4] = float("inf")
    t, dev = x["t"], x["dev"]
    skv.speechkv_pool_kv(t(x["k_raw"]), t(x["v_raw"]), x["spans"], case.w, t(x["u"]), case.layer, case.l0,
                         x["cache"])
    out = torch.full((1, x["S"], Hkv, D), float("nan"), device=dev)
    skv.speechkv_prefill_attn(t(x["q"]), x["cache"], x["spans"], case.w, case.layer, case.l0, out)
    torch.cuda.synchronize()
    assert torch.isposinf(out[0, 4:45]).all()
