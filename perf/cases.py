"""The work this library is used for, as cases that can be timed and checked.

A case is one pass through the public calls of paper_2607_06827_amd.speechkv, as
a speech LLM's program makes them: a decoding step, the prefill of a layer
(pool, then attend), the training of a layer (forward and backward), or the
pooling of hidden states.  Frames are 80 ms, so 375 are 30 s of audio, 750 are
60 s and 7500 are 10 minutes; heads and sizes are those of the workloads in
paper_2607_06827_amd.inputs unless a case says otherwise.
"""
import math

import torch

from paper_2607_06827_amd import inputs, speechkv as skv

_END, _START = skv.MASK_WINDOW_END, skv.MASK_WINDOW_START


def _case(name, kind, **kw):
    c = dict(name=name, kind=kind, dtype="bf16", batch=1, q_heads=16, kv_heads=8, dim=128, w=4,
             layers=1, l0=0, prefix=32, frames=375, suffix=0, generated=0, ragged=False, turns="",
             page=16, mask="end")
    c.update(kw)
    return c


def listed():
    return [
        # one user listening to an answer about 30 s of audio: the smallest
        # call there is, one layer's attention for one new token
        _case("decode_one_user", "decode", generated=40),
        # a serving step: one token for 64 users with 60 s of audio each,
        # through all 28 layers, the last 14 of them compressed
        _case("decode_stack_60s", "decode", batch=64, layers=28, l0=14, frames=750, generated=64),
        # the prompt of 32 users with 30 s of audio, one compressed layer
        _case("prefill_30s", "prefill", batch=32),
        # the prompt of 64 users with 60 s of audio, one layer below l0 (a
        # copy into the cache, then plain causal attention)
        _case("prefill_60s_full", "prefill", batch=64, frames=750, l0=1),
        # two users with 10 minutes of audio and a text question after it
        _case("prefill_10min", "prefill", batch=2, frames=7500, suffix=48),
        # a serving batch of unequal prompts, up to 45 s, odd lengths, four
        # query heads per KV head, bigger pages, window visible at its start
        _case("prefill_ragged", "prefill", batch=24, q_heads=32, w=2, prefix=21, frames=563,
              suffix=37, ragged=True, page=64, mask="start"),
        # two minutes of audio between a prompt and a question, pooled on the
        # fly inside the attention call
        _case("fused_2min", "fused", batch=8, frames=1500, suffix=64),
        # a conversation with three speech turns (30, 20 and 40 s)
        _case("turns", "turns", batch=16, turns="32+375,24+250,16+500,64+0"),
        # training one compressed layer on two minutes of audio: forward with
        # its log-sum-exp, gradients down to the raw K/V and the gate
        _case("train_2min", "train", batch=8, frames=1500, suffix=64),
        # training on short conversations of odd lengths, 64-wide heads, w = 3
        _case("train_turns", "train_turns", batch=6, q_heads=16, kv_heads=4, dim=64, w=3,
              turns="17+201,9+88,31+342,23+0"),
        # training in fp32 (a reference run, or a small model)
        _case("train_f32", "train", dtype="f32", batch=4, q_heads=8, kv_heads=4, dim=64,
              prefix=8, frames=600, suffix=24),
        # HS compression of 64 sequences with 60 s of audio, hidden size 2048
        _case("hidden_60s", "hidden", batch=64, frames=750),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["decode", "decode", "prefill", "prefill", "fused", "turns", "train",
                           "train", "train_turns", "hidden"])
        kv = rng.choice([2, 4, 8])
        c = _case("", kind, kv_heads=kv, q_heads=kv * rng.choice([1, 2, 2, 4, 8]),
                  dim=rng.choice([64, 128, 128]), w=rng.choice([2, 3, 4, 4, 8]),
                  batch=_logint(rng, 1, 64), prefix=rng.randint(0, 64),
                  frames=_logint(rng, 30, 7500), suffix=rng.choice([0, rng.randint(1, 96)]),
                  page=rng.choice([16, 16, 32, 64]), mask=rng.choice(["end", "end", "start"]),
                  ragged=rng.random() < 0.4, l0=rng.choice([0, 0, 1]))
        del c["name"]
        if kind != "fused":
            c["dtype"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
        if kind == "decode":
            c["generated"] = rng.randint(1, 256)
            c["layers"] = rng.choice([1, 4, 28])
            c["l0"] = rng.randint(0, c["layers"])
        if kind in ("turns", "train_turns"):
            n = rng.randint(1, 6)
            c["turns"] = ",".join("%d+%d" % (rng.randint(1, 40), _logint(rng, 10, 900)) for _ in range(n)) + ",20+0"
            c["prefix"] = c["frames"] = c["suffix"] = 0
            c["l0"] = 0
        if kind in ("train", "train_turns"):
            c["l0"] = 0
        if kind == "hidden":
            hidden = rng.choice([512, 1024, 2048, 4096])
            c.update(dim=128, q_heads=hidden // 128, kv_heads=hidden // 128, l0=0)
        w = work(c)
        slow = 16 if c["dtype"] == "f32" else 1  # fp32 products run on the fp32 matrix units
        if w["bytes"] <= 2.5e9 and w["flops"] * slow <= 1.0e11:
            return c


# ---------------------------------------------------------------- the layout

def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _w_eff(case, layer):
    return case["w"] if layer >= case["l0"] else 1


def _sequences(case):
    """Per sequence its [(text rows, speech frames), ...]; a ragged batch holds
    sequences of 30% to 100% of the full length."""
    if case["turns"]:
        full = [tuple(int(v) for v in t.split("+")) for t in case["turns"].split(",")]
    else:
        full = [(case["prefix"], case["frames"]), (case["suffix"], 0)]
    out = []
    for b in range(case["batch"]):
        f = 1.0
        if case["ragged"] and b:
            f = 0.3 + 0.7 * ((b * 0.6180339887) % 1.0)
        out.append([(int(t * f), int(s * f)) for t, s in full])
    return out


def _rows(segs):
    return sum(t + s for t, s in segs)


def _clen(segs, w):
    return sum(t + -(-s // w) for t, s in segs)


def _layout(segs, w, mask):
    """(first raw row, rows, visible from) of every cache slot of a sequence."""
    slots, row = [], 0
    for text, speech in segs:
        slots += [(row + i, 1, row + i) for i in range(text)]
        row += text
        for i in range(0, speech, w):
            n = min(w, speech - i)
            slots.append((row + i, n, row + i if mask == "start" else row + i + n - 1))
        row += speech
    return slots


def _pairs(case, w):
    """(row, visible key) pairs over the batch."""
    total = 0
    for segs in _sequences(case):
        rows = _rows(segs)
        total += sum(rows - tau for _, _, tau in _layout(segs, w, case["mask"]))
    return total


# ------------------------------------------------------------------ preparing

class _Draws:
    """Independent N(0, 1) tensors of one seed, on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.host = torch.Generator()
        self.host.manual_seed(seed)

    def normal(self, shape, dtype, scale=1.0):
        x = torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)
        return (x * scale if scale != 1.0 else x).to(dtype)

    def raw(self, case, seqs, heads, dim):
        """Raw rows [B, S, heads, dim]: text rows independent, the frames of a
        speech run correlated from one to the next (0.9), as speech is."""
        S = max(_rows(s) for s in seqs)
        x = torch.randn((len(seqs), S, heads * dim), generator=self.g, device="cuda")
        same = all(s == seqs[0] for s in seqs)
        for b in ([slice(None)] if same else range(len(seqs))):
            row = 0
            for text, speech in (seqs[0] if same else seqs[b]):
                row += text
                if speech:
                    part = x[b, row:row + speech]
                    x[b, row:row + speech] = inputs.ar1(part if same else part[None], 0.9).view_as(part)
                row += speech
        return x.view(len(seqs), S, heads, dim).to(_dt(case))

    def pages(self, count):
        return torch.randperm(count, generator=self.host).to(torch.int32)


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def _spans(case, seqs):
    p, t, n = ([s[0][0] for s in seqs], [s[0][1] for s in seqs], [s[1][0] for s in seqs])
    return skv.Spans(_i32(p), _i32(t), _i32(n), max(t), max(_rows(s) for s in seqs))


def _cache(case, d, seqs, w):
    per = max(1, -(-max(_clen(s, w) for s in seqs) // case["page"]))
    total = per * case["batch"]
    shape = (total, case["kv_heads"], case["page"], case["dim"])
    k = torch.zeros(shape, dtype=_dt(case), device="cuda")
    return skv.PagedKV(k, torch.zeros_like(k), d.pages(total).view(case["batch"], per).cuda())


def _prepare_decode(case, d):
    B, Hq, Hkv, D, ps, dt = (case["batch"], case["q_heads"], case["kv_heads"], case["dim"],
                             case["page"], _dt(case))
    seqs = _sequences(case)
    lens = [[_clen(s, _w_eff(case, layer)) + case["generated"] for s in seqs]
            for layer in range(case["layers"])]
    per = [-(-max(x) // ps) for x in lens]
    # one pool of pages for every layer, as a serving engine's allocator keeps it
    total = B * sum(per)
    k_pages = torch.empty((total, Hkv, ps, D), dtype=dt, device="cuda").normal_(generator=d.g)
    v_pages = torch.empty_like(k_pages).normal_(generator=d.g)
    ids, at, steps = d.pages(total), 0, []
    need = 16
    for layer in range(case["layers"]):
        table = ids[at:at + B * per[layer]].view(B, per[layer]).cuda()
        at += B * per[layer]
        longest = max(lens[layer])
        need = max(need, skv.speechkv_decode_workspace_bytes(B, Hq, Hkv, D, longest))
        steps.append((skv.PagedKV(k_pages, v_pages, table), _i32(lens[layer]), longest))
    n = case["layers"]
    return dict(case=case, steps=steps, k_pages=k_pages, v_pages=v_pages,
                q=d.normal((n, B, Hq, D), dt), k_new=d.normal((n, B, Hkv, D), dt),
                v_new=d.normal((n, B, Hkv, D), dt),
                out=torch.empty((n, B, Hq, D), dtype=dt, device="cuda"),
                workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))


def _prepare_layer(case, d):
    B, Hq, Hkv, D, dt = case["batch"], case["q_heads"], case["kv_heads"], case["dim"], _dt(case)
    seqs = _sequences(case)
    w = _w_eff(case, 0)
    S = max(_rows(s) for s in seqs)
    s = dict(case=case, k_raw=d.raw(case, seqs, Hkv, D), v_raw=d.raw(case, seqs, Hkv, D),
             gate=d.normal((Hkv, D), torch.float32, D ** -0.5), q=d.normal((B, S, Hq, D), dt),
             cache=_cache(case, d, seqs, w), out=torch.zeros((B, S, Hq, D), dtype=dt, device="cuda"),
             cache_len=torch.zeros(B, dtype=torch.int32, device="cuda"),
             mask=_END if case["mask"] == "end" else _START)
    if case["turns"]:
        s["where"] = skv.Segments.from_lists(seqs)
    else:
        s["where"] = _spans(case, seqs)
    if case["kind"].startswith("train"):
        cap = max(_clen(x, w) for x in seqs)
        f32 = dict(dtype=torch.float32, device="cuda")
        need = max(skv.speechkv_prefill_attn_bwd_workspace_bytes(B, Hq, S),
                   skv.speechkv_pool_kv_bwd_workspace_bytes(B, S, Hkv, D))
        s.update(dout=d.normal((B, S, Hq, D), dt), lse=torch.zeros((B, Hq, S), **f32),
                 dq=torch.zeros((B, S, Hq, D), dtype=dt, device="cuda"),
                 dk_hat=torch.zeros((B, cap, Hkv, D), **f32), dv_hat=torch.zeros((B, cap, Hkv, D), **f32),
                 dk_raw=torch.zeros_like(s["k_raw"]), dv_raw=torch.zeros_like(s["v_raw"]),
                 du=torch.zeros((Hkv, D), **f32),
                 workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))
    return s


def _prepare_hidden(case, d):
    seqs = _sequences(case)
    B, hidden, dt = case["batch"], case["q_heads"] * case["dim"], _dt(case)
    h = d.raw(case, seqs, 1, hidden).view(B, -1, hidden)
    rows = max(_clen(s, case["w"]) for s in seqs)
    return dict(case=case, h=h, gate=d.normal((hidden,), torch.float32, hidden ** -0.5),
                where=_spans(case, seqs), out=torch.zeros((B, rows, hidden), dtype=dt, device="cuda"),
                out_len=torch.zeros(B, dtype=torch.int32, device="cuda"))


def prepare(case, seed):
    d = _Draws(seed)
    if case["kind"] == "decode":
        return _prepare_decode(case, d)
    if case["kind"] == "hidden":
        return _prepare_hidden(case, d)
    return _prepare_layer(case, d)


# -------------------------------------------------------------------- running

def _run_decode(s):
    for i, (cache, lens, longest) in enumerate(s["steps"]):
        skv.speechkv_decode_attn(s["q"][i], cache, lens, longest, s["out"][i], k_new=s["k_new"][i],
                                 v_new=s["v_new"][i], workspace=s["workspace"])
    return [s["out"], s["k_pages"], s["v_pages"]]


def _run_layer(s):
    c, where, w, l0 = s["case"], s["where"], s["case"]["w"], s["case"]["l0"]
    turns = isinstance(where, skv.Segments)
    lse = s.get("lse")
    if c["kind"] == "fused":
        skv.speechkv_pool_prefill_attn(s["q"], s["k_raw"], s["v_raw"], where, w, s["gate"], 0, l0,
                                       s["cache"], s["out"], cache_len_out=s["cache_len"],
                                       mask_mode=s["mask"])
    else:
        pool = skv.speechkv_pool_kv_segments if turns else skv.speechkv_pool_kv
        attend = skv.speechkv_prefill_attn_segments if turns else skv.speechkv_prefill_attn
        pool(s["k_raw"], s["v_raw"], where, w, s["gate"], 0, l0, s["cache"], s["cache_len"])
        attend(s["q"], s["cache"], where, w, 0, l0, s["out"], mask_mode=s["mask"], lse=lse)
    if lse is None:
        return [s["out"], s["cache"].k_pages, s["cache"].v_pages, s["cache_len"]]
    attend_bwd = skv.speechkv_prefill_attn_bwd_segments if turns else skv.speechkv_prefill_attn_bwd
    pool_bwd = skv.speechkv_pool_kv_bwd_segments if turns else skv.speechkv_pool_kv_bwd
    attend_bwd(s["q"], s["cache"], where, w, 0, l0, s["out"], lse, s["dout"], s["dq"], s["dk_hat"],
               s["dv_hat"], s["workspace"], mask_mode=s["mask"])
    pool_bwd(s["k_raw"], s["v_raw"], where, w, s["gate"], 0, l0, s["dk_hat"], s["dv_hat"],
             s["dk_raw"], s["dv_raw"], s["du"], s["workspace"])
    return [s["out"], lse, s["dq"], s["dk_raw"], s["dv_raw"], s["du"]]


def run(state):
    kind = state["case"]["kind"]
    if kind == "decode":
        return _run_decode(state)
    if kind == "hidden":
        skv.speechkv_pool_hidden(state["h"], state["where"], state["case"]["w"], state["gate"],
                                 state["out"], state["out_len"])
        return [state["out"], state["out_len"]]
    return _run_layer(state)


# ------------------------------------------------------------------- counting

def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: two per
    multiply-add over every (row, visible key) pair of every query head, for
    q.k and p.v and, in training, the four gradient products."""
    B, Hq, Hkv, D = case["batch"], case["q_heads"], case["kv_heads"], case["dim"]
    e = 2 if case["dtype"] == "bf16" else 4
    seqs = _sequences(case)
    if case["kind"] == "decode":
        nbytes = flops = 0
        for layer in range(case["layers"]):
            keys = sum(_clen(s, _w_eff(case, layer)) + case["generated"] for s in seqs)
            # cached rows read, but for the new one, which is read and stored
            nbytes += 2 * Hkv * D * e * (keys - B) + 4 * B * Hkv * D * e + 2 * B * Hq * D * e
            flops += 4 * keys * Hq * D
        return {"bytes": nbytes, "flops": flops}
    w = _w_eff(case, 0)
    rows, keys = sum(_rows(s) for s in seqs), sum(_clen(s, w) for s in seqs)
    if case["kind"] == "hidden":
        return {"bytes": (rows + keys) * Hq * D * e, "flops": 4 * rows * Hq * D}
    pairs = _pairs(case, w)
    raw, q = 2 * rows * Hkv * D * e, rows * Hq * D * e
    if case["kind"].startswith("train"):
        # raw K/V, q, dO read; out, LSE, dQ, raw dK, dV written
        return {"bytes": 2 * raw + 4 * q + rows * Hq * 4, "flops": 12 * pairs * Hq * D}
    return {"bytes": raw + 2 * keys * Hkv * D * e + 2 * q, "flops": 4 * pairs * Hq * D}


def tolerance(case):
    """About four times the largest distance from exact() seen over the ranges
    of draw(): 2.9e-3 and 6.7e-2 in bf16 (gradients of raw K; the cache and the
    probabilities are rounded to bf16 on the way), 1.6e-6 and 1.9e-5 in fp32 on
    sums of 600 rows, with room for the sums of thousands."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    return {"rel": 1e-2, "max": 0.25}


# --------------------------------------------------------- plain 64-bit torch

def _pool64(case, segs, w, x, gate, weigh):
    """Eq. 4 for one sequence: x [rows, H, D] -> [slots, H, D], the windows'
    frames weighted by the softmax of their keys' (weigh) gate logits."""
    slots = _layout(segs, w, case["mask"])
    first = torch.tensor([a for a, _, _ in slots], device=x.device)
    count = torch.tensor([n for _, n, _ in slots], device=x.device)
    j = torch.arange(w, device=x.device)
    at = first[:, None] + torch.minimum(j[None], count[:, None] - 1)
    logits = (weigh * gate).sum(-1)[at]                                    # [slots, w, H]
    logits = logits.masked_fill((j[None] >= count[:, None])[..., None], -math.inf)
    return (torch.softmax(logits, 1)[..., None] * x[at]).sum(1)


def _attend64(case, segs, w, q, k, v):
    """Eq. 5 for one sequence: q [rows, Hq, D], k and v [slots, Hkv, D]."""
    tau = torch.tensor([t for _, _, t in _layout(segs, w, case["mask"])], device=q.device)
    G = case["q_heads"] // case["kv_heads"]
    rows = q.shape[0]
    outs, lses = [], []
    for h in range(case["q_heads"]):
        kh, vh = k[:, h // G], v[:, h // G]
        parts, stats = [], []
        for a in range(0, rows, 2048):
            p = torch.arange(a, min(rows, a + 2048), device=q.device)
            z = (q[a:a + 2048, h] @ kh.T) * case["dim"] ** -0.5
            z = z.masked_fill(tau[None] > p[:, None], -math.inf)
            top = z.detach().amax(1, keepdim=True)
            top = torch.where(torch.isinf(top), torch.zeros_like(top), top)
            e = torch.exp(z - top)
            total = e.sum(1, keepdim=True)
            parts.append((e @ vh) / torch.where(total > 0, total, torch.ones_like(total)))
            stats.append((total.log() + top)[:, 0])
        outs.append(torch.cat(parts))
        lses.append(torch.cat(stats))
    return torch.stack(outs, 1), torch.stack(lses)


def exact(case, seed):
    s = prepare(case, seed)
    seqs = _sequences(case)
    if case["kind"] == "decode":
        out = torch.zeros(s["out"].shape, dtype=torch.float64, device="cuda")
        G = case["q_heads"] // case["kv_heads"]
        for i, (cache, lens, _) in enumerate(s["steps"]):
            for b, n in enumerate(lens.tolist()):
                ids = cache.block_table[b].long()
                k, v = (x[ids].double().transpose(1, 2).reshape(-1, case["kv_heads"], case["dim"])[:n]
                        for x in (s["k_pages"], s["v_pages"]))
                k[n - 1], v[n - 1] = s["k_new"][i, b].double(), s["v_new"][i, b].double()
                k, v = k.repeat_interleave(G, 1).transpose(0, 1), v.repeat_interleave(G, 1).transpose(0, 1)
                z = (k @ s["q"][i, b].double()[..., None])[..., 0] * case["dim"] ** -0.5
                out[i, b] = (torch.softmax(z, 1)[:, None] @ v)[:, 0]
        return [out, None, None]
    if case["kind"] == "hidden":
        out = torch.zeros(s["out"].shape, dtype=torch.float64, device="cuda")
        for b, segs in enumerate(seqs):
            h = s["h"][b, :_rows(segs)].double()[:, None]
            out[b, :_clen(segs, case["w"])] = _pool64(case, segs, case["w"], h, s["gate"].double(), h)[:, 0]
        return [out, None]
    train = case["kind"].startswith("train")
    w = _w_eff(case, 0)
    f64 = lambda x: torch.zeros(x.shape, dtype=torch.float64, device="cuda")  # noqa: E731
    out, dq, dk, dv, du = f64(s["out"]), f64(s["q"]), f64(s["k_raw"]), f64(s["v_raw"]), f64(s["gate"])
    kp, vp = f64(s["cache"].k_pages), f64(s["cache"].v_pages)
    lse = f64(s["lse"]) if train else None
    for b, segs in enumerate(seqs):
        n = _rows(segs)
        if not n:
            continue
        q, k, v = (s[x][b, :n].double().requires_grad_(train) for x in ("q", "k_raw", "v_raw"))
        u = s["gate"].double().requires_grad_(train)
        pk, pv = _pool64(case, segs, w, k, u, k), _pool64(case, segs, w, v, u, k)
        o, l = _attend64(case, segs, w, q, pk, pv)
        out[b, :n] = o.detach()
        if train:
            lse[b, :, :n] = l.detach()
            g = torch.autograd.grad(o, (q, k, v, u), s["dout"][b, :n].double())
            dq[b, :n], dk[b, :n], dv[b, :n] = g[:3]
            du += g[3]
        else:
            c = torch.arange(pk.shape[0], device="cuda")
            page = s["cache"].block_table[b].long()[c // case["page"]]
            kp[page, :, c % case["page"]], vp[page, :, c % case["page"]] = pk, pv
    if train:
        return [out, lse, dq, dk, dv, du]
    return [out, kp, vp, None]
