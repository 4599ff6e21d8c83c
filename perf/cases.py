"""The work a user of this package has it do, as timed cases over the range of sizes it is used at.

Every case is a dialogue batch: `B` sequences of history rounds whose keys and values are N(0, 1), the keys of a
few rounds per sequence shifted towards the query (the rounds the selection is meant to find), and a current round
of its own (the question and the answer so far), which every real decode step and question has.  Inputs are drawn
on the GPU from the seed, in the library's own layout; `exact` reads that layout back by its definition
(include/round_attention.h) and evaluates the method in 64 bits with plain torch.

Kinds of pass (one `run`):
  step         round scores and selection at the watershed layer, then decode attention of one later layer
  decode       decode attention of one post-watershed layer over a selection made earlier (the call that every
               later layer and every further token makes)
  question     the same two calls for a question of several tokens (prefill)
  watershed    the fused call at the watershed layer (attention and scores in one pass), one token or a question
  rescore      answer tokens added to the running round distribution, and the coverage of the selection
  turn         a turn of the host-resident store: stage the selected rounds, decode over every staged layer,
               send the new round back to host memory
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2502_15294_amd as ra

ALPHA = 2.0  # shift of the relevant rounds' keys along the unit query direction


def listed():
    return [
        # one short fp32 dialogue with two KV heads: the smallest call, launches and round trips only
        dict(name="tiny_step", kind="step", dtype="f32", B=1, Hq=4, Hkv=2, d=64, R=8, lo=64, hi=64, paged=False, cur=24, n_rel=2),
        # one user's chat on an 8B-shaped model: a step of a single sequence, a handful of rounds
        dict(name="chat_step", kind="step", dtype="bf16", B=1, Hq=32, Hkv=8, d=128, R=12, lo=200, hi=1000, paged=False, cur=190, n_rel=2),
        # a small serving batch on the same model
        dict(name="small_batch_step", kind="step", dtype="bf16", B=8, Hq=32, Hkv=8, d=128, R=20, lo=200, hi=1000, paged=False, cur=350, n_rel=3),
        # the small models of the family have heads of 64 channels
        dict(name="head64_step", kind="step", dtype="bf16", B=16, Hq=32, Hkv=8, d=64, R=24, lo=100, hi=900, paged=False, cur=210, n_rel=3),
        # a large serving batch of a 70B-shaped layer slice over paged blocks
        dict(name="paged_batch_step", kind="step", dtype="bf16", B=64, Hq=64, Hkv=8, d=128, R=50, lo=300, hi=1000, paged=True, cur=260, n_rel=3),
        # one post-watershed layer over 128K-token dialogues, about a third of the rounds kept
        dict(name="long_context_decode", kind="decode", dtype="bf16", B=16, Hq=32, Hkv=8, d=128, R=200, lo=130, hi=1180, paged=False, cur=500, keep=0.32),
        # a short follow-up question, odd sizes
        dict(name="short_question", kind="question", dtype="bf16", B=3, Hq=64, Hkv=8, d=128, R=23, lo=60, hi=700, paged=True, q_len=19, cur=19, n_rel=3, half=False),
        # a question of 128 tokens over 32K-token dialogues
        dict(name="question", kind="question", dtype="bf16", B=4, Hq=32, Hkv=8, d=128, R=60, lo=80, hi=1012, paged=False, q_len=128, cur=128, n_rel=4, half=False),
        # decode at the watershed layer itself
        dict(name="watershed_decode", kind="watershed", dtype="bf16", B=16, Hq=64, Hkv=8, d=128, R=30, lo=300, hi=1000, paged=True, q_len=1, cur=130, n_rel=3),
        # a question at the watershed layer itself
        dict(name="watershed_question", kind="watershed", dtype="bf16", B=2, Hq=32, Hkv=8, d=128, R=41, lo=60, hi=900, paged=False, q_len=100, cur=100, n_rel=3),
        # three answer tokens re-scored while a small batch decodes
        dict(name="rescore", kind="rescore", dtype="bf16", B=8, Hq=32, Hkv=8, d=128, R=20, lo=200, hi=1000, paged=False, cur=77, tokens=3, n_rel=3),
        # a turn over the host-resident store
        dict(name="turn", kind="turn", dtype="bf16", B=4, Hq=32, Hkv=8, d=128, R=16, lo=150, hi=700, layers=6, cur=140, keep=0.25),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "step", "decode", "decode", "question", "question", "watershed", "rescore", "turn"])
    Hq, Hkv = rng.choice([(32, 8), (64, 8), (16, 8), (24, 8), (8, 8), (32, 2)])
    c = dict(kind=kind, dtype="bf16", Hq=Hq, Hkv=Hkv, d=128, paged=rng.random() < 0.4, n_rel=rng.randint(1, 4))
    c["lo"] = log(1, 400)
    c["hi"] = c["lo"] + log(40, 900)
    mean = (c["lo"] + c["hi"]) / 2
    if kind in ("step", "decode"):
        # head_dim 64 and fp32 run at the smaller models' sizes
        small = rng.random() < 0.3
        if small:
            c["dtype"], c["d"] = rng.choice([("bf16", 64), ("f32", 64), ("f32", 128)])
            c["Hq"], c["Hkv"] = rng.choice([(32, 8), (16, 8), (8, 8), (64, 8), (4, 2)])
        c["B"] = log(1, 24 if small else 64)
        c["R"] = log(4, 200 if kind == "decode" else 60)
        # no more history than the largest listed case of the kind
        most = 300e3 if small else 2.0e6
        c["R"] = max(4, min(c["R"], int(most / (c["B"] * mean))))
        c["cur"] = log(1, 600)
        c["n_rel"] = min(c["n_rel"], c["R"])
        if kind == "decode":
            c["keep"] = round(rng.uniform(0.06, 0.6), 2)
    elif kind in ("question", "watershed"):
        c["q_len"] = 1 if kind == "watershed" and rng.random() < 0.5 else log(2, 200)
        c["B"] = log(1, 16)
        c["R"] = log(4, 60)
        # rows times history tokens: no more than the listed questions
        rows = c["q_len"] * c["Hq"]
        most = min(300e3, 128 * 32 * 131e3 * (1.0 if kind == "question" else 0.4) / rows)
        c["R"] = max(4, min(c["R"], int(most / (c["B"] * mean))))
        if c["B"] * c["R"] * mean > most:
            c["B"] = max(1, int(most / (c["R"] * mean)))
        c["cur"] = c["q_len"] + (log(1, 60) if rng.random() < 0.4 else 0)
        c["n_rel"] = min(c["n_rel"], c["R"])
        if kind == "question":
            c["half"] = rng.random() < 0.2
    elif kind == "rescore":
        c["B"] = log(1, 16)
        c["R"] = max(4, min(log(4, 60), int(200e3 / (c["B"] * mean))))
        c["cur"] = log(2, 400)
        c["tokens"] = rng.randint(1, 3)
        c["n_rel"] = min(c["n_rel"], c["R"])
    else:
        c["B"] = log(1, 6)
        c["layers"] = rng.randint(2, 8)
        c["keep"] = round(rng.uniform(0.1, 0.4), 2)
        c["R"] = max(4, min(log(4, 40), int(200e3 / (c["B"] * c["layers"] * mean))))
        c["cur"] = log(4, 300)
        c["paged"] = False
    return c


# ---- inputs -------------------------------------------------------------------------------------------------------

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


class _Handle:
    """A context (or store) that is given back with the state that holds it."""

    def __init__(self, ptr, close):
        self.ptr, self._close = ptr, close

    def __del__(self):
        self._close(self.ptr)


def _lengths(case, rng):
    """Round lengths [B][R]."""
    return rng.integers(case["lo"], case["hi"] + 1, size=(case["B"], case["R"])).astype(np.int32)


def _layer(case, lens, gen, q=None, relevant=None, values=True):
    """One layer's history on the GPU in the library's layout: a dict with the raw tensors, the index and the view.
    q [B, q_len, Hq, d]: the queries that the keys of the `relevant` rounds lean towards."""
    B, R = lens.shape
    Hkv, d, dt = case["Hkv"], case["d"], _dtype(case)
    per_seq = lens.sum(axis=1)
    max_tokens = int(per_seq.max())
    L16 = (lens + 15) // 16 * 16
    table = None
    if case.get("paged"):
        blocks = L16 // 16
        off = np.cumsum(blocks, axis=1) - blocks
        width = int(blocks.sum(axis=1).max())
        n_blocks = int(blocks.sum())
        perm = torch.randperm(n_blocks, generator=gen, device="cuda").to(torch.int32)
        table = torch.full((B, width), -1, dtype=torch.int32, device="cuda")
        used = torch.arange(width, device="cuda")[None, :] < torch.from_numpy(blocks.sum(axis=1)).cuda()[:, None]
        table[used] = perm
        k = torch.randn((n_blocks, Hkv, 16, d), generator=gen, device="cuda", dtype=dt)
        v = torch.randn((n_blocks, Hkv, d, 16), generator=gen, device="cuda", dtype=dt) if values else None
        off_v = None
    else:
        flat = lens.reshape(-1).astype(np.int64)
        off = (np.cumsum(flat) - flat).reshape(B, R)
        flat16 = L16.reshape(-1).astype(np.int64)
        off_v = (np.cumsum(flat16) - flat16).reshape(B, R)
        k = torch.randn((int(flat.sum()) * Hkv * d,), generator=gen, device="cuda", dtype=dt)
        v = torch.randn((int(flat16.sum()) * Hkv * d,), generator=gen, device="cuda", dtype=dt) if values else None
    if q is not None:
        s = q.float().reshape(B, q.shape[1], Hkv, -1, d).sum(dim=(1, 3))
        lean = (ALPHA * s / s.norm(dim=-1, keepdim=True)).to(dt)  # [B, Hkv, d]
        for b in range(B):
            for r in relevant[b]:
                n, o = int(lens[b, r]), int(off[b, r])
                if n == 0:
                    continue
                if table is not None:
                    ids = table[b, o:o + (n + 15) // 16].long()
                    k[ids] += lean[b][None, :, None, :]
                else:
                    k[o * Hkv * d:(o + n) * Hkv * d].view(Hkv, n, d).add_(lean[b][:, None, :])
    view = ra.KVView(k, v, torch.from_numpy(off.astype(np.int64)).cuda(), torch.from_numpy(lens).cuda(),
                     torch.full((B,), R, dtype=torch.int32, device="cuda"), Hkv, d, max_tokens, block_table=table,
                     block_size=16 if table is not None else 0,
                     seg_off_v=None if off_v is None or not values else torch.from_numpy(off_v).cuda())
    return dict(k=k, v=v, off=off, off_v=off_v, lens=lens, table=table, view=view)


def _context(case, lens, q_len):
    ctx = _Handle(ra.ra_create(torch.cuda.current_device()), ra.ra_destroy)
    nbytes = ra.ra_workspace_bytes(case["B"], case["R"], case["Hq"], case["Hkv"], case["d"], q_len,
                                   ra.RA_F32 if case["dtype"] == "f32" else ra.RA_BF16,
                                   int(lens.sum(axis=1).max()) + case["cur"])
    workspace = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    ra.ra_set_workspace(ctx.ptr, workspace)
    return ctx, workspace


def _some_rounds(rng, B, R, n):
    return [np.sort(rng.choice(R, size=min(n, R), replace=False)) for _ in range(B)]


def _selection(sel, R):
    idx = np.full((len(sel), R), -1, dtype=np.int32)
    for b, s in enumerate(sel):
        idx[b, :len(s)] = s
    return torch.from_numpy(idx), torch.tensor([len(s) for s in sel], dtype=torch.int32)


def prepare(case, seed):
    rng = np.random.default_rng([2502, int(seed)])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dt, kind, B, Hq, Hkv, d, R = _dtype(case), case["kind"], case["B"], case["Hq"], case["Hkv"], case["d"], case["R"]

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dt)

    lens = _lengths(case, rng)
    s = dict(case=case, lens=lens)
    cur = case["cur"]
    if kind == "turn":
        return _prepare_turn(case, rng, gen, lens, s)
    q_len = case.get("q_len", 1)
    s["ctx"], s["workspace"] = _context(case, lens, q_len)
    if kind == "question" and case["half"]:
        ra.ra_set_prefill_precision(s["ctx"].ptr, ra.RA_PREFILL_P_F16)
    if kind == "decode":
        s["sel"] = _some_rounds(rng, B, R, max(1, round(case["keep"] * R)))
        s["sel_idx"], s["n_sel"] = (x.cuda() for x in _selection(s["sel"], R))
    else:
        relevant = _some_rounds(rng, B, R, case["n_rel"])
        s["q0"] = randn(B, q_len, Hq, d)
        s["layer0"] = _layer(case, lens, gen, s["q0"], relevant, values=kind == "watershed")
    if kind in ("step", "decode"):
        s["q1"] = randn(B, Hq, d)
        s["layer1"] = _layer(case, lens, gen)
        # sequences of a batch stand at different places of their answers
        cur_len = rng.integers(max(1, cur // 3), cur + 1, size=B).astype(np.int32)
        s["cur_len"] = torch.from_numpy(cur_len).cuda()
        s["ck"], s["cv"] = randn(B, cur, Hkv, d), randn(B, cur, Hkv, d)
    elif kind == "question":
        s["ck0"] = randn(B, cur, Hkv, d)
        s["q1"] = randn(B, q_len, Hq, d)
        s["layer1"] = _layer(case, lens, gen)
        s["ck"], s["cv"] = randn(B, cur, Hkv, d), randn(B, cur, Hkv, d)
    elif kind == "watershed":
        s["ck"], s["cv"] = randn(B, cur, Hkv, d), randn(B, cur, Hkv, d)
        s["cur_len"] = torch.full((B,), cur, dtype=torch.int32, device="cuda")
        if q_len == 1:
            s["q0"] = s["q0"][:, 0].contiguous()
    else:  # rescore: one query and one grown current round per answer token, a selection made from the question
        keys = randn(B, cur + case["tokens"], Hkv, d)
        s["tokens"] = [(randn(B, 1, Hq, d) if i else s["q0"], keys[:, :cur + i + 1].contiguous())
                       for i in range(case["tokens"])]
        s["sel_idx"], s["n_sel"] = (x.cuda() for x in _selection(relevant, R))
        s["acc"] = torch.zeros((B, Hq, R), dtype=torch.float32, device="cuda")
    return s


def _prepare_turn(case, rng, gen, lens, s):
    B, R, L, Hq, Hkv, d, cur, dt = (case["B"], case["R"], case["layers"], case["Hq"], case["Hkv"], case["d"], case["cur"],
                                    _dtype(case))
    s["sel"] = _some_rounds(rng, B, R, max(1, round(case["keep"] * R)))
    s["sel_idx"], s["n_sel"] = _selection(s["sel"], R + 1)
    sel_tokens = sum(int(lens[b, r] + (lens[b, r] + 15) // 16 * 16) for b in range(B) for r in s["sel"][b])
    new = np.array([max(1, cur - 7 * b * cur // 64) for b in range(B)], dtype=np.int32)  # the saved tensors' sizes are the case's
    new_tokens = sum(int(n + (n + 15) // 16 * 16) for n in new)
    elem = torch.empty((), dtype=dt).element_size()
    pool = (sel_tokens + new_tokens) * L * Hkv * d * elem
    s["store"] = _Handle(ra.ra_kv_store_create(torch.cuda.current_device(), L, B, R + 1, Hkv, d,
                                               ra.RA_F32 if dt == torch.float32 else ra.RA_BF16, pool), ra.ra_kv_store_destroy)
    s["ctx"], s["workspace"] = _context(dict(case, R=R + 1), lens, 1)
    # rounds that are not selected are never read: they share one buffer
    shared = torch.zeros(ra.ra_kv_store_round_bytes(s["store"].ptr, int(lens.max())), dtype=torch.uint8, pin_memory=True)
    s["host"] = {}
    for b in range(B):
        chosen = set(s["sel"][b].tolist())
        for r in range(R):
            n = int(lens[b, r])
            buf = shared
            if r in chosen:
                count = ra.ra_kv_store_round_bytes(s["store"].ptr, n) // elem
                buf = torch.empty(count, dtype=dt, pin_memory=True)
                buf.copy_(torch.randn((count,), generator=gen, device="cuda", dtype=dt))
                s["host"][b, r] = buf
            ra.ra_kv_store_register_round(s["store"].ptr, b, r, buf, n)
    s["shared"] = shared
    s["q"] = torch.randn((L, B, Hq, d), generator=gen, device="cuda", dtype=dt)
    s["ck"] = [torch.randn((B, cur, Hkv, d), generator=gen, device="cuda", dtype=dt) for _ in range(L)]
    s["cv"] = [torch.randn((B, cur, Hkv, d), generator=gen, device="cuda", dtype=dt) for _ in range(L)]
    s["new_len"] = torch.from_numpy(new)
    s["cur_len"] = s["new_len"].cuda()
    s["new_round"] = torch.full((B,), R, dtype=torch.int32)
    s["saved"] = [torch.empty(ra.ra_kv_store_round_bytes(s["store"].ptr, int(n)) // elem, dtype=dt, pin_memory=True) for n in new]
    s["side"] = torch.cuda.Stream()
    torch.cuda.synchronize()
    return s


# ---- one pass -----------------------------------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "turn":
        return _run_turn(s)
    ctx = s["ctx"].ptr
    if kind == "step":
        ph, p, sel, n = ra.ra_round_scores_select(ctx, s["q0"], s["layer0"]["view"])
        out, lse = ra.ra_round_sparse_attn_decode(ctx, s["q1"], s["layer1"]["view"], sel, n, s["ck"], s["cv"], s["cur_len"])
        return dict(scores_head=ph, scores=p, sel_idx=sel, n_sel=n, out=out, lse=lse)
    if kind == "decode":
        out, lse = ra.ra_round_sparse_attn_decode(ctx, s["q1"], s["layer1"]["view"], s["sel_idx"], s["n_sel"], s["ck"], s["cv"],
                                                  s["cur_len"])
        return dict(out=out, lse=lse)
    if kind == "question":
        ph, p, sel, n = ra.ra_round_scores_select(ctx, s["q0"], s["layer0"]["view"], cur_k=s["ck0"])
        out, lse = ra.ra_round_sparse_attn_prefill(ctx, s["q1"], s["layer1"]["view"], sel, n, s["ck"], s["cv"])
        return dict(scores_head=ph, scores=p, sel_idx=sel, n_sel=n, out=out, lse=lse)
    if kind == "watershed":
        if case["q_len"] == 1:
            out, lse, ph, p = ra.ra_watershed_attn_decode(ctx, s["q0"], s["layer0"]["view"], s["ck"], s["cv"], s["cur_len"])
        else:
            out, lse, ph, p = ra.ra_watershed_attn_prefill(ctx, s["q0"], s["layer0"]["view"], s["ck"], s["cv"])
        return dict(scores_head=ph, scores=p, out=out, lse=lse)
    s["acc"].zero_()
    cover = []
    for q, keys in s["tokens"]:
        ph, p = ra.ra_round_scores_accumulate(ctx, q, s["layer0"]["view"], s["acc"], cur_k=keys)
        cover.append(ra.ra_selection_coverage(ctx, p, s["sel_idx"], s["n_sel"]))
    return dict(acc=s["acc"], scores_head=ph, scores=p, cover=cover)


def _run_turn(s):
    case, store, ctx = s["case"], s["store"].ptr, s["ctx"].ptr
    compute = torch.cuda.current_stream()
    s["side"].wait_stream(compute)
    ra.ra_kv_store_stage(store, s["sel_idx"], s["n_sel"], ra.RA_STAGE_GROUPED, s["side"])
    outs = []
    for layer in range(case["layers"]):
        ra.ra_kv_store_wait_layer(store, layer, compute)
        view = ra.ra_kv_store_layer_view(store, layer)
        outs.append(ra.ra_round_sparse_attn_decode(ctx, s["q"][layer], view, None, None, s["ck"][layer], s["cv"][layer],
                                                   s["cur_len"])[0])
    ra.ra_kv_store_save_round(store, s["new_round"], s["new_len"], s["ck"], s["cv"], s["saved"], compute, s["side"])
    ra.ra_kv_store_save_wait(store)  # the turn ends when the new round is in host memory; the staged views are done then
    ra.ra_kv_store_release(store)
    return dict(out=outs, saved=s["saved"])


# ---- what a pass cannot do without --------------------------------------------------------------------------------

def work(case):
    """Bytes read and written once and operations, from the expected lengths (a selection keeps about a seventh of
    the rounds unless the case says)."""
    e = 4 if case["dtype"] == "f32" else 2
    B, Hq, Hkv, d, R, kind = case["B"], case["Hq"], case["Hkv"], case["d"], case["R"], case["kind"]
    tokens = B * R * (case["lo"] + case["hi"]) / 2
    row, q_len = Hkv * d * e, case.get("q_len", 1)
    rows = B * q_len * Hq
    kept = tokens * case.get("keep", max(case.get("n_rel", 1), R / 7) / R)
    per_q = rows * d * (e + 4) + rows * 4
    scores_out = B * (Hq + 1) * R * 4
    cur = B * case["cur"] * (2 / 3 if kind in ("step", "decode") else 0.75 if kind == "turn" else 1)

    def dots(n_tokens, products):
        return 2 * products * (n_tokens / B) * rows * d

    if kind == "step":
        return dict(bytes=tokens * row + rows * d * e + scores_out + (kept + cur) * 2 * row + per_q,
                    flops=dots(tokens, 1) + dots(kept + cur, 2))
    if kind == "decode":
        return dict(bytes=(kept + cur) * 2 * row + per_q, flops=dots(kept + cur, 2))
    if kind == "question":
        return dict(bytes=(tokens + cur) * row + rows * d * e + scores_out + (kept + cur) * 2 * row + per_q,
                    flops=dots(tokens + cur / 2, 1) + dots(kept + cur / 2, 2))
    if kind == "watershed":
        return dict(bytes=(tokens + cur) * 2 * row + per_q + scores_out, flops=dots(tokens + cur / 2, 2))
    if kind == "rescore":
        n = case["tokens"]
        return dict(bytes=n * ((tokens + cur) * row + rows * d * e + 2 * scores_out), flops=n * dots(tokens + cur, 1))
    L = case["layers"]  # turn: the staged bytes land in device memory and are read there; the new round is read and leaves
    return dict(bytes=L * (2 * kept * 2 * row + 2 * cur * 2 * row + per_q), flops=L * dots(kept + cur, 2))


def tolerance(case):
    """About four times the error seen against 64 bits: fp32 sums (4e-7 in the scores, 2e-7 with fp32 values or heads of
    64), the probabilities carried to 16 bits for bf16 values of 128 channels (1e-5, single outputs 6e-5), to 11 bits
    in the fp16 mode of a question (2e-4, single outputs 1.4e-3)."""
    if case["kind"] == "question" and case["half"]:
        return {"rel": 8e-4, "max": 6e-3}
    if case["kind"] == "rescore" or case["dtype"] == "f32" or case["d"] == 64:
        return {"rel": 1e-6, "max": 5e-6}
    return {"rel": 4e-5, "max": 2.5e-4}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------

def _keys(L, b, r, Hkv, d):
    """[Hkv, len, d] in double, by the definition of the layout."""
    n, o = int(L["lens"][b, r]), int(L["off"][b, r])
    if L["table"] is not None:
        ids = L["table"][b, o:o + (n + 15) // 16].long()
        return L["k"][ids].permute(1, 0, 2, 3).reshape(Hkv, -1, d)[:, :n].double()
    return L["k"][o * Hkv * d:(o + n) * Hkv * d].view(Hkv, n, d).double()


def _values(L, b, r, Hkv, d):
    n, tiles = int(L["lens"][b, r]), (int(L["lens"][b, r]) + 15) // 16
    if L["table"] is not None:
        o = int(L["off"][b, r])
        x = L["v"][L["table"][b, o:o + tiles].long()].permute(1, 0, 3, 2)
    else:
        o = int(L["off_v"][b, r])
        x = L["v"][o * Hkv * d:(o + tiles * 16) * Hkv * d].view(Hkv, tiles, d, 16).permute(0, 1, 3, 2)
    return x.reshape(Hkv, -1, d)[:, :n].double()


def _logits(q, k, scale):
    """q [q_len, Hq, d], k [Hkv, T, d] -> [Hkv, G, q_len, T] in double."""
    Hkv, G = k.shape[0], q.shape[1] // k.shape[0]
    x = q.double().reshape(q.shape[0], Hkv, G, -1).permute(1, 2, 0, 3)
    return torch.stack([(x[g].reshape(-1, x.shape[-1]) @ k[g].T).reshape(G, q.shape[0], -1) for g in range(Hkv)]) * scale


def _masked(x, n_hist, q_len):
    """-inf where a query token may not see a token of the current round (the columns from n_hist on)."""
    cur = x.shape[-1] - n_hist
    if cur:
        i, j = torch.arange(q_len, device="cuda")[:, None], torch.arange(cur, device="cuda")[None, :]
        x[..., n_hist:].masked_fill_(j > cur - q_len + i, -math.inf)
    return x


def _exact_masses(case, L, b, q, ck):
    """Round masses of Eq. 1 before the normalisation, [Hq, R]: summed over the query tokens."""
    Hkv, d, R = case["Hkv"], case["d"], case["R"]
    parts = [_keys(L, b, r, Hkv, d) for r in range(R)]
    n_hist = sum(p.shape[1] for p in parts)
    if ck is not None:
        parts.append(ck.transpose(0, 1).double())
    p = torch.softmax(_masked(_logits(q, torch.cat(parts, 1), d ** -0.5), n_hist, q.shape[0]), -1)[..., :n_hist].sum(2)
    owner = torch.repeat_interleave(torch.arange(R, device="cuda"), torch.from_numpy(L["lens"][b].astype(np.int64)).cuda())
    out = torch.zeros((Hkv, p.shape[1], R), dtype=torch.float64, device="cuda")
    return out.index_add_(2, owner, p).reshape(-1, R)


def _exact_select(scores):
    cut = scores.mean() + scores.std(unbiased=False)
    sel = torch.nonzero(scores > cut).flatten().tolist()
    return sel or [int(scores.argmax())]


def _exact_attention(case, L, b, rounds, q, ck, cv):
    """([q_len, Hq, d], [q_len, Hq]) in double."""
    Hkv, d = case["Hkv"], case["d"]
    k = [_keys(L, b, r, Hkv, d) for r in rounds] + [ck.transpose(0, 1).double()]
    v = torch.cat([_values(L, b, r, Hkv, d) for r in rounds] + [cv.transpose(0, 1).double()], 1)
    n_hist = sum(x.shape[1] for x in k[:-1])
    x = _masked(_logits(q, torch.cat(k, 1), d ** -0.5), n_hist, q.shape[0])
    lse = torch.logsumexp(x, -1)
    p = torch.softmax(x, -1)
    o = torch.stack([(p[g].reshape(-1, p.shape[-1]) @ v[g]).reshape(*p.shape[1:3], d) for g in range(Hkv)])
    return o.permute(2, 0, 1, 3).reshape(q.shape[0], -1, d), lse.permute(2, 0, 1).reshape(q.shape[0], -1)


def exact(case, seed):
    s = prepare(case, seed)
    kind, B, R, Hq = case["kind"], case["B"], case["R"], case["Hq"]
    if kind == "turn":
        return _exact_turn(case, s)
    one = lambda q: q if q.dim() == 4 else q[:, None]  # noqa: E731
    res = {}
    if kind == "rescore":
        acc, cover = torch.zeros((B, Hq, R), dtype=torch.float64, device="cuda"), []
        for q, keys in s["tokens"]:
            acc += torch.stack([_exact_masses(case, s["layer0"], b, q[b], keys[b]) for b in range(B)])
            head = acc / acc.sum(-1, keepdim=True)
            cover.append(torch.stack([head[b].mean(0)[s["sel_idx"][b, :s["n_sel"][b]].long()].sum() for b in range(B)]))
        return dict(acc=acc, scores_head=head, scores=head.mean(1), cover=cover)
    sel = s.get("sel")
    if kind != "decode":
        ck0 = s.get("ck0") if kind == "question" else s["ck"] if kind == "watershed" and case["q_len"] > 1 else None
        head = []
        for b in range(B):
            m = _exact_masses(case, s["layer0"], b, one(s["q0"])[b], None if ck0 is None else ck0[b])
            head.append(m / m.sum(-1, keepdim=True))
        res["scores_head"] = torch.stack(head)
        res["scores"] = res["scores_head"].mean(1)
    if kind == "watershed":
        sel, layer, q = [range(R)] * B, s["layer0"], one(s["q0"])
    else:
        layer, q = s["layer1"], one(s["q1"])
        if sel is None:
            sel = [_exact_select(x) for x in res["scores"]]
            res["sel_idx"], res["n_sel"] = _selection(sel, R)
    outs, lses = [], []
    for b in range(B):
        n = int(s["cur_len"][b]) if "cur_len" in s else case["cur"]
        o, l = _exact_attention(case, layer, b, sel[b], q[b], s["ck"][b, :n], s["cv"][b, :n])
        outs.append(o)
        lses.append(l)
    out, lse = torch.stack(outs), torch.stack(lses)
    single = case.get("q_len", 1) == 1
    res["out"], res["lse"] = (out[:, 0], lse[:, 0]) if single else (out, lse)
    return res


def _exact_turn(case, s):
    B, L, Hkv, d, lens = case["B"], case["layers"], case["Hkv"], case["d"], s["lens"]

    def slices(buf, n, layer):  # a host tensor: per layer the keys [Hkv][n][d], then the value tiles [Hkv][tiles][d][16]
        tiles = (n + 15) // 16
        x = buf.view(L, (n + tiles * 16) * Hkv * d)[layer].cuda().double()
        k, v = x[:n * Hkv * d], x[n * Hkv * d:]
        return k.view(Hkv, n, d), v.view(Hkv, tiles, d, 16).permute(0, 1, 3, 2).reshape(Hkv, -1, d)[:, :n]

    outs = []
    for layer in range(L):
        rows = []
        for b in range(B):
            n = int(s["new_len"][b])
            kv = [slices(s["host"][b, r], int(lens[b, r]), layer) for r in s["sel"][b].tolist()]
            kv.append((s["ck"][layer][b, :n].transpose(0, 1).double(), s["cv"][layer][b, :n].transpose(0, 1).double()))
            k, v = torch.cat([x[0] for x in kv], 1), torch.cat([x[1] for x in kv], 1)
            p = torch.softmax(_logits(s["q"][layer, b][None], k, d ** -0.5), -1)
            rows.append(torch.stack([p[g, :, 0] @ v[g] for g in range(Hkv)]).reshape(-1, d))
        outs.append(torch.stack(rows))
    saved = []
    for b in range(B):
        n = int(s["new_len"][b])
        tiles, parts = (n + 15) // 16, []
        for layer in range(L):
            k, v = s["ck"][layer][b, :n].transpose(0, 1), s["cv"][layer][b, :n].transpose(0, 1)
            v = torch.nn.functional.pad(v, (0, 0, 0, tiles * 16 - n)).reshape(Hkv, tiles, 16, d).transpose(2, 3)
            parts += [k.reshape(-1), v.reshape(-1)]
        saved.append(torch.cat(parts).double())
    return dict(out=outs, saved=saved)
