"""The finishing kernels and the selection at the sizes where their shape changes: 16, 32, 64 and 256 rounds (lanes and
rounds per head), head counts that leave segments or waves empty, rounds of more than four chunks, rows that do not
fit LDS, and selections on either side of one wave's 64 rounds."""
import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, to_device

pytestmark = pytest.mark.gpu
SCORE_TOL = 1e-5  # fp32 log-sum-exps of exact bf16 products: a few 1e-7, as in the other score tests


def _lens(R, seed):
    rng = np.random.default_rng(seed)
    return [rng.integers(0, 24, size=R).tolist(), rng.integers(1, 24, size=max(R - 1, 1)).tolist()]


CASES = [(R, Hq, Hkv, q_len) for R in (1, 15, 16, 17, 32, 33, 64, 65, 256, 257)
         for Hq, Hkv, q_len in ((3, 1, 1), (24, 8, 1), (18, 2, 5))] + [
    (R, Hq, Hkv, q_len) for R in (512, 513, 1024) for Hq, Hkv, q_len in ((3, 1, 1), (32, 8, 1), (18, 2, 5))] + [(50, 64, 8, 1), (50, 64, 8, 7), (40, 32, 8, 70)]


@pytest.mark.parametrize("R,Hq,Hkv,q_len", CASES)
def test_scores_and_selection(R, Hq, Hkv, q_len):
    cur_len = q_len + 3 if q_len > 1 else 0
    lens = _lens(R, R * 31 + Hq)
    lens[0][0] = 1500 if R <= 17 else lens[0][0] + 1  # six chunks: past the four that are read in one go
    w = make_workload("cfg2", B=2, Hq=Hq, Hkv=Hkv, q_len=q_len, cur_len=cur_len, lens=lens, n_relevant=1)
    eng = Engine(w)
    view = device_view(w, 0, with_v=False)
    q = to_device(w.q(0), w.dtype)
    ck = to_device(w.cur_k(0), w.dtype) if cur_len else None
    P, S, sel, n = ra.ra_round_scores_select(eng.ctx, q, view, ra.make_select_params(lam=0.5), cur_k=ck, scale=w.scale)
    P2, S2 = ra.ra_round_scores(eng.ctx, q, view, ck, scale=w.scale)
    acc = torch.zeros_like(P)
    P3, _ = ra.ra_round_scores_accumulate(eng.ctx, q, view, acc, cur_k=ck, scale=w.scale)
    torch.cuda.synchronize()
    assert torch.equal(P, P2) and torch.equal(S, S2)
    assert (P3 - P).abs().max().item() < 1e-6  # the same masses, normalised after having been stored
    P, S, sel, n = P.cpu().numpy(), S.cpu().numpy(), sel.cpu().numpy(), n.cpu().numpy()
    for b in range(w.B):
        Rb = w.n_rounds(b)
        rP, rS = pipeline.scores_for_sequence(w, b)
        assert np.abs(P[b, :, :Rb] - rP).max() < SCORE_TOL and np.abs(S[b, :Rb] - rS).max() < SCORE_TOL
        assert np.all(P[b, :, Rb:] == 0) and np.all(S[b, Rb:] == 0)
        assert sel[b, :n[b]].tolist() == ora.select_rounds([float(x) for x in S[b, :Rb]], lam=0.5)[0]
        assert np.all(sel[b, n[b]:] == -1)
    eng.close()


@pytest.mark.parametrize("q_len,chunks", [(1, 3000), (5, 500)])
def test_scores_with_a_capacity_whose_rows_do_not_fit_lds(q_len, chunks):
    """Four heads of 16 rounds with room declared for so many chunks that a workgroup's rows do not fit the finishing kernels'
    LDS: they are read from memory instead."""
    R, Hq, heads_per_wave = 16, 4, 4
    waves, limit = (4, 96 * 1024) if q_len == 1 else (8, 48 * 1024)  # one token per sequence; several, two workgroups a unit
    assert (R + 2) * 4 + waves * R * 4 + waves * heads_per_wave * chunks * 4 > limit
    assert q_len > 1 or Hq * chunks < 16384  # the one-token kernel, not the one that takes a head per workgroup
    cur_len = 9 if q_len > 1 else 0
    w = make_workload("cfg2", B=2, Hq=Hq, Hkv=1, q_len=q_len, cur_len=cur_len, lens=[[9, 600] * 8, [300] * 13], n_relevant=2)
    room = (chunks - R - (1 if cur_len else 0)) * 256
    eng = Engine(w, extra_tokens=room)
    view = device_view(w, 0)
    k, v, off, ln, nr, bt, off_v = view.tensors
    roomy = ra.KVView(k, v, off, ln, nr, view.Hkv, view.d, room, seg_off_v=off_v)
    q = to_device(w.q(0), w.dtype)
    ck = to_device(w.cur_k(0), w.dtype) if cur_len else None
    a = ra.ra_round_scores_select(eng.ctx, q, view, cur_k=ck, scale=w.scale)
    b = ra.ra_round_scores_select(eng.ctx, q, roomy, cur_k=ck, scale=w.scale)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    for i in range(w.B):
        rP, _ = pipeline.scores_for_sequence(w, i)
        assert np.abs(a[0][i, :, :w.n_rounds(i)].cpu().numpy() - rP).max() < SCORE_TOL
    eng.close()


@pytest.mark.parametrize("d", [128, 64])
def test_a_score_pass_of_two_launches(d):
    """Room declared for more chunks than one launch takes (65 535): the same scores, and the measured time is that of the
    whole pass (nearly all of it the first launch, whose workgroups find their chunk past the last one)."""
    w = make_workload("cfg2", B=1, d=d, lens=[[300, 7, 500]], n_relevant=1)
    eng = Engine(w, extra_tokens=66000 * 256)
    view = device_view(w, 0)
    k, v, off, ln, nr, bt, off_v = view.tensors
    q = to_device(w.q(0), w.dtype)
    want = ra.ra_round_scores(eng.ctx, q, view, scale=w.scale)
    ms = []
    ra.ra_profile_kernels(eng.ctx, True)
    for chunks in (65000, 66000):
        roomy = ra.KVView(k, v, off, ln, nr, view.Hkv, view.d, chunks * 256, seg_off_v=off_v)
        for _ in range(3):
            got = ra.ra_round_scores(eng.ctx, q, roomy, scale=w.scale)
        ms.append(ra.ra_profile_last_ms(eng.ctx))
        assert all((x - y).abs().max() < 1e-6 for x, y in zip(got, want))
    assert ms[1] > 0.5 * ms[0] > 0, ms
    eng.close()


@pytest.mark.parametrize("R", [1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 257, 511, 1024])
@pytest.mark.parametrize("kind", ["spread", "ties", "equal"])
def test_selection_sizes(R, kind):
    rng = np.random.default_rng(R)
    s = rng.random((4, R)).astype(np.float32)
    if kind == "ties":
        s = (np.round(s * 5) / 5).astype(np.float32)
    elif kind == "equal":
        s[:] = np.float32(1.0 / R)
    n_rounds = np.array([R, max(R - 1, 0), R // 2, 0], dtype=np.int32)
    ctx = ra.ra_create(0)
    ds, dn = torch.from_numpy(s).cuda(), torch.from_numpy(n_rounds).cuda()
    for kw in (dict(lam=1.0), dict(lam=0.0, ddof=1), dict(strategy=ra.RA_SEL_TOP_FRACTION, fraction=0.37),
               dict(strategy=ra.RA_SEL_THRESHOLD, threshold=0.8, min_rounds=2, keep_first=1, keep_last=2),
               dict(lam=-0.5, max_rounds=5)):
        idx, n = ra.ra_select_rounds(ctx, ds, dn, ra.make_select_params(**kw))
        idx, n = idx.cpu().numpy(), n.cpu().numpy()
        for b in range(4):
            want = ora.select_rounds([float(x) for x in s[b, :n_rounds[b]]], **kw)[0] if n_rounds[b] else []
            assert idx[b, :n[b]].tolist() == want and np.all(idx[b, n[b]:] == -1), (kw, b)
    ra.ra_destroy(ctx)
