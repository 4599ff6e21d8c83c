"""Questions at the sizes where their kernels change shape: row counts around the 16-row tiles and row blocks, batches that
the launch plans itself and ones planned by a kernel of their own, dialogues cut by themselves and ranges that cross from
one into the next, equal and by weight, dialogues without any key."""
import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, sel_to_device, to_device

pytestmark = pytest.mark.gpu
STREAM_TOL, SCORE_TOL = 5e-5, 1e-5  # the bars of the other parity tests: P carried to 16 bits, fp32 sums

ROWS = [(9, 32, 8), (8, 64, 8), (16, 64, 8), (17, 64, 8), (48, 32, 8), (65, 32, 8), (50, 24, 8), (30, 32, 2)]
BATCHES = {
    "long": dict(lens=[[900, 3, 700, 250], [17, 640, 33], [1000, 900, 800, 31, 5]]),      # about 170 tiles: equal ranges, or cut apart
    "short_paged": dict(lens=[[5, 16, 17, 0, 33], [64, 3], [0, 0]], block_size=16),
    "lists_of_1024": dict(B=64, R=16, length=("uniform", 0, 12)),                         # the most that is planned inline
    "planned_apart": dict(B=30, R=40, length=("uniform", 0, 9), block_size=16),
    # one dialogue of so many rounds that its lists leave room for fewer workgroups: the score pass, then both are planned apart
    "700_rounds": dict(B=1, R=700, length=("uniform", 0, 9)),
    "1000_rounds": dict(B=1, R=1000, length=("uniform", 0, 9), block_size=16),
    "planned_apart_65": dict(B=65, R=2, length=("uniform", 1, 40)),
}


@pytest.mark.parametrize("batch", list(BATCHES))
@pytest.mark.parametrize("q_len,Hq,Hkv", ROWS)
def test_question(batch, q_len, Hq, Hkv):
    over = dict(BATCHES[batch])
    if "lens" in over:
        over["B"] = len(over["lens"])
    cur_len = 0 if (batch, q_len) == ("short_paged", 16) else q_len + (q_len & 3)
    w = make_workload("cfg3", Hq=Hq, Hkv=Hkv, q_len=q_len, cur_len=cur_len, n_relevant=1, **over)
    eng = Engine(w)
    v0, v1 = device_view(w, 0), device_view(w, 1)
    dev = lambda x: None if x is None else to_device(x, "bf16")  # noqa: E731
    ck0, cv0, ck1, cv1 = dev(w.cur_k(0)), dev(w.cur_v(0)), dev(w.cur_k(1)), dev(w.cur_v(1))
    P, S, sel, n = ra.ra_round_scores_select(eng.ctx, dev(w.q(0)), v0, cur_k=ck0, scale=w.scale)
    rng = np.random.default_rng(q_len)
    sels = [sorted(rng.choice(w.n_rounds(b), size=(w.n_rounds(b) + 1) // 2, replace=False).tolist()) for b in range(w.B)]
    si, ns = sel_to_device(sels, v1.R_max)
    out, lse = ra.ra_round_sparse_attn_prefill(eng.ctx, dev(w.q(1)), v1, si, ns, ck1, cv1, scale=w.scale)
    again, _ = ra.ra_round_sparse_attn_prefill(eng.ctx, dev(w.q(1)), v1, si, ns, ck1, cv1, scale=w.scale)
    out2, _, P2, S2 = ra.ra_watershed_attn_prefill(eng.ctx, dev(w.q(0)), v0, ck0, cv0, scale=w.scale)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    P, S, out, lse, out2, S2 = (x.cpu().numpy() for x in (P, S, out, lse, out2, S2))
    for b in sorted({0, min(1, w.B - 1), w.B // 2, w.B - 1}):
        R = w.n_rounds(b)
        if w.total_tokens(b):
            rP, rS = pipeline.scores_for_sequence(w, b)
            assert np.abs(P[b, :, :R] - rP).max() < SCORE_TOL and np.abs(S[b, :R] - rS).max() < SCORE_TOL, b
            assert np.abs(S2[b, :R] - rS).max() < SCORE_TOL, b
        if w.total_tokens(b) + cur_len:
            assert ora.row_error(out2[b], pipeline.attention_for_sequence(w, b, 0, list(range(R)))[0]) < STREAM_TOL, b
        if sum(int(w.lens[b][r]) for r in sels[b]) + cur_len == 0:
            assert np.all(out[b] == 0) and np.all(np.isneginf(lse[b])), b
            continue
        ro, rl = pipeline.attention_for_sequence(w, b, 1, sels[b])
        assert ora.row_error(out[b], ro) < STREAM_TOL, b
        assert np.allclose(lse[b], rl, rtol=0, atol=2e-5 * max(1.0, np.abs(rl).max())), b
    eng.close()


@pytest.mark.parametrize("q_len,Hkv,tiles", [(100, 2, (17, 316, 17)), (128, 8, (60, 330, 60))])
def test_one_long_dialogue_between_two_short_ones(q_len, Hkv, tiles):
    """More than eight key tiles for every range that 256 compute units take.  100 tokens, 2 KV heads: 19 ranges, 26 items each;
    cut by the weights of the two classes of workgroups the long dialogue would meet 19 of them, and a row's partial
    results have room for 18.  128 tokens, 8 KV heads: 16 ranges in the attention kernel and 48 in the score kernel, by
    weight."""
    lens = [[32 * n] if n < 100 else [256] * (n // 8) + [32 * (n % 8)] * (n % 8 > 0) for n in tiles]
    w = make_workload("cfg3", B=3, Hq=32, Hkv=Hkv, q_len=q_len, cur_len=q_len, n_relevant=1, lens=lens)
    eng = Engine(w)
    v0, v1 = device_view(w, 0), device_view(w, 1)
    q0, q1, ck0, cv0, ck1, cv1 = (to_device(x, "bf16") for x in (w.q(0), w.q(1), w.cur_k(0), w.cur_v(0), w.cur_k(1), w.cur_v(1)))
    out, lse = ra.ra_round_sparse_attn_prefill(eng.ctx, q1, v1, None, None, ck1, cv1, scale=w.scale)
    again, lse2 = ra.ra_round_sparse_attn_prefill(eng.ctx, q1, v1, None, None, ck1, cv1, scale=w.scale)
    out2, _, _, S2 = ra.ra_watershed_attn_prefill(eng.ctx, q0, v0, ck0, cv0, scale=w.scale)
    _, S = ra.ra_round_scores(eng.ctx, q0, v0, ck0, scale=w.scale)
    torch.cuda.synchronize()
    assert torch.equal(out, again) and torch.equal(lse, lse2)
    for b in range(w.B):
        rounds = list(range(w.n_rounds(b)))
        for layer, o in ((1, out), (0, out2)):
            assert ora.row_error(o[b].cpu().numpy(), pipeline.attention_for_sequence(w, b, layer, rounds)[0]) < STREAM_TOL, (layer, b)
        rS = pipeline.scores_for_sequence(w, b)[1]
        for got in (S, S2):
            assert np.abs(got[b, :len(rounds)].cpu().numpy() - rS).max() < SCORE_TOL, b
    eng.close()


@pytest.mark.parametrize("q_len,Hq,Hkv", [(88, 256, 16), (112, 512, 32)])
def test_more_rows_than_the_chip_takes_ranges_of(q_len, Hq, Hkv):
    """Workgroups that stream several ranges one after the other, some of which cross from one dialogue into the next: 176
    items a range in the attention kernel (two ranges at a time on 256 units, four handed out), 224 in the score kernel."""
    w = make_workload("cfg3", B=3, Hq=Hq, Hkv=Hkv, q_len=q_len, cur_len=q_len + 3, n_relevant=1, lens=[[400, 33], [5, 500, 64], [100]])
    eng = Engine(w)
    v0, v1 = device_view(w, 0), device_view(w, 1)
    q0, q1, ck0, cv0, ck1, cv1 = (to_device(x, "bf16") for x in (w.q(0), w.q(1), w.cur_k(0), w.cur_v(0), w.cur_k(1), w.cur_v(1)))
    P, S = ra.ra_round_scores(eng.ctx, q0, v0, ck0, scale=w.scale)
    out, _ = ra.ra_round_sparse_attn_prefill(eng.ctx, q1, v1, None, None, ck1, cv1, scale=w.scale)
    out2, _, _, S2 = ra.ra_watershed_attn_prefill(eng.ctx, q0, v0, ck0, cv0, scale=w.scale)
    torch.cuda.synchronize()
    for b in range(w.B):
        rounds = list(range(w.n_rounds(b)))
        rP, rS = pipeline.scores_for_sequence(w, b)
        assert np.abs(P[b, :, :len(rounds)].cpu().numpy() - rP).max() < SCORE_TOL
        assert np.abs(S[b, :len(rounds)].cpu().numpy() - rS).max() < SCORE_TOL
        assert np.abs(S2[b, :len(rounds)].cpu().numpy() - rS).max() < SCORE_TOL
        for layer, o in ((1, out), (0, out2)):
            assert ora.row_error(o[b].cpu().numpy(), pipeline.attention_for_sequence(w, b, layer, rounds)[0]) < STREAM_TOL, (layer, b)
    eng.close()
