"""Question scores whose rounds are cut by the ranges of key tiles: one long round in many parts, rounds that end where a range
does, empty ones in between, more rounds than a lane has one of, batches planned apart, and a workspace without room for all
the parts that the launch would cut."""
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from synth import make_workload
from synth.device import Engine, device_view, to_device

pytestmark = pytest.mark.gpu
SCORE_TOL = 1e-5  # the bar of the other parity tests: fp32 sums

CASES = {
    "one_long_round": dict(q_len=40, Hq=32, Hkv=8, lens=[[9000], [0, 3, 31]]),
    "ends_of_ranges": dict(q_len=33, Hq=16, Hkv=8, lens=[[64] * 40, [32, 0, 0, 96, 1, 63, 0], [2048, 0, 2048]], block_size=16),
    "70_rounds": dict(q_len=9, Hq=32, Hkv=8, lens=[[33, 0, 700, 64, 1] * 14]),
    "300_rounds": dict(q_len=12, Hq=32, Hkv=8, lens=[[32, 5, 0] * 100]),
    "planned_apart": dict(q_len=20, Hq=16, Hkv=8, lens=[[300, 0, 17]] * 65 + [[4000, 100, 1]]),
    "one_kv_head": dict(q_len=17, Hq=16, Hkv=1, lens=[[3000, 40, 2500]]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_scores_of_cut_rounds(name):
    over = dict(CASES[name])
    w = make_workload("cfg3", B=len(over["lens"]), cur_len=over["q_len"] + 5, n_relevant=1, **over)
    eng = Engine(w)
    v, q, ck, cv = device_view(w, 0), *(to_device(x, "bf16") for x in (w.q(0), w.cur_k(0), w.cur_v(0)))
    P, S, sel, n = ra.ra_round_scores_select(eng.ctx, q, v, cur_k=ck, scale=w.scale)
    two = ra.ra_round_scores(eng.ctx, q, v, ck, scale=w.scale)
    _, _, P2, S2 = ra.ra_watershed_attn_prefill(eng.ctx, q, v, ck, cv, scale=w.scale)
    torch.cuda.synchronize()
    assert torch.equal(S, two[1]) and torch.equal(P, two[0])
    for b in sorted({0, 1 % w.B, w.B - 1}):
        R = w.n_rounds(b)
        rP, rS = (torch.from_numpy(x) for x in pipeline.scores_for_sequence(w, b))
        for gP, gS in ((P, S), (P2, S2)):
            assert (gP[b, :, :R].cpu() - rP).abs().max() < SCORE_TOL and (gS[b, :R].cpu() - rS).abs().max() < SCORE_TOL, b
    eng.close()


@pytest.mark.parametrize("parts", [1, 2, 3, 20])
def test_a_workspace_for_fewer_parts_is_enough(parts):
    """One round of 20 000 tokens, which a roomy workspace has cut into as many parts as there are ranges.  The least that the
    call takes holds one value per row and 256-token chunk."""
    w = make_workload("cfg3", B=1, q_len=24, cur_len=24, Hq=16, Hkv=8, n_relevant=1, lens=[[20000]])
    eng = Engine(w)
    v, q, ck = device_view(w, 0), to_device(w.q(0), "bf16"), to_device(w.cur_k(0), "bf16")
    roomy = ra.ra_round_scores(eng.ctx, q, v, ck, scale=w.scale)
    tokens = 20000 if parts == 20 else 256 * parts - 256  # (a caller that understates max_tokens gets NaN, and no write out of range)
    k, vv, seg_off, seg_len, n_rounds, _, seg_off_v = v.tensors
    small_view = ra.KVView(k, vv, seg_off, seg_len, n_rounds, v.Hkv, v.d, tokens, seg_off_v=seg_off_v)
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    rows, chunks = 24 * 16, tokens // 256 + 1 + 1
    least = 32768 + up(rows * chunks * 4) + up(16 * 4) + up((2 * 24 + 4 + 16 + 15) // 16 * 16)
    guard = torch.full((least + 4096,), 77, dtype=torch.uint8, device="cuda")
    ra.ra_set_workspace(eng.ctx, guard[:least])
    tight = ra.ra_round_scores(eng.ctx, q, small_view, ck, scale=w.scale)
    torch.cuda.synchronize()
    assert (guard[least:] == 77).all()
    if parts == 20:
        assert all((x - y).abs().max() < SCORE_TOL for x, y in zip(roomy, tight))
    else:
        assert torch.isnan(tight[1]).all()
    ra.ra_set_workspace(eng.ctx, guard[:least - 256])
    with pytest.raises(ra.RaError):
        ra.ra_round_scores(eng.ctx, q, small_view, ck, scale=w.scale)
    eng.close()
