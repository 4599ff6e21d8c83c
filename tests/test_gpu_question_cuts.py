"""Questions planned inside their launches at the sizes where the cut into ranges changes: as many key tiles as there are ranges
and one more or fewer, ranges of two to nine tiles, dialogues cut by themselves and ranges that cross, 32 (attention) and 96
(scores) ranges at a time for 8 KV heads."""
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, to_device

pytestmark = pytest.mark.gpu
STREAM_TOL, SCORE_TOL = 5e-5, 1e-5  # P carried to 16 bits, fp32 sums

TILES = [  # key tiles of every dialogue's history; the question's two come on top
    [1], [2], [30], [62], [63], [94], [95], [190], [192],
    [3, 5], [9, 10, 11], [62, 1], [30, 30, 30], [62, 62, 62], [40, 80, 70], [85, 86, 87], [5] * 16, [6] * 17, [1] * 40, [100, 1, 1, 1],
]


@pytest.mark.parametrize("tiles", TILES, ids=lambda t: "-".join(map(str, t)) if len(t) < 6 else f"{len(t)}x{t[0]}")
def test_question_cut(tiles):
    lens = [[32 * (n // 2), 32 * (n - n // 2) - 5] for n in tiles]
    w = make_workload("cfg3", B=len(lens), Hq=8, Hkv=8, q_len=40, cur_len=40, n_relevant=1, lens=lens)
    eng = Engine(w)
    v0, v1 = device_view(w, 0), device_view(w, 1)
    q0, q1, ck0, cv0, ck1, cv1 = (to_device(x, "bf16") for x in (w.q(0), w.q(1), w.cur_k(0), w.cur_v(0), w.cur_k(1), w.cur_v(1)))
    P, S = ra.ra_round_scores(eng.ctx, q0, v0, ck0, scale=w.scale)
    out, lse = ra.ra_round_sparse_attn_prefill(eng.ctx, q1, v1, None, None, ck1, cv1, scale=w.scale)
    out2, _, P2, S2 = ra.ra_watershed_attn_prefill(eng.ctx, q0, v0, ck0, cv0, scale=w.scale)
    torch.cuda.synchronize()
    for b in sorted({0, w.B // 2, w.B - 1}):
        R = w.n_rounds(b)
        rP, rS = (torch.from_numpy(x) for x in pipeline.scores_for_sequence(w, b))
        for gP, gS in ((P, S), (P2, S2)):
            assert (gP[b, :, :R].cpu() - rP).abs().max() < SCORE_TOL and (gS[b, :R].cpu() - rS).abs().max() < SCORE_TOL, b
        for layer, o in ((1, out), (0, out2)):
            ro, rl = pipeline.attention_for_sequence(w, b, layer, list(range(R)))
            assert ora.row_error(o[b].cpu().numpy(), ro) < STREAM_TOL, (layer, b)
        rl = torch.from_numpy(pipeline.attention_for_sequence(w, b, 1, list(range(R)))[1])
        assert (lse[b].cpu() - rl).abs().max() < 2e-5 * max(1.0, rl.abs().max().item()), b
    eng.close()
