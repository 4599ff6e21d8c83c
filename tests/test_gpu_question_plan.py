"""Questions planned inside their launches at the sizes where the plan takes more than one pass of a wave's lanes: dialogues
of about 64 and 128 segments, more than 64 ranges, list entries beyond one per thread."""
import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, sel_to_device, to_device

pytestmark = pytest.mark.gpu
STREAM_TOL, SCORE_TOL = 5e-5, 1e-5  # P carried to 16 bits, fp32 sums

CASES = {
    **{f"{R}_rounds": dict(B=2, R=R, q_len=9, Hq=32, Hkv=8, length=("uniform", 0, 60)) for R in (62, 63, 64, 127, 129)},
    "list_of_256": dict(B=4, R=64, q_len=17, Hq=16, Hkv=8, length=("uniform", 0, 20), block_size=16),
    "list_of_257": dict(B=1, R=257, q_len=17, Hq=16, Hkv=8, length=("uniform", 0, 20)),
    "many_ranges": dict(B=2, q_len=9, Hq=16, Hkv=1, lens=[[900, 5000, 33, 4000], [6000, 64, 5500]]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_question_plan(name):
    over = dict(CASES[name])
    w = make_workload("cfg3", cur_len=over["q_len"], n_relevant=1, **over)
    eng = Engine(w)
    v0, v1 = device_view(w, 0), device_view(w, 1)
    dev = lambda x: to_device(x, "bf16")  # noqa: E731
    ck0, cv0, ck1, cv1 = dev(w.cur_k(0)), dev(w.cur_v(0)), dev(w.cur_k(1)), dev(w.cur_v(1))
    P, S = ra.ra_round_scores(eng.ctx, dev(w.q(0)), v0, ck0, scale=w.scale)
    rng = np.random.default_rng(5)
    sels = [sorted(rng.choice(w.n_rounds(b), size=(2 * w.n_rounds(b) + 2) // 3, replace=False).tolist()) for b in range(w.B)]
    si, ns = sel_to_device(sels, v1.R_max)
    out, lse = ra.ra_round_sparse_attn_prefill(eng.ctx, dev(w.q(1)), v1, si, ns, ck1, cv1, scale=w.scale)
    out2, _, _, S2 = ra.ra_watershed_attn_prefill(eng.ctx, dev(w.q(0)), v0, ck0, cv0, scale=w.scale)
    torch.cuda.synchronize()
    P, S, out, lse, out2, S2 = (x.cpu().numpy() for x in (P, S, out, lse, out2, S2))
    for b in range(w.B):
        R = w.n_rounds(b)
        rP, rS = pipeline.scores_for_sequence(w, b)
        assert np.abs(P[b, :, :R] - rP).max() < SCORE_TOL and np.abs(S[b, :R] - rS).max() < SCORE_TOL, b
        assert np.abs(S2[b, :R] - rS).max() < SCORE_TOL, b
        assert ora.row_error(out2[b], pipeline.attention_for_sequence(w, b, 0, list(range(R)))[0]) < STREAM_TOL, b
        ro, rl = pipeline.attention_for_sequence(w, b, 1, sels[b])
        assert ora.row_error(out[b], ro) < STREAM_TOL, b
        assert np.allclose(lse[b], rl, rtol=0, atol=2e-5 * max(1.0, np.abs(rl).max())), b
    eng.close()
