"""fp32 calls at the edges of their 16-token units, tiles of values and 256-token chunks, for every number of heads per KV
head and both head dimensions, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, sel_to_device, to_device

pytestmark = pytest.mark.gpu
# fp32 products and sums of up to 128 channels and 1100 tokens: 4e-7 of a row; ten times that
OUT_TOL, SCORE_TOL = 4e-6, 1e-5

LENS = [[1, 15, 16, 17, 31, 0, 33], [255, 256, 257, 0, 3, 272, 64], [1030, 0, 0, 0, 0, 0, 5]]


@pytest.mark.parametrize("block_size", [0, 16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(3, 3), (4, 2), (8, 2), (16, 2)])
def test_fp32_step(Hq, Hkv, d, block_size):
    w = make_workload("cfg2", dtype="f32", B=3, Hq=Hq, Hkv=Hkv, d=d, lens=LENS, n_relevant=1, block_size=block_size, cur_len=19)
    eng = Engine(w)
    v0, v1 = device_view(w, 0, with_v=False), device_view(w, 1)
    q0, q1, ck, cv = (to_device(x, "f32") for x in (w.q(0), w.q(1)[:, 0], w.cur_k(1), w.cur_v(1)))
    cl = torch.full((w.B,), w.cur_len, dtype=torch.int32, device="cuda")
    sels = [[0, 2, 3, 6], [1, 2, 5], [0]]
    si, ns = sel_to_device(sels, v1.R_max)
    P, S = ra.ra_round_scores(eng.ctx, q0, v0, scale=w.scale)
    out, lse = ra.ra_round_sparse_attn_decode(eng.ctx, q1, v1, si, ns, ck, cv, cl, scale=w.scale)
    again, _ = ra.ra_round_sparse_attn_decode(eng.ctx, q1, v1, si, ns, ck, cv, cl, scale=w.scale)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    P, S, out, lse = (x.cpu().numpy() for x in (P, S, out, lse))
    for b in range(w.B):
        R = w.n_rounds(b)
        rP, rS = pipeline.scores_for_sequence(w, b)
        assert np.abs(P[b, :, :R] - rP).max() < SCORE_TOL and np.abs(S[b, :R] - rS).max() < SCORE_TOL
        ro, rl = pipeline.attention_for_sequence(w, b, 1, sels[b])
        assert ora.row_error(out[b], ro[0]) < OUT_TOL, b
        assert np.allclose(lse[b], rl[0], rtol=0, atol=1e-5)
    eng.close()
