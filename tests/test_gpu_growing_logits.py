"""Question kernels over keys whose logits grow along a round: the softmax reference is set by the first tile of a range and
raised again and again behind it, by a little, by much within one tile, and after mass has gathered just below the line."""
import math

import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, to_device
from synth.workloads import Workload, _store_round

pytestmark = pytest.mark.gpu
# A logit of at most 45 from 128 fp32 products is off by at most a few times sqrt(128) * 45 * 2^-24 = 3e-5, its exponential by as much
# of itself, and a share of the mass by half of that, in both directions
SCORE_TOL = 6e-5
# rows of the output: as above, and the weights carried to 16 bits (5e-5 in the other question tests)
OUT_TOL = 1.5e-4

PEAK = 40.0  # natural logarithms: the log-sum-exp of every profile's chunk
STEP = math.log(2.0)


def steps(*parts):
    return np.concatenate([np.full(n, level * STEP) for n, level in parts])


# logits along 256 tokens, a chunk of a round: eight tiles of 32
PROFILES = [
    # seven eighths of what raises the reference gathers below the line, then half as much again crosses it; twice
    steps((32, 0), (96, 12.5), (32, 13.5), (64, 26), (32, 27)),
    np.linspace(-100, 0, 256),                    # raised on every tile, by 2^18 each
    steps((32, -190), (5, -190), (27, 0), (192, 0)),  # beyond the range of fp32 within a tile
    np.linspace(0, -100, 256),                    # never raised again
    steps((200, 0), (56, 15)),
    steps((64, 0), (64, 9), (64, 18), (64, 27)),
]


class Growing(Workload):
    """Queries near one direction, keys along it: the logits follow the profiles, with a little noise."""

    def _direction(self):
        return np.where(np.arange(self.d) % 3 == 0, 1, -1).astype(np.float32) / np.float32(math.sqrt(self.d))

    def q(self, layer=0):
        return _store_round(np.float32(0.1) * super().q(layer) + np.float32(16) * self._direction(), self.dtype)

    def k_round(self, b, layer, r):
        noise = super().k_round(b, layer, r)
        p = PROFILES[(b + r) % len(PROFILES)]
        logit = np.resize(p - np.logaddexp.reduce(p) + PEAK + 0.2 * r, noise.shape[0])
        along = (logit / (self.scale * 16)).astype(np.float32)
        return _store_round(np.float32(0.1) * noise + along[:, None, None] * self._direction(), self.dtype)


# one chunk to a range; several of them; paged; a batch whose ranges cross dialogues
@pytest.mark.parametrize("B,chunks,block_size", [(1, 1, 0), (2, 3, 0), (2, 3, 16), (12, 2, 0)])
@pytest.mark.parametrize("q_len", [9, 40])
def test_growing_logits(B, chunks, block_size, q_len):
    w = make_workload("cfg3", B=B, Hq=8, Hkv=2, q_len=q_len, cur_len=q_len, n_relevant=0, block_size=block_size,
                      lens=[[256 * chunks - (7 if r == 4 else 0) for r in range(6)] for _ in range(B)])
    w.__class__ = Growing
    eng = Engine(w)
    v = device_view(w, 0)
    q, ck, cv = (to_device(x, "bf16") for x in (w.q(0), w.cur_k(0), w.cur_v(0)))
    P, S = ra.ra_round_scores(eng.ctx, q, v, ck, scale=w.scale)
    out, _, P2, S2 = ra.ra_watershed_attn_prefill(eng.ctx, q, v, ck, cv, scale=w.scale)
    torch.cuda.synchronize()
    P, S, out, P2, S2 = (x.cpu().numpy() for x in (P, S, out, P2, S2))
    for b in sorted({0, B // 2, B - 1}):
        rP, rS = pipeline.scores_for_sequence(w, b)
        assert np.sort(rS)[0] > 0.01  # every round's mass counts
        for p, s in ((P, S), (P2, S2)):
            assert np.abs(p[b] - rP).max() < SCORE_TOL and np.abs(s[b] - rS).max() < SCORE_TOL, b
        ro, _ = pipeline.attention_for_sequence(w, b, 0, list(range(6)))
        assert ora.row_error(out[b], ro) < OUT_TOL, b
    eng.close()
