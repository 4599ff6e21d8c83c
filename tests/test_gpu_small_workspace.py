"""Calls whose workspace has room for ranges of four key tiles and not for ones of two, or for few partial results of a question's
rows: they take longer ranges."""
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, to_device

pytestmark = pytest.mark.gpu
STREAM_TOL, SCORE_TOL = 5e-5, 1e-5  # the bars of the other parity tests


def _bytes_for(w, units, score_bytes):
    """Head, segment tables, and one record of 16 rows per (range or sequence, KV head, block of 16 rows)."""
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    tiles = w.B * (sum(w.lens[0]) // 32 + w.R_max + w.cur_len // 32 + 1)
    inner = w.Hkv * ((w.q_len * w.Hq // w.Hkv + 15) // 16)
    records = (tiles // units + w.B) * inner * 16
    plan = w.B * (((w.R_max + 1) * 24 + 4 + 16 + 15) // 16 * 16)
    return 32768 + up(plan) + up(records * w.d * 4) + up(records * 8) + score_bytes


@pytest.mark.parametrize("what", ["decode", "watershed_decode", "question", "watershed_question"])
def test_a_workspace_for_four_tile_ranges_is_enough(what):
    q_len = 5 if "question" in what else 1
    w = make_workload("cfg2", B=1, q_len=q_len, cur_len=q_len, lens=[[700, 33, 250]], n_relevant=1)
    layer = 0 if "watershed" in what else 1
    v, ck, cv = device_view(w, layer), to_device(w.cur_k(layer), "bf16"), to_device(w.cur_v(layer), "bf16")
    q = to_device(w.q(layer), "bf16")
    cl = torch.full((1,), w.cur_len, dtype=torch.int32, device="cuda")
    units = sum(w.lens[0]) // 32 + 3 + 1
    score_bytes = 0
    if layer == 0:
        score_bytes = (q_len * w.Hq * units * 4 + 255) // 256 * 256 + (w.Hq * 3 * 4 + 255) // 256 * 256 * (q_len > 1)

    def call(ctx):
        if what == "decode":
            return ra.ra_round_sparse_attn_decode(ctx, q[:, 0].contiguous(), v, None, None, ck, cv, cl, scale=w.scale)
        if what == "watershed_decode":
            return ra.ra_watershed_attn_decode(ctx, q[:, 0].contiguous(), v, ck, cv, cl, scale=w.scale)
        if what == "question":
            return ra.ra_round_sparse_attn_prefill(ctx, q, v, None, None, ck, cv, scale=w.scale)
        return ra.ra_watershed_attn_prefill(ctx, q, v, ck, cv, scale=w.scale)

    eng = Engine(w)
    roomy = call(eng.ctx)
    n = _bytes_for(w, 4, score_bytes)
    assert n < _bytes_for(w, 2, score_bytes) <= eng.workspace.numel()
    small = torch.empty(n, dtype=torch.uint8, device="cuda")
    ra.ra_set_workspace(eng.ctx, small)
    tight = call(eng.ctx)
    again = call(eng.ctx)
    torch.cuda.synchronize()
    ro, _ = pipeline.attention_for_sequence(w, 0, layer, [0, 1, 2])
    for got in (roomy, tight):
        assert ora.row_error(got[0][0].cpu().numpy().reshape(ro.shape), ro) < STREAM_TOL
    for x, y, z in zip(roomy, tight, again):
        assert torch.equal(y, z) and (x - y).abs().max() < max(STREAM_TOL, SCORE_TOL) * max(1.0, x.abs().max().item())
    ra.ra_set_workspace(eng.ctx, small[:n - 4096])
    with pytest.raises(ra.RaError):
        call(eng.ctx)
    eng.close()


@pytest.mark.parametrize("lens,parts", [([700, 33, 1250], 9), ([700, 33, 1250], 13), ([300, 20], 3), ([2] * 1000, 9)],
                         ids=["2000_9", "2000_13", "320_3", "1000_rounds"])
def test_a_question_with_room_for_a_few_parts(lens, parts):
    """160 query rows per KV head, the workspace with room for so many partial results of a row: ranges as short as those take."""
    w = make_workload("cfg3", B=1, q_len=40, cur_len=40, Hq=8, Hkv=2, lens=[lens], n_relevant=1)
    R, rows = len(lens), 40 * w.Hq
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    n = 32768 + up(((R + 1) * 24 + 4 + 16 + 15) // 16 * 16) + up(rows * parts * w.d * 4) + 2 * up(rows * parts * 4)
    n += up(rows * max(R + parts, sum(lens) // 256 + R + 1) * 4) + up(w.Hq * R * 4)
    eng = Engine(w)
    workspace = torch.empty(n, dtype=torch.uint8, device="cuda")
    ra.ra_set_workspace(eng.ctx, workspace)
    for layer in (0, 1):
        v, ck, cv = device_view(w, layer), to_device(w.cur_k(layer), "bf16"), to_device(w.cur_v(layer), "bf16")
        q = to_device(w.q(layer), "bf16")
        got = ra.ra_watershed_attn_prefill(eng.ctx, q, v, ck, cv, scale=w.scale) if layer == 0 else \
            ra.ra_round_sparse_attn_prefill(eng.ctx, q, v, None, None, ck, cv, scale=w.scale)
        torch.cuda.synchronize()
        ro, _ = pipeline.attention_for_sequence(w, 0, layer, list(range(R)))
        assert ora.row_error(got[0][0].cpu().numpy().reshape(ro.shape), ro) < STREAM_TOL
        if layer == 0:
            rP, rS = (torch.from_numpy(x) for x in pipeline.scores_for_sequence(w, 0))
            assert (got[2][0].cpu() - rP).abs().max() < SCORE_TOL and (got[3][0].cpu() - rS).abs().max() < SCORE_TOL
    eng.close()
