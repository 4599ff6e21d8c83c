"""Decode on the matrix cores where its prologue and its merge change form: batches whose tables take a quarter, a half or
all of a wave's lanes, or several passes of them; sequences cut into as many records as the merge has in flight, one more
and one less, with a workgroup per row and with several rows to one."""
import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, sel_to_device, to_device

pytestmark = pytest.mark.gpu
TOL = {128: 5e-5, 64: 2e-6}  # the weights carried to 16 bits; to 24 with 64 channels


def check(w, sels, check_b):
    eng = Engine(w)
    v = device_view(w, 1)
    q = to_device(w.q(1)[:, 0], "bf16")
    si, ns = sel_to_device(sels, v.R_max)
    ck = cv = cl = None
    if w.cur_len:
        ck, cv = to_device(w.cur_k(1), "bf16"), to_device(w.cur_v(1), "bf16")
        cl = torch.full((w.B,), w.cur_len, dtype=torch.int32, device="cuda")
    out, lse = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, si, ns, ck, cv, cl, scale=w.scale)
    again, _ = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, si, ns, ck, cv, cl, scale=w.scale)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    for b in check_b:
        ro, rl = pipeline.attention_for_sequence(w, b, 1, sels[b])
        assert ora.row_error(out[b], ro[0]) < TOL[w.d], b
        assert np.allclose(lse[b], rl[0], rtol=0, atol=1e-5)
    eng.close()


# (B, R): table entries R + 1 up to 16, 32, 64 and more; 256 and 257 .. 1024 list entries; 64 sequences
@pytest.mark.parametrize("B,R", [(1, 1), (5, 15), (4, 16), (9, 31), (8, 32), (3, 63), (4, 64), (2, 65), (64, 4), (64, 16), (13, 20), (10, 100)])
def test_the_inline_plan(B, R):
    rng = np.random.default_rng(B * 1000 + R)
    lens = [rng.choice([0, 1, 16, 31, 32, 33, 70], size=R).tolist() for _ in range(B)]
    for row in lens:
        row[rng.integers(R)] = 40
    w = make_workload("cfg2", B=B, Hq=8, Hkv=2, lens=lens, n_relevant=0, cur_len=0 if R == 15 else 21)
    sels = [sorted(rng.choice(R, size=max(1, 2 * R // 3), replace=False).tolist()) for _ in range(B)]
    for b in range(B):  # no empty key set (the oracle has none)
        if not any(lens[b][r] for r in sels[b]):
            sels[b] = [int(np.argmax(lens[b]))]
    check(w, sels, sorted({0, B // 2, B - 1}))


# one dialogue of one round: records = tiles / 2 up to 384 tiles, / 4 above; 64 (d = 64: 128) are in flight at a time
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (6, 2), (16, 1)])
@pytest.mark.parametrize("tiles", [1, 4, 18, 126, 129, 131, 255, 258, 384, 385])
def test_one_dialogue_in_many_records(tiles, Hq, Hkv, d):
    if d == 64 and Hq // Hkv not in (1, 2, 4, 8):
        Hq = 8 * Hkv
    w = make_workload("cfg2", B=1, Hq=Hq, Hkv=Hkv, d=d, lens=[[32 * tiles - 5]], n_relevant=0, cur_len=0)
    check(w, [[0]], [0])


# more rows than are merged by a workgroup each: 1, 2, 3, 4 and 8 of them to one
@pytest.mark.parametrize("B,Hq,Hkv", [(40, 32, 32), (40, 32, 16), (24, 48, 16), (40, 32, 8), (20, 64, 8)])
def test_many_rows_in_few_records(B, Hq, Hkv):
    w = make_workload("cfg2", B=B, Hq=Hq, Hkv=Hkv, lens=[[290 + 7 * b, 33] for b in range(B)], n_relevant=0, cur_len=9)
    check(w, [[0, 1]] * B, [0, B // 2, B - 1])


# more rows than are merged by a workgroup each, one dialogue of as many tiles as still allow ranges of two, or of one more
@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("B,Hq,Hkv,d,longest", [(17, 64, 8, 128, 96), (34, 32, 2, 128, 96), (64, 32, 8, 128, 191), (17, 64, 8, 64, 96), (64, 32, 8, 64, 192)])
def test_a_long_dialogue_among_short_ones(B, Hq, Hkv, d, longest, more):
    lens = [[32 * (longest + more) - 3]] + [[17]] * (B - 1)
    w = make_workload("cfg2", B=B, Hq=Hq, Hkv=Hkv, d=d, lens=lens, n_relevant=0, cur_len=0)
    check(w, [[0]] * B, [0, 1, B - 1])


# dialogues cut each by itself (up to a twelfth as many as there may be ranges) and one more than that, some of them empty
@pytest.mark.parametrize("B,Hq,Hkv,d", [(2, 16, 2, 128), (10, 32, 8, 128), (11, 32, 8, 128), (21, 32, 8, 64), (22, 32, 8, 64), (42, 16, 2, 128), (43, 16, 2, 128)])
def test_dialogues_cut_each_by_itself(B, Hq, Hkv, d):
    rng = np.random.default_rng(B)
    lens = rng.integers(0, 400, size=(B, 4)).tolist()
    lens[0] = [0, 0, 0, 1]
    lens[B // 2] = [0, 0, 0, 0]
    w = make_workload("cfg2", B=B, Hq=Hq, Hkv=Hkv, d=d, lens=lens, n_relevant=0, cur_len=0)
    check(w, [[0, 1, 3]] * B, [b for b in (0, 1, B - 1) if b != B // 2])


# ... and as far as their ranges are short: tiles of the batch for each range that there may be, and one more tile, which is cut
# as one list; 5 tiles and two dialogues of unequal length take the second of the lengths that are tried
@pytest.mark.parametrize("d,per_range,more", [(128, 5, 0), (128, 12, 0), (128, 12, 1), (64, 5, 0), (64, 5, 1)])
def test_dialogues_cut_each_by_itself_while_ranges_are_short(d, per_range, more):
    ranges = torch.cuda.get_device_properties(0).multi_processor_count * (4 if d == 128 else 8) // 8
    tiles = per_range * ranges + more
    first = 32 * (tiles // 3) - 7
    w = make_workload("cfg2", B=2, Hq=32, Hkv=8, d=d, lens=[[first], [32 * (tiles - tiles // 3) - 30]], n_relevant=0, cur_len=0)
    check(w, [[0], [0]], [0, 1])
