"""bf16 with 64 channels: the matrix-core kernels at the edges of their tiles and chunks, and the generic kernels that the
same calls fall back to (inputs that are not 16-byte aligned, many query rows), against the oracle."""
import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra
from oracle import pipeline
from oracle import round_attention as ora
from synth import make_workload
from synth.device import Engine, device_view, sel_to_device, to_device

pytestmark = pytest.mark.gpu
# fp32 sums of exact products of 64 channels, the probabilities carried to 24 bits: 2e-7 of a row, a few ulp of 2^-23
# at its worst entry; ten times that as the bar
OUT_TOL, SCORE_TOL = 2e-6, 1e-5

CASES = {
    "ragged": dict(B=3, lens=[[5, 16, 17, 0, 33, 1, 250], [64, 3, 0, 0, 15, 48, 31], [700, 1, 1, 1, 1, 1, 257]], cur_len=37),
    "ragged_paged": dict(B=2, lens=[[300, 17, 16, 1, 999, 50], [31, 32, 33, 0, 64, 5]], block_size=16, cur_len=1),
    "mha": dict(B=2, Hq=8, R=5, length=("uniform", 10, 200)),
    "g2_no_cur": dict(B=2, Hq=16, R=33, length=("uniform", 1, 60)),
    "g8_paged": dict(B=2, Hq=64, R=9, length=("uniform", 200, 600), block_size=16, cur_len=64),
    "many_rounds": dict(B=3, R=300, length=("uniform", 1, 40), cur_len=5),
    "planned_apart": dict(B=40, R=40, length=("uniform", 1, 90), cur_len=9),   # B * R_max above the inline plan's limit
}


def _offset(t, n):
    """The same values 2 * n bytes past an aligned address."""
    buf = torch.empty(t.numel() + 16, dtype=t.dtype, device=t.device)
    out = buf[n:n + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == 2 * n
    return out


@pytest.mark.parametrize("name", list(CASES))
def test_head64_matches_oracle(name):
    w = make_workload("cfg2", d=64, n_relevant=1, **CASES[name])
    eng = Engine(w)
    v0, v1 = device_view(w, 0, with_v=False), device_view(w, 1)
    q0, q1 = to_device(w.q(0), "bf16"), to_device(w.q(1)[:, 0], "bf16")
    rng = np.random.default_rng(3)
    sels = [sorted(rng.choice(w.n_rounds(b), size=max(1, w.n_rounds(b) // 3), replace=False).tolist()) for b in range(w.B)]
    si, ns = sel_to_device(sels, v1.R_max)
    ck = cv = cl = None
    if w.cur_len:
        ck, cv = to_device(w.cur_k(1), "bf16"), to_device(w.cur_v(1), "bf16")
        cl = torch.full((w.B,), w.cur_len, dtype=torch.int32, device="cuda")
    for q0x, q1x in ((q0, q1), (_offset(q0, 4), _offset(q1, 4))):  # matrix cores; generic kernels
        P, S = ra.ra_round_scores(eng.ctx, q0x, v0, scale=w.scale)
        out, lse = ra.ra_round_sparse_attn_decode(eng.ctx, q1x, v1, si, ns, ck, cv, cl, scale=w.scale)
        again, _ = ra.ra_round_sparse_attn_decode(eng.ctx, q1x, v1, si, ns, ck, cv, cl, scale=w.scale)
        noalloc = torch.empty_like(out)
        ra.ra_round_sparse_attn_decode_noalloc(eng.ctx, q1x, v1, noalloc, None, si, ns, ck, cv, cl, scale=w.scale)
        torch.cuda.synchronize()
        assert torch.equal(out, again) and torch.equal(out, noalloc)
        P, S, out, lse = P.cpu().numpy(), S.cpu().numpy(), out.cpu().numpy(), lse.cpu().numpy()
        for b in sorted({0, w.B // 2, w.B - 1}):
            R = w.n_rounds(b)
            rP, rS = pipeline.scores_for_sequence(w, b)
            assert np.abs(P[b, :, :R] - rP).max() < SCORE_TOL and np.abs(S[b, :R] - rS).max() < SCORE_TOL
            if sum(int(w.lens[b][r]) for r in sels[b]) + w.cur_len == 0:
                continue
            ro, rl = pipeline.attention_for_sequence(w, b, 1, sels[b])
            assert ora.row_error(out[b], ro[0]) < OUT_TOL, b
            assert np.allclose(lse[b], rl[0], rtol=0, atol=1e-5)
    eng.close()


@pytest.mark.parametrize("q_len,Hq", [(2, 32), (4, 32), (2, 64), (5, 32)])  # the last one: 20 rows, the generic kernel
def test_head64_scores_of_several_tokens(q_len, Hq):
    w = make_workload("cfg2", d=64, Hq=Hq, B=2, q_len=q_len, cur_len=q_len + 2, lens=[[300, 31, 0, 33], [17, 256, 257]], n_relevant=1)
    eng = Engine(w)
    P, S = ra.ra_round_scores(eng.ctx, to_device(w.q(0), "bf16"), device_view(w, 0, with_v=False), to_device(w.cur_k(0), "bf16"),
                              scale=w.scale)
    torch.cuda.synchronize()
    for b in range(w.B):
        R = w.n_rounds(b)
        rP, rS = pipeline.scores_for_sequence(w, b)
        assert np.abs(P[b, :, :R].cpu().numpy() - rP).max() < SCORE_TOL and np.abs(S[b, :R].cpu().numpy() - rS).max() < SCORE_TOL
    eng.close()


@pytest.mark.parametrize("last_len", [1, 16, 17, 33])
def test_head64_infinite_value_comes_out_infinite(last_len):
    """An infinite value of a selected token, with weights from exactly one downwards, makes its channel infinite and
    changes no other channel; its place (the last token) is read a second time by a half tile past the round's end."""
    w = make_workload("cfg2", d=64, n_relevant=0, B=1, lens=[[40, last_len]], cur_len=0)
    eng = Engine(w)
    v = device_view(w, 1)
    q = to_device(w.q(1)[:, 0], "bf16")
    for sel in ([1], [0, 1]):
        si, ns = sel_to_device([sel], v.R_max)
        ref, ref_lse = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, si, ns, scale=w.scale)
        nblk, first = (last_len + 15) // 16, 48 * w.Hkv * 64        # round 0 fills 48 tokens of values
        last = v.tensors[1].view(torch.bfloat16).view(-1)[first:first + w.Hkv * nblk * 16 * 64].view(w.Hkv, nblk, 64, 16)
        keep = last.clone()
        last[:, nblk - 1, 7, (last_len - 1) % 16] = float("inf")
        out, lse = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, si, ns, scale=w.scale)
        torch.cuda.synchronize()
        last.copy_(keep)
        assert torch.equal(lse, ref_lse)
        assert torch.isposinf(out[..., 7]).all()
        others = [c for c in range(64) if c != 7]
        assert torch.isfinite(ref).all() and torch.equal(out[..., others], ref[..., others])
    eng.close()


@pytest.mark.parametrize("bits", [20, 40, 60, 80, 90, 100, 110, 120, 125])
def test_head64_infinite_value_with_a_tiny_weight(bits):
    """Two tokens, one 2^-bits of the other and with an infinite value: infinite as long as the weight is not zero, from
    the matrix cores as from the generic kernel."""
    w = make_workload("cfg2", d=64, n_relevant=0, B=1, lens=[[2]], cur_len=0)
    eng = Engine(w)
    v = device_view(w, 1)
    q = torch.zeros((1, w.Hq, 64), dtype=torch.bfloat16, device="cuda")
    q[..., 0] = 1
    keys = v.tensors[0].view(-1)[:w.Hkv * 2 * 64].view(w.Hkv, 2, 64)
    keys.zero_()
    keys[:, 1, 0] = -bits  # exact in bf16
    values = v.tensors[1].view(-1)[:w.Hkv * 64 * 16].view(w.Hkv, 64, 16)
    values[:, 7, 1] = float("inf")
    scale = float(np.log(2.0))
    out, lse = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, scale=scale)
    generic, _ = ra.ra_round_sparse_attn_decode(eng.ctx, _offset(q, 4), v, scale=scale)
    torch.cuda.synchronize()
    others = [c for c in range(64) if c != 7]
    assert torch.isposinf(generic[..., 7]).all() and torch.isposinf(out[..., 7]).all()
    assert (out[..., others] - generic[..., others]).abs().max() < OUT_TOL * generic[..., others].abs().max()
    assert lse.abs().max() < 2.0 ** -bits + 1e-7
    eng.close()
