"""The kernel that merges the partial results of split rows (fp32 decode, the 64-channel fallback, questions of many rows)
at the piece counts around the four it has in flight."""
import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra
from synth import make_workload
from synth.device import Engine, device_view, to_device

pytestmark = pytest.mark.gpu
PIECES = [2, 3, 4, 5, 6, 7, 9]


def _decode_case(dtype, d, pieces, last=128):
    """One dialogue of one round cut into `pieces` pieces of 128 tokens (eight 16-token units, the smallest piece)."""
    w = make_workload("cfg2", dtype=dtype, d=d, B=1, lens=[[128 * (pieces - 1) + last]], n_relevant=0, cur_len=0)
    q = to_device(w.q(1)[:, 0], dtype)
    if dtype == "bf16":  # off a 16-byte boundary: the generic kernels
        q = torch.empty(q.numel() + 8, dtype=q.dtype, device="cuda")[4:4 + q.numel()].view(q.shape).copy_(q)
    return w, Engine(w), device_view(w, 1), q


@pytest.mark.parametrize("pieces", PIECES)
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
def test_an_infinite_value_of_the_last_piece_comes_out_infinite(dtype, d, pieces):
    w, eng, v, q = _decode_case(dtype, d, pieces)
    ref, ref_lse = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, scale=w.scale)
    v.tensors[1].view(-1)[:w.Hkv * 128 * pieces * d].view(w.Hkv, 8 * pieces, d, 16)[:, -1, 7, 15] = float("inf")
    out, lse = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, scale=w.scale)
    torch.cuda.synchronize()
    others = [c for c in range(d) if c != 7]
    assert torch.isposinf(out[..., 7]).all()
    assert torch.isfinite(ref).all() and torch.equal(out[..., others], ref[..., others]) and torch.equal(lse, ref_lse)
    eng.close()


@pytest.mark.parametrize("d", [64, 128])
def test_the_output_may_lie_anywhere(d):
    """A buffer of floats that starts 4, 8 or 12 bytes past a 16-byte boundary."""
    w, eng, v, q = _decode_case("f32", d, 3)
    ref, ref_lse = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, scale=w.scale)
    for n in (1, 2, 3):
        buf = torch.full((ref.numel() + 8,), 5.0, device="cuda")
        out, lse = ra.ra_round_sparse_attn_decode(eng.ctx, q, v, scale=w.scale, out=buf[n:n + ref.numel()].view(ref.shape))
        torch.cuda.synchronize()
        assert out.data_ptr() % 16 == 4 * n and torch.equal(out, ref) and torch.equal(lse, ref_lse)
        assert (buf[:n] == 5).all() and (buf[n + ref.numel():] == 5).all()
    eng.close()


@pytest.mark.parametrize("pieces", PIECES)
def test_an_infinite_value_of_a_question_comes_out_infinite(pieces):
    """A dialogue of one round and a question of 20 tokens: 8 key tiles a piece (with room declared for more tokens, or the
    cut would be into fewer), the question's own tile the last one.  The token with the infinite value has a key of zeros,
    so that no row takes its weight, exactly one then, as reference."""
    n = 32 * (8 * pieces - 1)
    w = make_workload("cfg3", B=1, Hq=32, Hkv=8, q_len=20, cur_len=20, lens=[[n]], n_relevant=0)
    eng = Engine(w, extra_tokens=4096)
    k, values, off, ln, nr, _, off_v = device_view(w, 1).tensors
    v = ra.KVView(k, values, off, ln, nr, w.Hkv, w.d, n + 4096, seg_off_v=off_v)
    q, ck, cv = to_device(w.q(1), "bf16"), to_device(w.cur_k(1), "bf16"), to_device(w.cur_v(1), "bf16")
    v.tensors[0].view(-1)[:w.Hkv * n * w.d].view(w.Hkv, n, w.d)[:, -1] = 0
    ref, ref_lse = ra.ra_round_sparse_attn_prefill(eng.ctx, q, v, None, None, ck, cv, scale=w.scale)
    v.tensors[1].view(-1)[:w.Hkv * n * w.d].view(w.Hkv, n // 16, w.d, 16)[:, -1, 7, 15] = float("inf")
    out, lse = ra.ra_round_sparse_attn_prefill(eng.ctx, q, v, None, None, ck, cv, scale=w.scale)
    torch.cuda.synchronize()
    others = [c for c in range(w.d) if c != 7]
    assert torch.isposinf(out[..., 7]).all()
    assert torch.isfinite(ref).all() and torch.equal(out[..., others], ref[..., others]) and torch.equal(lse, ref_lse)
    eng.close()


@pytest.mark.parametrize("pieces", PIECES)
@pytest.mark.parametrize("d", [64, 128])
def test_the_merged_output_is_the_correctly_rounded_quotient(d, pieces):
    """With a query of zeros every weight is one, and sums of small whole numbers are exact: what is left to round is the
    division by the sum of the weights."""
    w, eng, v, q = _decode_case("f32", d, pieces, last=77)
    n, tiles = 128 * (pieces - 1) + 77, 8 * pieces - 3
    values = v.tensors[1].view(-1)[:w.Hkv * tiles * 16 * d].view(w.Hkv, tiles, d, 16)
    values.copy_(torch.randint(-50, 200, values.shape, generator=torch.Generator().manual_seed(pieces)))
    out, _ = ra.ra_round_sparse_attn_decode(eng.ctx, torch.zeros_like(q), v, scale=w.scale)
    total = values.permute(0, 1, 3, 2).reshape(w.Hkv, -1, d)[:, :n].double().sum(1).float()
    want = (total.cpu().numpy() / np.float32(n)).repeat(w.Hq // w.Hkv, axis=0)
    assert np.array_equal(out[0].cpu().numpy(), want)
    eng.close()
