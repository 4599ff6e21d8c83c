"""The extension module that the compute calls go through: what it refuses, and how, without a GPU."""
import ctypes

import pytest
import torch

import paper_2502_15294_amd as ra


def view(B=1, R=3, Hkv=2, d=64):
    k = torch.zeros(B * R * 16 * Hkv * d)
    lens = torch.full((B, R), 16, dtype=torch.int32)
    off = (torch.arange(R) * 16).repeat(B, 1)
    return ra.KVView(k, k.clone(), off, lens, torch.full((B,), R, dtype=torch.int32), Hkv, d, R * 16)


CALLS = {
    "scores": (ra.ra_round_scores, 4), "scores_select": (ra.ra_round_scores_select, 4), "decode": (ra.ra_round_sparse_attn_decode, 3),
    "watershed_decode": (ra.ra_watershed_attn_decode, 3), "prefill": (ra.ra_round_sparse_attn_prefill, 4),
    "watershed_prefill": (ra.ra_watershed_attn_prefill, 4),
}


@pytest.mark.parametrize("name", CALLS)
def test_errors_reach_the_caller(name):
    call, dims = CALLS[name]
    q = torch.zeros((1, 2, 4, 64) if dims == 4 else (1, 4, 64))
    with pytest.raises(ra.RaError, match="ctx is NULL") as e:  # a status of the library
        call(None, q, view(), stream=0)
    assert e.value.code == ra.RA_ERR_INVALID_ARG
    with pytest.raises(ra.RaError, match="ctx is NULL"):  # a context handle that holds nothing
        call(ctypes.c_void_p(), q, view(), stream=0)
    with pytest.raises(AssertionError, match="contiguous"):
        call(None, q.transpose(1, 2), view(), stream=0)
    with pytest.raises(ValueError):
        call(None, q[0], view(), stream=0)
    with pytest.raises(TypeError):
        call(None, q.numpy(), view(), stream=0)
    with pytest.raises(AttributeError):
        call(None, q, None, stream=0)
    with pytest.raises(TypeError):
        call(None, q, view(), scale="1", stream=0)


def test_accumulate_and_coverage_errors():
    q, v = torch.zeros(1, 1, 4, 64), view()
    for acc in (torch.zeros(1, 4, 2), torch.zeros(1, 4, 3, dtype=torch.float64)):
        with pytest.raises(AssertionError, match="acc"):
            ra.ra_round_scores_accumulate(None, q, v, acc, stream=0)
    with pytest.raises(ra.RaError):
        ra.ra_round_scores_accumulate(None, q, v, torch.zeros(1, 4, 3), stream=0)
    with pytest.raises(ra.RaError):
        ra.ra_selection_coverage(None, torch.zeros(1, 3), torch.zeros(1, 3, dtype=torch.int32), torch.zeros(1, dtype=torch.int32),
                                 stream=0)


def test_structures_are_checked():
    q = torch.zeros(1, 1, 4, 64)
    with pytest.raises(TypeError):
        ra.ra_round_scores_select(None, q, view(), params=ctypes.c_int(0), stream=0)

    class Other:
        c = ctypes.c_int(0)

    with pytest.raises(TypeError):
        ra.ra_round_scores(None, q, Other(), stream=0)


@pytest.mark.gpu
def test_outputs_are_the_callers_or_new():
    from synth import make_workload
    from synth.device import Engine, device_view, to_device
    w = make_workload("cfg2", B=2, R=6, length=("uniform", 20, 200))
    eng = Engine(w)
    q, v = to_device(w.q(0), w.dtype), device_view(w, 0, with_v=False)
    new = ra.ra_round_scores_select(eng.ctx, q, v, scale=w.scale)
    assert [t.dtype for t in new] == [torch.float32, torch.float32, torch.int32, torch.int32]
    assert [tuple(t.shape) for t in new] == [(2, w.Hq, 6), (2, 6), (2, 6), (2,)]
    given = [torch.empty_like(t) for t in new]
    got = ra.ra_round_scores_select(eng.ctx, q, v, None, None, w.scale, *given)
    assert all(a is b for a, b in zip(got, given))
    assert all(torch.equal(a, b) for a, b in zip(got, new))
    with pytest.raises(AssertionError, match="contiguous"):
        ra.ra_round_scores(eng.ctx, q, v, scores=torch.empty(6, 2, device="cuda").T)
    eng.close()
