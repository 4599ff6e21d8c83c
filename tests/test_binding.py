"""The extension module that the compute calls go through: what it refuses, and how, without a GPU."""
import ctypes
import threading
import time

import numpy as np
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


class Adapter:
    def __init__(self, value):
        self._as_parameter_ = value


class Handle(ctypes.c_void_p):
    pass


class View(ra.ra_kv_view):
    pass


class Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


# what ctypes takes as a handle or a number, and what it refuses although it has memory of the right size; all handles are null,
# so that the library itself ends every call that gets through
@pytest.mark.parametrize("ctx", [0, 1 << 64, Handle(), ctypes.POINTER(ctypes.c_int)(), Adapter(None), Adapter(ctypes.c_void_p())])
def test_handles_that_are_taken(ctx):
    with pytest.raises(ra.RaError, match="ctx is NULL"):
        ra.ra_round_scores(ctx, torch.zeros(1, 1, 4, 64), view(), stream=0)


@pytest.mark.parametrize("ctx", [np.zeros(1, np.int64), view().c, ra.ra_problem(), bytearray(8), 1.5, [0]])
def test_handles_that_are_refused(ctx):
    with pytest.raises(ctypes.ArgumentError):
        ra.ra_round_scores(ctx, torch.zeros(1, 1, 4, 64), view(), stream=0)
    with pytest.raises(ctypes.ArgumentError):
        ra.ra_round_scores(None, torch.zeros(1, 1, 4, 64), view(), stream=Stream(ctx))


@pytest.mark.parametrize("given", [dict(stream=Stream(ctypes.c_void_p())), dict(stream=(1 << 64) + 8), dict(stream=0, scale=ctypes.c_float(1)),
                                   dict(stream=0, scale=Adapter(1.0)), dict(stream=0, scale=np.float32(1)), dict(stream=0, scale=1)])
def test_streams_and_scales_that_are_taken(given):
    with pytest.raises(ra.RaError, match="ctx is NULL"):
        ra.ra_round_scores(None, torch.zeros(1, 1, 4, 64), view(), **given)


@pytest.mark.parametrize("scale", ["1", 1j, ctypes.c_double(1), pytest.param(10**400, id="huge")])
def test_scales_that_are_refused(scale):
    with pytest.raises(ctypes.ArgumentError):
        ra.ra_round_scores(None, torch.zeros(1, 1, 4, 64), view(), scale=scale, stream=0)


def test_structures_are_known_by_their_type():
    q = torch.zeros(1, 1, 4, 64)
    size = max(ctypes.sizeof(ra.ra_kv_view), ctypes.sizeof(ra.ra_select_params))
    for params in (view().c, bytes(size), bytearray(size), ctypes.pointer(ra.make_select_params()), (ra.ra_select_params * 2)()):
        with pytest.raises(TypeError):
            ra.ra_round_scores_select(None, q, view(), params=params, stream=0)
    v = view()
    for c in (bytes(size), bytearray(size), None, ctypes.pointer(v.c), (ra.ra_kv_view * 1)(), np.zeros(size, np.uint8)):
        v.c = c
        with pytest.raises(TypeError):
            ra.ra_round_scores(None, q, v, stream=0)
    v.c = View.from_buffer_copy(view().c)
    with pytest.raises(ra.RaError, match="ctx is NULL"):
        ra.ra_round_scores(None, q, v, stream=0)


def test_other_threads_run_while_outputs_are_allocated():
    """An allocation that takes long (here: one that is filled) does not hold the interpreter."""
    heads, rounds = 2048, 131072  # 1 GB of round scores
    v = view()
    v.c.R_max = v.R_max = rounds
    q = torch.zeros(1, 1, heads, 64)
    stop, ticks = threading.Event(), []

    def watch():
        while not stop.is_set():
            time.sleep(0.001)
            ticks.append(time.perf_counter())

    before = torch.are_deterministic_algorithms_enabled()
    torch.use_deterministic_algorithms(True)  # torch.empty then fills what it returns
    watcher = threading.Thread(target=watch)
    watcher.start()
    try:
        while not ticks:
            time.sleep(0.001)
        t0 = time.perf_counter()
        with pytest.raises(ra.RaError, match="ctx is NULL"):
            ra.ra_round_scores(None, q, v, scale=1.0, stream=0)
        t1 = time.perf_counter()
    finally:
        torch.use_deterministic_algorithms(before)
        stop.set()
        watcher.join()
    during = [t0] + [t for t in ticks if t0 < t < t1] + [t1]
    assert max(b - a for a, b in zip(during, during[1:])) < (t1 - t0) / 2, (len(during), t1 - t0)


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
