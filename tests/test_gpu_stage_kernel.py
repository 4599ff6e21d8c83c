"""Staging: the kernel that reads pinned host memory against asynchronous copies of the same bytes (host tensors at addresses that
the kernel cannot read in 16-byte pieces), for every order, rounds of a token and of none, and more rounds than a wave looks up at
once; and rounds on both sides of the sizes from which a slice is copied, against the rounds themselves."""
import numpy as np
import pytest
import torch

import paper_2502_15294_amd as ra

pytestmark = pytest.mark.gpu

LENS = {
    "few": [[700, 0, 1, 33], [16, 17, 250, 0]],
    "130_short": [[1 + i % 3 for i in range(130)], [5] * 130],
    "unit_ends": [[32, 64, 31, 480], [1, 96, 2000, 4]],  # a unit of 16 KB is 32 tokens' keys and values of one layer at 2 KV heads
}


def _stage(lens, layers, order, offset):
    """(outputs of a decode over every staged layer, bytes staged): the host tensors begin `offset` bytes into their buffers."""
    B, R, Hkv, d = len(lens), len(lens[0]), 2, 64
    rng = np.random.default_rng(1)
    store = ra.ra_kv_store_create(0, layers, B, R, Hkv, d, ra.RA_BF16, 128 << 20)
    keep = []
    for b in range(B):
        for r in range(R):
            n = ra.ra_kv_store_round_bytes(store, lens[b][r])
            buf = torch.zeros(n + 64, dtype=torch.uint8, pin_memory=True)
            if n:
                buf[offset:offset + n] = torch.from_numpy(rng.normal(size=n // 2).astype(np.float32)).to(torch.bfloat16).view(torch.uint8)
            keep.append(buf)
            ra.ra_kv_store_register_round(store, b, r, buf[offset:], lens[b][r])
    sel = torch.arange(R, dtype=torch.int32).repeat(B, 1)
    sel[:, -1] = -1  # all rounds but the last
    side = torch.cuda.Stream()
    ra.ra_kv_store_stage(store, sel, torch.full((B,), R - 1, dtype=torch.int32), order, side)
    ctx = ra.ra_create(0)
    ws = torch.empty(ra.ra_workspace_bytes(B, R, 8, Hkv, d, 1, ra.RA_BF16, max(sum(x) for x in lens)), dtype=torch.uint8, device="cuda")
    ra.ra_set_workspace(ctx, ws)
    q = torch.randn((B, 8, d), generator=torch.Generator("cuda").manual_seed(2), device="cuda", dtype=torch.bfloat16)
    outs = []
    for layer in range(layers):
        ra.ra_kv_store_wait_layer(store, layer)
        outs.append(ra.ra_round_sparse_attn_decode(ctx, q, ra.ra_kv_store_layer_view(store, layer))[0])
    torch.cuda.synchronize()
    staged = ra.ra_kv_store_stats(store)[0]
    ra.ra_kv_store_release(store)
    ra.ra_kv_store_destroy(store)
    ra.ra_destroy(ctx)
    return torch.stack(outs).cpu(), staged, q, keep


@pytest.mark.parametrize("name", list(LENS))
@pytest.mark.parametrize("order,layers", [(ra.RA_STAGE_ROUND_MAJOR, 3), (ra.RA_STAGE_LAYER_MAJOR, 7), (ra.RA_STAGE_GROUPED, 9), (ra.RA_STAGE_GROUPED, 1)])
def test_kernel_and_copies_stage_the_same_bytes(name, order, layers):
    lens = LENS[name]
    by_kernel, n = _stage(lens, layers, order, 16)[:2]
    by_copies, m = _stage(lens, layers, order, 8)[:2]
    assert n == m == sum((x + (x + 15) // 16 * 16) * 2 * 64 * 2 * layers for row in lens for x in row[:-1])
    assert torch.isfinite(by_kernel).all() and torch.equal(by_kernel, by_copies)


@pytest.mark.parametrize("order", [ra.RA_STAGE_ROUND_MAJOR, ra.RA_STAGE_LAYER_MAJOR, ra.RA_STAGE_GROUPED])
def test_large_and_small_rounds_arrive_before_their_layer_is_read(order):
    """Slices of 4 MB and more are copied (a token of a layer: 512 bytes; groups of one, two or six layers), the others come by the
    kernel."""
    lens, layers, Hkv, d, offset = [[8192, 3, 8191, 1361, 1], [1360, 4096, 40, 8208, 9]], 6, 2, 64, 16
    for _ in range(3):
        out, _, q, bufs = _stage(lens, layers, order, offset)
        for b, row in enumerate(lens):
            ks, vs = [], []
            for r, n in enumerate(row[:-1]):
                tiles = (n + 15) // 16
                x = bufs[b * len(row) + r][offset:offset + (n + tiles * 16) * Hkv * d * 2 * layers].view(torch.bfloat16).view(layers, -1).cuda().double()
                ks.append(x[:, :n * Hkv * d].view(layers, Hkv, n, d))
                vs.append(x[:, n * Hkv * d:].view(layers, Hkv, tiles, d, 16).transpose(3, 4).reshape(layers, Hkv, tiles * 16, d)[:, :, :n])
            p = torch.softmax(q[b].double().view(Hkv, -1, d) @ torch.cat(ks, 2).transpose(2, 3).contiguous() * d ** -0.5, -1)
            exact = (p @ torch.cat(vs, 2)).view(layers, -1, d)
            assert (out[:, b].cuda().double() - exact).norm() < 1e-5 * exact.norm(), b  # fp32 sums: 2e-7


@pytest.mark.parametrize("new", [[300, 1, 0, 47, 16, 33], [2000, 400, 0, 410, 5, 420]], ids=["small", "large"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_saved_rounds_are_the_same_bytes_by_kernel_and_by_copies(dtype, new):
    """Sequences of 1 to 300 tokens, one without any and one skipped; several layers in one gather.  2 000 tokens and, of those of
    400 to 420, the longer: tensors of a megabyte and more, which are copied."""
    L, Hkv, d, cap = 5, 2, 64, max(new)
    B, skip = len(new), 4
    gen = torch.Generator("cuda").manual_seed(3)
    ks, vs = ([torch.randn((B, cap, Hkv, d), generator=gen, device="cuda").to(dtype) for _ in range(L)] for _ in range(2))
    results = []
    for offset in (16, 8):
        store = ra.ra_kv_store_create(0, L, B, 1, Hkv, d, ra.RA_BF16 if dtype == torch.bfloat16 else ra.RA_F32, 64 << 20)
        sizes = [ra.ra_kv_store_round_bytes(store, n) for n in new]
        bufs = [torch.full((n + 64,), 77, dtype=torch.uint8, pin_memory=True) for n in sizes]
        rounds = torch.tensor([-1 if b == skip else 0 for b in range(B)], dtype=torch.int32)
        ra.ra_kv_store_save_round(store, rounds, torch.tensor(new, dtype=torch.int32), ks, vs, [x[offset:] for x in bufs], None,
                                  torch.cuda.Stream())
        assert ra.ra_kv_store_save_wait(store) == sum(n for b, n in enumerate(sizes) if b != skip)
        results.append([x[offset:offset + n].clone() for x, n in zip(bufs, sizes)])
        assert all((x[:offset] == 77).all() and (x[offset + n:] == 77).all() for x, n in zip(bufs, sizes))
        assert (bufs[skip] == 77).all()
        ra.ra_kv_store_destroy(store)
    assert all(torch.equal(x, y) for x, y in zip(*results))
    for b, n in enumerate(new):  # the layout by its definition
        if b == skip or n == 0:
            continue
        tiles, parts = (n + 15) // 16, []
        for k, v in zip(ks, vs):
            padded = torch.nn.functional.pad(v[b, :n].transpose(0, 1), (0, 0, 0, tiles * 16 - n))
            parts += [k[b, :n].transpose(0, 1).reshape(-1), padded.reshape(Hkv, tiles, 16, d).transpose(2, 3).reshape(-1)]
        assert torch.equal(results[0][b], torch.cat(parts).view(torch.uint8).cpu())
