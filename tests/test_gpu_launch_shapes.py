"""GPU parity where the launch shape can go wrong: how many work items there
are, in which of the queues, and how they fall on the workgroups.

Against the float64 oracle at the fixed bounds of gpu_util.check.
"""
import numpy as np
import pytest
import torch

import paper_2607_23250_amd as pl
from oracle import attention as oa
import workloads as wl
from gpu_util import DEV, LSE_TOL, check, say, to_np

pytestmark = pytest.mark.gpu


def _tiles(spans):
    """Tiles (q_begin, q_end, head_begin, head_end), rows at their positions."""
    t = np.zeros(len(spans), dtype=pl.TILE_DTYPE)
    for i, (a, b, h0, h1) in enumerate(spans):
        t[i]["q_begin"], t[i]["q_end"], t[i]["q_row"] = a, b, a
        t[i]["head_begin"], t[i]["head_end"] = h0, h1
    return t


def _check(lengths, tiles, h_q, h_kv, d, seed=5):
    """fwd + accumulate-mode bwd of `tiles` (which cover one range of heads on all rows)."""
    n = sum(lengths)
    q, k, v, do = wl.tensors(seed, n, n, h_q, h_kv, d)
    qd, kd, vd, dod = (t.to(DEV) for t in (q, k, v, do))
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)).to(DEV)
    td = pl.tiles_to_device(tiles, DEV)
    o, lse = pl.libra_attn_fwd(qd, kd, vd, cu, td)
    dq, dk, dv = pl.libra_attn_bwd(qd, kd, vd, o, lse, dod, cu, td, accumulate=True)
    torch.cuda.synchronize()
    h0, h1 = int(tiles["head_begin"].min()), int(tiles["head_end"].max())
    g0, g1 = h0 * h_kv // h_q, (h1 - 1) * h_kv // h_q + 1
    G = h_q // h_kv
    assert h0 % G == 0 and h1 % G == 0, "whole KV groups"
    sl = (slice(None), slice(h0, h1))
    kv = (slice(None), slice(g0, g1))
    pos = np.arange(n)
    O, LSE = oa.attention_fwd(q[sl], k[kv], v[kv], lengths, pos)
    dQ, dK, dV = oa.attention_bwd(q[sl], k[kv], v[kv], do[sl], lengths, pos)
    check("O", to_np(o)[sl], O, bf16_out=True)
    check("LSE", to_np(lse)[h0:h1], LSE, (LSE_TOL, 1e-4))
    check("dQ", to_np(dq)[sl], dQ, bf16_out=True)
    check("dK fp32", to_np(dk)[kv], dK)
    check("dV fp32", to_np(dv)[kv], dV)
    other = [g for g in range(h_kv) if not g0 <= g < g1]
    assert not to_np(dk)[:, other].any() and not to_np(dv)[:, other].any()


@pytest.mark.parametrize("n_items", (1, 32, 33, 64, 65, 96, 97, 700, 1025, 2048))
def test_one_queue_holds_every_item(n_items):
    """One of eight heads (no grouping): all items lie in one queue.  With more
    of them than its own workgroups (96 of the forward at d = 64, 32 of the
    backward) the others have to come from the seven empty queues; with fewer,
    every workgroup has to find its way out.  From 1025 samples on their extents, and
    from 2048 on their offsets, stay in memory during the preparation."""
    lengths = [int(x) for x in np.random.default_rng(n_items).integers(1, 60, n_items)]
    n = sum(lengths)
    say(f"[one queue] {n_items} items of one head, {n} rows")
    _check(lengths, _tiles([(0, n, 3, 4)]), 8, 8, 64)


@pytest.mark.parametrize("d", (64, 128))
@pytest.mark.parametrize("cuts", ((0, 4, 8), (0, 2, 4, 8), (0, 1, 4, 7, 8), (0, 3, 8)))
def test_head_ranges_and_shared_row_blocks(cuts, d):
    """Two KV heads of four query heads each, the heads cut into ranges of even
    and odd widths (a dK / dV step takes two heads, or one) and the rows into
    tiles that end inside 32-row blocks, differently for each range; samples of
    1 to 300 rows, the last block of the buffer not full."""
    lengths = [1, 300, 31, 33, 129, 64, 2, 95]
    n = sum(lengths)
    spans = []
    for i, (a, b) in enumerate(zip(cuts[:-1], cuts[1:])):
        rows = list(range(0, n, 37 + 11 * i)) + [n]
        spans += [(x, y, a, b) for x, y in zip(rows[:-1], rows[1:])]
    say(f"[head ranges] {cuts} d={d} rows={n} tiles={len(spans)}")
    _check(lengths, _tiles(spans), 8, 2, d)


@pytest.mark.parametrize("h_q,h_kv,d,n", [(2, 1, 64, 480), (2, 1, 64, 481), (2, 1, 64, 511),
                                          (4, 2, 128, 513), (3, 1, 64, 1200), (2, 2, 128, 2049),
                                          (8, 2, 64, 4096)])
def test_few_long_kv_items_split_rows(h_q, h_kv, d, n):
    """One or two samples and few KV heads: the dK / dV items are longer than
    the share of a workgroup and are cut into row ranges whose partial sums are
    merged, from 481 rows on (16 row blocks, two parts).  Tiles that end inside
    the parts; both output modes; the same bits from one call to the next."""
    lengths = [n, 77]
    rows = n + 77
    spans = [(a, min(a + 301, rows), 0, h_q) for a in range(0, rows, 301)]
    tiles = _tiles(spans)
    say(f"[row split] heads=({h_q},{h_kv}) d={d} rows={rows}")
    _check(lengths, tiles, h_q, h_kv, d)
    q, k, v, do = (t.to(DEV) for t in wl.tensors(5, rows, rows, h_q, h_kv, d))
    cu = torch.tensor([0, n, rows], dtype=torch.int64, device=DEV)
    td = pl.tiles_to_device(tiles, DEV)
    o, lse = pl.libra_attn_fwd(q, k, v, cu, td)
    ws = pl.alloc_workspace(pl.libra_attn_workspace_size(len(tiles), 2, rows, rows, h_q, h_kv, d,
                                                         True), DEV)
    a, b = (pl.libra_attn_bwd(q, k, v, o, lse, do, cu, td, workspace=ws) for _ in range(2))
    torch.cuda.synchronize()
    assert (int(ws[24:28].view(torch.int32)) > 0) == (n > 480)   # header slot kBwdSplits
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    _, dK, dV = oa.attention_bwd(q.cpu(), k.cpu(), v.cpu(), do.cpu(), lengths, np.arange(rows))
    check("dK", to_np(a[1]), dK, bf16_out=True)
    check("dV", to_np(a[2]), dV, bf16_out=True)


def test_overflow_of_the_dq_items_is_reported():
    """200 copies of a tile make more dQ items than the workspace holds (it is
    sized for tiles that do not overlap): the ones that fit run, and the count of
    skipped tiles says so, once for the forward list, once for the dQ list."""
    n, T = 4096, 200
    tiles = _tiles([(0, n, 0, 1)] * T)
    q, k, v, do = (t.to(DEV) for t in wl.tensors(5, n, n, 1, 1, 64))
    cu = torch.tensor([0, n], dtype=torch.int64, device=DEV)
    td = pl.tiles_to_device(tiles, DEV)
    assert T * (n // 128) > n // 64 + (T + 1) * 2 + 1 + 3072
    ws = pl.alloc_workspace(max(pl.libra_attn_workspace_size(T, 1, n, n, 1, 1, 64, b)
                                for b in (False, True)), DEV)
    say(f"[overflow] {T} copies of a tile of {n} rows")
    for _ in range(3):
        o, lse = pl.libra_attn_fwd(q, k, v, cu, td, workspace=ws)
        assert pl.libra_attn_skipped_tiles(ws) == 1
        pl.libra_attn_bwd(q, k, v, o, lse, do, cu, td, workspace=ws)
        assert pl.libra_attn_skipped_tiles(ws) == 1


@pytest.mark.parametrize("d", (64, 128))
def test_tiles_past_the_last_sample(d):
    """K and V buffers longer than the samples, and tiles that reach past them: the
    rows there attend nothing and leave the others' gradients alone, whatever the
    workspace held before."""
    n, rows, h_q, h_kv = 200, 300, 4, 2
    tiles = _tiles([(0, 90, 0, 4), (90, rows, 0, 4)])
    q, k, v, do = wl.tensors(5, rows, rows, h_q, h_kv, d)
    qd, kd, vd, dod = (t.to(DEV) for t in (q, k, v, do))
    cu = torch.tensor([0, 70, n], dtype=torch.int64, device=DEV)
    td = pl.tiles_to_device(tiles, DEV)
    o = torch.zeros_like(qd)
    lse = torch.zeros((h_q, rows), dtype=torch.float32, device=DEV)
    dq = torch.zeros_like(qd)
    ws = pl.alloc_workspace(max(pl.libra_attn_workspace_size(2, 2, rows, rows, h_q, h_kv, d, b)
                                for b in (False, True)), DEV)
    say(f"[past the samples] d={d}")
    pl.libra_attn_fwd(qd, kd, vd, cu, td, o=o, lse=lse, workspace=ws)
    ws.fill_(0xFF)
    _, dk, dv = pl.libra_attn_bwd(qd, kd, vd, o, lse, dod, cu, td, dq=dq, workspace=ws)
    torch.cuda.synchronize()
    dQ, dK, dV = oa.attention_bwd(q[:n], k[:n], v[:n], do[:n], [70, n - 70], np.arange(n))
    check("dQ", to_np(dq)[:n], dQ, bf16_out=True)
    check("dK", to_np(dk)[:n], dK, bf16_out=True)
    check("dV", to_np(dv)[:n], dV, bf16_out=True)
    assert not to_np(dq)[n:].any() and not to_np(dk)[n:].any() and not to_np(dv)[n:].any()
