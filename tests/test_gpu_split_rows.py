"""The dK / dV items of a backward call, read back from its workspace: which are
cut into row ranges, that the ranges hold covered rows, and parity where the
tiles cover only part of a sample's rows.

Parity against the float64 oracle at the fixed bounds of gpu_util.check.
"""
import numpy as np
import pytest
import torch

import paper_2607_23250_amd as pl
from oracle import attention as oa
import workloads as wl
from gpu_util import DEV, check, say, to_np

pytestmark = pytest.mark.gpu

KEYS, ROWS, MIN_BLOCKS = 128, 32, 8          # kBwdBK, kRows, kBwdSplitMinBlocks
HEADER, SPLITS_SLOT, QUEUES_SLOT = 1280, 6, 32   # kHdrBytes, kBwdSplits, kBwdQ
ITEM = np.dtype([(n, "<i4") for n in ("sample", "kb", "g", "slot", "r0", "r1", "p0", "p1")])


def _align(x):
    return -(-x // 256) * 256


def bwd_items(ws, n):
    """(items, split items) of the last backward that used `ws`, n samples."""
    raw = ws.cpu().numpy()
    hdr = raw[:HEADER].view("<i4")
    counts = hdr[QUEUES_SLOT + 8:QUEUES_SLOT + 16]
    at = _align(_align(HEADER + 4 * n) + 8 * n)
    items = raw[at:at + int(counts.sum()) * ITEM.itemsize].view(ITEM)
    return items, int(hdr[SPLITS_SLOT])


def covered(lengths, tiles, h_q, h_kv):
    """{(sample, KV head): steps that every row of the sample takes part in (two
    heads of one tile make one)}."""
    G, cu, out = h_q // h_kv, np.concatenate([[0], np.cumsum(lengths)]), {}
    for t in tiles:
        for j in range(len(lengths)):
            a, b = max(t["q_begin"], cu[j]) - cu[j], min(t["q_end"], cu[j + 1]) - cu[j]
            for g in range(h_kv if a < b else 0):
                nh = min(t["head_end"], (g + 1) * G) - max(t["head_begin"], g * G)
                if nh > 0:
                    out.setdefault((j, g), np.zeros(lengths[j], dtype=np.int64))[a:b] += (nh + 1) // 2
    return out


def check_items(items, splits, lengths, cov):
    """Every (sample, key block, KV head) once, whole or as adjoining row ranges
    that each hold covered rows; the steps of the longest item and in all."""
    by = {}
    for it in items:
        by.setdefault((int(it["sample"]), int(it["kb"]), int(it["g"])), []).append(it)
    reach = {}
    for (j, _), c in cov.items():
        reach[j] = max(reach.get(j, 0), int(np.nonzero(c)[0].max()) + 1)
    want = {(j, kb, g) for (j, g) in cov for kb in range(-(-reach[j] // KEYS))}
    assert set(by) == want
    assert splits == sum(len(p) > 1 for p in by.values())
    longest = work = 0
    for (j, kb, g), parts in by.items():
        c, parts = cov[j, g], sorted(parts, key=lambda p: p["r0"])
        assert len({int(p["slot"]) for p in parts}) == len(parts)
        assert (len(parts) == 1) == (parts[0]["slot"] < 0)
        work += int(c[kb * KEYS:].sum()) / ROWS
        for p, nxt in zip(parts, parts[1:] + [None]):
            lo, hi = max(int(p["r0"]), kb * KEYS), min(int(p["r1"]), len(c))
            rows = int(c[lo:hi].sum()) / ROWS
            longest = max(longest, rows)
            if len(parts) > 1:
                assert rows > 0, f"a part without rows: {p}"
                assert nxt is None or nxt["r0"] == p["r1"]
        assert parts[0]["r0"] <= kb * KEYS and parts[-1]["r1"] >= len(c)
    return longest, work


def _share(lengths, cp):
    n = sum(lengths)
    c = n // (2 * cp)
    return [(0, c), (n - c, n)]


CALLS = {
    # name: lengths, query ranges (None: all), B, H, heads, d, are items cut?
    "late tile of a long sample": ([32768], [(32256, 32768)], 512, 1, (2, 1), 64, False),
    "late tile": ([12288], [(10240, 12288)], 2048, 1, (4, 1), 64, True),
    "late tile, another sample after it": ([5120, 1024], [(4096, 5120)], 1024, 1, (8, 2), 128, True),
    "share": ([700, 684, 6808], _share([700, 684, 6808], 4), 256, 2, (4, 2), 64, True),
    "share, one head to a group": ([300, 7892], _share([300, 7892], 4), 512, 1, (2, 2), 128, True),
    "gaps": ([4096], [(0, 512), (1536, 2048), (2560, 2816), (3840, 4096)], 256, 1, (6, 2), 64,
             True),
    "one head to a tile": ([6000, 2192], _share([6000, 2192], 4), 512, 4, (4, 2), 64, True),
    # more samples than the counts in LDS are kept for
    "many samples": ([4] * 1100 + [6000], [(0, 400), (9600, 10400)], 400, 1, (2, 1), 64, True),
    # one row block below two parts (no merge is launched), and two
    "480 rows": ([480], None, 480, 1, (2, 1), 64, False),
    "481 rows": ([481, 1], None, 482, 1, (2, 1), 64, True),
    "all rows": ([4096, 512], None, 300, 2, (8, 2), 64, True),
}


@pytest.mark.parametrize("name", CALLS)
def test_parts_hold_covered_rows(name):
    lengths, ranges, B, H, (h_q, h_kv), d, cut = CALLS[name]
    keys, n = sum(lengths), len(lengths)
    tiles, _ = pl.libra_plan(lengths, [keys], block_tokens=B, head_shards=H, cp=1, num_q_heads=h_q,
                             num_kv_heads=h_kv, head_dim=d, q_ranges=ranges)
    pos = np.concatenate([np.arange(a, b) for a, b in ranges or [(0, keys)]])
    q, k, v, do = wl.tensors(11, len(pos), keys, h_q, h_kv, d)
    qd, kd, vd, dod = (t.to(DEV) for t in (q, k, v, do))
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)).to(DEV)
    td = pl.tiles_to_device(tiles, DEV)
    say(f"[split rows] {name}: heads=({h_q},{h_kv}) d={d} rows={len(pos)} keys={keys}")
    ws = pl.alloc_workspace(pl.libra_attn_workspace_size(len(tiles), n, len(pos), keys, h_q, h_kv,
                                                         d, True), DEV)
    ws.fill_(0xFF)
    o, lse = pl.libra_attn_fwd(qd, kd, vd, cu, td)
    dq, dk, dv = pl.libra_attn_bwd(qd, kd, vd, o, lse, dod, cu, td, workspace=ws)
    torch.cuda.synchronize()
    items, splits = bwd_items(ws, n)
    cov = covered(lengths, tiles, h_q, h_kv)
    longest, work = check_items(items, splits, lengths, cov)
    grid = torch.cuda.get_device_properties(0).multi_processor_count
    block = KEYS / ROWS * max(int(c.max()) for c in cov.values())
    chunk = max(17 / 16 * work / grid + 1, MIN_BLOCKS, block)
    say(f"  {len(items)} items, {splits} cut, longest {longest:.1f} steps, C {chunk:.1f}")
    assert (splits > 0) == cut
    if cut:   # a cut lies within a key block of its place
        assert longest <= chunk + block
    dQ, dK, dV = oa.attention_bwd(q, k, v, do, lengths, pos)
    check("dQ", to_np(dq), dQ, bf16_out=True)
    check("dK", to_np(dk), dK, bf16_out=True)
    check("dV", to_np(dv), dV, bf16_out=True)
    again = pl.libra_attn_bwd(qd, kd, vd, o, lse, dod, cu, td, workspace=ws)
    assert all(torch.equal(a, b) for a, b in zip((dq, dk, dv), again))
