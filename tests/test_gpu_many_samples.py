"""Calls of very many short samples: their cost is in the work queues and in the
preparation, not in the products.  The bounds lie between what the calls take
and what they took with the fault that each test names (MI355X)."""
import pytest
import torch

import paper_2607_23250_amd as pl
import workloads as wl
from gpu_util import DEV, say

pytestmark = pytest.mark.gpu


def _inputs(samples, rows, h_q=8, h_kv=2, d=64, B=4096):
    n = samples * rows
    tiles, _ = pl.libra_plan([rows] * samples, [n], block_tokens=B, head_shards=1, cp=1,
                             num_q_heads=h_q, num_kv_heads=h_kv, head_dim=d)
    q, k, v, do = (t.to(DEV) for t in wl.tensors(7, n, n, h_q, h_kv, d))
    cu = torch.arange(samples + 1, dtype=torch.int64, device=DEV) * rows
    ws = pl.alloc_workspace(max(pl.libra_attn_workspace_size(len(tiles), samples, n, n, h_q, h_kv,
                                                             d, b) for b in (False, True)), DEV)
    return q, k, v, do, cu, pl.tiles_to_device(tiles, DEV), ws


def _ms(fn, reps=5):
    fn()
    best = float("inf")
    for _ in range(reps):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_forward_queue_heads_do_not_serialise():
    """131072 forward items of one key block: 1.6 ms.  With the heads of all
    queues on one cache line every item waited for its turn there: 8.3 ms."""
    q, k, v, _, cu, td, ws = _inputs(65536, 16)
    o, lse = pl.libra_attn_fwd(q, k, v, cu, td, workspace=ws)
    ms = _ms(lambda: pl.libra_attn_fwd(q, k, v, cu, td, o=o, lse=lse, workspace=ws))
    say(f"[many samples] forward of 65536 samples of 16 rows: {ms:.3f} ms")
    assert ms < 4.0


def test_backward_preparation_of_many_samples():
    """What a backward of 65536 samples does beside its dK / dV and dQ kernels:
    4.5 ms.  With a wave looking up every sample of the dK / dV items by itself,
    the preparation alone took 8 ms, 11.9 in all."""
    q, k, v, do, cu, td, ws = _inputs(65536, 16)
    o, lse = pl.libra_attn_fwd(q, k, v, cu, td, workspace=ws)
    out = pl.libra_attn_bwd(q, k, v, o, lse, do, cu, td, workspace=ws)

    def call():
        pl.libra_attn_bwd(q, k, v, o, lse, do, cu, td, dq=out[0], dk=out[1], dv=out[2],
                          workspace=ws)

    pl.libra_timing_enable(True)
    ms = _ms(call, reps=1)
    (kv, n), (dq, _) = pl.libra_timing_read(1), pl.libra_timing_read(2)
    pl.libra_timing_enable(False)
    rest = ms - (kv + dq) / n
    say(f"[many samples] backward of 65536 samples of 16 rows: {ms:.3f} ms, {rest:.3f} beside "
        "its two kernels")
    assert rest < 8.5
