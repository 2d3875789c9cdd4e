"""The planner binding takes lengths as lists, tuples or arrays, of ints or of
numbers NumPy converts, and sizes its tile array without a counting call when
every query row is present: all of it gives what the plain way gives."""
import numpy as np
import pytest

import paper_2607_23250_amd as pl

PLAN = dict(block_tokens=48, head_shards=2, cp=2, num_q_heads=8, num_kv_heads=2, head_dim=64)


def _plan(lengths, **kw):
    return pl.libra_plan(lengths, [256, 128], with_bytes=True, **{**PLAN, **kw})


def _same(a, b):
    return all(np.array_equal(x, y) and x.dtype == y.dtype for x, y in zip(a, b))


@pytest.mark.parametrize("form", (tuple, np.array, lambda x: np.array(x, dtype=np.int32),
                                  lambda x: [np.int64(v) for v in x], lambda x: [float(v) for v in x],
                                  lambda x: np.repeat(np.array(x), 2)[::2]))
def test_length_forms(form):
    lengths = [100, 1, 155, 60, 68]
    assert _same(_plan(lengths), _plan(form(lengths)))
    packs = [[100, 1, 155], [60, 68], [], [7]]
    assert _same(pl.libra_vrsp(packs, 2), pl.libra_vrsp([form(p) for p in packs], 2))


@pytest.mark.parametrize("block", (1, 7, 127, 128, 129, 4096))
def test_tile_count_without_a_counting_call(block):
    lengths = [100, 1, 155, 60, 68]
    every = [(0, 256), (256, 384)]   # the same rows named as ranges: counted by a call
    a, b = _plan(lengths, block_tokens=block), _plan(lengths, block_tokens=block, q_ranges=every)
    assert len(a[0]) and _same(a, b)


@pytest.mark.parametrize("lengths,kw", [([], {}), ([384], {}), ([256, 128], dict(block_tokens=0)),
                                        ([256, 128], dict(head_shards=3)), ([256, 0, 128], {}),
                                        ([256, 127], {})])
def test_refused_inputs_stay_refused(lengths, kw):
    with pytest.raises(pl.LibraError) as e:
        _plan(lengths, **kw)
    assert e.value.code == pl.LIBRA_EINVAL
