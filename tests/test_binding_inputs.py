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


@pytest.mark.parametrize("limit", (0, 1, 767, 768, 1 << 20))
def test_more_tiles_than_one_call_sizes(limit, monkeypatch):
    """384 one-token blocks in two shards: above the bound the library counts
    them, and the plan is the same."""
    lengths = [100, 1, 155, 60, 68]
    want = _plan(lengths, block_tokens=1)
    assert len(want[0]) == 768
    monkeypatch.setattr(pl, "_PLAN_ONE_CALL", limit)
    assert _same(want, _plan(lengths, block_tokens=1))


def test_block_tokens_as_the_library_sees_them():
    """The library's fields have 32 bits; the tile count follows them."""
    lengths = [100, 1, 155, 60, 68]
    assert _same(_plan(lengths, block_tokens=48), _plan(lengths, block_tokens=48 + (1 << 32)))


@pytest.mark.parametrize("kw", (dict(cp=-1), dict(cp=0), dict(cp=1 << 30),
                                dict(cp=1 << 30, block_tokens=1), dict(head_shards=1 << 30)))
def test_refused_before_anything_is_allocated(kw, monkeypatch):
    def zeros(shape, *a, **k):
        assert int(np.prod(shape)) < 1 << 16, "array for a refused plan"
        return real(shape, *a, **k)
    real = np.zeros
    monkeypatch.setattr(pl.np, "zeros", zeros)
    with pytest.raises(pl.LibraError) as e:
        _plan([100, 1, 155, 60, 68], **kw)
    assert e.value.code == pl.LIBRA_EINVAL


@pytest.mark.parametrize("lengths,kw", [([], {}), ([384], {}), ([256, 128], dict(block_tokens=0)),
                                        ([256, 128], dict(head_shards=3)), ([256, 0, 128], {}),
                                        ([256, 127], {})])
def test_refused_inputs_stay_refused(lengths, kw):
    with pytest.raises(pl.LibraError) as e:
        _plan(lengths, **kw)
    assert e.value.code == pl.LIBRA_EINVAL
