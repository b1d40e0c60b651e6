"""Map edits at the edges of the removal bitmap's 64-slot words: maps and new
counts of whole words and one slot either side, holes in the first, the last and
every word, tails with one survivor and with none, in the single call and in the
call for several maps, with and without an id record: equal to the oracle."""
import ctypes as ct

import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_map import _points, _same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_batch_frames=1, max_map_points=4096, max_inflight=1))


def removals(n):
    """Slots removed from a map of n points, by what the edit does."""
    odd = np.arange(n)[1::2]
    yield "first half", np.arange(n // 2)
    yield "last half", np.arange(n - n // 2, n)
    yield "odd slots, downwards", odd[::-1]
    yield "all but one", np.delete(np.arange(n), n - 1)
    yield "all", np.arange(n)
    for keep in (63, 64, 65, 128):
        if keep < n:
            yield f"the first down to {keep} left", np.arange(n - keep)
            yield f"a hole in the last word, {keep} left", np.concatenate([[keep - 1], np.arange(keep + 1, n)])


@pytest.mark.parametrize("ids", [False, True])
@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 640, 1000])
def test_words_equal_oracle(ft, ctx, n, many, ids):
    for tag, remove in removals(n):
        remove = np.ascontiguousarray(remove, np.int32)
        m = 5
        mp, ins = _points(n, 31, 0), _points(m, 32, 9000)
        cap = n + m
        want = oracle.map_update(mp, cap, remove.tolist(), ins)
        dm = ft.DeviceMap(mp, cap)
        rec, new_ids, given = None, None, remove
        if ids:      # point ids 3 * slot + 1, inserted ids 3 j
            slot_id, slot_of = np.full(cap, -1, np.int32), np.full(3 * cap + 2, -1, np.int32)
            slot_id[:n] = 3 * np.arange(n) + 1
            slot_of[slot_id[:n]] = np.arange(n)
            rec = ft.ft_map_ids(slot_id.ctypes.data, slot_of.ctypes.data, len(slot_of))
            new_ids = np.ascontiguousarray(3 * np.arange(m), np.int32)
            given = np.ascontiguousarray(3 * remove + 1, np.int32)
        dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in ins.items()}
        src = ft.ft_map_points(m, *(dev[k].data_ptr() for k in ("pos", "normal", "dmin", "dmax", "desc")))
        if many:
            ed = ft.ft_map_edit(len(given), given.ctypes.data if len(given) else None, src,
                                new_ids.ctypes.data if ids else None, ct.pointer(rec) if ids else None)
            ctx.ft_map_update_many([dm.struct], [cap], [ed])
        else:
            ctx.ft_map_update(dm.struct, cap, given, src, ids=rec, insert_ids=new_ids)
        torch.cuda.synchronize()
        assert dm.n == len(want["dmin"]), tag
        _same(dm.host(), want, (n, tag))
        if ids:
            # dmin is the point's tag: its old slot, or 9000 + j
            tags = want["dmin"].astype(np.int64)
            expect = np.where(tags >= 9000, 3 * (tags - 9000), 3 * tags + 1)
            assert np.array_equal(slot_id[:dm.n], expect), tag
            assert np.array_equal(slot_of[expect], np.arange(dm.n)), tag
            assert (np.delete(slot_of, expect) == -1).all(), tag
