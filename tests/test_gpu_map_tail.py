"""Map edits at the ends of the one-launch edit kernel, against the oracle: the
tail and the inserted points shorter and longer than one another, at the edges
of its workgroups, no survivor in the tail, and points inserted from the map's
own arrays (after every move, before no append)."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_map import _points, _same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_batch_frames=1, max_inflight=1))


@pytest.mark.parametrize("n,remove,m", [(600, range(0, 257), 256), (600, range(0, 255), 300), (600, range(345, 600), 1),
                                        (600, range(0, 600, 2), 0), (1, [0], 1), (513, range(511, 513), 257), (600, [], 256),
                                        (600, list(range(0, 100)) + list(range(500, 600)), 200)])
def test_tail_and_inserts_equal_oracle(ft, ctx, n, remove, m):
    mp, ins = _points(n, 11, 0), _points(m, 12, 5000)
    want = oracle.map_update(mp, 1000, list(remove), ins)
    dm = ft.DeviceMap(mp, 1000)
    dm.edit(ctx, list(remove), ins)
    torch.cuda.synchronize()
    _same(dm.host(), want, f"{n} {m}")


def test_points_inserted_from_the_map_itself(ft, ctx):
    mp = _points(600, 21, 0)
    remove = list(range(10, 310))
    dm = ft.DeviceMap(mp, 1000)
    t, k = dm.t, 40                                    # inserted: slots 10 .. 49, which the moves fill first
    src = ft.ft_map_points(k, *(t[f][10:].data_ptr() for f in ("pos", "normal", "dmin", "dmax", "desc")))
    ctx.ft_map_update(dm.struct, 1000, remove, src)
    torch.cuda.synchronize()
    moved = oracle.map_update(mp, 1000, remove, _points(0, 1, 0))
    want = {f: np.concatenate([v, v[10:10 + k]]) for f, v in moved.items()}
    assert dm.n == 340
    _same(dm.host(), want, "own arrays")
