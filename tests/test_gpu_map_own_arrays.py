"""Points inserted from the edited map's own arrays, at the two ends of what the
call allows: their slots end right below the slots they are written to, or begin
right above them; with moves in the edit and without; in the single call and in
the call for several maps: the moves first, then the inserted points."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_map import _points, _same

pytestmark = pytest.mark.gpu
FIELDS = ("pos", "normal", "dmin", "dmax", "desc")


@pytest.fixture(scope="module")
def ctx(ft):
    return ft.Context(ft.default_limits(max_batch_frames=1, max_map_points=4096, max_inflight=1))


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("moves", [True, False])
@pytest.mark.parametrize("k,below", [(1, True), (1, False), (40, True), (40, False), (257, True), (257, False)])
def test_sources_beside_the_appended_slots(ft, ctx, k, below, moves, many):
    mp = _points(1400, 21, 0)
    remove = list(range(10, 710)) if moves else list(range(700, 1400))
    n1 = 700
    start = n1 - k if below else n1 + k
    dm = ft.DeviceMap(mp, 2000)
    src = ft.ft_map_points(k, *(dm.t[f][start:].data_ptr() for f in FIELDS))
    if many:
        rem = np.array(remove, np.int32)
        ctx.ft_map_update_many([dm.struct], [2000], [ft.ft_map_edit(len(rem), rem.ctypes.data, src, None, None)])
    else:
        ctx.ft_map_update(dm.struct, 2000, remove, src)
    torch.cuda.synchronize()
    assert dm.n == n1 + k
    moved = oracle.map_update(mp, 2000, remove, _points(0, 1, 0))
    read = {f: np.concatenate([moved[f], mp[f][n1:]])[start:start + k] for f in FIELDS}   # (moves leave the tail as it is)
    _same(dm.host(), {f: np.concatenate([moved[f], read[f]]) for f in FIELDS}, (k, below, moves, many))
