"""dd_pic_sort with and without room for the places of its particles: the room is
laid out by the first particle call (at least 2^22 particles), a larger ordering
draws the places from cursors; both captured into a graph and replayed beside
eager calls on the same context."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from workloads.mesh import cube_mesh
from workloads.partition import box_partition

pytestmark = pytest.mark.gpu

ROOM = 1 << 22


def _check(cell, perm, nt):
    cell, perm = cell.cpu().numpy(), perm.cpu().numpy()
    assert np.array_equal(np.bincount(perm, minlength=len(cell)), np.ones(len(cell)))
    k = cell[perm]
    k = np.where((k < 0) | (k >= nt), nt, k)
    assert np.all(np.diff(k) >= 0)


@pytest.mark.parametrize("captured,eager", [(5000, ROOM + 3), (ROOM + 3, 5000), (ROOM, ROOM)])
def test_captured_and_eager_orderings(captured, eager):
    from paper_2204_13254_amd.solver import DDSolver, _dev_i32
    n = 5
    c, t, _ = cube_mesh(n)
    nt = len(t)
    assert 8 * nt < ROOM
    st = torch.cuda.Stream()
    g = torch.Generator(device="cuda").manual_seed(captured)

    def draw(size):
        v = torch.randint(-2, nt + 3, (size,), generator=g, device="cuda", dtype=torch.int32)
        v[: size // 3] = torch.sort(v[: size // 3]).values
        return v

    with torch.cuda.stream(st):
        st.wait_stream(torch.cuda.default_stream())
        s = DDSolver(c, t, box_partition(n, 2), np.ones(nt), dt=0.05, factor=False, stream=st)
        first = draw(100)
        _check(first, s.pic_sort(first), nt)
        cell = draw(captured)
        perm = torch.full((captured,), -7, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            assert s.lib.dd_pic_sort(s.h, captured, _dev_i32(cell), _dev_i32(perm)) == 0
        for _ in range(3):
            other = draw(eager)
            _check(other, s.pic_sort(other), nt)
            cell.copy_(draw(captured))
            perm.fill_(-7)
            graph.replay()
            _check(cell, perm, nt)
