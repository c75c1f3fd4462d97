"""Shapes where the launch rules of the solve change: problems smaller than a
full reduction grid, right-hand-side counts on either side of each product
form, against the monolithic oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.newmark import NewmarkOracle
from workloads.mesh import cube_mesh
from workloads.partition import box_partition
from workloads.sources import dense_random_source

pytestmark = pytest.mark.gpu


def _steps(n, parts, nrhs, precision, N=2, **opt):
    """Relative error of N Newmark steps from rest, largest over steps and RHS."""
    from paper_2204_13254_amd.solver import DDSolver
    c, t, _ = cube_mesh(n)
    p = box_partition(n, parts)
    eps = np.random.default_rng(n).uniform(1, 4, len(t))
    dt = 0.4 / n
    o = NewmarkOracle(c, t, eps=eps, dt=dt)
    J = dense_random_source(o.d.n_e, ~o.d.pec, N, dt, dt, dt, seed=1, nrhs=nrhs)
    Eo = o.run(J)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s = DDSolver(c, t, p, eps, dt=dt, nrhs=nrhs, precision=precision, stream=st,
                     cg_tol=1e-13 if precision == "fp64" else 1e-6, **opt)
        Jd = torch.tensor(J, device="cuda")
        z = torch.zeros((nrhs, s.n_edges), dtype=torch.float64, device="cuda")
        E = [z, z.clone()]
        for k in range(N):
            E.append(s.step(Jd[k], Jd[k - 1] if k else z, E[-1], E[-2]))
        out = torch.stack(E[2:]).cpu().numpy()
    return max(np.linalg.norm(out[k] - Eo[k + 1], axis=1).max() / np.linalg.norm(Eo[k + 1], axis=1).min()
               for k in range(N))


# the bars of the parity tests: 1e-10 in FP64, 1e-8 with FP32 factors
BAR = {"fp64": 1e-10, "fp32_refine": 1e-8}


@pytest.mark.parametrize("nrhs", [1, 2, 3, 7, 13, 31])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_reductions_of_a_few_workgroups(nrhs, precision):
    assert _steps(5, (2, 2, 1), nrhs, precision) <= BAR[precision]


@pytest.mark.parametrize("opt", [dict(precond=0), dict(method="dp2")])
@pytest.mark.parametrize("nrhs", [1, 5])
def test_reductions_of_the_other_solvers(opt, nrhs):
    assert _steps(5, (1, 2, 2), nrhs, "fp64", **opt) <= BAR["fp64"]


@pytest.mark.parametrize("nrhs", [1, 2, 5, 16, 19])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_rows_shared_by_four_waves(nrhs, precision):
    # 16^3 in 64 boxes: coarse rows of up to 16 tiles, a few dozen rows
    assert _steps(16, (4, 4, 4), nrhs, precision) <= BAR[precision]


@pytest.mark.parametrize("n,parts", [(3, (1, 1, 1)), (4, (2, 1, 1)), (9, (2, 2, 2)), (14, (2, 1, 2))])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_factorisation_levels(n, parts, precision):
    # one block without interface or corners; no corners; several levels with
    # corner rows; blocks of 30 and more tile rows; then new materials on the
    # same context (the work lists are kept, the zero pattern may change)
    from paper_2204_13254_amd.solver import DDSolver
    c, t, _ = cube_mesh(n)
    p = box_partition(n, parts)
    dt = 0.4 / n
    rng = np.random.default_rng(n)
    s = DDSolver(c, t, p, np.ones(len(t)), dt=dt, nrhs=2, precision=precision,
                 cg_tol=1e-13 if precision == "fp64" else 1e-6)
    for eps in (np.ones(len(t)), rng.uniform(1, 4, len(t)), np.ones(len(t))):
        s.set_eps(eps)
        s.factor()
        o = NewmarkOracle(c, t, eps=eps, dt=dt)
        J = dense_random_source(o.d.n_e, ~o.d.pec, 1, dt, dt, dt, seed=2, nrhs=2)
        want = o.run(J)[1]
        z = torch.zeros((2, s.n_edges), dtype=torch.float64, device="cuda")
        got = s.step(torch.tensor(J[0], device="cuda"), z, z, z.clone()).cpu().numpy()
        assert np.linalg.norm(got - want) <= BAR[precision] * np.linalg.norm(want)


@pytest.mark.parametrize("n,parts,nrhs", [(12, 3, 1), (12, 3, 2), (12, 3, 31), (20, 4, 16), (20, 4, 19)])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_iteration_short_and_long(n, parts, nrhs, precision):
    # 324 workgroups in a reduction at 12^3 and 31 RHS, 170 at 20^3 and 16 RHS:
    # the short form; more than 512 at 19 RHS: the long one
    assert _steps(n, (parts,) * 3, nrhs, precision) <= BAR[precision]


@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_solves_repeat_with_other_loads(precision):
    # dd_solve on one context with a graph-capable stream: eager, captured and
    # replayed solves of loads that need different iteration counts (a smooth
    # load, single entries, zero, a non-finite one between), each against the
    # residual of the assembled matrix
    from paper_2204_13254_amd.solver import DDSolver
    n = 8
    c, t, _ = cube_mesh(n)
    dt = 0.4 / n
    o = NewmarkOracle(c, t, dt=dt)
    free = np.flatnonzero(~o.d.pec)
    rng = np.random.default_rng(0)
    loads = [rng.standard_normal((2, o.d.n_e)), np.zeros((2, o.d.n_e)), np.ones((2, o.d.n_e))]
    loads[1][0, free[7]] = 1.0
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s = DDSolver(c, t, box_partition(n, (2, 2, 2)), np.ones(len(t)), dt=dt, nrhs=2, precision=precision,
                     cg_tol=1e-13 if precision == "fp64" else 1e-6, stream=st, use_graph=True)
        for k in (0, 0, 0, 1, 0, 2, 2, 1, 0):
            b = torch.tensor(loads[k], device="cuda")
            x = s.solve(b).cpu().numpy()[:, free]
            if k == 2:
                bad = b.clone()
                bad[1, free[3]] = float("nan")
                with pytest.raises(Exception, match="non-finite"):
                    s.solve(bad)
            want = loads[k][:, free]
            r = (o.A @ x.T).T - want
            assert np.linalg.norm(r) <= BAR[precision] * np.linalg.norm(want)


@pytest.mark.parametrize("m", [1, 63, 64, 65, 1000, 40001])
def test_ordering_with_and_without_room_for_places(m):
    # a first call, one within the room of the last, one captured that needs
    # more than the context has (it does without), replayed beside eager calls
    from paper_2204_13254_amd.solver import DDSolver
    n = 5
    c, t, _ = cube_mesh(n)
    nt = len(t)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s = DDSolver(c, t, box_partition(n, 2), np.ones(nt), dt=0.05, factor=False, stream=st)
        rng = np.random.default_rng(m)

        def check(cell, perm):
            cell, perm = cell.cpu().numpy(), perm.cpu().numpy()
            assert np.array_equal(np.sort(perm), np.arange(len(cell)))
            k = cell[perm]
            k = np.where((k < 0) | (k >= nt), nt, k)
            assert np.all(np.diff(k) >= 0)

        def draw(size):
            v = rng.integers(-2, nt + 3, size).astype(np.int32)
            v[: size // 3] = np.sort(v[: size // 3])
            return torch.tensor(v, device="cuda")

        for size in (m, max(1, m // 2), m):
            cell = draw(size)
            check(cell, s.pic_sort(cell))
        big = draw(2 * m + 5)
        perm = torch.full((2 * m + 5,), -7, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            from paper_2204_13254_amd.solver import _dev_i32
            assert s.lib.dd_pic_sort(s.h, big.numel(), _dev_i32(big), _dev_i32(perm)) == 0
        for _ in range(3):
            big.copy_(draw(2 * m + 5))
            perm.fill_(-7)
            g.replay()
            check(big, perm)
            cell = draw(4 * m + 9)                 # the room grows between replays
            check(cell, s.pic_sort(cell))
