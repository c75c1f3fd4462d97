"""dd_solve, dd_step_mixed and dd_adjoint_step with FP32 factors on a graph-capable
stream: the first call is launched from the host, later ones run as a captured
graph whose iteration count comes from the calls before.  A call's status,
result and counts are those of its inputs alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from workloads.mesh import cube_mesh
from workloads.partition import box_partition

pytestmark = pytest.mark.gpu


class _Calls:
    """One context and the three calls on it, each returning its result."""

    def __init__(self, n, parts, nrhs, **opt):
        from paper_2204_13254_amd.solver import DDSolver
        c, t, _ = cube_mesh(n)
        eps = np.random.default_rng(n).uniform(1, 4, len(t))
        self.stream = torch.cuda.Stream()
        with torch.cuda.stream(self.stream):
            self.s = DDSolver(c, t, box_partition(n, parts), eps, dt=0.4 / n, nrhs=nrhs, precision="fp32_refine",
                              stream=self.stream, use_graph=True, **opt)
        self.s.faces()

    def __call__(self, kind, load, face):
        s, z = self.s, torch.zeros_like(load)
        with torch.cuda.stream(self.stream):
            self.out = out = z.clone()
            if kind == "solve":
                s.solve(load, out)
            elif kind == "mixed":
                s.step_mixed(load, z, face, E_next=out, stats=True)
            else:
                s.adjoint_step(load, None, None, None, None, None, None, g_out=out)
        return out


def _loads(c):
    """A random load, a single entry and zero, with faces to match."""
    g = torch.Generator(device="cuda").manual_seed(1)
    e, pec = c.s.edges()
    shape, fshape = (c.s.nrhs, c.s.n_edges), (c.s.nrhs, c.s.n_faces)
    free = torch.as_tensor(~pec, device="cuda").double()
    hard = (2 * torch.rand(shape, generator=g, dtype=torch.float64, device="cuda") - 1) * free
    one = torch.zeros_like(hard)
    one[0, int(np.flatnonzero(~pec)[7])] = 1.0
    face = 2 * torch.rand(fshape, generator=g, dtype=torch.float64, device="cuda") - 1
    zero = torch.zeros_like(face)
    torch.cuda.synchronize()
    return [(hard, face), (one, zero), (torch.zeros_like(hard), zero)]


@pytest.mark.parametrize("kind", ["solve", "mixed", "adjoint"])
@pytest.mark.parametrize("cap", [2, 3])
def test_the_iteration_cap_is_reported_by_every_call(kind, cap):
    # cg_tol is out of reach of `cap` iterations, the refinement gets there all the same
    from paper_2204_13254_amd._lib import DDError
    c = _Calls(8, 2, 2, cg_tol=1e-6, cg_max_iter=cap, refine_max=60)
    load, face = _loads(c)[0]
    first = None
    for call in range(4):
        with pytest.raises(DDError, match="NO_CONVERGENCE"):
            c(kind, load, face)
            print(f"{kind} cap {cap}: call {call} reported success", flush=True)
        first = c.out if first is None else first
        assert bool(torch.isfinite(c.out).all()) and torch.equal(c.out, first)


@pytest.mark.parametrize("kind,n,parts,nrhs,opt", [
    ("solve", 8, 2, 2, {}), ("mixed", 8, 2, 2, {}), ("adjoint", 8, 2, 2, {}),
    ("solve", 9, 3, 1, {}),
    ("solve", 20, 4, 19, {}),              # reductions of more than 512 workgroups
    ("solve", 9, 3, 5, dict(precond=0)),
    ("solve", 9, 3, 4, dict(check_every=1)),
])
def test_results_do_not_depend_on_the_calls_before(kind, n, parts, nrhs, opt):
    # a random load needs a dozen iterations, zero none; each order of them gives
    # what a context gives whose first call has that load
    def counts(s):
        return [list(s.stats.cg_iters[:nrhs]), list(s.stats.cg_relres[:nrhs]), s.stats.refine_sweeps]

    want, stats = [], []
    for k in range(3):
        c = _Calls(n, parts, nrhs, cg_tol=1e-6, **opt)
        load, face = _loads(c)[k]
        want.append(c(kind, load, face))
        stats.append(counts(c.s))
    c = _Calls(n, parts, nrhs, cg_tol=1e-6, **opt)
    loads = _loads(c)
    for call, k in enumerate((2, 2, 0, 0, 2, 1, 0, 1, 1, 2, 2, 0, 1, 0)):
        got = c(kind, *loads[k])
        d = float((got - want[k]).abs().max())
        assert torch.equal(got, want[k]), f"call {call}, load {k}: largest difference {d:.3e}"
        if kind != "adjoint":
            assert counts(c.s) == stats[k], f"call {call}, load {k}"


def test_a_refinement_sweep_left_unfinished():
    # single entries need as many iterations in both solves as the first solve of a
    # random load, whose sweep needs more: the graph ends behind the first check
    def solve_iters(s):
        return tuple(s.stats.solve_iters)

    opt = dict(cg_tol=1e-6)
    c = _Calls(8, 2, 2, **opt)
    _, (one, _), _ = _loads(c)
    c("solve", one, None)
    few = max(solve_iters(c.s))
    e, pec = c.s.edges()
    free = np.flatnonzero(~pec)
    for seed in range(8):
        load = torch.zeros_like(one)
        load[:, torch.as_tensor(free, device="cuda")] = torch.tensor(
            np.random.default_rng(seed).standard_normal((2, len(free))), device="cuda")
        torch.cuda.synchronize()
        fresh = _Calls(8, 2, 2, **opt)
        want = fresh("solve", load, None)
        iters = solve_iters(fresh.s)
        if iters[0] <= few < iters[1]:
            break
    else:
        pytest.fail(f"no load of that kind (single entries {few}, the last one {iters})")
    for _ in range(2):
        c("solve", one, None)
    got = c("solve", load, None)
    assert torch.equal(got, want) and solve_iters(c.s) == iters
    assert c.s.stats.refine_sweeps == fresh.s.stats.refine_sweeps
