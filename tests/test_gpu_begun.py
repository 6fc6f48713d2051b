"""Begun solves (sso_solve_begin) under the library's automatic choice of solver: what they leave
behind at every end, and the calls that follow."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def settled(mesh, seed=5):
    """The structure with supports that moved by some millimetres."""
    rng = np.random.default_rng(seed)
    return mesh.copy(u_prescribed=1e-3 * rng.standard_normal((mesh.n_nodes, 6)))


@pytest.mark.parametrize("moved", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
def test_ended_before_a_launch(mixed, moved):
    """A begun solve that no launch took ends with u = 0 on the free DOFs and SSO_ENOTCONV; the
    adjoints that may follow are solved, by the standard recurrences, to the same bits as where
    those are named."""
    import paper_2407_20026_amd as sso
    print(f"[gpu] ended before a launch, mixed {mixed}, moved supports {moved}", flush=True)
    # its own weight: without displacements the load's part is what is left of a gradient
    mesh = meshgen.shell(13, seed=3).copy(unit_weight=25e3)
    mesh = settled(mesh) if moved else mesh
    a = np.zeros((mesh.n_nodes, 6))
    free = np.flatnonzero((mesh.fixed == 0).all(axis=1))
    a[free[len(free) // 2], 2] = 1.0
    out = []
    for solver in (sso.SOLVER_AUTO, sso.SOLVER_STANDARD):
        o = sso.Options(rtol=1e-10, solver=solver,
                        precision=sso.PREC_MIXED if mixed else sso.PREC_FP64)
        with sso.Problem(mesh, o) as p:
            p.solve_begin()
            u, _ = p.solve_end(check=False)
            assert p.last_status == sso.SSO_ENOTCONV
            assert not u[free].any()
            g = [p.adjoint("linear", dg_du=a)["dg_dxyz"], p.adjoint("compliance")["dg_dxyz"]]
            for noalloc in (False, True):
                z = p.size_objective(1.0, 1e-3, 0.05, noalloc=noalloc)
                g += [z["dg_dxyz"], z["dg_dt"]]
            out.append(g)
            u, _ = p.solve()                    # and the problem is none the worse for it
            assert p.last_status == sso.SSO_OK and u[free].any()
    for x, y in zip(*out):
        assert torch.isfinite(x).all() and torch.equal(x, y)
    assert out[0][0].any()


def arch():
    return meshgen.arch_bridge(20, n_spans=40)


def floating():
    """A shell without supports under vertical forces in balance at its corners: K has six zero
    eigenvalues, the load lies in its range."""
    m = meshgen.shell(12, seed=6)
    n = 13
    m.fixed[:] = 0
    m.f_nodal[:] = 0.0
    m.f_nodal[[0, n - 1, n * n - n, n * n - 1], 2] = [1e3, -1e3, -1e3, 1e3]
    return m


def _alone(sso, mesh, o):
    with sso.Problem(mesh, o) as p:
        u, st = p.solve(check=False)
        return u, st, p.last_status


ENDS = {
    # met by the first solution, or after refinement
    "shell": (lambda: meshgen.shell(15, seed=3), 1e-10, "direct"),
    "arch": (arch, 3e-13, "direct"),
    # below what refinement reaches: corrections by PCG
    "floor": (lambda: meshgen.gridshell(11, seed=0), 1e-15, "direct"),
    # a pivot too small: PCG from the start
    "floating": (floating, 1e-6, "pcg"),
}


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("name", list(ENDS))
def test_one_call_ends_a_begun_solve(name, mixed):
    """One launch with max_it iterations brings a begun solve to its end, at once and on its own or
    beside another problem, to the bits and the status of a solve alone."""
    import paper_2407_20026_amd as sso
    print(f"[gpu] one call, {name}, mixed {mixed}", flush=True)
    make, rtol, way = ENDS[name]
    mesh = make()
    o = sso.Options(rtol=rtol, max_it=3000, precision=sso.PREC_MIXED if mixed else sso.PREC_FP64)
    u, st, status = _alone(sso, mesh, o)
    assert (st["solver"] == sso.SOLVER_AUTO) == (way == "direct")
    other = meshgen.shell(9, seed=2)
    for beside in (False, True):
        with sso.Problem(mesh, o) as p, sso.Problem(other, sso.Options(rtol=1e-9)) as q:
            b = sso.Batch(p.stream)
            ps = [p, q] if beside else [p]
            for x in ps:
                x.solve_begin()
            done = all(b.iterate(ps, o.max_it))
            if mixed and way == "pcg":      # by PCG, mixed precision takes one inner solve a call
                for _ in range(100):
                    done = done or all(b.iterate(ps, o.max_it))
            assert done
            v, sv = p.solve_end(check=False)
            assert p.last_status == status and sv["solver"] == st["solver"]
            assert torch.equal(u, v)
            if beside:
                q.solve_end()
            b.close()


def test_iterations_are_refinement_steps():
    """Calls of one iteration each are one substitution each, and end where one call ends."""
    import paper_2407_20026_amd as sso
    print("[gpu] one iteration a call", flush=True)
    o = sso.Options(rtol=3e-13, precision=sso.PREC_MIXED)
    u, st, status = _alone(sso, arch(), o)
    with sso.Problem(arch(), o) as p:
        b = sso.Batch(p.stream)
        p.solve_begin()
        calls, done = 0, False
        while not done and calls < 20:
            done = b.iterate([p], 1)[0]
            calls += 1
        v, sv = p.solve_end(check=False)
        b.close()
    assert calls == sv["refine_steps"] == st["refine_steps"]
    assert p.last_status == status and torch.equal(u, v)


def test_samples_are_of_the_last_solve():
    """A direct solve has no iterations to time: no samples of an earlier solve are reported."""
    import paper_2407_20026_amd as sso
    print("[gpu] timing samples", flush=True)
    with sso.Problem(meshgen.shell(20, seed=1),
                     sso.Options(rtol=1e-9, solver=sso.SOLVER_STANDARD, profile_every=8)) as p:
        _, st = p.solve()
        assert st["spmv_samples"] > 0 and st["spmv_us"] > 0.0
        p.set_options(sso.Options(rtol=1e-9, profile_every=8))
        _, st = p.solve()
        assert st["solver"] == sso.SOLVER_AUTO
        assert st["spmv_samples"] == 0 and st["spmv_us"] == 0.0
