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
