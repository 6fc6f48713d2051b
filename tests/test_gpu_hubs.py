"""The direct solver on structures that one node holds together: ribs and spokes, whose elimination
joins many pieces under fronts that own no nodes."""
import numpy as np
import pytest
import scipy.sparse as sp

import meshgen
from oracle import solve

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def ribs(count, length):
    """Arched ribs of `length` members from one crown to clamped feet on a circle."""
    a = 2.0 * np.pi * np.arange(count) / count
    t = np.arange(1, length + 1) / length
    r = 10.0 * np.sin(0.5 * np.pi * t)
    xyz = np.stack([np.cos(a)[:, None] * r, np.sin(a)[:, None] * r,
                    np.broadcast_to(6.0 * np.cos(0.5 * np.pi * t), (count, length))], axis=-1)
    ids = 1 + np.arange(count * length).reshape(count, length)
    beams = np.stack([np.hstack([np.zeros((count, 1), int), ids[:, :-1]]), ids], axis=-1)
    n = 1 + count * length
    fixed = np.zeros((n, 6), np.uint8)
    fixed[ids[:, -1]] = 1
    f = np.zeros((n, 6))
    f[:, 2] = -1e3
    prop = np.tile([2.1e11, 8.1e10, 1e-3, 1e-6, 1e-6, 2e-6], (count * length, 1))
    return meshgen.Mesh(xyz=np.vstack([[[0.0, 0.0, 6.0]], xyz.reshape(-1, 3)]), fixed=fixed,
                        f_nodal=f, beam_nodes=beams.reshape(-1, 2).astype(np.int32),
                        beam_prop=prop, name="ribs")


# spokes of one member (nine or fewer are cut like any part), of a leaf's nodes and more, and a dome
@pytest.mark.parametrize("count,length", [(9, 2), (12, 1), (25, 3), (11, 10), (13, 11), (96, 20)])
def test_ribs_from_one_crown(count, length):
    """Solved directly, to the target in long double (1 % for the sums of squares in 64 bits), the
    load's solution and a general objective's alike."""
    import paper_2407_20026_amd as sso
    print(f"[gpu] {count} ribs of {length}", flush=True)
    mesh = ribs(count, length)
    a = np.zeros((mesh.n_nodes, 6))
    a[0] = 1.0
    with sso.Problem(mesh, sso.Options(rtol=1e-9)) as p:
        u, st = p.solve()
        assert st["solver"] == sso.SOLVER_AUTO and st["iters"] == 0
        assert p.adjoint("linear", dg_du=a)["stats"]["iters"] == 0
        vals, f = p.matrix()
        pat = {k: v.cpu().numpy() for k, v in p.pattern().items()}
        n = 6 * p.n_nodes
        K = sp.csr_matrix((vals.cpu().numpy(), pat["col"], pat["row_ptr"]), shape=(n, n))
    f = f.cpu().numpy().ravel()
    r = solve.residual_ld(K, u.cpu().numpy().ravel(), f)
    assert np.sqrt(np.sum(r * r)) <= 1.01e-9 * np.linalg.norm(f)
