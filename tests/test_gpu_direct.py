"""The direct solver that sso_solve's automatic choice takes (FP64): at the sizes where its tiles
end and begin, on every kind of structure, and where it hands over to PCG."""
import numpy as np
import pytest
import scipy.sparse as sp

import meshgen
from oracle import solve

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def rect_shell(mx, my, seed):
    """A rectangular cut of the seeded square shell: mx x my quads."""
    m = max(mx, my)
    s = meshgen.shell(m, seed=seed)
    n = m + 1
    keep = (np.arange(n * n) % n <= mx) & (np.arange(n * n) // n <= my)
    new = np.full(n * n, -1)
    new[keep] = np.arange(keep.sum())
    q = keep[s.quad_nodes].all(axis=1)
    s.quad_nodes = new[s.quad_nodes[q]].astype(np.int32)
    s.quad_prop = s.quad_prop[q].copy()
    s.xyz, s.f_nodal = s.xyz[keep].copy(), s.f_nodal[keep].copy()
    s.fixed = s.fixed[keep].copy()
    s.fixed[[0, mx, keep.sum() - 1, keep.sum() - 1 - mx], :3] = 1
    return s


def two_pieces():
    """A grid-shell and a shell that share no node, numbered one after the other."""
    a, b = meshgen.gridshell(9, seed=3), meshgen.shell(7, seed=4)
    n = a.n_nodes
    m = b.copy()
    m.xyz = np.vstack([a.xyz, b.xyz + [50.0, 0.0, 0.0]])
    m.fixed = np.vstack([a.fixed, b.fixed])
    m.f_nodal = np.vstack([a.f_nodal, b.f_nodal])
    m.beam_nodes, m.beam_prop = a.beam_nodes.copy(), a.beam_prop.copy()
    m.quad_nodes = (b.quad_nodes + n).astype(np.int32)
    return m


def renumbered(mesh, seed):
    """The same structure with its nodes numbered at random."""
    p = np.random.default_rng(seed).permutation(mesh.n_nodes)      # old -> new
    m = mesh.copy()
    for k in ("xyz", "fixed", "f_nodal"):
        v = np.empty_like(getattr(mesh, k))
        v[p] = getattr(mesh, k)
        setattr(m, k, v)
    m.quad_nodes = p[mesh.quad_nodes].astype(np.int32)
    m.beam_nodes = p[mesh.beam_nodes].astype(np.int32)
    return m


def soft_and_stiff(m=24):
    """Per-element stiffness scales over six decades."""
    s = meshgen.shell(m, seed=12)
    s.quad_scale = np.random.default_rng(3).uniform(0.01, 1.0, s.n_quads) ** 3
    return s


CASES = {
    # one front alone (10 nodes), then a separator; a panel of 60 and of 66 own DOFs
    "grid2x2": lambda: meshgen.gridshell(2, seed=1),
    "grid3x3": lambda: meshgen.gridshell(3, seed=1),
    "grid4x4": lambda: meshgen.gridshell(4, seed=1),
    "shell2x2": lambda: meshgen.shell(2, seed=1),
    # separators of 10, 11, 12, 21, 22 and 33 nodes (60, 66, 72, 126, 132 and 198 own DOFs)
    "shell9x9": lambda: meshgen.shell(9, seed=2),
    "shell10x10": lambda: meshgen.shell(10, seed=2),
    "shell11x11": lambda: meshgen.shell(11, seed=2),
    "shell20x31": lambda: rect_shell(20, 31, 5),
    "shell21x21": lambda: meshgen.shell(21, seed=2),
    "shell32x64": lambda: rect_shell(32, 64, 6),
    "grid43x43": lambda: meshgen.gridshell(43, seed=7),
    "strip3x90": lambda: rect_shell(3, 90, 8),
    "arch11": lambda: meshgen.arch_bridge(11, n_spans=30),
    "renumbered": lambda: renumbered(meshgen.shell(19, seed=9), 4),
    "pieces": two_pieces,
    "soft_and_stiff": soft_and_stiff,
}


def _residual(p, u):
    """|f - K u| / |f| of the free equations in long double, under the problem's own K (|f - K u|
    itself without a load: every loaded DOF of the 2 x 2 grid-shell is held)."""
    vals, f = p.matrix()
    pat = {k: v.cpu().numpy() for k, v in p.pattern().items()}
    n = 6 * p.n_nodes
    K = sp.csr_matrix((vals.cpu().numpy(), pat["col"], pat["row_ptr"]), shape=(n, n))
    f = f.cpu().numpy().ravel()
    r = solve.residual_ld(K, u.cpu().numpy().ravel(), f)
    return float(np.sqrt(np.sum(r * r)) / (np.linalg.norm(f) or 1.0))


@pytest.mark.parametrize("name", list(CASES))
def test_residual_and_agreement_with_pcg(name):
    """The residual target is met in long double; u and a general objective's gradient agree with
    those of the standard recurrences at the same target.  Two solutions with residuals of
    rtol |f| differ by at most 2 rtol |K^-1| |f|; |K^-1| |f| / |u| stays below 10^3 on these
    structures (5 x 10^2 on the 60 x 60 shell), so 2e-7 bounds u at rtol 1e-10, and the gradient,
    bilinear in u and lambda, 10 times that."""
    import paper_2407_20026_amd as sso
    mesh = CASES[name]()
    print(f"[gpu] direct {name}", flush=True)
    a = np.zeros((mesh.n_nodes, 6))
    a[mesh.n_nodes // 2, 2] = 1.0
    out = []
    for solver in (sso.SOLVER_AUTO, sso.SOLVER_STANDARD):
        with sso.Problem(mesh, sso.Options(rtol=1e-10, max_it=200000, solver=solver)) as p:
            u, st = p.solve()
            g = p.adjoint("linear", dg_du=a)
            if solver == sso.SOLVER_AUTO:
                assert st["solver"] == sso.SOLVER_AUTO and st["iters"] == 0
                assert g["stats"]["iters"] == 0
                # the reported residual is the long-double one to rounding
                assert _residual(p, u) <= 1.01e-10
                u2, _ = p.solve()
                assert torch.equal(u, u2)
            out.append((u.cpu().numpy(), g["dg_dxyz"].cpu().numpy()))
    (u, g), (v, h) = out
    assert np.linalg.norm(u - v) <= 2e-7 * np.linalg.norm(v)
    assert np.abs(g - h).max() <= 2e-6 * np.abs(h).max()


def test_supports_moved_and_an_update():
    """Prescribed displacements hold exactly, and new coordinates are factored anew."""
    import paper_2407_20026_amd as sso
    rng = np.random.default_rng(5)
    mesh = meshgen.shell(13, seed=3)
    mesh = mesh.copy(u_prescribed=1e-3 * rng.standard_normal((mesh.n_nodes, 6)))
    fixed = mesh.fixed != 0
    x2 = mesh.xyz + rng.normal(0.0, 0.01, mesh.xyz.shape)
    with sso.Problem(mesh, sso.Options(rtol=1e-10)) as p:
        p.solve()
        p.update(xyz=x2)
        u, st = p.solve()
        assert st["solver"] == sso.SOLVER_AUTO
    np.testing.assert_array_equal(u.cpu().numpy()[fixed], mesh.u_prescribed[fixed])
    with sso.Problem(mesh.copy(xyz=x2), sso.Options(rtol=1e-10)) as q:
        v, _ = q.solve()
    assert torch.equal(u, v)


def lattice(n):
    """Members along the edges of an n x n x n lattice, one face clamped."""
    i, j, k = (v.ravel() for v in np.meshgrid(*3 * [np.arange(n)], indexing="ij"))
    ids = np.arange(n ** 3).reshape(n, n, n)
    beams = np.concatenate([np.stack([ids[:-1].ravel(), ids[1:].ravel()], 1),
                            np.stack([ids[:, :-1].ravel(), ids[:, 1:].ravel()], 1),
                            np.stack([ids[:, :, :-1].ravel(), ids[:, :, 1:].ravel()], 1)])
    fixed = np.zeros((n ** 3, 6), np.uint8)
    fixed[k == 0] = 1
    f = np.zeros((n ** 3, 6))
    f[k == n - 1, 2] = -1e3
    prop = np.tile([2.1e11, 8.1e10, 1e-3, 1e-6, 1e-6, 2e-6], (len(beams), 1))
    return meshgen.Mesh(xyz=np.stack([i, j, k], 1).astype(float), fixed=fixed, f_nodal=f,
                        beam_nodes=beams.astype(np.int32), beam_prop=prop, name="lattice")


def test_a_lattice_that_fills_too_much_stays_with_pcg():
    import paper_2407_20026_amd as sso
    print("[gpu] lattice", flush=True)
    with sso.Problem(lattice(11), sso.Options(rtol=1e-9)) as p:
        _, st = p.solve()
    assert st["solver"] == sso.SOLVER_FUSED and st["iters"] > 0


def test_a_target_below_the_floor_keeps_its_status():
    """A residual that 64 bits cannot reach ends as it does in PCG: not converged, with the best
    displacements kept."""
    import paper_2407_20026_amd as sso
    mesh = meshgen.gridshell(11, seed=0)
    with sso.Problem(mesh, sso.Options(rtol=1e-15, max_it=20000)) as p:
        u, st = p.solve(check=False)
        assert p.last_status == sso.SSO_ENOTCONV and st["rel_residual"] < 1e-9
        assert _residual(p, u) < 1e-9


def clique(n, seed=2):
    """Members between every two of n nodes: one front, which no separator cuts."""
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(n, 1)
    fixed = np.zeros((n, 6), np.uint8)
    fixed[0] = 1
    f = np.zeros((n, 6))
    f[1:, 2] = -1e3
    prop = np.tile([2.1e11, 8.1e10, 1e-3, 1e-6, 1e-6, 2e-6], (len(i), 1))
    return meshgen.Mesh(xyz=rng.uniform(0.0, 3.0, (n, 3)), fixed=fixed, f_nodal=f,
                        beam_nodes=np.stack([i, j], 1).astype(np.int32), beam_prop=prop,
                        name="clique")


# own DOFs 18 .. 132: up to, at and past the 16-column panels of a pivot block and its 64 columns
@pytest.mark.parametrize("n", [3, 5, 8, 9, 10, 11, 13, 16, 19, 21, 22])
def test_pivot_blocks_of_every_width(n):
    """K of a clique is factored without a fallback and the residual target met in long double
    (1 % for the sum of squares in 64 bits), at a right-hand side other than the load as well."""
    import paper_2407_20026_amd as sso
    print(f"[gpu] clique {n}", flush=True)
    mesh = clique(n)
    a = np.zeros((n, 6))
    a[n // 2] = 1.0
    with sso.Problem(mesh, sso.Options(rtol=1e-12)) as p:
        u, st = p.solve()
        assert st["solver"] == sso.SOLVER_AUTO and st["iters"] == 0
        assert _residual(p, u) <= 1.01e-12
        assert p.adjoint("linear", dg_du=a)["stats"]["iters"] == 0


# 1, 15, 16, 17 and 33 elements: 16 lanes an element, 4 a wave and 16 a workgroup
@pytest.mark.parametrize("mx,my", [(1, 1), (3, 5), (4, 4), (1, 17), (3, 11)])
def test_shell_elements(mx, my):
    """K and the adjoint's element terms against the oracle, for the same displacements.  An entry
    of K is a sum over at most four elements of some 400 rounded terms, none above the largest
    entry: 400 x 1.1e-16 x 4 < 2e-13.  A derivative has some 1000, of products of displacements
    that exceed what the strains leave of them by up to 10^3: 1e-10 of the largest."""
    import paper_2407_20026_amd as sso
    from oracle import assembly, sensitivity
    print(f"[gpu] elements {mx} x {my}", flush=True)
    mesh = rect_shell(mx, my, 11)
    rng = np.random.default_rng(1)
    mesh.xyz = mesh.xyz + rng.normal(0.0, 0.03, mesh.xyz.shape)
    mesh.quad_scale = rng.uniform(0.3, 1.0, mesh.n_quads)
    K, f = assembly.assemble(mesh), assembly.load_vector(mesh)
    ref = assembly.masked_system(mesh, K, f)[0].tocsr()
    ref.sort_indices()
    with sso.Problem(mesh, sso.Options(rtol=1e-10)) as p:
        u, _ = p.solve()
        g = p.adjoint("compliance")
        vals, _ = p.matrix()
    assert np.abs(vals.cpu().numpy() - ref.data).max() <= 2e-13 * np.abs(ref.data).max()
    u = u.cpu().numpy().ravel()
    gb, gq = sensitivity.element_terms(mesh, u, u, 1.0, 1.0)
    for got, want in zip((g["dg_dxyz"], g["dg_dt"], g["dg_dscale"]),
                         sensitivity.gather(mesh, gb, gq)):
        assert np.abs(got.cpu().numpy() - want).max() <= 1e-10 * np.abs(want).max()
