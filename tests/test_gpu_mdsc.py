"""GPU two-level column semicoarsening preconditioner (fo_mdsc_*) against the oracle: the
aggregation hierarchy bit for bit, the collapse weights, plane operators and Chebyshev bounds
element by element, one application on random vectors, and Newton solves preconditioned by
it against the oracle's direct-solve Newton."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

from fo_inputs import config0_slab, smooth_velocity, structured_box
from fo_inputs.meshgen import ExtrudedMesh, _dome_fields, ellipse_mesh
from oracle import fo_oracle as fo
from oracle import mdsc, solve

from gpu_util import gpu_jacobian, gpu_mesh, to_dev

pytestmark = pytest.mark.gpu


def _cap(n_points, L=6, seed=11, elem="wedge", sigma=None, a=70e3, b=40e3):
    rng = np.random.default_rng(seed)
    xy, tri = ellipse_mesh(n_points, a, b, rng)
    s, H, beta = _dome_fields(xy, a, b, rng, 2000.0, 300.0, 500.0, 1.0, 15e3, 60e3)
    sig = np.linspace(0, 1, L + 1) if sigma is None else sigma
    return ExtrudedMesh(elem, xy, tri, s, H, beta, sig, A=1e-16)


def _case(name):
    if name == "cap400_wedge":
        m = _cap(400)
    elif name == "cap3000_wedge_L10":
        m = _cap(3000, L=10, seed=5, a=250e3, b=120e3)
    elif name == "slab_hex":
        m, U = config0_slab()
        return m, U
    elif name == "cap400_tet":
        m = _cap(400, L=4, elem="tet")
    elif name == "tiny_exact_plane":
        m = _cap(50, L=3, seed=2)
    elif name == "single_layer":
        m = _cap(600, L=1, seed=3)
    elif name == "cap500_wedge_L24":
        # 24 layers: the weights and J P0 kernels run fewer columns (blocks) per workgroup to
        # keep their LDS staging within 64 KB
        m = _cap(500, L=24, seed=9)
    elif name == "graded_sigma":
        m = _cap(500, L=8, seed=4, sigma=np.linspace(0, 1, 9) ** 1.7)
    elif name in ("box_plane_64", "box_plane_65"):
        # 64 base vertices: the whole plane is the coarsest level (its inverse has the largest
        # size, 128 dofs); 65: one smoothing level above it
        nx, ny = (7, 7) if name == "box_plane_64" else (4, 12)
        xy, cells, sig = structured_box(nx, ny, 3, 20e3, 30e3, elem="wedge")
        m = _slab_fields(xy, cells, sig, seed=6)
    elif name == "islands_100":
        # 100 separate triangles: every aggregate of the first coarse level is isolated, so the
        # next level groups them 8 at a time
        rng = np.random.default_rng(7)
        base = np.array([[0.0, 0.0], [3e3, 0.0], [1e3, 2.5e3]])
        xy = np.concatenate([base + np.array([10e3 * (i % 10), 10e3 * (i // 10)]) for i in range(100)])
        xy += rng.uniform(-200.0, 200.0, xy.shape)
        cells = np.arange(300, dtype=np.int32).reshape(100, 3)
        m = _slab_fields(xy, cells, np.linspace(0, 1, 4), seed=8)
    else:
        raise KeyError(name)
    return m, solve.sia_guess(m) + smooth_velocity(m, np.random.default_rng(1), u_scale=5.0)


def _slab_fields(xy, cells, sigma, seed):
    rng = np.random.default_rng(seed)
    x, y = xy[:, 0], xy[:, 1]
    H = 800.0 + 100.0 * np.sin(x / 7e3) * np.cos(y / 9e3) + rng.uniform(-5.0, 5.0, len(x))
    bed = -0.01 * x
    beta = 1000.0 * (1.0 + 0.5 * np.sin(y / 5e3))
    return ExtrudedMesh("wedge", xy, cells, bed + H, H, beta, sigma, A=1e-16)


CASES = ["cap400_wedge", "cap3000_wedge_L10", "slab_hex", "cap400_tet", "tiny_exact_plane", "single_layer",
         "graded_sigma", "box_plane_64", "box_plane_65", "islands_100", "cap500_wedge_L24"]


def _oracle_levels(m):
    """Graphs and aggregates of every plane level, by the oracle's rules."""
    nbrs = mdsc.plane_graph(m)
    out = []
    while True:
        if len(nbrs) <= mdsc.COARSEST_MAX:
            out.append((nbrs, None))
            return out
        agg, n_agg = mdsc.aggregate(nbrs)
        out.append((nbrs, agg))
        nbrs = mdsc.coarse_graph(nbrs, agg, n_agg)


def _blocks_of(A, ptr, idx):
    """The 2x2 blocks of a scalar plane matrix at a block pattern: [nnzb, 4]."""
    A = sp.csr_matrix(A)
    rows = np.repeat(np.arange(len(ptr) - 1), np.diff(ptr))
    out = np.empty((len(idx), 4))
    for c in range(2):
        for d in range(2):
            out[:, 2 * c + d] = np.asarray(A[2 * rows + c, 2 * idx + d]).ravel()
    return out


@pytest.fixture(scope="module", params=CASES)
def setup_case(request):
    from paper_2204_04321_amd.api import Mdsc
    name = request.param
    m, U = _case(name)
    print(f"\n[mdsc] case {name}: V {m.n_verts} L {m.n_layers} elem {m.elem}", flush=True)
    M = gpu_mesh(m)
    P = Mdsc(M)
    _, Jg = gpu_jacobian(M, U)
    _, Jvals = M.jacobian(to_dev(U))
    P.setup(Jvals)
    torch.cuda.synchronize()
    _, Jo = fo.assemble(m, U)
    H = mdsc.Hierarchy(m, Jo.tocsr())
    return name, m, U, M, P, H, Jvals


def test_hierarchy_graphs_and_aggregates(setup_case):
    name, m, U, M, P, H, _ = setup_case
    want = _oracle_levels(m)
    assert P.n_levels == len(want) - 1 == len(H.levels), name
    for lvl, (nbrs, agg) in enumerate(want):
        ptr, idx, gagg = P.graph(lvl)
        assert np.array_equal(np.diff(ptr), [len(l) for l in nbrs]), (name, lvl)
        assert np.array_equal(idx, np.concatenate(nbrs)), (name, lvl)
        if agg is None:
            assert gagg is None
        else:
            assert np.array_equal(gagg, agg), (name, lvl)


def test_weights_plane_operators_and_bounds(setup_case):
    """FP64 setup against the oracle: the weights within 1e-11 of each weight vector's largest
    entry (a recursion against a dense solve of the same column, both backward stable: the
    difference is bounded by the column block's condition number times rounding, and the
    bar leaves room for condition numbers up to ~1e4), the plane blocks within 1e-10 of each
    level's largest block entry (sums of those weights times Jacobian values), the Gershgorin
    bounds within 1e-10 relative."""
    name, m, U, M, P, H, _ = setup_case
    W = P.export("weights").reshape(H.W.shape)
    scale = np.abs(H.W).max(axis=(1, 2))[:, None, None, :]
    err_w = (np.abs(W - H.W) / scale).max()
    errs = [err_w]
    for lvl in range(P.n_levels + 1):
        ptr, idx, _ = P.graph(lvl)
        A_g = P.export("plane", lvl).reshape(-1, 4)
        A_o = _blocks_of(H.levels[lvl]["A"] if lvl < len(H.levels) else H.A_coarse, ptr, idx)
        e = np.abs(A_g - A_o).max() / np.abs(A_o).max()
        errs.append(e)
        assert e <= 1e-10, (name, lvl, e)
        if lvl < P.n_levels:
            g = P.export("bound", lvl)[0]
            assert abs(g - H.levels[lvl]["g"]) <= 1e-10 * H.levels[lvl]["g"], (name, lvl)
    print(f"[mdsc] {name}: weights {err_w:.1e}, plane levels " + " ".join(f"{e:.1e}" for e in errs[1:]))
    assert err_w <= 1e-11, (name, err_w)


def test_apply_matches_oracle(setup_case):
    """z = M^-1 r for random r against the oracle's application of the same hierarchy.  Both
    store the column factors in FP32 from FP64 recursions that agree to rounding, so a factor
    can round to neighbouring FP32 values on the two sides (a relative change of 6e-8 in one
    factor); the bar 1e-6 of max |z| allows that change times the column solve's
    amplification.  Two vectors, the second after a second setup of the same Jacobian (the
    numeric state is rebuilt, not accumulated)."""
    name, m, U, M, P, H, Jvals = setup_case
    rng = np.random.default_rng(3)
    for rep in range(2):
        if rep == 1:
            P.setup(Jvals)
        r = rng.normal(size=m.n_dofs)
        z = P.apply(to_dev(r)).cpu().numpy()
        want = H.apply(r)
        err = np.abs(z - want).max() / np.abs(want).max()
        print(f"[mdsc] {name}: apply {err:.1e}")
        assert err <= 1e-6, (name, err)


@pytest.fixture(scope="module")
def cap_solution():
    m = _cap(400)
    U_ref, info = solve.newton_solve(m, solve.sia_guess(m), tol=1e-11)
    assert info["status"] == "converged"
    return m, U_ref, gpu_mesh(m)


@pytest.mark.parametrize("jdt", ["f64", "f32"])
def test_newton_with_mdsc_matches_oracle_solution(cap_solution, jdt):
    from paper_2204_04321_amd.api import Mdsc
    m, U_ref, M = cap_solution
    P = Mdsc(M)
    U = to_dev(solve.sia_guess(m))
    rep = M.newton_solve(U, tol=1e-8, jac_dtype=jdt, preconditioner="mdsc", mdsc=P)
    U0 = to_dev(solve.sia_guess(m))
    base = M.newton_solve(U0, tol=1e-8, jac_dtype=jdt)
    print(f"\n[newton mdsc {jdt}] its {rep['newton_its']} gmres {rep['lin_its']} (column: {base['newton_its']} / "
          f"{base['lin_its']}) res {rep['final_rel']:.2e}")
    assert rep["status"] == 0, rep
    Ug = U.cpu().numpy()
    f0 = np.linalg.norm(fo.residual(m, np.zeros_like(Ug)))
    assert np.linalg.norm(fo.residual(m, Ug)) <= 1.01e-8 * f0
    diff = np.abs(Ug - U_ref).max() / np.abs(U_ref).max()
    assert diff <= 1e-6, diff
    assert rep["lin_its"] < base["lin_its"], (rep["lin_its"], base["lin_its"])


@pytest.mark.parametrize("which", ["tet_cap", "marine_fronts", "hex_slab", "cap_24_layers"])
def test_newton_with_mdsc_other_meshes(which):
    """Tetrahedral extrusion, a marine sheet with a floating shelf (beta = 0) and ocean fronts,
    the hexahedral slab and a cap with 24 layers: Newton with the two-level preconditioner
    against the oracle's direct-solve Newton."""
    from paper_2204_04321_amd.api import Mdsc
    if which == "tet_cap":
        m = _cap(300, L=5, seed=21).with_fields(elem="tet")
    elif which == "cap_24_layers":
        m = _cap(150, L=24, seed=22)
    elif which == "marine_fronts":
        from fo_inputs import marine_sheet
        m, _ = marine_sheet(seed=5, n_points=400, n_layers=5)
    else:
        m, _ = config0_slab()
    print(f"\n[newton mdsc {which}] V {m.n_verts} L {m.n_layers} elem {m.elem}", flush=True)
    U_ref, info = solve.newton_solve(m, solve.sia_guess(m), tol=1e-11)
    assert info["status"] == "converged", info
    M = gpu_mesh(m)
    P = Mdsc(M)
    U = to_dev(solve.sia_guess(m))
    rep = M.newton_solve(U, tol=1e-8, preconditioner="mdsc", mdsc=P)
    print(f"[newton mdsc {which}] its {rep['newton_its']} gmres {rep['lin_its']} res {rep['final_rel']:.2e}")
    assert rep["status"] == 0, rep
    Ug = U.cpu().numpy()
    f0 = np.linalg.norm(fo.residual(m, np.zeros_like(Ug)))
    assert np.linalg.norm(fo.residual(m, Ug)) <= 1.01e-8 * f0
    diff = np.abs(Ug - U_ref).max() / np.abs(U_ref).max()
    print(f"[newton mdsc {which}] max |U - U_oracle| / max |U_oracle| = {diff:.2e}")
    assert diff <= 1e-6


def _icesheet_patch(n_points, seed=1):
    """The ice-sheet configuration (dome, bed and log-normal beta fields, 10 layers) on an
    ellipse scaled down with the point count, so the base spacing stays the ice sheet's."""
    rng = np.random.default_rng(seed)
    sc = (n_points / 125_000) ** 0.5
    a, b = 750e3 * sc, 350e3 * sc
    xy, tri = ellipse_mesh(n_points, a, b, rng)
    s, H, beta = _dome_fields(xy, a, b, rng, 3000.0, 500.0, 500.0, 1.0, 30e3 * sc, 200e3 * sc)
    return ExtrudedMesh("wedge", xy, tri, s, H, beta, np.linspace(0, 1, 11), A=1e-16)


def test_mdsc_cuts_gmres_iterations_on_an_icesheet_patch():
    """6000 base points at the ice sheet's spacing, 10 layers: fewer GMRES iterations per
    Newton step than the column preconditioner."""
    from paper_2204_04321_amd.api import Mdsc
    m = _icesheet_patch(6000)
    M = gpu_mesh(m)
    P = Mdsc(M)
    out = {}
    for prec in ("column", "mdsc"):
        U = to_dev(solve.sia_guess(m))
        kw = {"preconditioner": "mdsc", "mdsc": P} if prec == "mdsc" else {}
        rep = M.newton_solve(U, tol=1e-8, **kw)
        assert rep["status"] == 0, (prec, rep)
        out[prec] = rep
        print(f"\n[newton patch6000 {prec}] its {rep['newton_its']} gmres {rep['lin_its']} "
              f"({rep['lin_its'] / max(rep['newton_its'], 1):.1f} per step) lin {rep['ms_linear_solve']:.1f} ms")
    per = {k: v["lin_its"] / max(v["newton_its"], 1) for k, v in out.items()}
    assert per["mdsc"] < 0.8 * per["column"], per


def test_mdsc_argument_errors():
    from paper_2204_04321_amd.api import Mdsc
    from paper_2204_04321_amd._lib import FoError
    m = _cap(120, L=2, seed=8)
    M, M2 = gpu_mesh(m), gpu_mesh(m)
    P = Mdsc(M)
    U = to_dev(solve.sia_guess(m))
    with pytest.raises(FoError, match="no successful fo_mdsc_setup"):
        P.apply(torch.zeros_like(U))
    with pytest.raises(FoError, match="no successful fo_mdsc_setup"):
        P.export("weights")
    rep = M2.newton_solve(U.clone(), preconditioner="mdsc", mdsc=P)
    assert rep["status"] == -1 and "created on this mesh" in rep["message"]
    rep = M.newton_solve(U.clone(), preconditioner="mdsc", mdsc=P, linear_solver="pcg")
    assert rep["status"] == -1 and "not symmetric" in rep["message"]
    rep = M.newton_solve(U.clone(), preconditioner="mdsc", mdsc=None)
    assert rep["status"] == -1
    # a non-finite Jacobian value makes a plane diagonal block non-finite: reported, no apply
    _, J = M.jacobian(U)
    J[0] = float("nan")
    with pytest.raises(FoError, match="singular or not finite"):
        P.setup(J)
    with pytest.raises(FoError, match="no successful fo_mdsc_setup"):
        P.apply(torch.zeros_like(U))
    r = torch.zeros_like(U)
    with pytest.raises(FoError, match="aliased"):
        from paper_2204_04321_amd import _lib
        _lib.check(_lib.lib().fo_mdsc_apply(P.handle, r.data_ptr(), r.data_ptr(), None))


def test_icesheet_two_level_full_size():
    """Ice-sheet configuration (125k base vertices, 10 layers) in the benchmark's launch
    configuration: every plane level's graph and aggregates bit for bit against the oracle's
    rules; the collapse weights of 64 seeded columns and of their neighbours, and the plane
    blocks of the seeded columns, against the oracle's from the Jacobian rows it assembles
    around them; one application linear and bitwise repeatable; the Newton solve with the
    two-level preconditioner reaching the column-preconditioned solution."""
    from fo_inputs import config1_icesheet
    from paper_2204_04321_amd.api import Mdsc
    m, U = config1_icesheet()
    print(f"\n[case] icesheet two-level: V {m.n_verts} dofs {m.n_dofs}", flush=True)
    M = gpu_mesh(m)
    P = Mdsc(M)
    _, Jv = M.jacobian(to_dev(U))
    P.setup(Jv)
    torch.cuda.synchronize()
    want = _oracle_levels(m)
    assert P.n_levels == len(want) - 1
    for lvl, (nbrs, agg) in enumerate(want):
        ptr, idx, gagg = P.graph(lvl)
        assert np.array_equal(np.diff(ptr), [len(l) for l in nbrs]) and np.array_equal(idx, np.concatenate(nbrs))
        assert (gagg is None) == (agg is None) and (agg is None or np.array_equal(gagg, agg)), lvl
    print(f"[icesheet two-level] levels {P.level_verts} equal the oracle's", flush=True)

    L1 = m.n_layers + 1
    nb = 2 * L1
    rng = np.random.default_rng(5)
    seeds = rng.choice(m.n_verts, 64, replace=False)
    ptr0, idx0, _ = P.graph(0)
    cols = np.unique(np.concatenate([idx0[ptr0[v]:ptr0[v + 1]] for v in seeds]))
    pos = {int(c): i for i, c in enumerate(cols)}
    dofs = (cols[:, None] * nb + np.arange(nb)[None, :]).ravel()
    _, Jr, _ = fo.assemble_rows(m, U, dofs)
    Jr = sp.csr_matrix(Jr)
    blocks = np.stack([Jr[i * nb:(i + 1) * nb][:, c * nb:(c + 1) * nb].toarray() for i, c in enumerate(cols)])
    Wo = mdsc.vertical_weights(blocks)
    Wg = P.export("weights").reshape(m.n_verts, L1, 2, 2)[cols]
    err_w = (np.abs(Wg - Wo) / np.abs(Wo).max(axis=(1, 2))[:, None, None, :]).max()
    A_g = P.export("plane", 0).reshape(-1, 4)
    err_a = 0.0
    for v in seeds:
        i = pos[int(v)]
        Jrow = Jr[i * nb:(i + 1) * nb]
        Pv = Wo[i].reshape(nb, 2)
        Ao = np.stack([(Pv.T @ Jrow[:, w * nb:(w + 1) * nb].toarray() @ Wo[pos[int(w)]].reshape(nb, 2)).ravel()
                       for w in idx0[ptr0[v]:ptr0[v + 1]]])
        err_a = max(err_a, np.abs(A_g[ptr0[v]:ptr0[v + 1]] - Ao).max() / np.abs(Ao).max())
    print(f"[icesheet two-level] weights of {len(cols)} columns {err_w:.1e}, plane rows of 64 columns {err_a:.1e}",
          flush=True)
    assert err_w <= 1e-11 and err_a <= 1e-10

    g = torch.Generator(device="cpu").manual_seed(9)
    r1 = torch.randn(m.n_dofs, generator=g, dtype=torch.float64).cuda()
    r2 = torch.randn(m.n_dofs, generator=g, dtype=torch.float64).cuda()
    z1, z2 = P.apply(r1), P.apply(r2)
    z3 = P.apply(2.0 * r1 - 3.0 * r2)
    z1b = P.apply(r1)
    torch.cuda.synchronize()
    lin = ((z3 - (2.0 * z1 - 3.0 * z2)).abs().max() / z3.abs().max()).item()
    print(f"[icesheet two-level] linearity {lin:.1e}", flush=True)
    assert torch.equal(z1, z1b) and lin <= 1e-10

    sols = {}
    for prec in ("column", "mdsc"):
        Ug = to_dev(solve.sia_guess(m))
        kw = {"preconditioner": "mdsc", "mdsc": P} if prec == "mdsc" else {}
        rep = M.newton_solve(Ug, tol=1e-8, **kw)
        assert rep["status"] == 0 and rep["final_rel"] <= 1e-8, (prec, rep)
        sols[prec] = (Ug.cpu().numpy(), rep)
        print(f"[icesheet newton {prec}] its {rep['newton_its']} gmres {rep['lin_its']} "
              f"res {rep['final_rel']:.1e}", flush=True)
    Uc, rc = sols["column"]
    Um, rm = sols["mdsc"]
    diff = np.abs(Um - Uc).max() / np.abs(Uc).max()
    print(f"[icesheet newton] max |U_two_level - U_column| / max |U_column| = {diff:.1e}", flush=True)
    assert rm["newton_its"] == rc["newton_its"] and rm["lin_its"] < 0.75 * rc["lin_its"]
    assert diff <= 1e-6


@pytest.mark.parametrize("name", ["cap400_wedge", "cap400_tet", "slab_hex"])
def test_setup_from_fp32_values_matches_oracle(name):
    """The FP32-value setup path on the oracle's own Jacobian rounded to FP32 (written into the
    library's layout through its CSR pattern, which equals the oracle's): weights, plane
    operators and one application against the oracle's hierarchy of the same rounded values,
    at the bars of the FP64 path."""
    from paper_2204_04321_amd.api import Mdsc
    m, U = _case(name)
    M = gpu_mesh(m)
    rowptr, colidx = M.pattern()
    _, Jo = fo.assemble(m, U)
    Jo = sp.csr_matrix(Jo)
    assert np.array_equal(rowptr.cpu().numpy(), Jo.indptr) and np.array_equal(colidx.cpu().numpy(), Jo.indices)
    J32 = Jo.data.astype(np.float32)
    Jr = sp.csr_matrix((J32.astype(np.float64), Jo.indices, Jo.indptr), shape=Jo.shape)
    P = Mdsc(M)
    P.setup(torch.from_numpy(J32).cuda())
    H = mdsc.Hierarchy(m, Jr)
    W = P.export("weights").reshape(H.W.shape)
    err_w = (np.abs(W - H.W) / np.abs(H.W).max(axis=(1, 2))[:, None, None, :]).max()
    errs = []
    for lvl in range(P.n_levels + 1):
        ptr, idx, _ = P.graph(lvl)
        A_o = _blocks_of(H.levels[lvl]["A"] if lvl < len(H.levels) else H.A_coarse, ptr, idx)
        errs.append(np.abs(P.export("plane", lvl).reshape(-1, 4) - A_o).max() / np.abs(A_o).max())
    r = np.random.default_rng(4).normal(size=m.n_dofs)
    z = P.apply(to_dev(r)).cpu().numpy()
    want = H.apply(r)
    err_z = np.abs(z - want).max() / np.abs(want).max()
    print(f"\n[mdsc fp32 values] {name}: weights {err_w:.1e}, plane {max(errs):.1e}, apply {err_z:.1e}")
    assert err_w <= 1e-11 and max(errs) <= 1e-10 and err_z <= 1e-6


def test_weights_fallback_columns_match_oracle():
    """Columns whose block-tridiagonal solve gives a weight vector with non-positive mean
    (here: the column blocks of every seventh column negated, so they are negative definite)
    take the plain vertical average e_c on both sides; the rest of the setup is unaffected.
    The Jacobian is the oracle's, written into the library's layout through its pattern."""
    from paper_2204_04321_amd.api import Mdsc
    m, U = _case("cap400_wedge")
    M = gpu_mesh(m)
    _, Jo = fo.assemble(m, U)
    Jo = sp.csr_matrix(Jo).tocoo()
    nb = 2 * (m.n_layers + 1)
    col = Jo.row // nb
    flip = ((col % 7) == 0) & (col == Jo.col // nb)
    data = np.where(flip, -Jo.data, Jo.data)
    Jm = sp.csr_matrix((data, (Jo.row, Jo.col)), shape=Jo.shape)
    Jm.sort_indices()
    rowptr, colidx = M.pattern()
    assert np.array_equal(rowptr.cpu().numpy(), Jm.indptr) and np.array_equal(colidx.cpu().numpy(), Jm.indices)
    P = Mdsc(M)
    P.setup(torch.from_numpy(Jm.data.copy()).cuda())
    H = mdsc.Hierarchy(m, Jm)
    W = P.export("weights").reshape(H.W.shape)
    e = np.zeros((m.n_layers + 1, 2, 2))
    e[:, 0, 0] = e[:, 1, 1] = 1.0
    fell = [v for v in range(m.n_verts) if np.array_equal(H.W[v], e)]
    assert len(fell) >= m.n_verts // 7 - 1
    assert all(np.array_equal(W[v], e) for v in fell)
    err_w = (np.abs(W - H.W) / np.abs(H.W).max(axis=(1, 2))[:, None, None, :]).max()
    ptr, idx, _ = P.graph(0)
    A_o = _blocks_of(H.levels[0]["A"] if H.levels else H.A_coarse, ptr, idx)
    err_a = np.abs(P.export("plane", 0).reshape(-1, 4) - A_o).max() / np.abs(A_o).max()
    print(f"\n[mdsc fallback] {len(fell)} columns on e_c; weights {err_w:.1e}, plane {err_a:.1e}")
    assert err_w <= 1e-11 and err_a <= 1e-10


@pytest.mark.parametrize("name,sizes", [("islands_512", [1536, 512, 64]), ("islands_513", [1539, 513, 65, 9]),
                                        ("strip", [2000, 334, 112, 38])])
def test_apply_where_levels_are_one_matrix(name, sizes):
    """Planes whose coarser levels lie at the largest size that is applied as one matrix, just above it,
    and below it twice over (a strip, which coarsens three- to sixfold): one application against the
    oracle's V-cycle.  The FP32 column factors bound the difference as in
    test_apply_matches_oracle (the matrix itself is FP64): the same 1e-6."""
    from paper_2204_04321_amd.api import Mdsc
    if name == "strip":
        xy, cells, sig = structured_box(999, 1, 2, 999 * 2e3, 2e3, elem="wedge")
        m = _slab_fields(xy, cells, sig, seed=9)
    else:
        n = int(name.split("_")[1])
        base = np.array([[0.0, 0.0], [3e3, 0.0], [1e3, 2.5e3]])
        xy = np.concatenate([base + np.array([10e3 * (i % 32), 10e3 * (i // 32)]) for i in range(n)])
        m = _slab_fields(xy, np.arange(3 * n, dtype=np.int32).reshape(n, 3), np.linspace(0, 1, 3), seed=10)
    M = gpu_mesh(m)
    P = Mdsc(M)
    got = [len(P.graph(lvl)[0]) - 1 for lvl in range(P.n_levels + 1)]
    print(f"\n[mdsc matrix] {name}: levels {got}", flush=True)
    assert got == sizes
    U = solve.sia_guess(m) + smooth_velocity(m, np.random.default_rng(1), u_scale=5.0)
    _, Jo = fo.assemble(m, U)
    Jo = sp.csr_matrix(Jo)
    P.setup(torch.from_numpy(Jo.data.copy()).cuda())
    H = mdsc.Hierarchy(m, Jo)
    r = np.random.default_rng(4).normal(size=m.n_dofs)
    z = P.apply(to_dev(r)).cpu().numpy()
    want = H.apply(r)
    err = np.abs(z - want).max() / np.abs(want).max()
    print(f"[mdsc matrix] {name}: apply {err:.1e}")
    assert err <= 1e-6
