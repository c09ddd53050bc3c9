"""Kernel variants chosen by size: each at the edges of its range."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _handle(p, **opt):
    from paper_1602_03641_amd import vag
    opt.setdefault("max_iter", 20000)
    opt.setdefault("cfl", p.cfl)
    h = vag.Handle(p, **opt)
    return h, h.solve_pressure()


@pytest.mark.parametrize("dims,B", [((9, 7, 6), 2), ((9, 7, 6), 129), ((13, 4, 3), 64), ((12, 11, 9), 512),
                                    ((12, 11, 9), 900), ((12, 11, 9), 2048)])
def test_ilu_substitutions(dims, B):
    """Block sizes on both sides of what fits in LDS, last blocks ragged,
    levels of more rows than a wavefront takes at once: z = M^-1 r element by
    element against the oracle's block-Jacobi ILU(0) of its own system.  Each
    entry of z is a sum of about 10^2 terms per block row, so 1e-11 of max |z|
    leaves 10^3 over the rounding of the substitutions."""
    from paper_1602_03641_amd import vag
    from oracle import ilu
    p = synth.random_problem(dims, 21, n_patches=4, n_steps=0, ratios=(1e2, 1e4))
    h, info = _handle(p, rtol=1e-8, precond=vag.VAG_PC_BJILU0, krylov=vag.VAG_BICGSTAB, ilu_block_rows=B,
                      eliminate_frac_faces=0)
    A, _ = oracle.system(p)
    rows = ilu.bj_ilu0(A, B)
    r = np.random.default_rng(22).standard_normal(A.shape[0])
    z, zr = h.apply_preconditioner(r), ilu.bj_ilu0_apply(rows, r)
    assert np.abs(z - zr).max() <= 1e-11 * np.abs(zr).max()
    h.close()


def _fan(sectors, layers):
    """Wedges around an axis: its nodes couple to every node of three layers."""
    k, i = np.meshgrid(np.arange(layers), np.arange(sectors), indexing="ij")
    k, i = k.ravel(), i.ravel()
    at = lambda k, i: k * (sectors + 1) + 1 + i % sectors  # noqa: E731
    axis = k * (sectors + 1)
    up = sectors + 1
    cells = np.stack([axis, at(k, i), at(k, i + 1), axis + up, at(k, i) + up, at(k, i + 1) + up], 1)
    a = 2 * np.pi * np.arange(sectors) / sectors
    ring = np.concatenate([[[0.0, 0.0]], np.stack([np.cos(a), np.sin(a)], 1)])
    xyz = np.concatenate([np.c_[ring, np.full(sectors + 1, 0.3 * z)] for z in range(layers + 1)])
    cfp, cf, fnp, fn, _ = synth.faces_of_cells(cells)
    z = np.repeat(np.arange(layers + 1), sectors + 1)
    nc = len(cells)
    perm = np.zeros((nc, 6))
    perm[:, :3] = np.random.default_rng(3).uniform(0.5, 2.0, (nc, 1))
    return synth.GeneralProblem(
        name="fan", xyz=xyz, cells=cells, cell_face_ptr=cfp, cell_faces=cf, face_node_ptr=fnp, face_nodes=fn,
        frac_face_ids=np.zeros(0, np.int32), frac_width=np.zeros(0), frac_perm=np.zeros(0), frac_poro=np.zeros(0),
        perm=perm, poro=np.ones(nc), mu=1.0, dirichlet=((z == 0) | (z == layers)).astype(np.uint8),
        p_bar=1.0 - z / layers, c_bar=(z == 0).astype(float))


@pytest.mark.parametrize("mesh,coarse", [((5, 4, 4), 8), ((14, 12, 11), 6), ((26, 24, 22), 12), ("fan", 12)])
def test_classical_products(mesh, coarse):
    """Classical hierarchies coarsened far down; on the fan, rows of A P and
    R A P with more columns than a wavefront holds in LDS: every coarse operator
    is P^T A P of the level above.  An entry sums at most ~10^4 products, each
    rounded relative to max |A|: 1e-12 max |A|."""
    from paper_1602_03641_amd import vag
    import scipy.sparse as sp
    p = _fan(120, 14) if mesh == "fan" else synth.random_problem(mesh, 23, n_patches=5, n_steps=0, ratios=(1e2, 1e4))
    h, info = _handle(p, rtol=1e-8, precond=vag.VAG_PC_AMG, amg_kind=1, amg_coarse_size=coarse)
    mats = []
    for d in (h.amg_level(l) for l in range(info["amg_levels"])):
        n = len(d["A"][0]) - 1
        A = sp.csr_matrix((d["A"][2], d["A"][1], d["A"][0]), shape=(n, n))
        P = sp.csr_matrix((d["P"][2], d["P"][1], d["P"][0]), shape=(n, d["n_coarse"])) if d["P"] is not None else None
        mats.append((A, P))
    wide = []
    for (A, P), (Ac, _) in zip(mats, mats[1:]):
        assert abs(P.T @ A @ P - Ac).max() <= 1e-12 * abs(A).max()
        wide.append((int((abs(A).sign() @ P.getnnz(axis=1)).max()), int(Ac.getnnz(axis=1).max())))
    print("most contributions to a row of A P, most columns of R A P, per level:", wide)
    h.close()


@pytest.mark.parametrize("dims", [(6, 5, 4), (17, 16, 15), (66, 50, 48)])
def test_noalloc_step_counts(dims):
    """Step counts on both sides of where vag_transport_noalloc builds the
    operator, wells included, on meshes below and above 2^18 control volumes:
    the state of vag_transport within the 1e-12 of the order of additions."""
    p = synth.random_problem(dims, 25, n_patches=5, n_steps=0, ratios=(1e2, 1e4))
    synth.add_wells(p, 4, n_inj=1, n_prod=1)
    h, _ = _handle(p, rtol=1e-8, precond=1)
    rng = np.random.default_rng(26)
    c0 = {k: rng.uniform(0, 1, n) for k, n in (("c_cell", p.n_cells), ("c_frac", p.n_frac), ("c_node", p.n_nodes))}
    from paper_1602_03641_amd import vag
    for n in (0, 1, 3, 4, 11, 12, 13):
        h.transport(n_steps=n, c0=c0)
        ref = vag.to_numpy(h.concentration())
        got = vag.to_numpy(h.transport_noalloc(n_steps=n, c0=c0)[0])
        for k in ref:
            assert np.abs(got[k] - ref[k]).max(initial=0.0) <= 1e-12, (n, k)
        # the operator lives in the local matrices: the next solve is unharmed
    u = vag.to_numpy(h.pressure())
    h.solve_pressure()
    for k, v in vag.to_numpy(h.pressure()).items():
        assert np.array_equal(v, u[k]), k
    h.close()


@pytest.mark.parametrize("dims", [(3, 3, 3), (8, 4, 2), (16, 15, 3), (51, 48, 50), (53, 49, 50)])
@pytest.mark.parametrize("opt", ["cg", "cg mixed", "cg V", "jacobi", "bicgstab"])
def test_krylov_rows_per_block(dims, opt):
    """Fewer unknowns than a wavefront's rows, ragged last slices, and both
    sides of 131072 unknowns, where rows go from four lanes to one; hierarchies
    of several levels, K-cycles and V-cycles.  The systems' condition numbers
    are below 50^2 times the contrast of 10^3: rtol 1e-12 leaves 1e-6 of max
    |u|.  A second solve gives the same bits."""
    from paper_1602_03641_amd import vag
    kw = {"cg": dict(precond=vag.VAG_PC_AMG, amg_coarse_size=12),
          "cg mixed": dict(precond=vag.VAG_PC_AMG, amg_coarse_size=12, precision=vag.VAG_MIXED),
          "cg V": dict(precond=vag.VAG_PC_AMG, amg_coarse_size=12, amg_kcycle=0),
          "jacobi": dict(precond=vag.VAG_PC_JACOBI),
          "bicgstab": dict(precond=vag.VAG_PC_AMG, amg_coarse_size=12, krylov=vag.VAG_BICGSTAB)}[opt]
    p = synth.random_problem(dims, 27, n_patches=5, n_steps=0, ratios=(1e2, 1e3))
    od = oracle.solve_darcy(p, rtol=1e-13)
    h, info = _handle(p, rtol=1e-12, eliminate_frac_faces=0, **kw)
    assert info["status"] == 0 and info["n_unknowns"] == oracle.system(p)[0].shape[0]
    u = vag.to_numpy(h.pressure())
    for k in ("u_node", "u_frac"):
        assert np.abs(u[k] - od[k]).max(initial=0.0) <= 1e-6 * np.abs(od["u_node"]).max(), k
    h.solve_pressure()
    for k, v in vag.to_numpy(h.pressure()).items():
        assert np.array_equal(v, u[k]), k
    h.close()


@pytest.mark.parametrize("restart", [5, 8, 9, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("dims,opt", [((16, 15, 3), "jacobi"), ((53, 49, 50), "mixed"), ((16, 15, 3), "mixed_ir")])
def test_gmres_basis_sizes(dims, opt, restart):
    """Cycle lengths on both sides of 8, 16 and 32 basis vectors, which the
    orthogonalisation holds at once, and of two such sets: the pressures of the
    oracle.  Condition numbers below 50^2 times the contrast of 10: rtol 1e-11
    leaves 1e-6 of max |u|."""
    from paper_1602_03641_amd import vag
    kw = {"jacobi": dict(precond=vag.VAG_PC_JACOBI), "mixed": dict(precond=vag.VAG_PC_AMG, precision=vag.VAG_MIXED),
          "mixed_ir": dict(precond=vag.VAG_PC_AMG, precision=vag.VAG_MIXED_IR, inner_rtol=1e-6)}[opt]
    p = synth.random_problem(dims, 29, n_patches=3, n_steps=0, ratios=(1e1, 1e1))
    od = oracle.solve_darcy(p, rtol=1e-13)
    h, info = _handle(p, rtol=1e-11, krylov=vag.VAG_GMRES, gmres_restart=restart, **kw)
    assert info["status"] == 0
    print("iterations", info["iterations"])
    u = vag.to_numpy(h.pressure())
    for k in ("u_node", "u_frac"):
        assert np.abs(u[k] - od[k]).max(initial=0.0) <= 1e-6 * np.abs(od["u_node"]).max(), k
    h.close()


def _star(sectors, layers, dirichlet_axis):
    """A prism of hexahedra around an axis: an axis node has `sectors` cells in
    each layer.  Fracture faces on vertical planes through the axis (they meet
    there: one group of many faces per layer) and horizontal ones off it."""
    n = 2 * sectors
    t = np.arange(n) * (2 * np.pi / n)
    rad = np.where(np.arange(n) % 2 == 0, 1.0, 1.35)
    inner = np.c_[rad * np.cos(t), rad * np.sin(t)]
    ring = np.concatenate([[[0.0, 0.0]], inner, 2.0 * inner])
    m = len(ring)
    xyz = np.concatenate([np.c_[ring, np.full(m, 0.4 * z)] for z in range(layers + 1)])
    quads = [(0, 1 + 2 * i, 2 + 2 * i, 1 + (2 * i + 2) % n) for i in range(sectors)]
    quads += [(1 + i, 1 + n + i, 1 + n + (i + 1) % n, 1 + (i + 1) % n) for i in range(n)]
    hex8 = np.array([[a + m * z for a in q] + [a + m * (z + 1) for a in q] for z in range(layers) for q in quads],
                    np.int32)
    frac = [(0 + m * z, 1 + 2 * i + m * z, 1 + 2 * i + m * (z + 1), 0 + m * (z + 1))
            for z in range(layers) for i in (0, 2, 5)]
    frac += [tuple(a + m for a in quads[sectors + i]) for i in (1, 2, 7)]
    z = np.repeat(np.arange(layers + 1), m)
    d = (z == 0) | (z == layers)
    if dirichlet_axis:
        d |= np.tile(np.arange(m) == 0, layers + 1)
    perm = np.zeros((len(hex8), 6))
    perm[:, :3] = np.random.default_rng(5).uniform(0.5, 2.0, (len(hex8), 3))
    nf = len(frac)
    return synth.Problem(
        name="star", dims=None, xyz=xyz, hex8=hex8, frac_nodes=np.array(frac, np.int32), frac_width=np.full(nf, 0.01),
        frac_perm=np.geomspace(10.0, 1e3, nf), frac_poro=np.ones(nf), perm=perm, poro=np.ones(len(hex8)), mu=1.0,
        dirichlet=d.astype(np.uint8), p_bar=1.0 - z / layers, c_bar=(z == 0).astype(float))


@pytest.mark.parametrize("mesh", [(6, 3, False), (12, 3, False), (13, 4, False), (7, 3, True), (5, 4, 3)])
@pytest.mark.parametrize("eliminate", [0, 1])
def test_assembled_rows(mesh, eliminate):
    """Nodes of 6, 12 and 13 cells a layer (lists of 8 in one, two and four
    pieces, rows of more slots than LDS holds), Dirichlet nodes among their
    columns, fracture faces kept and eliminated in groups of one and of many:
    the oracle's system, and its Schur complement on what is kept.  An entry
    sums below 10^3 terms of at most max |A|, the complement two products more:
    1e-12 max |A|."""
    from paper_1602_03641_amd import vag
    import scipy.sparse as sp
    p = (synth.random_problem(mesh, 31, n_patches=9, n_steps=0, ratios=(1e1, 1e3)) if mesh == (5, 4, 3)
         else _star(*mesh))
    h, info = _handle(p, rtol=1e-12, precond=vag.VAG_PC_AMG, eliminate_frac_faces=eliminate)
    d = h.amg_level(0)
    got = sp.csr_matrix((d["A"][2], d["A"][1], d["A"][0])).toarray()
    A = oracle.system(p)[0].toarray()
    n = len(got)
    assert n < len(A) if eliminate else n == len(A)
    nfree = len(A) - p.n_frac
    if eliminate:
        assert n == nfree  # every group is small enough
        S = A[:n, :n] - A[:n, n:] @ np.linalg.solve(A[n:, n:], A[n:, :n])
    else:
        S = A
    assert np.abs(got - S).max() <= 1e-12 * np.abs(A).max()
    od = oracle.solve_darcy(p, rtol=1e-13)
    u = vag.to_numpy(h.pressure())
    for k in ("u_node", "u_frac"):
        assert np.abs(u[k] - od[k]).max(initial=0.0) <= 1e-6 * np.abs(od["u_node"]).max(), k
    h.close()


@pytest.mark.parametrize("mesh,coarse,hops,theta", [((5, 4, 4), 8, 2, 0.08), ((14, 12, 11), 6, 2, 0.08),
                                                    ((26, 24, 22), 12, 1, 0.08), ((26, 24, 22), 4, 2, 1e-9),
                                                    ("fan", 12, 1, 0.08), ("fan", 12, 1, 0.3)])
def test_aggregation_products(mesh, coarse, hops, theta):
    """Aggregation hierarchies coarsened far down; on the fan, rows with more
    aggregates than ap_collapse's registers and coarse rows of more columns than
    the hashed kernel's 256: every coarse operator is P^T A P
    of the level above.  An entry sums at most ~10^4 products, each rounded
    relative to max |A|: 1e-12 max |A|."""
    from paper_1602_03641_amd import vag
    import scipy.sparse as sp
    p = _fan(120, 14) if mesh == "fan" else synth.random_problem(mesh, 33, n_patches=5, n_steps=0, ratios=(1e2, 1e4))
    h, info = _handle(p, rtol=1e-8, precond=vag.VAG_PC_AMG, amg_coarse_size=coarse, amg_aggregate_hops=hops,
                      amg_theta=theta)
    mats = []
    for d in (h.amg_level(l) for l in range(info["amg_levels"])):
        n = len(d["A"][0]) - 1
        A = sp.csr_matrix((d["A"][2], d["A"][1], d["A"][0]), shape=(n, n))
        P = sp.csr_matrix((d["P"][2], d["P"][1], d["P"][0]), shape=(n, d["n_coarse"])) if d["P"] is not None else None
        mats.append((A, P))
    assert len(mats) >= 2
    wide = []
    for (A, P), (Ac, _) in zip(mats, mats[1:]):
        assert np.all(np.diff(P.indptr) == 1)
        assert abs(P.T @ A @ P - Ac).max() <= 1e-12 * abs(A).max()
        AP = abs(A).sign() @ P
        wide.append((int(AP.getnnz(axis=1).max()), int((P.T @ AP.sign()).sum(axis=1).max()),
                     int(Ac.getnnz(axis=1).max())))
    print("most aggregates of a row, candidates and columns of a coarse row, per level:", wide)
    h.close()


@pytest.mark.parametrize("dims,share", [((2, 2, 1), 0.6), ((3, 3, 3), 0.0), ((5, 4, 4), 0.3), ((9, 8, 7), 0.5)])
def test_tetrahedra_fracture_faces(dims, share):
    """Tetrahedra with none to all four of their faces fractures (ratio 10, so
    that pressures and fluxes are compared relative to their largest at 1e-9:
    condition numbers below 10^4 at a residual of 1e-13), faces in any order
    and orientation; sums of incidence lists shorter and longer than a batch."""
    from oracle import general_cells as gc
    from paper_1602_03641_amd import vag
    from test_gpu_general import oracle_fluxes_flat, oracle_mesh
    p = synth.general_problem("tet", dims, 35, aniso_sigma=0.5, n_steps=9)
    rng = np.random.default_rng(36)
    two = np.nonzero(np.bincount(p.cell_faces, minlength=len(p.face_node_ptr) - 1) == 2)[0]
    p.frac_face_ids = np.sort(rng.choice(two, int(share * len(two)), replace=False)).astype(np.int32)
    nf = len(p.frac_face_ids)
    p.frac_width, p.frac_perm, p.frac_poro = np.full(nf, 0.01), rng.uniform(5.0, 10.0, nf), np.ones(nf)
    per_cell = np.isin(p.cell_faces, p.frac_face_ids).reshape(-1, 4).sum(axis=1)
    print("cells by fracture faces:", np.bincount(per_cell))
    h, info = _handle(p, rtol=1e-13, precond=vag.VAG_PC_JACOBI)
    m = oracle_mesh(p)
    sol = gc.solve_darcy(m)
    g, gf = vag.to_numpy(h.pressure()), vag.to_numpy(h.fluxes())
    for k in ("u_node", "u_cell", "u_frac"):
        assert np.abs(g[k] - np.asarray(sol[k])).max(initial=0.0) <= 1e-9, k
    of = oracle_fluxes_flat(p, sol)
    scale = max(np.abs(of["F_cell"]).max(), np.abs(of["F_frac"]).max(initial=0.0))
    for k in ("F_cell", "F_cell_frac", "F_frac"):
        assert np.abs(gf[k] - of[k]).max(initial=0.0) <= 1e-9 * scale, k
    phi, gphi = gc.porous_volumes(m, sol), vag.to_numpy(h.porous_volumes())
    for k in ("phi_cell", "phi_frac", "phi_node"):
        np.testing.assert_allclose(gphi[k], phi[k], rtol=1e-13, atol=1e-18, err_msg=k)
    h.set_fluxes(of)
    t = h.transport(n_steps=p.n_steps)
    oc = gc.transport(m, sol, phi, t["dt"], p.n_steps)
    c = vag.to_numpy(h.concentration())
    for k in ("c_cell", "c_frac", "c_node"):
        assert np.abs(c[k] - oc[k]).max(initial=0.0) <= 1e-12, k
    h.close()


@pytest.mark.parametrize("dims,n", [((2, 1, 1), 4), ((2, 8, 6), 63), ((2, 7, 7), 64), ((2, 12, 4), 65),
                                    ((3, 7, 7), 128), ((2, 42, 2), 129), ((2, 32, 30), 1023), ((2, 31, 31), 1024)])
def test_dense_inverse(dims, n):
    """Hierarchies of one level, whose V-cycle is the dense inverse: one tile,
    last tiles of one row and of all but one, an odd and an even number of
    steps, the most rows there are.  Condition numbers below 10^5: 1e-10 of
    max |z|."""
    from paper_1602_03641_amd import vag
    p = synth.random_problem(dims, 37, n_patches=0, n_steps=0, ratios=(1e2,))
    h, info = _handle(p, rtol=1e-10, precond=vag.VAG_PC_AMG, amg_coarse_size=1024)
    assert info["amg_levels"] == 1 and info["n_unknowns"] == n
    A = oracle.system(p)[0].toarray()
    r = np.random.default_rng(38).standard_normal(n)
    z, zr = h.apply_preconditioner(r), np.linalg.solve(A, r)
    print("condition", np.linalg.cond(A))
    assert np.abs(z - zr).max() <= 1e-10 * np.abs(zr).max()
    h.close()


@pytest.mark.parametrize("dims,B", [((9, 7, 6), 15), ((9, 7, 6), 16), ((9, 7, 6), 17), ((3, 2, 2), 128),
                                    ((12, 11, 9), 33), ((12, 11, 9), 128), ((12, 11, 9), 400), ((12, 11, 9), 1600)])
def test_ilu_block_sizes(dims, B):
    """Blocks of more sizes, of fewer rows than asked for, ragged last ones, and
    on both sides of what fits in LDS: as test_ilu_substitutions."""
    from paper_1602_03641_amd import vag
    from oracle import ilu
    p = synth.random_problem(dims, 39, n_patches=4, n_steps=0, ratios=(1e2, 1e4))
    h, info = _handle(p, rtol=1e-8, precond=vag.VAG_PC_BJILU0, krylov=vag.VAG_BICGSTAB, ilu_block_rows=B,
                      eliminate_frac_faces=0)
    A, _ = oracle.system(p)
    rows = ilu.bj_ilu0(A, B)
    r = np.random.default_rng(40).standard_normal(A.shape[0])
    z, zr = h.apply_preconditioner(r), ilu.bj_ilu0_apply(rows, r)
    print("distance", np.abs(z - zr).max() / np.abs(zr).max())
    assert np.abs(z - zr).max() <= 1e-11 * np.abs(zr).max()
    h.close()


@pytest.mark.parametrize("dims,patches", [((12, 11, 10), 6), ((43, 44, 45), 0), ((43, 44, 45), 40), ((300, 9, 16), 12)])
def test_transport_column_codes(dims, patches):
    """Operators whose columns lie in one cluster, in two (fracture faces more
    than 65536 away from the cells' nodes) and, at wells, in neither form: two
    steps of a random state against the same steps without the operator, within
    the 1e-12 of the order of additions."""
    from paper_1602_03641_amd import vag
    p = synth.random_problem(dims, 41, n_patches=patches, n_steps=0, ratios=(1e1, 1e4))
    if patches:
        synth.add_wells(p, 4, n_inj=1, n_prod=1)
    h, _ = _handle(p, rtol=1e-8, precond=vag.VAG_PC_AMG)
    rng = np.random.default_rng(42)
    c0 = {k: rng.uniform(0, 1, n) for k, n in (("c_cell", p.n_cells), ("c_frac", p.n_frac), ("c_node", p.n_nodes))}
    h.transport(n_steps=2, c0=c0)
    ref = vag.to_numpy(h.concentration())
    got = vag.to_numpy(h.transport_noalloc(n_steps=2, c0=c0)[0])
    for k in ref:
        assert np.abs(got[k] - ref[k]).max(initial=0.0) <= 1e-12, k
    h.close()


@pytest.mark.parametrize("mesh,patches", [((4, 1, 1), 0), ((64, 1, 1), 0), ((24, 20, 2), 3), ((9, 8, 7), 5), ((18, 18, 18), 6),
                                          ((27, 26, 25), 8), ((31, 31, 31), 9), ((32, 32, 31), 5), ("star", 0)])
def test_transport_many_steps(mesh, patches):
    """Calls of many steps on small meshes, several steps per launch on parts of
    the mesh: one part, parts whose halos allow eight steps or fewer, rows wider
    than a part holds (step by step), meshes on both sides of the size limit,
    wells, step counts around where it starts and whole and shortened last
    steps: the bits of the same steps in calls of one."""
    from paper_1602_03641_amd import vag
    if mesh == "star":
        p = _star(13, 4, False)
    else:
        p = synth.random_problem(mesh, 43, n_patches=patches, n_steps=0, ratios=(1e1, 1e4))
    if patches:
        synth.add_wells(p, 4, n_inj=1, n_prod=1)
    h, _ = _handle(p, rtol=1e-8, precond=vag.VAG_PC_JACOBI)
    rng = np.random.default_rng(44)
    c0 = {k: rng.uniform(0, 1, n) for k, n in (("c_cell", p.n_cells), ("c_frac", p.n_frac), ("c_node", p.n_nodes))}
    for steps in (31, 33, 101, 104):
        h.transport(n_steps=1, c0=c0)
        for k in range(1, steps):
            t = h.transport(n_steps=1)
        ref = vag.to_numpy(h.concentration())
        info = h.transport(n_steps=steps, c0=c0)
        got = vag.to_numpy(h.concentration())
        assert info["n_steps"] == steps
        for k in ref:
            assert np.array_equal(got[k], ref[k]), (steps, k)
    # to a final time: 120 steps, the last one shortened
    end = 119.25 * t["dt"]
    h.transport(n_steps=119, c0=c0)
    h.transport(t_final=end - 119 * t["dt"])
    ref = vag.to_numpy(h.concentration())
    info = h.transport(t_final=end, c0=c0)
    got = vag.to_numpy(h.concentration())
    assert info["n_steps"] == 120
    for k in ref:
        assert np.abs(got[k] - ref[k]).max(initial=0.0) <= 1e-12, k
    h.close()


@pytest.mark.parametrize("later", [128, 16, 2])
def test_ilu_handles_of_different_blocks(later):
    """A handle whose blocks take most of a CU's LDS, used again after another
    one with smaller blocks was built: the same bits as before."""
    from paper_1602_03641_amd import vag
    kw = dict(rtol=1e-8, precond=vag.VAG_PC_BJILU0, krylov=vag.VAG_BICGSTAB, eliminate_frac_faces=0)
    p = synth.random_problem((24, 23, 22), 45, n_patches=4, n_steps=0, ratios=(1e2, 1e4))
    h, info = _handle(p, ilu_block_rows=768, **kw)  # 136 KB
    r = np.random.default_rng(46).standard_normal(info["n_unknowns"])
    z = h.apply_preconditioner(r)
    q = synth.random_problem((6, 5, 4), 47, n_patches=2, n_steps=0, ratios=(1e2,))
    h2, _ = _handle(q, ilu_block_rows=later, **kw)
    assert np.array_equal(h.apply_preconditioner(r), z)
    assert h.solve_pressure()["status"] == 0
    h2.close()
    h.close()


@pytest.mark.parametrize("B", [16, 128, 200])
@pytest.mark.parametrize("scale", [0, 505, -505])
def test_ilu_quotients_of_any_size(B, scale):
    """Nodes numbered by the parities of their place: a block of unknowns of one
    class has no couplings, so its z is r / diagonal, to the bit, whatever the
    sizes: right-hand sides from the least subnormal number to the largest and
    infinities, pivots about 2^scale.  Then with couplings: where the oracle's z
    is finite, infinite or neither."""
    from paper_1602_03641_amd import vag
    from oracle import ilu
    import scipy.sparse as sp
    dims = (16, 15, 14)
    p = synth.random_problem(dims, 49, n_patches=0, n_steps=0, ratios=(1e2,))
    i, j, k = (a.ravel(order="F") for a in np.meshgrid(*(np.arange(n + 1) for n in dims), indexing="ij"))
    old = np.lexsort((np.arange(len(i)), i % 2 + 2 * (j % 2) + 4 * (k % 2)))
    new = np.empty(len(old), np.int32)
    new[old] = np.arange(len(old))
    p.hex8, p.xyz, p.dirichlet, p.p_bar, p.c_bar = (new[p.hex8], p.xyz[old], p.dirichlet[old], p.p_bar[old],
                                                    p.c_bar[old])
    p.mu = 2.0 ** -scale
    kw = dict(rtol=1e-2, max_iter=3, eliminate_frac_faces=0)
    g, _ = _handle(p, precond=vag.VAG_PC_AMG, **kw)
    d = g.amg_level(0)["A"]
    g.close()
    A = sp.csr_matrix((d[2], d[1], d[0]))
    n = A.shape[0]
    h, info = _handle(p, precond=vag.VAG_PC_BJILU0, krylov=vag.VAG_BICGSTAB, ilu_block_rows=B, **kw)
    assert info["n_unknowns"] == n
    c = A.tocoo()
    alone = np.ones((n + B - 1) // B, bool)
    alone[(c.row // B)[(c.row // B == c.col // B) & (c.row != c.col)]] = False
    own = np.repeat(alone, B)[:n]
    assert own.sum() > n // 4
    rng = np.random.default_rng(50)
    r = np.ldexp(rng.uniform(1.0, 2.0, n), rng.integers(-1074, 1024, n)) * rng.choice([-1.0, 1.0], n)
    r[rng.choice(n, n // 20)] = rng.choice([np.inf, -np.inf, 0.0, -0.0], n // 20)
    z = h.apply_preconditioner(r)
    with np.errstate(all="ignore"):
        q = r / A.diagonal()
    assert np.array_equal(z[own].view(np.int64), q[own].view(np.int64))
    # the entry that a block's other rows take last, and nothing else in r
    r = np.zeros(n)
    r[np.arange(B - 1, n, 3 * B)] = np.inf
    z = h.apply_preconditioner(r)
    with np.errstate(all="ignore"):
        zr = ilu.bj_ilu0_apply(ilu.bj_ilu0(A, B), r)
    assert np.array_equal(np.isnan(z), np.isnan(zr)) and np.array_equal(np.isinf(z), np.isinf(zr))
    h.close()


@pytest.mark.parametrize("dims", [(8, 8, 9), (9, 9, 9), (10, 9, 10), (4, 15, 16)])
@pytest.mark.parametrize("opt", ["fp64", "mixed", "mixed_ir", "gmres"])
def test_footprint_of_small_handles(dims, opt):
    """About a thousand unknowns, where the dense inverse and its workspace are
    most of a handle: within the estimate that a server admits it by."""
    from paper_1602_03641_amd import vag
    kw = {"fp64": {}, "mixed": dict(precision=vag.VAG_MIXED), "mixed_ir": dict(precision=vag.VAG_MIXED_IR),
          "gmres": dict(precision=vag.VAG_MIXED, krylov=vag.VAG_GMRES)}[opt]
    kw.update(precond=vag.VAG_PC_AMG, rtol=1e-8)
    p = synth.random_problem(dims, 51, n_patches=6, n_steps=0, ratios=(1e2, 1e4))
    h, info = _handle(p, **kw)
    assert info["amg_levels"] == 1
    h.transport(n_steps=2)
    used, est = vag.load().vag_footprint_bytes(h.h), vag.estimate_footprint(p, **kw)
    print(used, est)
    assert used <= est
    h.close()


@pytest.mark.parametrize("sectors", [120, 200, 300])
def test_noalloc_at_wide_nodes(sectors):
    """An axis node of 246, 406 and 606 fluxes, of which about half flow in: past
    the 255 entries that a row of the upwind operator counts, the allocation-free
    transport gathers at any step count.  Against the oracle's steps on the
    library's fluxes, within the 1e-10 that its other tests take."""
    from paper_1602_03641_amd import vag
    p = _star(sectors, 2, False)
    h, _ = _handle(p, rtol=1e-10, precond=vag.VAG_PC_JACOBI)
    flux, phi = vag.to_numpy(h.fluxes()), vag.to_numpy(h.porous_volumes())
    into = np.bincount(p.hex8.ravel(), weights=(flux["F_cell"].ravel() > 0).astype(float), minlength=p.n_nodes)
    assert (into[p.dirichlet == 0].max() > 255) == (sectors == 300)
    rng = np.random.default_rng(52)
    c0 = {k: rng.uniform(0, 1, n) for k, n in (("c_cell", p.n_cells), ("c_frac", p.n_frac), ("c_node", p.n_nodes))}
    c0o = dict(c0, c_node=np.where(p.dirichlet == 1, p.c_bar, c0["c_node"]))
    for n in (11, 13, 40):
        print("sectors", sectors, "steps", n, flush=True)
        got, info = h.transport_noalloc(n_steps=n, c0=c0)
        ref = oracle.transport(p, flux, phi, info["dt"], n, c0=c0o)
        for k, v in vag.to_numpy(got).items():
            assert np.abs(v - ref[k]).max(initial=0.0) <= 1e-10, (n, k)
    h.close()


@pytest.mark.parametrize("sectors", [200, 300])
def test_transport_at_wide_nodes(sectors):
    """The same nodes in vag_transport and through the serving loop: rows of more
    than 255 entries are gathered; calls of many steps, a last step shortened."""
    from paper_1602_03641_amd import vag
    p = _star(sectors, 2, False)
    opt = dict(rtol=1e-10, precond=vag.VAG_PC_JACOBI, max_iter=20000, cfl=p.cfl)
    h, _ = _handle(p, **opt)
    flux, phi = vag.to_numpy(h.fluxes()), vag.to_numpy(h.porous_volumes())
    rng = np.random.default_rng(53)
    c0 = {k: rng.uniform(0, 1, n) for k, n in (("c_cell", p.n_cells), ("c_frac", p.n_frac), ("c_node", p.n_nodes))}
    c0o = dict(c0, c_node=np.where(p.dirichlet == 1, p.c_bar, c0["c_node"]))
    for n, part in ((1, 0.0), (50, 0.0), (50, 0.25)):
        print("sectors", sectors, "steps", n, part, flush=True)
        dt = h.transport(n_steps=1, c0=c0)["dt"]
        info = h.transport(n_steps=n, c0=c0) if not part else h.transport(t_final=(n - 1 + part) * dt, c0=c0)
        assert info["n_steps"] == n
        ref = oracle.transport(p, flux, phi, info["dt"], n, last_dt=info["last_dt"] if part else 0.0, c0=c0o)
        for k, v in vag.to_numpy(h.concentration()).items():
            assert np.abs(v - ref[k]).max(initial=0.0) <= 1e-10, (n, k)
    # a job starts from zero
    h.solve_pressure()
    h.transport(n_steps=20)
    lone = vag.to_numpy(h.concentration())
    h.close()
    srv = vag.Server(n_workers=1)
    res = srv.wait(srv.submit(p, n_steps=20, **opt))
    srv.close()
    assert res["status"] == 0
    for k, v in lone.items():
        assert np.array_equal(res[k], v), k


@pytest.mark.parametrize("dims", [(43, 43, 43), (43, 44, 43)])
@pytest.mark.parametrize("opt", ["cg", "cg mixed", "cg V", "jacobi", "bicgstab"])
def test_krylov_rows_at_the_line(dims, opt):
    """Systems on both sides of 81920 unknowns: the fused kernels with four lanes
    per row, and one lane per row around a finest level whose coarse levels keep
    theirs.  Tolerance and bits as in test_krylov_rows_per_block."""
    test_krylov_rows_per_block(dims, opt)


@pytest.mark.parametrize("dims,steps", [((17, 16, 15), (15, 16, 17)), ((33, 32, 32), (11, 12)),
                                        ((40, 41, 40), (7, 8)), ((66, 50, 48), (5, 6)), ((64, 65, 64), (3, 4))])
def test_noalloc_where_the_operator_starts(dims, steps):
    """The step counts from which the allocation-free transport builds the
    operator, in each range of sizes: against the oracle's steps on the library's
    fluxes, within the 1e-10 that its other tests take."""
    from paper_1602_03641_amd import vag
    p = synth.random_problem(dims, 54, n_patches=4, n_steps=0, ratios=(1e2, 1e3))
    synth.add_wells(p, 4, n_inj=1, n_prod=1)
    h, _ = _handle(p, rtol=1e-8, precond=vag.VAG_PC_AMG)
    flux, phi = vag.to_numpy(h.fluxes()), vag.to_numpy(h.porous_volumes())
    flux["well_rate"] = h.well_rates()
    rng = np.random.default_rng(55)
    c0 = {k: rng.uniform(0, 1, n) for k, n in (("c_cell", p.n_cells), ("c_frac", p.n_frac), ("c_node", p.n_nodes))}
    c0o = dict(c0, c_node=np.where(p.dirichlet == 1, p.c_bar, c0["c_node"]))
    for n in steps:
        got, info = h.transport_noalloc(n_steps=n, c0=c0)
        ref = oracle.transport(p, flux, phi, info["dt"], n, c0=c0o)
        for k, v in vag.to_numpy(got).items():
            assert np.abs(v - ref[k]).max(initial=0.0) <= 1e-10, (n, k)
    h.close()


@pytest.mark.parametrize("dims,rows", [((35, 35, 35), 1500), ((35, 36, 36), 1500), ((48, 48, 48), 128), ((48, 49, 49), 128)])
def test_bicgstab_rows_at_its_lines(dims, rows):
    """BiCGStab on both sides of 45056 unknowns, its line with an ILU that is
    solved from global memory, and of 114688, its line otherwise: the oracle's
    pressures as in test_krylov_rows_per_block, and the same bits twice."""
    from paper_1602_03641_amd import vag
    p = synth.random_problem(dims, 56, n_patches=5, n_steps=0, ratios=(1e2, 1e3))
    od = oracle.solve_darcy(p, rtol=1e-13)
    h, info = _handle(p, rtol=1e-12, precond=vag.VAG_PC_BJILU0, krylov=vag.VAG_BICGSTAB, ilu_block_rows=rows,
                      eliminate_frac_faces=0)
    print(dims, info["n_unknowns"], flush=True)
    assert info["status"] == 0
    u = vag.to_numpy(h.pressure())
    for k in ("u_node", "u_frac"):
        assert np.abs(u[k] - od[k]).max(initial=0.0) <= 1e-6 * np.abs(od["u_node"]).max(), k
    h.solve_pressure()
    for k, v in vag.to_numpy(h.pressure()).items():
        assert np.array_equal(v, u[k]), k
    h.close()


def test_fan_has_the_wide_rows():
    """What test_classical_products and test_aggregation_products mean by wide:
    the fan's rows outgrow the limits of the kernels that most rows take."""
    import os
    import re
    from paper_1602_03641_amd import vag
    import scipy.sparse as sp
    csrc = os.path.join(os.path.dirname(vag.__file__), "csrc")
    limit = {}
    for f in ("amg.hip", "amg_classical.hip"):
        with open(os.path.join(csrc, f)) as src:
            limit.update({k: int(v) for k, v in re.findall(r"\b(k\w+) = (\d+)[,;]", src.read())})
    for kind, names in ((1, ("kApCand", "kRapCols")), (0, ("kSet", "kGalDistinct"))):
        h, _ = _handle(_fan(120, 14), rtol=1e-8, precond=vag.VAG_PC_AMG, amg_kind=kind, amg_coarse_size=12,
                       amg_aggregate_hops=1, amg_theta=0.3)
        a, b = h.amg_level(0), h.amg_level(1)
        A = sp.csr_matrix((np.ones(len(a["A"][2])), a["A"][1], a["A"][0]))
        P = sp.csr_matrix((np.ones(len(a["P"][2])), a["P"][1], a["P"][0]), shape=(A.shape[0], a["n_coarse"]))
        # contributions to a row of A P (classical), its columns (aggregation); columns of a coarse row
        most = int((A @ P.getnnz(axis=1)).max()) if kind else int((A @ P).getnnz(axis=1).max())
        assert most > limit[names[0]] and np.diff(b["A"][0]).max() > limit[names[1]], (kind, most, limit)
        h.close()
