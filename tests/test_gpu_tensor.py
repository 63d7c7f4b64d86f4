"""The step kernel in tensor-product form, the FP64 default: against the
oracle where its tiles, planes and column groups end.

Tiles hold a few cells along x and y and all vectors in groups of 16; a
workgroup walks a range of cell layers along z.  The meshes have fewer cells
than a tile, whole tiles and remainders, every degree, Dirichlet and periodic
axes (the halo of a tile wraps or is absent), and 1, 15, 16, 17 columns past
the last group.  Bars as for the other FP64 kernels: 1e-13 for one product,
1e-12 for a filter, relative per vector."""
import math

import numpy as np
import pytest

import oracle as O
from paper_2504_00998_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

D, P = W.DIRICHLET, W.PERIODIC
CASES = [
    # p, cells, bc, N, ld - N
    (1, (17, 9, 5), (P, P, D), 16, 0),
    (1, (4, 4, 4), (D, D, D), 3, 1),
    (2, (9, 7, 5), (P, P, P), 31, 0),
    (2, (8, 4, 2), (D, P, D), 33, 3),
    (3, (1, 1, 1), (D, D, D), 5, 0),
    (3, (2, 2, 2), (P, P, P), 17, 0),
    (3, (5, 7, 3), (P, D, P), 48, 2),
    (4, (2, 2, 1), (P, P, D), 3, 0),
    (4, (5, 3, 7), (P, P, D), 17, 1),
    (4, (9, 5, 2), (D, D, P), 40, 0),
    (5, (4, 4, 4), (P, P, D), 16, 0),
    (5, (7, 3, 4), (D, P, P), 15, 5),
    (6, (3, 5, 5), (P, P, D), 18, 0),
    (6, (4, 4, 4), (D, D, D), 3, 0),
    (7, (3, 5, 5), (P, P, D), 7, 0),
    (7, (4, 4, 4), (P, P, P), 33, 0),
]


@pytest.mark.parametrize("p,cells,bc,N,pad", CASES)
def test_tensor_kernel_matches_oracle(p, cells, bc, N, pad):
    import paper_2504_00998_amd as fe
    wl = W.small_slab(cells, p=p, N=N, m=6, bc=bc, **({"E": 0.0} if bc[2] == P else {}))
    print("case: tensor", p, cells, bc, N, pad, flush=True)
    om = O.Mesh.from_workload(wl)
    Vq = W.workload_potential(wl, om.quad_points())
    op = O.Operator(om, Vq, wl.E, wl.z0)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(Vq).cuda(), wl.E, wl.z0)
    Xh = wl.X(op.n)
    buf = torch.full((op.n, N + pad), float("nan"), dtype=torch.float64, device="cuda")
    buf[:, :N] = torch.from_numpy(Xh).cuda()
    out = torch.full_like(buf, float("nan"))
    X, Y = buf[:, :N], out[:, :N]

    def err(Yd, R):
        return (np.linalg.norm(Yd.cpu().numpy() - R, axis=0) / np.linalg.norm(R, axis=0)).max()

    assert err(gm.hx(X, Y), op.apply(Xh)) < 1e-13
    first = Y.clone()
    assert torch.equal(gm.hx(X, Y), first)
    if op.n > N:
        a0, b, _ = O.lanczos_bounds(op.apply, wl.lanczos_start(op.n), min(10, op.n))
        a = O.weyl_cut(a0, b, N, op.n)
        for a0s in (a0, math.nan):
            assert err(gm.cheb_filter(X, wl.m, a, b, a0s, Y=Y), op.filter(Xh, wl.m, a, b, a0s)) < 1e-12
    assert torch.isnan(out[:, N:]).all()  # the columns beside the block are left alone
    # a column's result does not depend on the columns beside it
    if N > 3:
        gm.hx(X, Y)
        part = gm.hx(X[:, 1:].contiguous())
        assert torch.equal(part, Y[:, 1:])


@pytest.mark.parametrize("p,cells,N", [(1, (5, 9, 4), 3), (2, (4, 7, 5), 9), (3, (3, 2, 7), 8), (4, (5, 5, 3), 1),
                                       (5, (2, 5, 3), 7), (6, (3, 3, 2), 2), (7, (2, 2, 3), 9)])
def test_tensor_kernel_bloch_matches_oracle(p, cells, N):
    """The k.G term of complex vectors at every degree (one, eight and a few
    vectors past a group of eight; tiles with remainders along x and y)."""
    import paper_2504_00998_amd as fe
    wl = W.small_slab(cells, p=p, N=N, m=5)
    print("case: tensor bloch", p, cells, N, flush=True)
    om = O.Mesh.from_workload(wl)
    Vq = W.workload_potential(wl, om.quad_points())
    op = O.Operator(om, Vq, wl.E, wl.z0)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(Vq).cuda(), wl.E, wl.z0)
    k = (0.37, -0.61)
    gm.set_kpoint(*k)
    B = O.BlochOperator(op, om, k)
    Xh = wl.Xc(op.n)
    X = torch.from_numpy(Xh).cuda()
    Y = gm.hx_k(X)
    assert torch.equal(gm.hx_k(X), Y)
    for Yd, R, bar in ((Y, B.apply(Xh), 1e-13),
                       (gm.cheb_filter_k(X, 5, 3.0, 900.0, -1.0), B.filter(Xh, 5, 3.0, 900.0, -1.0), 1e-12)):
        assert (np.linalg.norm(Yd.cpu().numpy() - R, axis=0) / np.linalg.norm(R, axis=0)).max() < bar


N_ = W.NEUMANN


@pytest.mark.parametrize("p,cells,bc,N,pad", [
    (1, (33, 9, 4), (P, P, D), 1, 0), (1, (8, 8, 16), (N_, D, N_), 2, 1),
    (2, (17, 7, 9), (D, P, N_), 1, 2), (3, (9, 8, 15), (P, N_, P), 2, 0),
    (4, (8, 8, 16), (D, D, D), 1, 0), (4, (9, 7, 17), (P, P, N_), 1, 1), (4, (2, 16, 32), (P, P, P), 2, 0),
    (5, (5, 13, 16), (P, D, D), 1, 0), (6, (4, 9, 29), (N_, P, N_), 1, 0), (7, (5, 9, 23), (P, P, D), 2, 3)])
def test_single_vector_kernel_matches_oracle(p, cells, bc, N, pad):
    """One and two columns on meshes of 1024 cells and more: tiles with
    remainders, a mesh of two cells along x, and zero-Neumann faces (reflected)
    on each axis, for the bare product and with the previous iterate."""
    import paper_2504_00998_amd as fe
    wl = W.small_slab(cells, p=p, N=N, m=4, bc=bc, **({"E": 0.0} if bc[2] == P else {}))
    print("case: single vector", p, cells, bc, N, pad, flush=True)
    om = O.Mesh.from_workload(wl)
    Vq = W.workload_potential(wl, om.quad_points())
    op = O.Operator(om, Vq, wl.E, wl.z0)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(Vq).cuda(), wl.E, wl.z0)
    Xh = wl.X(op.n)
    buf = torch.full((op.n, N + pad), float("nan"), dtype=torch.float64, device="cuda")
    buf[:, :N] = torch.from_numpy(Xh).cuda()
    out = torch.full_like(buf, float("nan"))
    X, Y = buf[:, :N], out[:, :N]

    def err(Yd, R):
        return (np.linalg.norm(Yd.cpu().numpy() - R, axis=0) / np.linalg.norm(R, axis=0)).max()

    assert err(gm.hx(X, Y), op.apply(Xh)) < 1e-13
    first = Y.clone()
    assert torch.equal(gm.hx(X, Y), first)
    if N == 2:
        assert torch.equal(gm.hx(X[:, 1:].contiguous()), Y[:, 1:])
    assert err(gm.cheb_filter(X, 4, 3.0, 900.0, -1.0, Y=Y), op.filter(Xh, 4, 3.0, 900.0, -1.0)) < 1e-12
    assert torch.isnan(out[:, N:]).all()


@pytest.mark.parametrize("prec,m,stride,pad", [("f64", 2, 1, 0), ("f64", 3, 2, 3), ("f32", 2, 1, 3), ("f32", 4, 2, 0)])
def test_adjoint_step_takes_the_block_before_last(prec, m, stride, pad):
    """The reverse sweep's three-block rotation where the cotangent itself is
    one of the blocks (m = 2 and past it), over checkpoint segments and rows
    wider than the block, in FP64 and with FP32 products (whose second step
    takes a copy).  FP32: sums of 64 rounded products (64 eps = 4e-6) over up
    to four steps."""
    import paper_2504_00998_amd as fe
    wl = W.small_slab((4, 3, 3), p=3, N=33, m=m)
    print("case: adjoint", prec, m, stride, pad, flush=True)
    om = O.Mesh.from_workload(wl)
    Vq = W.workload_potential(wl, om.quad_points())
    op = O.Operator(om, Vq, wl.E, wl.z0)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(Vq).cuda(), wl.E, wl.z0)
    Xh = wl.X(op.n)
    Gh = np.random.default_rng(3).standard_normal(Xh.shape)
    a0, b, _ = O.lanczos_bounds(op.apply, wl.lanczos_start(op.n), 10)
    a = O.weyl_cut(a0, b, wl.N, op.n)
    wide = torch.zeros((2, op.n, wl.N + pad), dtype=torch.float64, device="cuda")
    X, G = wide[0, :, :wl.N], wide[1, :, :wl.N]
    X.copy_(torch.from_numpy(Xh))
    G.copy_(torch.from_numpy(Gh))
    Xb, Vb, _ = gm.cheb_filter_vjp(X, G, m, a, b, a0, prec=prec, ckpt_stride=stride)
    R, g = op.filter_vjp(Xh, Gh, m, a, b, a0)
    bar = 1e-12 if prec == "f64" else 2e-5
    assert (np.linalg.norm(Xb.cpu().numpy() - R, axis=0) / np.linalg.norm(R, axis=0)).max() < bar
    Rv = op.potential_vjp(g)[0]
    assert np.abs(Vb.cpu().numpy() - Rv).max() / np.abs(Rv).max() < 10 * bar


@pytest.mark.parametrize("p,cells,k", [(1, (3, 3, 3), 1), (2, (3, 4, 5), 8), (3, (4, 4, 3), 9), (4, (9, 9, 13), 17),
                                       (3, (4, 4, 8), 64)])
def test_lanczos_bounds_match_oracle(p, cells, k):
    """One column to 64 (whole and broken groups of eight, one workgroup and
    many) of the reorthogonalisation; the bounds' error is held against the
    norm of H~: k steps of products and sums each good to about 1e-14."""
    import paper_2504_00998_amd as fe
    wl = W.small_slab(cells, p=p, N=2, m=4)
    print("case: lanczos", p, cells, k, flush=True)
    om = O.Mesh.from_workload(wl)
    Vq = W.workload_potential(wl, om.quad_points())
    op = O.Operator(om, Vq, wl.E, wl.z0)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(Vq).cuda(), wl.E, wl.z0)
    v0 = wl.lanczos_start(op.n)
    a0, b, _ = O.lanczos_bounds(op.apply, v0, k)
    v = torch.from_numpy(v0).cuda()
    got = gm.lanczos_bounds(v, k)
    assert abs(got[0] - a0) < 1e-11 * b and abs(got[1] - b) < 1e-11 * b
    assert gm.lanczos_bounds(v, k) == got


@pytest.mark.parametrize("p,cells,bc,N", [(2, (1, 32, 33), (N_, P, D), 1), (3, (33, 1, 32), (P, N_, N_), 2),
                                          (4, (32, 33, 1), (P, P, N_), 1), (1, (1, 1, 1030), (N_, N_, D), 1)])
def test_single_vector_kernel_on_a_neumann_axis_of_one_cell(p, cells, bc, N):
    """One cell along a zero-Neumann axis: the nodes that the extension reaches
    past either face are the other face's, which carries the face factor too."""
    import paper_2504_00998_amd as fe
    wl = W.small_slab(cells, p=p, N=N, m=4, bc=bc)
    print("case: one Neumann cell", p, cells, bc, N, flush=True)
    om = O.Mesh.from_workload(wl)
    Vq = W.workload_potential(wl, om.quad_points())
    op = O.Operator(om, Vq, wl.E, wl.z0)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(Vq).cuda(), wl.E, wl.z0)
    Xh = wl.X(op.n)
    X = torch.from_numpy(Xh).cuda()

    def err(Yd, R):
        return (np.linalg.norm(Yd.cpu().numpy() - R, axis=0) / np.linalg.norm(R, axis=0)).max()

    assert err(gm.hx(X), op.apply(Xh)) < 1e-13
    assert err(gm.cheb_filter(X, 4, 3.0, 900.0, -1.0), op.filter(Xh, 4, 3.0, 900.0, -1.0)) < 1e-12
    v0 = wl.lanczos_start(op.n)
    a0, b, _ = O.lanczos_bounds(op.apply, v0, 8)
    got = gm.lanczos_bounds(torch.from_numpy(v0).cuda(), 8)
    assert abs(got[0] - a0) < 1e-11 * b and abs(got[1] - b) < 1e-11 * b


@pytest.mark.parametrize("p,cells,bc", [(2, (1, 4, 3), (N_, P, D)), (3, (3, 1, 2), (P, N_, N_)), (4, (2, 3, 1), (P, P, N_)),
                                        (5, (1, 1, 3), (N_, N_, D)), (2, (4, 1, 6), (P, N_, N_))])
def test_poisson_on_a_neumann_axis_of_one_cell(p, cells, bc):
    """The solves on such axes, with the bar of the other Poisson cases; where z
    has room for conductors, the constrained solve too."""
    import paper_2504_00998_amd as fe
    print("case: poisson, one Neumann cell", p, cells, bc, flush=True)
    L = tuple(float(c) for c in cells)
    om, gm = O.Mesh(L, cells, p, bc), fe.Mesh(L, cells, p, bc)
    s = np.random.default_rng(11).standard_normal(om.n)
    sd = torch.from_numpy(s).cuda()
    ref = O.poisson(om, s)
    phi, it, rel = gm.poisson(sd, tol=1e-13)
    assert rel <= 1e-13 and it > 0
    assert np.abs(phi.cpu().numpy() - ref).max() <= 1e-8 * np.abs(ref).max()
    if cells[2] >= 6:
        ref = O.poisson_cpd(om, s, np.zeros(om.n), 1.2, 4.9, 0.3)
        phi, it, rel = gm.poisson_cpd(sd, 1.2, 4.9, 0.3, tol=1e-13)
        assert rel <= 1e-13 and np.abs(phi.cpu().numpy() - ref).max() <= 1e-8 * np.abs(ref).max()


@pytest.mark.parametrize("p,cells,bc,N", [(4, (5, 5, 6), (P, P, D), 1), (4, (4, 3, 5), (P, P, D), 2), (4, (8, 8, 16), (P, P, D), 1),
                                          (4, (8, 8, 16), (P, P, D), 2), (4, (8, 8, 16), (P, P, D), 3),
                                          (2, (16, 17, 4), (P, P, N_), 2), (6, (4, 16, 16), (P, D, P), 2),
                                          (3, (16, 8, 8), (D, D, D), 1), (5, (4, 4, 4), (P, P, D), 2)])
def test_gamma_point_equals_real_path_at_every_width(p, cells, bc, N):
    """One to three complex vectors at k = 0, on both sides of the 1024 cells from
    which one and two vectors take the single-vector kernel: bit for bit the
    real entry points on the real and imaginary parts."""
    import paper_2504_00998_amd as fe
    wl = W.small_slab(cells, p=p, N=N, m=5, bc=bc, **({"E": 0.0} if bc[2] == P else {}))
    print("case: gamma", p, cells, bc, N, flush=True)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(W.workload_potential(wl, gm.quad_points())).cuda(), wl.E, wl.z0)
    X = torch.from_numpy(wl.Xc(gm.n)).cuda()
    Xr, Xi = X.real.contiguous(), X.imag.contiguous()
    Y = gm.hx_k(X)
    assert torch.equal(Y.real, gm.hx(Xr)) and torch.equal(Y.imag, gm.hx(Xi))
    Y = gm.cheb_filter_k(X, 5, 3.0, 900.0, -1.0)
    assert torch.equal(Y.real, gm.cheb_filter(Xr, 5, 3.0, 900.0, -1.0))
    assert torch.equal(Y.imag, gm.cheb_filter(Xi, 5, 3.0, 900.0, -1.0))


@pytest.mark.parametrize("gib", [0.9, 1.1, 1.9])
def test_gamma_point_equals_real_path_at_wide_rows(gib):
    """Three vectors in rows so wide that a z plane of the real block has 0.9, 1.1
    and 1.9 GiB (twice that the complex one): both take the same kernel on
    either side of the line, and the values are those of narrow rows."""
    import paper_2504_00998_amd as fe
    wl = W.small_slab((2, 2, 1), p=3, N=3)
    plane = 36
    ld = int(gib * 2**30) // (8 * plane)
    print("case: gamma, wide rows", gib, ld, flush=True)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(W.workload_potential(wl, gm.quad_points())).cuda(), wl.E, wl.z0)
    assert gm.n == 2 * plane
    Xc = torch.from_numpy(wl.Xc(gm.n)).cuda()
    X = torch.empty((gm.n, ld), dtype=torch.complex128, device="cuda")[:, :3]
    X.copy_(Xc)
    Y = gm.hx_k(X).contiguous()
    del X
    narrow = gm.hx_k(Xc)
    assert float((Y - narrow).abs().max()) < 1e-13 * float(narrow.abs().max())
    Xr = torch.empty((gm.n, ld), dtype=torch.float64, device="cuda")[:, :3]
    Xr.copy_(Xc.real)
    assert torch.equal(Y.real, gm.hx(Xr).contiguous())
    Xr.copy_(Xc.imag)
    assert torch.equal(Y.imag, gm.hx(Xr).contiguous())
    torch.cuda.empty_cache()


def _device_mesh(p, cells, bc):
    import paper_2504_00998_amd as fe
    gm = fe.Mesh(tuple(float(c) for c in cells), cells, p, bc)
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * p + cells[2])
    gm.set_potential(torch.randn((gm.n_cells, gm.nc), generator=g, dtype=torch.float64, device="cuda"), 0.0, 0.0)
    return gm, g


def _against_one_cell_kernel(gm, X, m=4):
    """Product and filter against variant 1 (itself held to 1e-13 and 1e-12 of the
    oracle, as the kernel under test is: twice that between the two)."""
    def err(A, B):
        return float(((A - B).norm(dim=0) / B.norm(dim=0)).max())

    got = gm.hx(X), gm.cheb_filter(X, m, 3.0, 900.0, -1.0)
    gm.set_kernel(1)
    ref = gm.hx(X), gm.cheb_filter(X, m, 3.0, 900.0, -1.0)
    gm.set_kernel(0)
    assert err(got[0], ref[0]) < 2e-13 and err(got[1], ref[1]) < 2e-12


@pytest.mark.parametrize("p,cells,bc,N,pad", [(1, (64, 63, 17), (P, P, D), 64, 0), (2, (30, 31, 17), (P, P, P), 64, 0),
                                              (3, (24, 25, 17), (D, P, D), 64, 0), (4, (24, 22, 13), (P, P, D), 64, 0),
                                              (5, (12, 13, 11), (P, D, P), 64, 0), (6, (12, 11, 11), (P, P, D), 64, 0),
                                              (7, (16, 31, 9), (P, P, D), 64, 0), (2, (30, 31, 17), (P, P, D), 50, 3),
                                              (7, (16, 31, 9), (P, P, P), 50, 3)])
def test_tensor_kernel_walks_several_layers(p, cells, bc, N, pad):
    """More (tile, column group, layer) items than workgroups at once, so that a
    workgroup closes several of its own layers: sums carried from one to the
    next, the previous iterate's register sets in turn, and several column
    groups on whole and on ragged 128-byte rows."""
    print("case: layers", p, cells, bc, N, pad, flush=True)
    gm, g = _device_mesh(p, cells, bc)
    X = torch.randn((gm.n, N + pad), generator=g, dtype=torch.float64, device="cuda")[:, :N]
    _against_one_cell_kernel(gm, X)


@pytest.mark.parametrize("p,cells,bc", [(1, (64, 63, 400), (P, P, D)), (2, (64, 65, 127), (P, P, N_)), (3, (48, 49, 65), (N_, P, P)),
                                        (4, (48, 47, 65), (P, P, D)), (6, (16, 33, 81), (P, D, N_)), (7, (16, 33, 81), (P, P, D))])
def test_single_vector_kernel_walks_several_layers(p, cells, bc):
    """The same for one vector."""
    print("case: layers, one vector", p, cells, bc, flush=True)
    gm, g = _device_mesh(p, cells, bc)
    _against_one_cell_kernel(gm, torch.randn((gm.n, 1), generator=g, dtype=torch.float64, device="cuda"))


@pytest.mark.parametrize("p,cells,bc", [(1, (3, 4, 5), (P, N_, P)), (6, (2, 3, 2), (P, P, N_)), (7, (2, 2, 3), (N_, P, D)),
                                        (7, (2, 3, 2), (P, P, N_))])
def test_poisson_at_the_other_degrees(p, cells, bc):
    """Conjugate gradients with the product's own partial sums at p = 1, 6 and 7."""
    import paper_2504_00998_amd as fe
    print("case: poisson", p, cells, bc, flush=True)
    L = tuple(float(c) for c in cells)
    om, gm = O.Mesh(L, cells, p, bc), fe.Mesh(L, cells, p, bc)
    s = np.random.default_rng(12).standard_normal(om.n)
    ref = O.poisson(om, s)
    phi, it, rel = gm.poisson(torch.from_numpy(s).cuda(), tol=1e-13)
    assert rel <= 1e-13 and it > 0
    assert np.abs(phi.cpu().numpy() - ref).max() <= 1e-8 * np.abs(ref).max()


@pytest.mark.parametrize("p,cells,bc", [(1, (64, 63, 129), (P, P, D)), (2, (64, 63, 65), (P, P, D)), (4, (48, 47, 49), (P, P, N_)),
                                        (7, (16, 33, 40), (P, P, D)), (1, (1056, 250, 2), (P, P, D))])
def test_poisson_with_more_layers_than_partial_sums(p, cells, bc):
    """More (tile, layer) items than partial sums of p.Hp, so that a workgroup walks
    several layers, and (last) more tiles than partial sums, where the product
    and its dot product are launches of their own: the residual of the scaled
    equation H0 x = 2 pi M^1/2 s by the one-cell kernel.  The solve's recurrence
    ends at 1e-11; the residual formed anew differs from it by the rounding of
    the iterates, eps |H0| |x| / |b| an iteration at most and less than 1e-9 over
    all (|H0| below 2e3, |x| / |b| about 10 for random charges)."""
    import paper_2504_00998_amd as fe
    print("case: poisson, layers", p, cells, bc, flush=True)
    L = tuple(float(c) for c in cells)
    gm = fe.Mesh(L, cells, p, bc)
    g = torch.Generator(device="cuda")
    g.manual_seed(p)
    s = torch.randn(gm.n, generator=g, dtype=torch.float64, device="cuda")
    phi, it, rel = gm.poisson(s, tol=1e-11)
    print("iterations", it, "relres", rel, flush=True)
    assert 0 < it < 100000 and rel <= 1e-11
    root = torch.from_numpy(np.sqrt(O.Mesh(L, cells, p, bc).mass())).cuda()
    b = 2.0 * math.pi * root * s
    if D not in bc:
        e = root / root.norm()
        b -= (e @ b) * e
        assert abs(float(root @ (root * phi))) < 1e-10 * float(phi.abs().max()) * float(root @ root)
    gm.set_potential(None, 0.0, 0.0)
    gm.set_kernel(1)
    r = gm.hx((root * phi).reshape(-1, 1)).reshape(-1) - b
    assert float(r.norm() / b.norm()) < 1e-9


@pytest.mark.parametrize("p,cells,bc,variant", [(p, (3, 2, 3), (P, P, D), 1) for p in range(1, 8)] +
                         [(3, (3, 4, 3), (P, P, N_), 0), (5, (2, 3, 2), (P, D, N_), 0), (4, (4, 4, 4), (P, P, P), 6)])
def test_bloch_row_owner_kernel_matches_oracle(p, cells, bc, variant):
    """Bloch mode where the tensor-product kernel is not taken: the other variants
    at every degree, and a zero-Neumann z axis by default."""
    import paper_2504_00998_amd as fe
    wl = W.small_slab(cells, p=p, N=9, m=4, bc=bc, **({"E": 0.0} if bc[2] == P else {}))
    print("case: bloch, row owner", p, cells, bc, variant, flush=True)
    om = O.Mesh.from_workload(wl)
    Vq = W.workload_potential(wl, om.quad_points())
    op = O.Operator(om, Vq, wl.E, wl.z0)
    gm = fe.Mesh.from_workload(wl)
    gm.set_potential(torch.from_numpy(Vq).cuda(), wl.E, wl.z0)
    gm.set_kernel(variant)
    k = (0.37, -0.61 if bc[1] == P else 0.0)
    gm.set_kpoint(*k)
    B = O.BlochOperator(op, om, k)
    Xh = wl.Xc(op.n)
    X = torch.from_numpy(Xh).cuda()
    for Yd, R, bar in ((gm.hx_k(X), B.apply(Xh), 1e-13),
                       (gm.cheb_filter_k(X, 4, 3.0, 900.0, -1.0), B.filter(Xh, 4, 3.0, 900.0, -1.0), 1e-12)):
        assert (np.linalg.norm(Yd.cpu().numpy() - R, axis=0) / np.linalg.norm(R, axis=0)).max() < bar
