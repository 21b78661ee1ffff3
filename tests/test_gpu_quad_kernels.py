"""The kernels of the pipelined and coloured forms on the quadratic level, each
in turn: variant 0 takes the one that suits the mesh, 1 single elements, 2
fans of tetrahedra (wide patches at up to four cases).  On the meshes of short
fans, ragged wide patches and chains, so that each meets the shapes where it
can go wrong whichever the default is."""
import numpy as np
import pytest
import torch

from oracle import fem
from paper_1710_08679_amd import ebe, meshgen
from tests.helpers import assert_close_bound, kappa_max, oracle_K, parity_mesh, tol_factor
from tests.test_gpu_fans import DT, checkered, interleaved

pytestmark = pytest.mark.gpu

KERNELS = [(f, v) for f in (ebe.FORM_PIPELINED, ebe.FORM_COLOURED) for v in (0, 1, 2)]


@pytest.fixture(scope="module", params=["checkered", "interleaved", "ragged"])
def case(request, gpu_lib):
    m = parity_mesh(*((9, 5, 7) if request.param == "ragged" else (4, 4, 4)), seed=5, bc=True)
    m = {"checkered": checkered, "interleaved": interleaved}.get(request.param, lambda m: m)(m)
    return m, ebe.Mesh.from_generated(m), oracle_K(m), kappa_max(m)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nrhs", range(1, 17))
def test_products_in_each_kernel(case, dtype, nrhs):
    """K x, P K P x and y += K x against the oracle, then K x with an infinite and a NaN entry in x,
    which reach the nodes of their elements and no others."""
    m, gm, K, kap = case
    rng = meshgen.rng_for(98, nrhs)
    x, y0 = (rng.standard_normal((m.n_nodes, 3, nrhs)).astype(dtype) for _ in range(2))
    xr, xd = x.astype(np.float64), torch.from_numpy(x).cuda()
    ref = (K @ xr.reshape(-1, nrhs)).reshape(x.shape)
    bound = tol_factor(dtype, kap) * (abs(K) @ np.abs(xr).reshape(-1, nrhs)).reshape(x.shape)
    refb, total = fem.matvec_bc(K, xr, m.fixed), y0 + ref
    bad = x.copy()
    bad[0, 0, 0], bad[m.n_nodes - 1, 2, nrhs - 1] = np.inf, np.nan
    touched = np.zeros((m.n_nodes, nrhs), dtype=bool)
    for node, r in ((0, 0), (m.n_nodes - 1, nrhs - 1)):
        touched[np.unique(m.conn[(m.conn == node).any(axis=1)]), r] = True
    for form, variant in KERNELS:
        what = f"n={nrhs} form={form} variant={variant}"
        gm.set_form(0, DT[dtype], nrhs, form)
        gm.set_variant(0, DT[dtype], nrhs, variant)
        assert gm.form(0, DT[dtype], nrhs) == form
        assert_close_bound(gm.matvec(xd).cpu().numpy().astype(np.float64), ref, abs(K), xr, dtype, kap, what)
        assert_close_bound(gm.matvec(xd, apply_bc=True).cpu().numpy().astype(np.float64), refb, abs(K), xr, dtype, kap,
                           "P K P " + what)
        y = torch.from_numpy(y0).cuda()
        gm.matvec_add(xd, y)
        assert np.all(np.abs(y.cpu().numpy() - total) <= bound + 2 * np.finfo(dtype).eps * np.abs(total)), what
        y = gm.matvec(torch.from_numpy(bad).cuda()).cpu().numpy()
        assert np.all(np.isfinite(y) | touched[:, None, :]), what
        assert not np.isfinite(y[0, :, 0]).any() and not np.isfinite(y[m.n_nodes - 1, :, nrhs - 1]).any(), what


@pytest.fixture(scope="module")
def middle(gpu_lib):
    """3000 patches: no chains; the sizes at which some numbers of cases keep the geometry in LDS."""
    m = meshgen.crust_mesh(40, 30, 20)
    return m, ebe.Mesh.from_generated(m)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nrhs", [2, 4, 6, 7, 9, 10, 11])
def test_kernels_agree_on_a_middle_sized_mesh(middle, dtype, nrhs):
    m, gm = middle
    dt = DT[dtype]
    g = torch.Generator(device="cuda").manual_seed(99)
    x, y0 = (torch.randn((m.n_nodes, 3, nrhs), generator=g, device="cuda", dtype=dt) for _ in range(2))

    def products(form, variant):
        gm.set_form(0, dt, nrhs, form)
        gm.set_variant(0, dt, nrhs, variant)
        y = y0.clone()
        gm.matvec_add(x, y)
        return [v.double() for v in (gm.matvec(x), gm.matvec(x, apply_bc=True), y)]

    ref = products(ebe.FORM_GATHER, 0)
    for form, variant in KERNELS:
        for k, (a, b) in enumerate(zip(products(form, variant), ref)):
            # both sum a few hundred products a row, which cancel to a tenth of their size
            assert (a - b).abs().max() <= 100 * np.finfo(dtype).eps * b.abs().max(), (form, variant, k)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nrhs", [3, 5, 16])
def test_tuned_variant_gives_the_same_product(middle, dtype, nrhs):
    m, gm = middle
    dt = DT[dtype]
    x = torch.randn((m.n_nodes, 3, nrhs), generator=torch.Generator(device="cuda").manual_seed(100), device="cuda",
                    dtype=dt)
    gm.set_form(0, dt, nrhs, ebe.FORM_GATHER)
    ref = gm.matvec(x).double()
    gm.autotune(0, dt, nrhs)
    assert gm.variant(0, dt, nrhs) in (0, 1, 2)
    assert (gm.matvec(x).double() - ref).abs().max() <= 100 * np.finfo(dtype).eps * ref.abs().max()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("nrhs", [1, 2])
def test_untuned_form_of_the_smallest_meshes(gpu_lib, dtype, nrhs):
    """Untuned, a mesh of one patch (up to 48 elements, one launch either way) takes the gather form;
    one of several patches that make one wide patch the pipelined one, captured into a graph or not."""
    dt = DT[dtype]
    for grid, form in (((1, 1, 1), ebe.FORM_GATHER), ((2, 2, 2), ebe.FORM_GATHER), ((3, 3, 2), ebe.FORM_PIPELINED),
                       ((4, 4, 4), ebe.FORM_PIPELINED)):
        m = parity_mesh(*grid, seed=7, bc=True)
        gm, K, kap = ebe.Mesh.from_generated(m), oracle_K(m), kappa_max(m)
        assert gm.form(0, dt, nrhs) == form, grid
        x = torch.zeros((m.n_nodes, 3, nrhs), dtype=dt, device="cuda")
        y = gm.matvec(x, apply_bc=True)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            gm.matvec(x, apply_bc=True, out=y)
        for rep in range(3):
            xh = meshgen.rng_for(102 + rep, nrhs).standard_normal(tuple(x.shape)).astype(dtype)
            x.copy_(torch.from_numpy(xh))
            xr = xh.astype(np.float64)
            ref = fem.matvec_bc(K, xr, m.fixed)
            graph.replay()
            for v in (y, gm.matvec(x, apply_bc=True)):
                assert_close_bound(v.cpu().numpy().astype(np.float64), ref, abs(K), xr, dtype, kap, f"{grid} {rep}")
