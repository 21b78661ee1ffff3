"""(x, K x) as the patch kernels form it beside y = K x: the CG step lengths of
every solve rest on it, and no entry point returns it, so these tests call the
library's own launcher.

A tetrahedron's forces sum to zero, so a translation common to its nodes does
not change (x, K x); the kernels must not let the rounding of the forces,
times that translation, into the sum.  Rounding of the forces is c kappa u
|K_e||x_e| (tests/helpers.py), and only the nodes' differences d_e from the
tetrahedron's first corner may multiply it:
    |gamma - gamma_ref| <= c kappa u sum_e (|K_e||x_e|) . |d_e|.
"""
import ctypes

import numpy as np
import pytest
import torch

from oracle import fem
from paper_1710_08679_amd import ebe, meshgen
from tests.helpers import kappa_max, parity_mesh, tol_factor

pytestmark = pytest.mark.gpu

DT = {np.float64: torch.float64, np.float32: torch.float32}
FORMS = [(ebe.FORM_GATHER, 0), (ebe.FORM_STAGED, 0), (ebe.FORM_PIPELINED, 0), (ebe.FORM_PIPELINED, 1),
         (ebe.FORM_PIPELINED, 2), (ebe.FORM_COLOURED, 2),
         (ebe.FORM_COLOURED, 0), (ebe.FORM_COLOURED, 1)]


def product_and_energy(gm, x, bc=False):
    """y = K x and gamma[j] = (x_j, K x_j) in the mesh's current form."""
    gm.matvec(x)  # prepares what the form needs
    fn = ctypes.CDLL(ebe.LIB_PATH)["_ZN3ebe10launch_ebeEPK8ebe_meshiiiPKvPvbbbPKiP12ihipStream_tPd"]
    fn.restype = ctypes.c_int
    p, i, b = ctypes.c_void_p, ctypes.c_int, ctypes.c_bool
    fn.argtypes = [p, i, i, i, p, p, b, b, b, p, p, p]
    y, gamma = torch.empty_like(x), torch.zeros(16, dtype=torch.float64, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    n = x.shape[2]
    assert fn(gm._h, 2, 0 if x.dtype == torch.float64 else 1, n, x.data_ptr(), y.data_ptr(), False, bc, False, None,
              stream, gamma.data_ptr()) == 0
    return y, gamma[:n].cpu().numpy()


@pytest.fixture(scope="module", params=[(4, 4, 4), (9, 5, 7)])
def case(request, gpu_lib):
    m = parity_mesh(*request.param, seed=11)
    return m, ebe.Mesh.from_generated(m), fem.element_stiffness_p2(m.xyz[m.conn], m.young, m.poisson), kappa_max(m)


@pytest.mark.parametrize("dtype, size", [(np.float64, 1e-8), (np.float32, 5e-3)])
@pytest.mark.parametrize("nrhs", range(1, 17))
def test_energy_of_translated_fields(case, dtype, size, nrhs):
    """x = 1000 + values of the given size."""
    m, gm, Ke, kap = case
    x = (1000.0 + size * meshgen.rng_for(95, nrhs).standard_normal((m.n_nodes, 3, nrhs))).astype(dtype)
    xe = x[m.conn].astype(np.float64)
    d = (xe - xe[:, :1]).reshape(-1, 30, nrhs)
    ref = (d * (Ke @ d)).sum((0, 1))
    bound = tol_factor(dtype, kap) * (np.abs(d) * (np.abs(Ke) @ np.abs(xe.reshape(-1, 30, nrhs)))).sum((0, 1))
    xd = torch.from_numpy(x).cuda()
    for form, variant in FORMS:
        gm.set_form(0, DT[dtype], nrhs, form)
        gm.set_variant(0, DT[dtype], nrhs, variant)
        g = product_and_energy(gm, xd)[1]
        assert np.all(np.abs(g - ref) <= bound), (form, variant, float(np.max(np.abs(g - ref) / bound)))


@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 5, 8, 9, 10, 12, 16])
def test_energy_as_accurate_as_from_strains(case, nrhs):
    """Linear fields beside a translation ten times their size, FP32: the root mean square of the
    error over 192 fields or more is no larger than the gather form's, which sums strains times
    stresses (1.25: five standard deviations of the quotient of two such estimates)."""
    m, gm, Ke, _ = case
    rng = meshgen.rng_for(97, nrhs)
    err = {f: [] for f in FORMS}
    for _ in range(-(-192 // nrhs)):
        A, t = rng.standard_normal((3, 3, nrhs)), rng.choice([-10.0, 10.0], (3, nrhs))
        x = (t + (m.xyz @ A.reshape(3, -1)).reshape(m.n_nodes, 3, nrhs)).astype(np.float32)
        xe = x[m.conn].astype(np.float64)
        d = (xe - xe[:, :1]).reshape(-1, 30, nrhs)
        ref = (d * (Ke @ d)).sum((0, 1))
        xd = torch.from_numpy(x).cuda()
        for form, variant in FORMS:
            gm.set_form(0, torch.float32, nrhs, form)
            gm.set_variant(0, torch.float32, nrhs, variant)
            err[form, variant] += list((product_and_energy(gm, xd)[1] - ref) / ref)
    rms = {f: float(np.sqrt(np.mean(np.square(e)))) for f, e in err.items()}
    print(f"[energy n={nrhs}] {rms}", flush=True)
    assert all(r <= 1.25 * rms[FORMS[0]] for r in rms.values()), rms


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_energy_on_chained_patches(gpu_lib, dtype):
    """A mesh whose patches hand accumulator rows on.  |x|.|K_e||x| <= 30 sum_i K_ii x_i^2
    in each tetrahedron (K_e is positive semidefinite), summed by the assembled diagonal."""
    m = meshgen.crust_mesh(53, 47, 25)
    gm = ebe.Mesh.from_generated(m)
    diag = gm.diag_blocks(0).diagonal(dim1=1, dim2=2)[:, :, None]
    factor = 30 * tol_factor(dtype, kappa_max(m))
    gen = torch.Generator(device="cuda").manual_seed(96)
    for nrhs in (1, 3, 4, 5, 8, 9, 10, 12, 16):
        x = torch.randn((m.n_nodes, 3, nrhs), generator=gen, device="cuda", dtype=DT[dtype])
        x64 = x.double()
        gm.set_form(0, torch.float64, nrhs, ebe.FORM_GATHER)
        ref = (x64 * gm.matvec(x64)).sum((0, 1)).cpu().numpy()
        bound = factor * (x64.square() * diag).sum((0, 1)).cpu().numpy()
        for form, variant in FORMS[2:]:
            gm.set_form(0, DT[dtype], nrhs, form)
            gm.set_variant(0, DT[dtype], nrhs, variant)
            g = product_and_energy(gm, x)[1]
            assert np.all(np.abs(g - ref) <= bound), (nrhs, form, variant, float(np.max(np.abs(g - ref) / bound)))
