"""The adjoint element gradient by single elements, which meshes of 2^25 nodes or
more take (too large for a test), small ones at some numbers of cases: called
here through the library's own launcher, against the oracle; and the entry
point on either side of the size from which it goes by fans."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import adjoint
from paper_1710_08679_amd import ebe, meshgen
from tests.helpers import parity_mesh

pytestmark = pytest.mark.gpu


def by_elements(gm, u, lam):
    fn = ctypes.CDLL(ebe.LIB_PATH)["_ZN3ebe14launch_adjointEPK8ebe_meshiiPKvS4_PvP12ihipStream_tb"]
    fn.restype = ctypes.c_int
    p, i = ctypes.c_void_p, ctypes.c_int
    fn.argtypes = [p, i, i, p, p, p, p, ctypes.c_bool]
    g = torch.empty((gm.n_elem,), dtype=u.dtype, device="cuda")
    assert fn(gm._h, 0 if u.dtype == torch.float64 else 1, u.shape[2], u.data_ptr(), lam.data_ptr(), g.data_ptr(),
              torch.cuda.current_stream().cuda_stream, True) == 0
    return g


@pytest.fixture(scope="module")
def case(gpu_lib):
    m = parity_mesh(6, 5, 4, seed=12, bc=True)
    return m, ebe.Mesh.from_generated(m)


@pytest.mark.parametrize("dtype, tol", [(np.float64, 1e-12), (np.float32, 2e-5)])
@pytest.mark.parametrize("nrhs", range(1, 17))
def test_gradient_by_elements(case, dtype, tol, nrhs):
    m, gm = case
    rng = meshgen.rng_for(101, nrhs)
    u, lam = (rng.standard_normal((m.n_nodes, 3, nrhs)).astype(dtype) for _ in range(2))
    free = 1.0 - m.fixed[:, :, None].astype(np.float64)
    ref = adjoint.element_gradient(m.xyz, m.conn, m.poisson, u * free, lam * free)
    ud, ld = torch.from_numpy(u).cuda(), torch.from_numpy(lam).cuda()
    for g in (by_elements(gm, ud, ld), gm.adjoint_grad(ud, ld)):
        assert np.max(np.abs(g.cpu().numpy() - ref)) <= tol * np.max(np.abs(ref))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_sixteen_cases_by_elements_are_spread_over_lanes(gpu_lib, dtype):
    """Sixteen cases take less time than fifteen, which one work-item goes through in turn (4 to 5
    times less: 77 us against 306 in FP64 on this mesh, 48 against 222 in FP32)."""
    m = meshgen.crust_mesh(29, 23, 17)
    gm = ebe.Mesh.from_generated(m)
    times = {}
    for n in (15, 16):
        u, lam = (torch.randn((m.n_nodes, 3, n), device="cuda", dtype=dtype) for _ in range(2))
        runs = []
        for _ in range(7):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                by_elements(gm, u, lam)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b))
        times[n] = min(runs)
    assert times[16] < times[15], times


@pytest.mark.parametrize("dtype, tol", [(np.float64, 1e-12), (np.float32, 2e-5)])
@pytest.mark.parametrize("nrhs, grid", [(1, (23, 24, 24)), (1, (24, 24, 24)), (1, (25, 26, 25)), (4, (14, 15, 15)),
                                        (4, (15, 15, 15)), (4, (16, 16, 16)), (16, (8, 9, 11)), (16, (9, 10, 10)),
                                        (16, (10, 10, 11))])
def test_gradient_around_the_size_of_a_resident_mesh(gpu_lib, dtype, tol, nrhs, grid):
    """80000 (FP64) or 96000 elements times cases: below and above, by the entry point and by elements."""
    m = meshgen.crust_mesh(*grid)
    gm = ebe.Mesh.from_generated(m)
    rng = meshgen.rng_for(103, nrhs)
    u, lam = (rng.standard_normal((m.n_nodes, 3, nrhs)).astype(dtype) for _ in range(2))
    free = 1.0 - m.fixed[:, :, None].astype(np.float64)
    ref = adjoint.element_gradient(m.xyz, m.conn, m.poisson, u * free, lam * free)
    ud, ld = torch.from_numpy(u).cuda(), torch.from_numpy(lam).cuda()
    for g in (by_elements(gm, ud, ld), gm.adjoint_grad(ud, ld)):
        assert np.max(np.abs(g.cpu().numpy() - ref)) <= tol * np.max(np.abs(ref))
