"""Solves whose quadratic products, which also form (p, K p), are forced into each
kernel of the pipelined and coloured forms, at case counts that divide a
wavefront and that do not; and on a mesh whose patches hand rows on."""
import numpy as np
import pytest
import torch

from oracle import fem, solve
from paper_1710_08679_amd import ebe, meshgen

pytestmark = pytest.mark.gpu

KERNELS = [(f, v) for f in (ebe.FORM_PIPELINED, ebe.FORM_COLOURED) for v in (0, 1, 2)]


def force(gm, n, form, variant):
    for dt in (torch.float64, torch.float32):
        gm.set_form(0, dt, n, form)
        gm.set_variant(0, dt, n, variant)


@pytest.fixture(scope="module")
def crust(gpu_lib):
    m = meshgen.crust_mesh(7, 6, 5)
    f, _ = meshgen.dislocation_pair_loads(m, meshgen.rng_for(3, 7), nrhs=16)
    K = fem.assemble(m.xyz, m.conn, m.young, m.poisson)
    return m, ebe.Mesh.from_generated(m), f, solve.sparse_solve(K, f, m.fixed)


@pytest.mark.parametrize("precond, mode, tol, bound", [(ebe.PREC_PCGE, ebe.MODE_FP64, 1e-11, 1e-8),
                                                       (ebe.PREC_MG2, ebe.MODE_MIXED, 1e-8, 1e-6)])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 5, 7, 9, 12])
def test_solves_in_each_kernel(crust, precond, mode, tol, bound, nrhs):
    m, gm, f, ud = crust
    fd = torch.from_numpy(np.ascontiguousarray(f[:, :, :nrhs])).cuda()
    ref = ud[:, :, :nrhs]
    for form, variant in KERNELS:
        force(gm, nrhs, form, variant)
        u, st = gm.solve(fd, precond=precond, mode=mode, tol=tol)
        assert st["status"] == ebe.OK and st["max_rel_res"] <= tol, (form, variant, st)
        err = float(np.linalg.norm(u.cpu().numpy() - ref) / np.linalg.norm(ref))
        assert err <= bound, (form, variant, err)


@pytest.mark.parametrize("nrhs", [5, 8])
def test_solve_on_chained_patches(gpu_lib, nrhs):
    """The pipelined form on more than 768 patches a range against the gather form: the same
    solution, and outer iterations that differ by no more than one."""
    m = meshgen.crust_mesh(53, 47, 25)
    gm = ebe.Mesh.from_generated(m)
    f, _ = meshgen.dislocation_pair_loads(m, meshgen.rng_for(3, 8), nrhs=nrhs)
    fd = torch.from_numpy(np.ascontiguousarray(f)).cuda()
    out = []
    for form in (ebe.FORM_GATHER, ebe.FORM_PIPELINED):
        force(gm, nrhs, form, 0)
        u, st = gm.solve(fd, precond=ebe.PREC_MG2, mode=ebe.MODE_MIXED, tol=1e-8)
        assert st["status"] == ebe.OK and st["max_rel_res"] <= 1e-8, st
        out.append((u, st["outer_iters"]))
        print(f"[chained n={nrhs} form={form}] {st}", flush=True)
    (a, ia), (b, ib) = out
    assert abs(ia - ib) <= 1
    assert float((a - b).norm() / a.norm()) <= 1e-6
