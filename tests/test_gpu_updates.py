"""The CG's vector updates (x beside p, r in the last hop) at the edges of their kernels: rhs
counts that do not divide a 16-byte element, columns that are done before the others or from
the start, checks that fall between updates, and caps inside a block of iterations."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_00850_amd.synth import Synth, bc_phases
from tests._util import assert_close, rel

pytestmark = pytest.mark.gpu

cola = pytest.importorskip("paper_2302_00850_amd.cola")

DIMS, KAPPA = (6, 4, 4, 10), 0.12
ANTI = bc_phases((0, 0, 0, np.pi))


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def fields():
    s = Synth(55)
    return s.gauge(DIMS, mix=0.4).numpy(), s.gaussian_spinor(DIMS, 5).numpy()


@pytest.mark.parametrize("nrhs", [1, 3, 5])
@pytest.mark.parametrize("system", [cola.COLA_SYS_MDAGM, cola.COLA_SYS_SCHUR])
@pytest.mark.parametrize("n", [1, 4, 7])
def test_fixed_iterations_match_oracle(fields, nrhs, system, n):
    """n FP64 iterations with a check every third: rounding only."""
    U, b = fields
    sysid = 0 if system == cola.COLA_SYS_MDAGM else 1
    lat = cola.Lattice(DIMS, KAPPA, ANTI)
    lat.set_gauge(_cuda(U))
    x, info = lat.cg(_cuda(b[:nrhs]), system=system, scheme=cola.COLA_CG_FP64, tol=1e-300,
                     max_iter=n, check_interval=3)
    assert info["iterations"] == n
    for q in range(nrhs):
        want, _, _ = oracle.cg(U, b[q], KAPPA, ANTI, system=sysid, fixed_iters=n)
        assert_close(x.cpu().numpy()[q], want, 1e-12, (q,))
    lat.close()


@pytest.mark.parametrize("scheme", [cola.COLA_CG_FP64, cola.COLA_CG_FP32_RELIABLE,
                                    cola.COLA_CG_FP16_DEFECT, cola.COLA_CG_FP32_DEFECT])
@pytest.mark.parametrize("check", [1, 3, 8])
def test_columns_that_end_apart(fields, scheme, check):
    """A zero column (done from the start) and one smooth source among the rest: every column
    reaches the tolerance, the zero one stays zero."""
    U, b = fields
    src = b.copy()
    src[1] = 0
    src[3] = 1.0
    lat = cola.Lattice(DIMS, KAPPA, ANTI)
    lat.set_gauge(_cuda(U))
    x, info = lat.cg(_cuda(src), system=cola.COLA_SYS_MDAGM, scheme=scheme, tol=1e-10,
                     check_interval=check)
    assert info["status"] == cola.COLA_OK, info
    xs = x.cpu().numpy()
    assert not xs[1].any()
    for q in (0, 2, 3, 4):
        ax = oracle.apply_M(U, oracle.apply_M(U, xs[q], KAPPA, ANTI), KAPPA, ANTI, dagger=True)
        assert rel(ax, src[q]) <= 1.05e-10, (q, info)
    lat.close()
