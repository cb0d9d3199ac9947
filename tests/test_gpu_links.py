"""Link kernels at the edges of their blocks and site orders, against the oracle: lattices
whose parity volume is not a multiple of a 64-site block, whose y and z extents take each of
the tile orders (8, 4 or 2 by 4 or 2), and extents of 2, where both neighbours coincide."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_00850_amd.synth import Synth, bc_phases
from tests._util import assert_close

pytestmark = pytest.mark.gpu

cola = pytest.importorskip("paper_2302_00850_amd.cola")

ANTI = bc_phases((0, 0, 0, np.pi))
# (tile 8 x 4, 4 x 4, 4 x 2, 2 x 4, 2 x 2), extents of 2, partial 64-site blocks
LATTICES = [(4, 8, 4, 4), (6, 4, 4, 10), (2, 4, 6, 4), (4, 6, 8, 2), (6, 10, 2, 6)]


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("dims", LATTICES)
def test_clover_blocks_match_oracle(dims):
    """M and S (A and A^-1) with c_sw = 1 in FP64: rounding only, as the plain operators."""
    kappa = 0.118
    s = Synth(77)
    U, psi = s.gauge(dims).numpy(), s.gaussian_spinor(dims).numpy()
    A = oracle.clover(U, kappa, 1.0)
    lat = cola.Lattice(dims, kappa, ANTI, 1.0)
    lat.set_gauge(_cuda(U))
    pin = lat.pack(_cuda(psi), cola.COLA_FP64, -1)
    out = lat.empty_packed(cola.COLA_FP64, 1, -1)
    lat.dslash(out, pin, cola.COLA_OP_M, -1, cola.COLA_FP64, 1)
    got = lat.unpack(out, cola.COLA_FP64, 1, -1).cpu().numpy()[0]
    assert_close(got, oracle.apply_M(U, psi[0], kappa, ANTI, clover=A), 1e-13, dims)
    even = np.where(oracle.parity_mask(dims)[..., None, None], psi[0], 0)
    pe = lat.pack(_cuda(even[None]), cola.COLA_FP64, 0)
    oe = lat.empty_packed(cola.COLA_FP64, 1, 0)
    lat.dslash(oe, pe, cola.COLA_OP_SCHUR, 0, cola.COLA_FP64, 1)
    got = lat.unpack(oe, cola.COLA_FP64, 1, 0).cpu().numpy()[0]
    ref = oracle.apply_schur(U, even, kappa, ANTI, clover=A, clover_inv=oracle.site_inverse(A))
    assert_close(got, ref, 1e-13, dims)
    lat.close()
