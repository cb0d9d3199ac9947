"""The hop with a wavefront per direction (the default of small launches) against the hop
with one lane per site, pinned by COLA_HOP_SHAPE: the outputs agree bitwise, in every
precision it takes, for every epilogue an operator uses, with right-hand sides that do not
fill a 64-lane block, parity volumes that leave a partial block, extents of 2 and complex
boundary phases."""
import numpy as np
import pytest
import torch

from paper_2302_00850_amd.synth import Synth, bc_phases

pytestmark = pytest.mark.gpu

cola = pytest.importorskip("paper_2302_00850_amd.cola")

ANTI = bc_phases((0, 0, 0, np.pi))
GENERIC = bc_phases((0.3, -0.5, 0.7, np.pi))


@pytest.mark.parametrize("dims", [(6, 4, 4, 10), (2, 2, 4, 2)])
@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("nrhs", [1, 3, 12, 16])
@pytest.mark.parametrize("csw", [0.0, 1.0])
def test_bitwise_as_one_lane_per_site(dims, prec, nrhs, csw, monkeypatch):
    s = Synth(31)
    U, psi = s.gauge(dims).cuda(), s.gaussian_spinor(dims, nrhs).cuda()
    for bc in (ANTI, GENERIC):
        lat = cola.Lattice(dims, 0.118, bc, csw)
        lat.set_gauge(U)
        for op, parity in ((cola.COLA_OP_HOP, 1), (cola.COLA_OP_M, -1), (cola.COLA_OP_MDAG, -1),
                           (cola.COLA_OP_SCHUR, 0), (cola.COLA_OP_SCHUR_DAG, 0)):
            pin = lat.pack(psi, prec, 1 - parity if op == cola.COLA_OP_HOP else parity)
            outs = []
            for shape in (f"1,{64 // nrhs},0,1,0,0,2", "1,8,0,1,0,0,0"):
                monkeypatch.setenv("COLA_HOP_SHAPE", shape)
                out = lat.empty_packed(prec, nrhs, parity)
                lat.dslash(out, pin, op, parity, prec, nrhs)
                outs.append(out)
            assert torch.equal(*outs), (op, parity)
        lat.close()
