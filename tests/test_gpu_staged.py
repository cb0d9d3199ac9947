"""Hops with the links staged in LDS where both parities are one launch (M, M^H), from four
right-hand sides up, and the hop of one parity at counts that do not fill a wavefront: bitwise
the kernel that loads links per lane, in tiles, time chunks and partly filled blocks, and by
the oracle to the precision's tolerance."""
import numpy as np
import pytest
import torch

import oracle
from paper_2302_00850_amd.synth import Synth, bc_phases
from tests._util import assert_close

pytestmark = pytest.mark.gpu

cola = pytest.importorskip("paper_2302_00850_amd.cola")

DIMS = (6, 4, 4, 10)
GENERIC = bc_phases((0.3, -0.5, 0.7, np.pi))
TOL = {cola.COLA_FP32: 2e-6, cola.COLA_FP16: 4e-3}  # of test_gpu_parity.py's same operators


@pytest.mark.parametrize("prec", [cola.COLA_FP32, cola.COLA_FP16])
@pytest.mark.parametrize("nrhs", [4, 5, 8, 11, 16])
@pytest.mark.parametrize("csw", [0.0, 1.0])
def test_staged_links_with_both_parities(prec, nrhs, csw, monkeypatch):
    kappa = 0.118 if csw else 0.12
    s = Synth(303)
    U, psi = s.gauge(DIMS), s.gaussian_spinor(DIMS, nrhs)
    lat = cola.Lattice(DIMS, kappa, GENERIC, csw)
    lat.set_gauge(U.cuda())
    clover = oracle.clover(U.numpy(), kappa, csw) if csw else None
    T = max(t for t in (4, 8, 16, 32) if t * nrhs <= 256)
    for op, parity in ((cola.COLA_OP_M, -1), (cola.COLA_OP_MDAG, -1), (cola.COLA_OP_HOP, 1)):
        src = 1 - parity if parity >= 0 else -1
        pin = lat.pack(psi.cuda(), prec, src)
        monkeypatch.setenv("COLA_HOP_SHAPE", "1,8,0,1,0,0,0")
        ref = lat.empty_packed(prec, nrhs, parity)
        lat.dslash(ref, pin, op, parity, prec, nrhs)
        # whole and halved blocks, plain order and tiles, chunks walked or not, a grid that loops
        for shape in (f"1,{T},0,1,0,0,1", f"1,{T},0,2,0,0,1", f"1,{T},0,1,2,4,1",
                      f"1,{T},0,2,4,2,1", f"1,{T // 2},0,5,2,2,1", f"1,{T},3,1,2,2,1",
                      f"1,{T},-1,2,4,4,1"):
            monkeypatch.setenv("COLA_HOP_SHAPE", shape)
            out = lat.empty_packed(prec, nrhs, parity)
            lat.dslash(out, pin, op, parity, prec, nrhs)
            assert torch.equal(out, ref), (op, shape)
        if parity < 0:
            got = lat.unpack(ref, prec, nrhs, -1).cpu().numpy()
            x = lat.unpack(pin, prec, nrhs, -1).cpu().numpy()
            for q in (0, nrhs - 1):
                want = oracle.apply_M(U.numpy(), x[q], kappa, GENERIC, clover=clover,
                                      dagger=op == cola.COLA_OP_MDAG)
                assert_close(got[q], want, TOL[prec], (op, q))
    lat.close()
