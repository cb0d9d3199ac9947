"""Device memory that a handle keeps: smearing and the trajectory share their packed link
fields."""
import numpy as np
import pytest
import torch

from paper_2302_00850_amd.synth import Synth, bc_phases

pytestmark = pytest.mark.gpu

cola = pytest.importorskip("paper_2302_00850_amd.cola")


def test_smearing_and_trajectory_share_link_fields():
    """Two packed link fields and the momenta: 3 fields of 75 MB at 16^3 x 32, not 5; half a
    field of slack for the allocator and the kernels' code."""
    dims = (16, 16, 16, 32)
    s = Synth(91, device="cuda", rng="torch")
    U, P = s.gauge(dims), s.momenta(dims)
    field = U.numel() * 16
    small = cola.Lattice((4, 4, 4, 4), 0.12, bc_phases((0, 0, 0, np.pi)))
    Us = Synth(92).gauge((4, 4, 4, 4)).cuda()
    small.ape_smear(Us, 0.7, 2)  # the kernels are loaded
    small.hmc_trajectory(Us, torch.zeros_like(Us), 5.6, 0.01, 1)
    small.close()
    lat = cola.Lattice(dims, 0.12, bc_phases((0, 0, 0, np.pi)))
    F = torch.empty_like(U)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    cola.cola_ape_smear(lat.h, F.data_ptr(), U.data_ptr(), 0.7, 2,
                        torch.cuda.current_stream().cuda_stream)
    lat.hmc_trajectory(U, P, 5.6, 0.01, 2)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    assert used <= 3.5 * field, used / field
    # and one does not disturb the other
    again = torch.empty_like(F)
    cola.cola_ape_smear(lat.h, again.data_ptr(), F.data_ptr(), 0.7, 1,
                        torch.cuda.current_stream().cuda_stream)
    want = cola.Lattice(dims, 0.12, bc_phases((0, 0, 0, np.pi)))
    assert torch.equal(again, want.ape_smear(F, 0.7, 1))
    want.close()
    lat.close()


@pytest.mark.parametrize("nsweeps", [1, 2, 3])
def test_smearing_in_place(nsweeps):
    """F may be U: the links are copied before the last sweep writes its result; same bits."""
    dims = (6, 10, 4, 6)
    lat = cola.Lattice(dims, 0.12, bc_phases((0, 0, 0, np.pi)))
    U = Synth(94).gauge(dims, mix=0.5).cuda()
    want = lat.ape_smear(U, 0.7, nsweeps)
    cola.cola_ape_smear(lat.h, U.data_ptr(), U.data_ptr(), 0.7, nsweeps,
                        torch.cuda.current_stream().cuda_stream)
    assert torch.equal(U, want)
    lat.close()
