"""The kernel that holds a lattice in one workgroup skips directions one node
wide: what the stage kernel reports of them is reported all the same."""
import numpy as np
import pytest

import olb_inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1), (1, 5), (5, 1)], ids=lambda v: f"{v[0]}x{v[1]}")
def test_an_infinite_pressure_is_reported(shape):
    """A finite density whose square overflows: the van der Waals pressure is
    infinite, its difference from itself not a number, also along a direction
    that holds one node."""
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a visible GPU")
    from paper_1702_01690_amd import olb
    nx, ny = shape
    p = dict(nx=nx, ny=ny, ds=1 / 64, dt=5e-4, tau=0.01, a=I.VDW_A, b=I.VDW_B, sigma=1e-4, bc_x=0, bc_y=0)
    one = np.ones((ny, nx))
    for by in (None, 8):          # the lattice's own kernel, and the stage kernel
        lat = olb.Lattice(p)
        if by:
            lat.set_tile(by)
        lat.set_fields(2.0 * one, 0.0 * one, 0.0 * one, one)
        f = np.array(lat.get_f()).reshape(25, ny, nx)
        f[7, 0, 0] = 1e290
        lat.set_f(f)
        lat.step(2)
        with pytest.raises(olb.OlbError) as e:
            lat.sync()
        assert e.value.code == olb.OLB_E_NONFINITE
        lat.close()
