"""16-bit states do not depend on the launch shape that the library picks: the
default shape against the tiles that the width alone gives."""
import pytest

from gpu_util import say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,scale", [("f16s", 2.0 ** -13), ("f16su", 2.0 ** -13)])
@pytest.mark.parametrize("Q", [19, 27])
@pytest.mark.parametrize("force", [(0.0, 0.0, 0.0), (2e-5, -1e-5, 3e-5)])
@pytest.mark.parametrize("shape,sites,walls", [((64, 16, 52), 1, False), ((192, 85, 76), 1, False),
                                               ((128, 158, 42), 2, False), ((64, 73, 242), 1, True)])
def test_default_shape_keeps_the_words(storage, scale, Q, force, shape, sites, walls):
    import torch
    from paper_2609_09160_amd import Solver
    say(f"words {storage} Q{Q} {force} {shape}")
    g = torch.Generator(device="cuda").manual_seed(3)
    nx, ny, nz = shape
    m0 = 0.01 * torch.randn((10, nz, ny, nx), generator=g, device="cuda")
    m0[4:] *= 0.01
    out = []
    for launch in (None, (8, 0, sites)):
        s = Solver(shape, 0.8, lattice=Q, storage=storage, bc=(0, int(walls), 0), force=force,
                   scale=[scale] * 4 + [scale / 8] * 6)
        if launch:
            s.set_launch(*launch)
        s.set_moments(m0)
        s.step(6)
        out.append(s.moments(dtype=torch.float32))
        s.close()
    assert torch.equal(out[0], out[1])
