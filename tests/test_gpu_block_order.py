"""The order of the workgroups changes no result: the checkpointed run and the
adjoint sweep in marches, and the two-component step."""
import numpy as np
import pytest

from gpu_util import say
from paper_2609_09160_amd import _lib, inputs

pytestmark = pytest.mark.gpu
SHAPE = (131, 50, 37)  # odd, a ragged last tile each way, columns no multiple of 8


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("Q", [19, 27])
@pytest.mark.parametrize("every", [1, 2])
def test_checkpoints_and_gradients(storage, Q, every):
    import torch
    from paper_2609_09160_amd import Solver
    say(f"block order, adjoint {storage} Q{Q} every {every}")
    g = torch.Generator(device="cuda").manual_seed(7)
    out = []
    lam = None
    for order in (0, 1, 2):
        s = Solver(SHAPE, 0.8, lattice=Q, storage=storage)
        _lib.check(s.lib.lbfast_set_form(s.h, _lib.LBF_FORM_MARCH))
        s.set_block_order(order)
        s.set_force_field(torch.as_tensor(inputs.random_force(SHAPE, seed=3, std=1e-4),
                                          device="cuda"))
        s.set_moments(inputs.random_state(SHAPE, seed=4))
        if lam is None:
            lam = torch.randn(10 * s.N, generator=g, device="cuda", dtype=s.compute_dtype)
        ck = s.forward_checkpointed(3, every)
        out.append((ck, s.moments()) + tuple(s.adjoint(3, every, ck, lam)))
        s.close()
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert torch.equal(a, b)


@pytest.mark.parametrize("storage,Q", [("f32", 19), ("f32", "27h"), ("f64", 19), ("f64", 27),
                                       ("f16s", 19)])
@pytest.mark.parametrize("contrast", [False, True])
def test_two_component_step(storage, Q, contrast):
    from paper_2609_09160_amd import Solver
    say(f"block order, two components {storage} Q{Q} contrast={contrast}")
    nx, ny, nz = SHAPE
    phi = np.random.default_rng(5).uniform(0.2, 0.8, (nz, ny, nx))
    out = []
    for order in (0, 1, 2):
        s = Solver(SHAPE, 0.8, lattice=Q, storage=storage,
                   scale=[2.0 ** -13] * 10 if storage == "f16s" else None)
        s.set_moments(inputs.random_state(SHAPE, seed=4))
        s.enable_two_phase(0.03, 4.0, 0.1, **(dict(rho=(0.5, 1.5), tau=(0.65, 1.7))
                                              if contrast else {}))
        _lib.check(s.lib.lbfast_set_form(s.h, _lib.LBF_FORM_MARCH))
        s.set_block_order(order)
        s.set_phase(phi)
        s.step(3)
        out.append((s.moments_host(), s.phase().cpu().numpy()))
        s.close()
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)
