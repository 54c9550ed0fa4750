"""The one-plane form of the step and of the adjoint step, which small grids
take by default, against the march of the same grid (an explicit launch
shape), and so against the oracle where the march is."""
import numpy as np
import pytest

from gpu_util import group_rel_err, say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu

# one plane and two (a plane is its own neighbour), a lane more than a tile, a
# row more and less than one, several workgroups per CU
SHAPES = [(1, 1, 1), (5, 3, 1), (64, 4, 2), (65, 5, 3), (127, 2, 5), (33, 70, 40)]
TOL = {"f64": 1e-12, "f32": 2e-6, "f16s": 0.0}


def _step(shape, storage, Q, walls, force, launch, phase=None, steps=3):
    import torch
    from paper_2609_09160_amd import Solver
    Fu = (2e-5, -1e-5, 3e-5) if force == "uniform" else (0.0, 0.0, 0.0)
    s = Solver(shape, 0.7, lattice=Q, storage=storage, bc=(0, int(walls), 0), force=Fu,
               scale=[2.0 ** -13] * 10 if storage == "f16s" else None)
    s.set_moments(inputs.random_state(shape, seed=sum(shape)))
    if phase is not None:
        kw = dict(rho=(0.5, 1.5), tau=(0.65, 1.7)) if phase == "contrast" else {}
        s.enable_two_phase(0.03, 4.0, 0.1, **kw)
    if launch:
        s.set_launch(*launch)
    if phase is not None:
        nx, ny, nz = shape
        s.set_phase(np.random.default_rng(5).uniform(0.2, 0.8, (nz, ny, nx)))
    if force == "field":
        F = inputs.random_force(shape, seed=7, std=1e-4)
        s.set_force_field(torch.as_tensor(F, device="cuda"))
    s.step(steps)
    out = s.moments_host()
    s.close()
    return out


@pytest.mark.parametrize("storage,Q", [("f64", 19), ("f64", 27), ("f64", "27h"), ("f32", 19),
                                       ("f32", 27), ("f32", "27h"), ("f16s", 19), ("f16s", 27)])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("force", ["none", "uniform", "field"])
@pytest.mark.parametrize("walls", [False, True])
def test_step(storage, Q, shape, force, walls):
    """Three steps from an off-equilibrium state; FP16 words bit for bit."""
    if walls and shape[1] < 2:
        pytest.skip("a walled axis needs >= 2 sites")
    say(f"one plane {storage} Q{Q} {shape} {force} walls={walls}")
    want = _step(shape, storage, Q, walls, force, (4, 2, 1))
    got = _step(shape, storage, Q, walls, force, None)
    assert group_rel_err(got, want) <= TOL[storage]


@pytest.mark.parametrize("storage,Q", [("f64", 19), ("f64", 27), ("f64", "27h"), ("f32", 19)])
@pytest.mark.parametrize("shape", SHAPES[1:])
@pytest.mark.parametrize("phase", ["equal", "contrast"])
@pytest.mark.parametrize("walls", [False, True])
def test_two_component_step(storage, Q, shape, phase, walls):
    """The same with the phase field's force and stencils (a random field, so
    that every neighbour counts)."""
    say(f"one plane, two components {storage} Q{Q} {shape} {phase} walls={walls}")
    want = _step(shape, storage, Q, walls, "uniform", (4, 2, 1), phase)
    got = _step(shape, storage, Q, walls, "uniform", None, phase)
    assert group_rel_err(got, want) <= 10 * TOL[storage]


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("Q", [19, 27])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("walls,field", [(False, True), (True, True), (True, False)])
def test_adjoint_step(storage, Q, shape, walls, field):
    """Gradients of a linear objective over three steps, with a per-site or a
    uniform force."""
    import torch
    from paper_2609_09160_amd import Solver
    if walls and shape[1] < 2:
        pytest.skip("a walled axis needs >= 2 sites")
    say(f"one plane, adjoint {storage} Q{Q} {shape} walls={walls} field={field}")
    nx, ny, nz = shape
    lam = np.random.default_rng(9).standard_normal((10, nz, ny, nx))
    out = []
    for march in (True, False):
        s = Solver(shape, 0.7, lattice=Q, storage=storage, bc=(0, int(walls), 0),
                   force=(2e-5, -1e-5, 3e-5))
        if march:
            s.set_launch(4, 2, 1)
            s.set_adjoint_launch(1, 6)
        if field:
            s.set_force_field(torch.as_tensor(inputs.random_force(shape, seed=7, std=1e-4),
                                              device="cuda"))
        s.set_moments(inputs.random_state(shape, seed=4))
        ck = s.forward_checkpointed(3, 2)
        gF, l0 = s.adjoint(3, 2, ck, torch.as_tensor(lam, device="cuda"))
        out.append((gF.double().cpu().numpy(), l0.double().cpu().numpy()))
        s.close()
    for want, got in zip(*out):
        assert np.abs(got - want).max() <= TOL[storage] * np.abs(want).max()
