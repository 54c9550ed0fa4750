"""Every one-plane form against the march of the same grid, each form set
explicitly, so that no case compares a kernel with itself; in both orders of
the workgroups (several per CU in the largest grid)."""
import numpy as np
import pytest

from gpu_util import group_rel_err, say
from paper_2609_09160_amd import _lib, inputs

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (5, 3, 1), (65, 5, 3), (33, 70, 40)]
# three steps of the same formulas, compiled twice
TOL = {"f64": 1e-12, "f32": 2e-6}
FORMS = [(_lib.LBF_FORM_MARCH, 0), (_lib.LBF_FORM_ONE_PLANE, 1), (_lib.LBF_FORM_ONE_PLANE, 2)]


def _solver(shape, storage, Q, walls, force=(0.0, 0.0, 0.0)):
    from paper_2609_09160_amd import Solver
    s = Solver(shape, 0.7, lattice=Q, storage=storage, bc=(0, int(walls), 0), force=force)
    s.set_moments(inputs.random_state(shape, seed=sum(shape)))
    return s


def _set(s, form, order):
    _lib.check(s.lib.lbfast_set_form(s.h, form))
    s.set_block_order(order)


def _field(s, shape):
    import torch
    s.set_force_field(torch.as_tensor(inputs.random_force(shape, seed=7, std=1e-4), device="cuda"))


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("Q", [19, 27, "27h"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("force", ["none", "uniform", "field"])
@pytest.mark.parametrize("walls", [False, True])
def test_step(storage, Q, shape, force, walls):
    if walls and shape[1] < 2:
        pytest.skip("a walled axis needs >= 2 sites")
    say(f"one-plane form {storage} Q{Q} {shape} {force} walls={walls}")
    out = []
    for form, order in FORMS:
        s = _solver(shape, storage, Q, walls,
                    (2e-5, -1e-5, 3e-5) if force == "uniform" else (0.0, 0.0, 0.0))
        if force == "field":
            _field(s, shape)
        _set(s, form, order)
        s.step(3)
        out.append(s.moments_host())
        s.close()
    assert group_rel_err(out[1], out[0]) <= TOL[storage]
    assert np.array_equal(out[1], out[2])


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("Q", [19, 27, "27h"])
@pytest.mark.parametrize("shape", SHAPES[2:])
@pytest.mark.parametrize("phase", ["equal", "contrast"])
@pytest.mark.parametrize("walls", [False, True])
def test_two_component_step(storage, Q, shape, phase, walls):
    say(f"one-plane form, two components {storage} Q{Q} {shape} {phase} walls={walls}")
    nx, ny, nz = shape
    phi = np.random.default_rng(5).uniform(0.2, 0.8, (nz, ny, nx))
    out = []
    for form, order in FORMS:
        s = _solver(shape, storage, Q, walls, (2e-5, -1e-5, 3e-5))
        s.enable_two_phase(0.03, 4.0, 0.1, **(dict(rho=(0.5, 1.5), tau=(0.65, 1.7))
                                              if phase == "contrast" else {}))
        s.set_phase(phi)
        _set(s, form, order)
        s.step(3)
        out.append(s.moments_host())
        s.close()
    assert group_rel_err(out[1], out[0]) <= 10 * TOL[storage]
    assert np.array_equal(out[1], out[2])


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("Q", [19, 27])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("walls,field", [(False, True), (True, True), (True, False)])
def test_adjoint_step(storage, Q, shape, walls, field):
    import torch
    if walls and shape[1] < 2:
        pytest.skip("a walled axis needs >= 2 sites")
    say(f"one-plane form, adjoint {storage} Q{Q} {shape} walls={walls} field={field}")
    nx, ny, nz = shape
    lam = torch.as_tensor(np.random.default_rng(9).standard_normal((10, nz, ny, nx)), device="cuda")
    out = []
    for form, order in FORMS:
        s = _solver(shape, storage, Q, walls, (2e-5, -1e-5, 3e-5))
        if field:
            _field(s, shape)
        _set(s, form, order)
        ck = s.forward_checkpointed(3, 2)
        gF, l0 = s.adjoint(3, 2, ck, lam)
        out.append((gF.double().cpu().numpy(), l0.double().cpu().numpy()))
        s.close()
    for march, one, again in zip(*out):
        assert np.abs(one - march).max() <= TOL[storage] * np.abs(march).max()
        assert np.array_equal(one, again)


@pytest.mark.parametrize("storage", ["f16s", "bf16s", "f16su"])
def test_16bit_storage_has_no_one_plane_form(storage):
    from paper_2609_09160_amd import LbfastError, Solver
    s = Solver((8, 8, 8), 0.8, storage=storage)
    with pytest.raises(LbfastError):
        _lib.check(s.lib.lbfast_set_form(s.h, _lib.LBF_FORM_ONE_PLANE))
    _lib.check(s.lib.lbfast_set_form(s.h, _lib.LBF_FORM_MARCH))
    s.close()
