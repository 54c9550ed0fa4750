"""Where the checkpointed forward run and the adjoint keep their states: the
slots, the caller's lambda arrays and the handle's own state."""
import ctypes

import numpy as np
import pytest

from gpu_util import say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu
SHAPE = (33, 9, 7)


def _solver(storage="f32"):
    import torch
    from paper_2609_09160_amd import Solver
    s = Solver(SHAPE, 0.8, storage=storage)
    F = torch.as_tensor(inputs.random_force(SHAPE, seed=3, std=1e-4), device="cuda",
                        dtype=s.compute_dtype)
    s.set_force_field(F)
    s.set_moments(inputs.random_state(SHAPE, seed=4))
    return s


@pytest.mark.parametrize("nsteps,every", [(1, 2), (2, 2), (3, 2), (6, 2), (6, 3), (7, 3), (5, 9)])
def test_checkpoints_are_the_states(nsteps, every):
    """Slot k holds the state at t = k every, and the handle the final one, bit
    for bit those of a plain run."""
    import torch
    say(f"checkpoints {nsteps} steps every {every}")
    a, b = _solver(), _solver()
    nb = a.buffer_bytes()
    ck = a.forward_checkpointed(nsteps, every)
    for t in range(nsteps + 1):
        state = b.moments(dtype=torch.float32).view(torch.uint8).reshape(-1)
        if t < nsteps and t % every == 0:
            k = t // every
            assert torch.equal(ck[k * nb:(k + 1) * nb], state), t
        if t < nsteps:
            b.step(1)
    assert torch.equal(a.moments(dtype=torch.float32), b.moments(dtype=torch.float32))
    a.close()
    b.close()


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("nsteps,every", [(1, 1), (1, 3), (2, 1), (5, 2)])
@pytest.mark.parametrize("how", ["apart", "one array", "unaligned"])
def test_lambda_arrays_where_they_lie(storage, nsteps, every, how):
    """lambda_T and lambda0 as separate arrays, as one array, and off a 16-byte
    boundary: the same gradients bit for bit, and lambda_T left as it was
    where it is an array of its own."""
    import torch
    from paper_2609_09160_amd import _lib
    say(f"lambda {storage} {nsteps}/{every} {how}")
    s = _solver(storage)
    dt, n = s.compute_dtype, 10 * s.N
    g = torch.Generator(device="cuda").manual_seed(7)
    lam = torch.randn(n, generator=g, device="cuda", dtype=dt)
    ck = s.forward_checkpointed(nsteps, every)
    gF_ref, l0_ref = s.adjoint(nsteps, every, ck, lam)
    pad = 1 if how == "unaligned" else 0
    lT = torch.empty(n + pad, dtype=dt, device="cuda")[pad:]
    lT.copy_(lam)
    l0 = lT if how == "one array" else torch.empty(n + pad, dtype=dt, device="cuda")[pad:]
    gF = torch.empty(3 * s.N, dtype=dt, device="cuda")
    work = torch.empty(s.lib.lbfast_adjoint_work_bytes(s.h, every), dtype=torch.uint8,
                       device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    _lib.check(s.lib.lbfast_adjoint(s.h, nsteps, every, p(ck), p(lT), p(gF), p(l0), p(work)))
    s.sync()
    assert np.array_equal(gF.cpu().numpy(), gF_ref.cpu().numpy().reshape(-1))
    assert np.array_equal(l0.cpu().numpy(), l0_ref.cpu().numpy().reshape(-1))
    if how != "one array":
        assert torch.equal(lT, lam)
    s.close()
