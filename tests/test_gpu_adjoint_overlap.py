"""lambda_T and lambda0 in memory that the gradient also uses for its
checkpoints, recomputed states or force: the gradients are those of arrays of
their own, bit for bit."""
import ctypes

import pytest

from gpu_util import say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu
SHAPE = (32, 9, 7)  # 40 N and 80 N are multiples of 16: every slot is aligned


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("nsteps,every", [(1, 1), (1, 2), (2, 2), (3, 1), (5, 2), (6, 3)])
@pytest.mark.parametrize("where", ["work 0", "work 1", "lambda 0", "lambda 1"])
def test_lambda_T_in_the_work_area(storage, nsteps, every, where):
    _check(storage, nsteps, every, T=where)


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("nsteps,every", [(1, 1), (1, 2), (2, 2), (3, 1), (5, 2), (6, 3)])
@pytest.mark.parametrize("where", ["work 0", "lambda 0", "lambda 1", "checkpoint 0",
                                   "checkpoint 1", "force"])
def test_lambda_0_over_what_is_read(storage, nsteps, every, where):
    _check(storage, nsteps, every, zero=where)


def _check(storage, nsteps, every, T=None, zero=None):
    import torch
    from paper_2609_09160_amd import Solver, _lib
    say(f"overlap {storage} {nsteps}/{every} T={T} 0={zero}")
    s = Solver(SHAPE, 0.8, storage=storage)
    dt, N, nb = s.compute_dtype, s.N, s.buffer_bytes()
    # the force field at the head of an array that a whole state fits in
    room = torch.zeros(10 * N, dtype=dt, device="cuda")
    room[:3 * N] = torch.as_tensor(inputs.random_force(SHAPE, seed=3, std=1e-4),
                                   device="cuda").to(dt).reshape(-1)
    s.set_force_field(room[:3 * N])
    s.set_moments(inputs.random_state(SHAPE, seed=4))
    g = torch.Generator(device="cuda").manual_seed(7)
    lam = torch.randn(10 * N, generator=g, device="cuda", dtype=dt)
    ck = s.forward_checkpointed(nsteps, every)
    gF_ref, l0_ref = s.adjoint(nsteps, every, ck, lam)
    ck = torch.cat([ck, torch.zeros(2 * nb, dtype=torch.uint8, device="cuda")])
    work = torch.zeros((every + 2) * nb, dtype=torch.uint8, device="cuda")
    gF = torch.empty(3 * N, dtype=dt, device="cuda")

    def array(where):
        if where is None:
            return torch.empty(10 * N, dtype=dt, device="cuda")
        if where == "force":
            return room
        kind, k = where.split()
        k = int(k) + (every if kind == "lambda" else 0)
        return (ck if kind == "checkpoint" else work)[k * nb:(k + 1) * nb].view(dt)

    lT, l0 = array(T), array(zero)
    lT.copy_(lam)
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    torch.cuda.synchronize()
    _lib.check(s.lib.lbfast_adjoint(s.h, nsteps, every, p(ck), p(lT), p(gF), p(l0), p(work)))
    s.sync()
    assert torch.equal(gF, gF_ref.reshape(-1))
    assert torch.equal(l0, l0_ref.reshape(-1))
    s.close()
