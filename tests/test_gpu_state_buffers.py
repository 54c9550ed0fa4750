"""Which of the two state buffers holds the current state: a program that
recorded launches (a captured graph of steps) relies on it."""
import pytest

from gpu_util import say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu
SHAPE = (33, 9, 7)


@pytest.mark.parametrize("nsteps,every", [(1, 3), (2, 2), (3, 2), (4, 2), (6, 2), (7, 2), (6, 3),
                                          (7, 3), (10, 3), (5, 9)])
def test_checkpointed_run_ends_where_steps_end(nsteps, every):
    """A checkpointed run of n steps leaves the state in the buffer that n
    plain steps leave it in."""
    from paper_2609_09160_amd import Solver
    say(f"final buffer {nsteps} steps every {every}")
    s = Solver(SHAPE, 0.8)
    s.set_moments(inputs.random_state(SHAPE, seed=4))
    at = [b.data_ptr() for b in s._bufs]
    first = at.index(s.state_ptr())
    s.forward_checkpointed(nsteps, every)
    assert at.index(s.state_ptr()) == first ^ (nsteps & 1)
    s.close()


def test_captured_steps_after_a_checkpointed_run():
    """Two steps captured in a graph, replayed with checkpointed runs between:
    each replay advances the current state, bit for bit as plain steps do."""
    import torch
    from paper_2609_09160_amd import Solver
    say("captured steps after checkpointed runs")
    m0 = inputs.random_state(SHAPE, seed=4)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s = Solver(SHAPE, 0.8)
        s.set_moments(m0)
        s.step(2)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            s.step(2)
    ref = Solver(SHAPE, 0.8)
    ref.set_moments(m0)
    ref.step(2)
    for nsteps, every in ((4, 2), (6, 3), (6, 2), (2, 5)):
        with torch.cuda.stream(side):
            graph.replay()
            s.forward_checkpointed(nsteps, every)
            graph.replay()
        side.synchronize()
        ref.step(2 + nsteps + 2)
        assert torch.equal(s.moments(), ref.moments()), (nsteps, every)
    s.close()
    ref.close()
