"""The launch shapes that the library chooses by itself, and the forms that
only large states take (non-temporal stores with one site per lane)."""
import numpy as np
import pytest

from gpu_util import gpu_run, group_rel_err, lattice_number, oracle_run, say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu

# chunks of one and two planes, single tiles with idle lanes and rows, a tail
# in every direction, and enough columns for tall tiles and contiguous order
SHAPES = [(1, 1, 1), (3, 2, 1), (8, 40, 8), (65, 9, 2), (33, 17, 5), (96, 30, 7), (131, 45, 37),
          (192, 26, 11)]


@pytest.mark.parametrize("Q", [19, 27, "27h"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("walls", [False, True])
def test_default_shape_fp64(Q, shape, walls):
    """The default launch against the oracle: off-equilibrium random state,
    uniform force, 5 steps, FP64: <= 1e-12 of each moment group."""
    if walls and shape[1] < 2:
        pytest.skip("a walled axis needs >= 2 sites")
    bc = (0, 1 if walls else 0, 0)
    m0 = inputs.random_state(shape, seed=sum(shape) + lattice_number(Q))
    F = (2e-5, -1e-5, 3e-5)
    say(f"default shape fp64 Q{Q} {shape} walls={walls}")
    got = gpu_run(shape, 0.7, m0, 5, lattice=Q, bc=bc, force=F)
    want = oracle_run(shape, 0.7, m0, 5, lattice=Q, bc=bc, force=np.array(F))
    assert group_rel_err(got, want) <= 1e-12


@pytest.mark.parametrize("storage,shape", [("f32", (161, 160, 120)), ("f16s", (161, 160, 240)),
                                           ("f64", (161, 80, 120))])
@pytest.mark.parametrize("rows", [6, 8, 14])
def test_states_beyond_the_cache(storage, shape, rows):
    """States larger than the last-level cache holds twice (above 120 MB) take
    the forms with non-temporal stores; the same tiles on a quarter of the grid
    take those with plain stores.  A field of four equal quarters along z,
    advanced 3 steps, has to give the small grid's state four times: the same
    formulas compiled twice, so within 4 ulp of the largest value of the state
    per step (FP32 and FP64), and the same 16-bit words but for values that
    fall on the other side of a rounding (one unit of binary16 there)."""
    nx, ny, nz = shape
    small = (nx, ny, nz // 4)
    m0 = inputs.random_state(small, seed=rows)
    kw = dict(storage=storage, launch=(rows, 8, 1))
    if storage == "f16s":
        kw["scale"] = [2.0 ** -13] * 4 + [2.0 ** -16] * 6
    say(f"beyond the cache {storage} {shape} rows={rows}")
    want = gpu_run(small, 0.7, m0, 3, **kw)
    got = gpu_run(shape, 0.7, np.concatenate([m0] * 4, axis=1), 3, **kw)
    top = np.abs(want).max()
    tol = {"f32": 12 * 2.0 ** -24, "f64": 12 * 2.0 ** -53, "f16s": 2.0 ** -10}[storage] * top
    for q in range(4):
        part = got[:, q * (nz // 4):(q + 1) * (nz // 4)]
        assert np.abs(part - want).max() <= tol


@pytest.mark.parametrize("storage,Q,shape", [("f32", 27, (201, 97, 113)), ("f32", 19, (48, 48, 48)),
                                             ("f64", 19, (152, 247, 151)), ("f16s", 19, (112, 112, 112))])
def test_block_orders_agree_on_default_shapes(storage, Q, shape):
    """The workgroup order does not move the default launch shape: automatic
    and explicit orders give bitwise the same state."""
    from paper_2609_09160_amd import Solver
    m0 = inputs.random_state(shape, seed=sum(shape) + Q)
    out = []
    for order in (0, 1, 2):
        s = Solver(shape, 0.65, lattice=Q, storage=storage)
        s.set_block_order(order)
        s.set_moments(m0)
        s.step(3)
        out.append(s.moments_host())
        s.close()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
