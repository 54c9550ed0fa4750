"""set_moments and moments of whole states in device memory (one pass over
the state) against the plane-by-plane route that host arrays take."""
import numpy as np
import pytest

from gpu_util import say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s", "bf16s", "f16su"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 7), (2, 9, 11), (64, 8, 4), (33, 31, 40)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_whole_state_equals_planes(storage, shape, dtype):
    """Odd and even site counts, one to many workgroups: the stored bytes after
    set_moments from a device array equal those from a host array, and a device
    read-out equals a host one, bit for bit; so does a device array that is
    not 16-byte aligned."""
    import torch
    from paper_2609_09160_amd import Solver
    nx, ny, nz = shape
    say(f"state io {storage} {shape} {np.dtype(dtype)}")
    m = inputs.random_state(shape, seed=nx + ny).astype(dtype)
    kw = dict(storage=storage, scale=[2.0 ** -13] * 10 if "16" in storage else None)
    a, b, c = (Solver(shape, 0.7, **kw) for _ in range(3))
    a.set_moments(m)
    dev = torch.as_tensor(m, device="cuda")
    b.set_moments(dev)
    shifted = torch.empty(m.size + 1, dtype=dev.dtype, device="cuda")[1:].view(dev.shape)
    shifted.copy_(dev)
    c.set_moments(shifted)
    assert torch.equal(a._bufs[0], b._bufs[0])
    assert torch.equal(a._bufs[0], c._bufs[0])
    want = a.moments_host(dtype=dtype)
    got = b.moments(dtype=dev.dtype).cpu().numpy()
    odd = torch.empty(m.size + 1, dtype=dev.dtype, device="cuda")[1:].view(dev.shape)
    assert np.array_equal(got, want)
    assert np.array_equal(c.moments(out=odd).cpu().numpy(), want)
    for s in (a, b, c):
        s.close()


@pytest.mark.parametrize("storage,quarter", [("f32", (128, 128, 32)), ("f64", (64, 40, 6))])
def test_phase_update_in_tall_and_low_tiles(storage, quarter):
    """A droplet in a quarter box along z (4-row tiles, short chunks) and four
    of them in one box (FP32: 16-row tiles): three steps keep the quarters equal
    to the small box, to 4 ulp of the largest value per step."""
    import torch
    from paper_2609_09160_amd import Solver
    nx, ny, nz = quarter
    r = np.sqrt(sum((np.arange(n).reshape(v) - n / 2.0) ** 2
                    for n, v in ((nz, (-1, 1, 1)), (ny, (1, -1, 1)), (nx, (1, 1, -1)))))
    phi = 0.5 * (1.0 - np.tanh((r - 0.3 * min(quarter)) / 2.0))
    m0 = inputs.random_state(quarter, seed=3)
    out = []
    for n in (1, 4):
        s = Solver((nx, ny, nz * n), 1.0, storage=storage)
        s.set_moments(np.concatenate([m0] * n, axis=1))
        s.enable_two_phase(0.03, 4.0, 0.1)
        s.set_phase(np.concatenate([phi] * n, axis=0))
        s.step(3)
        out.append((s.moments_host(), s.phase(dtype=torch.float64).cpu().numpy()))
        s.close()
    eps = 12 * (2.0 ** -24 if storage == "f32" else 2.0 ** -53)
    for small, big in zip(*out):
        top = np.abs(small).max()
        for q in range(4):
            part = big[..., q * nz:(q + 1) * nz, :, :]
            assert np.abs(part - small).max() <= eps * max(top, 1.0)
