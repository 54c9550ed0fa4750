"""Whole states in device arrays that start on a 16-byte boundary and no wider
one, the least that the one-pass conversions ask for."""
import numpy as np
import pytest

from gpu_util import say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s", "bf16s", "f16su"])
@pytest.mark.parametrize("shape", [(3, 5, 7), (64, 8, 4)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_arrays_on_16_byte_boundaries(storage, shape, dtype):
    import torch
    from paper_2609_09160_amd import Solver
    say(f"16-byte boundary {storage} {shape} {np.dtype(dtype)}")
    m = inputs.random_state(shape, seed=2).astype(dtype)
    kw = dict(storage=storage, scale=[2.0 ** -13] * 10 if "16" in storage else None)
    a, b = Solver(shape, 0.7, **kw), Solver(shape, 0.7, **kw)
    a.set_moments(m)
    pad = 16 // m.itemsize

    def shifted():
        t = torch.empty(m.size + pad, device="cuda", dtype=torch.from_numpy(m).dtype)[pad:]
        assert t.data_ptr() % 32 == 16
        return t.view(m.shape)

    src, out = shifted(), shifted()
    src.copy_(torch.from_numpy(m))
    b.set_moments(src)
    assert torch.equal(a._bufs[0], b._bufs[0])
    assert np.array_equal(b.moments(out=out).cpu().numpy(), a.moments_host(dtype=dtype))
    a.close()
    b.close()
