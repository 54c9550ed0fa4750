"""What the library launches by default, form by form (no GPU needed)."""
import ctypes

import pytest

from launch_util import CONTRAST, EQUAL, default_launch
from paper_2609_09160_amd import _lib

SMALL = [(1, 1, 1), (5, 3, 1), (64, 4, 2), (65, 5, 3), (127, 2, 5), (32, 32, 32)]


@pytest.mark.parametrize("shape", SMALL)
@pytest.mark.parametrize("Q", [19, 27, "27h"])
@pytest.mark.parametrize("storage", ["f32", "f64"])
def test_small_grids_take_the_one_plane_form(shape, Q, storage):
    kinds = [{}, {"field": True}, {"phase": EQUAL}, {"phase": CONTRAST}]
    if Q != "27h":
        kinds.append({"field": True, "what": _lib.LBF_LAUNCH_ADJOINT})
    for kind in kinds:
        got = default_launch(shape, Q, storage, **kind)
        assert got["one_plane"] == 1 and got["z_chunk"] == 1 and got["lane_sites"] == 1, kind
        nx, ny, nz = shape
        assert got["blocks"] == -(-nx // 64) * -(-ny // got["tile_rows"]) * nz


@pytest.mark.parametrize("storage", ["f16s", "bf16s", "f16su"])
@pytest.mark.parametrize("shape", SMALL)
def test_16bit_storage_marches(storage, shape):
    assert default_launch(shape, 19, storage)["one_plane"] == 0


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("what", [_lib.LBF_LAUNCH_STEP, _lib.LBF_LAUNCH_ADJOINT])
def test_large_grids_march(storage, what):
    assert default_launch((192, 192, 192), 19, storage, field=True, what=what)["one_plane"] == 0


def test_what_cannot_be_launched_is_refused():
    out = _lib.LbfastLaunchInfo()
    lib = _lib.load()

    def rc(what, field=0, **kw):
        p = _lib.make_params((8, 8, 8), 0.8, **kw)
        return lib.lbfast_default_launch(ctypes.byref(p), 0, field, None, what, ctypes.byref(out))

    assert rc(_lib.LBF_LAUNCH_STEP) == _lib.LBF_OK
    assert rc(99) == _lib.LBF_E_ARG
    assert rc(_lib.LBF_LAUNCH_ADJOINT, storage="f16s") == _lib.LBF_E_UNSUPPORTED
    assert rc(_lib.LBF_LAUNCH_ADJOINT, lattice="27h") == _lib.LBF_E_UNSUPPORTED
    assert lib.lbfast_default_launch(None, 0, 0, None, 0, ctypes.byref(out)) == _lib.LBF_E_ARG
    assert lib.lbfast_set_form(None, 1) == _lib.LBF_E_ARG


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s", "bf16s", "f16su"])
@pytest.mark.parametrize("what", [_lib.LBF_LAUNCH_SET_F64, _lib.LBF_LAUNCH_SET_F32,
                                  _lib.LBF_LAUNCH_GET_F64, _lib.LBF_LAUNCH_GET_F32])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 7), (512, 512, 512), (1000, 1000, 858),
                                   (1000, 1000, 859),
                                   (1024, 1024, 1024), (1201, 1200, 1200), (1580, 1590, 1590)])
def test_whole_state_conversions_stay_within_the_launch_limit(storage, what, shape):
    """HIP takes fewer than 2^32 work-items per launch; larger states go plane
    by plane.  Every launch covers its state."""
    got = default_launch(shape, 19, storage, what=what)
    n = shape[0] * shape[1] * shape[2]
    assert got["blocks"] * got["block_threads"] < 2 ** 32
    wide = storage == "f64" if what <= _lib.LBF_LAUNCH_SET_F32 else what == _lib.LBF_LAUNCH_GET_F64
    per = (2 if wide else 4) if storage in ("f64", "f32") else (1 if n % 2 else 2)
    items = 10 * n if storage in ("f64", "f32") else n
    if got["blocks"]:
        assert got["blocks"] * got["block_threads"] * per >= items
    else:
        assert items / per > 2 ** 32 - 512


@pytest.mark.parametrize("storage,phase,shape,most,least", [
    ("f32", EQUAL, (256, 256, 256), 32, 512), ("f16s", EQUAL, (256, 256, 256), 32, 512),
    ("f32", EQUAL, (256, 64, 400), 17, 384), ("f32", EQUAL, (128, 128, 128), 8, 256),
    ("f64", EQUAL, (128, 128, 128), 8, 256), ("f32", CONTRAST, (128, 128, 128), 8, 256),
    ("f64", CONTRAST, (256, 256, 256), 64, 256)])
def test_force_march_keeps_the_device_busy(storage, phase, shape, most, least):
    """The chunks are no longer, and the workgroups no fewer, than those that
    the times of a sweep over chunk lengths ask for."""
    got = default_launch(shape, 19, storage, phase=phase, what=_lib.LBF_LAUNCH_FORCE)
    assert got["z_chunk"] <= most and got["blocks"] >= least, got


@pytest.mark.parametrize("storage,Q,shape,rows", [("f64", 27, (64, 64, 64), 4),
                                                  ("f32", 27, (16, 32, 72), 0),
                                                  ("f32", 19, (16, 168, 24), 0),
                                                  ("f32", 19, (128, 128, 128), 8),
                                                  ("f64", 19, (96, 96, 96), 6)])
def test_adjoint_shapes_in_the_cache(storage, Q, shape, rows):
    """The adjoint step has no kernels with plain stores: shapes and forms are
    compared with their stores counted (0: one plane per workgroup).  The one
    that a sweep found to be the fastest, by 6% or more."""
    got = default_launch(shape, Q, storage, field=True, what=_lib.LBF_LAUNCH_ADJOINT)
    assert got["plain_stores"] == got["one_plane"]
    assert (0 if got["one_plane"] else got["tile_rows"]) == rows


@pytest.mark.parametrize("storage,Q,shape,equal,contrast", [
    ("f32", 19, (201, 97, 113), 1, 1), ("f32", 27, (180, 90, 60), 1, 1),
    ("f64", 19, (100, 100, 100), 1, 1), ("f64", 27, (64, 200, 100), 1, 1),
    ("f64", 19, (128, 128, 128), 1, 0), ("f64", 19, (256, 256, 256), 1, 0),
    ("f64", 27, (512, 256, 100), 1, 0), ("f32", 27, (256, 256, 256), 0, 0),
    ("f64", 27, (256, 256, 256), 0, 0), ("f16s", 19, (112, 112, 112), 0, 0)])
def test_block_order_of_the_two_component_step(storage, Q, shape, equal, contrast):
    """Contiguous where the state is in the last-level cache, and for FP64 with
    equal properties and D3Q19 or many columns beyond it; 16-bit storage keeps
    the hardware's order."""
    assert default_launch(shape, Q, storage, phase=EQUAL)["contiguous"] == equal
    assert default_launch(shape, Q, storage, phase=CONTRAST)["contiguous"] == contrast


@pytest.mark.parametrize("storage,Q,shape,kind,one_plane", [
    ("f64", 19, (176, 256, 8), {"field": True}, 0), ("f32", 19, (192, 232, 24), {"field": True}, 0),
    ("f32", 19, (61, 253, 170), {"phase": CONTRAST}, 0),
    ("f32", 19, (224, 184, 32), {"phase": CONTRAST}, 0), ("f32", 19, (248, 232, 16), {}, 0),
    ("f32", 27, (16, 72, 48), {"field": True}, 1), ("f32", 27, (16, 56, 104), {}, 1),
    ("f32", 19, (8, 56, 112), {"field": True}, 1), ("f32", 27, (16, 24, 296), {}, 1)])
def test_one_plane_form_against_its_memory_time(storage, Q, shape, kind, one_plane):
    """The form that both forms' times name, by 15% or more: the one-plane form
    reads three planes for one, which decides on larger grids."""
    assert default_launch(shape, Q, storage, **kind)["one_plane"] == one_plane


@pytest.mark.parametrize("what,phase", [(_lib.LBF_LAUNCH_STEP, None),
                                        (_lib.LBF_LAUNCH_ADJOINT, None),
                                        (_lib.LBF_LAUNCH_PHASE, EQUAL),
                                        (_lib.LBF_LAUNCH_FORCE, EQUAL)])
@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("shape", [(64, 64, 64), (128, 128, 128), (160, 150, 140)])
def test_a_partition_with_fewer_compute_units(what, phase, storage, shape):
    """A device partition of 32 compute units gets no more workgroups than the
    whole device, and chunks at least as long."""
    whole = default_launch(shape, 19, storage, phase=phase, what=what)
    part = default_launch(shape, 19, storage, phase=phase, what=what, cus=32)
    assert default_launch(shape, 19, storage, phase=phase, what=what, cus=256) == whole
    assert part["blocks"] <= whole["blocks"] and part["z_chunk"] >= whole["z_chunk"]
    assert part["blocks"] < whole["blocks"]
