"""What the library launches by default, as plain values."""
import ctypes

from paper_2609_09160_amd import _lib

EQUAL = dict(rho=(1.0, 1.0), tau=(0.8, 0.8))
CONTRAST = dict(rho=(0.5, 1.5), tau=(0.65, 1.7))


def default_launch(shape, Q=19, storage="f32", walls=False, force=(0.0, 0.0, 0.0), field=False,
                   phase=None, what=_lib.LBF_LAUNCH_STEP, cus=0):
    p = _lib.make_params(shape, 0.8, lattice=Q, storage=storage, bc=(0, int(walls), 0), force=force)
    pp = None
    if phase is not None:
        pp = _lib.LbfastPhaseParams()
        pp.struct_size = ctypes.sizeof(pp)
        pp.sigma, pp.width, pp.diffusivity = 0.03, 4.0, 0.1
        (pp.rho_l, pp.rho_h), (pp.tau_l, pp.tau_h) = phase["rho"], phase["tau"]
    out = _lib.LbfastLaunchInfo()
    _lib.check(_lib.load().lbfast_default_launch(ctypes.byref(p), cus, int(field),
                                                 ctypes.byref(pp) if pp else None, what,
                                                 ctypes.byref(out)))
    return {name: getattr(out, name) for name, _ in out._fields_}
