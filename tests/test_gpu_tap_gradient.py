"""The implicit gradient B d of the direct kernels.  No C entry returns it
(the nonlinear solver's line search reads it on the domain), so the library's
own launcher is called by its C++ name."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_taps import DEV, domain, fc

pytestmark = pytest.mark.gpu

# launch_tap<double, double>(Ctx, mode, in, out, mask_in, mask_out, rows, vol, nrhs, stream, cg)
LAUNCH = "_ZN6fcrkpm10launch_tapIddEEvRKNS_3CtxEiPKT0_PS4_PKhS9_PKT_SC_iP12ihipStream_tPKNS_5TapCgE"
GRADIENT = 4


@pytest.mark.parametrize("dims,at,degree", [((70, 48), 2.5, 1), ((36, 35), 3.0, 2), ((40, 36), 4.0, 3),
                                            ((36, 30, 28), 2.5, 1), ((72, 56, 40), 3.0, 2), ((35, 16, 18), 3.5, 2)])
def test_every_component_is_written_at_every_node(dims, at, degree):
    """A ball leaves planes of its tile columns, and whole columns, outside the
    domain: the gradient is zero there in every component.  Its energy is
    d . K d (Eq 57): terms of one sign, so the sums agree to rounding."""
    print(f"\n[taps gradient] {dims} support {at} degree {degree}", flush=True)
    f = fc()
    h, chi, dirichlet, vol = domain(dims, at, "ball")
    g = f.Problem(dims, h, (at,) * len(dims), degree, chi, dirichlet, vol, device=DEV)
    ba = g.coeffs("balpha")
    mask = torch.from_numpy(chi).to(DEV)
    d = torch.from_numpy(np.random.default_rng(11).standard_normal(chi.shape)).to(DEV)
    launch = getattr(f.load_library(), LAUNCH)
    launch.restype = None
    ptr = lambda t: C.c_void_p(t.data_ptr())

    def gradient(fill):
        out = torch.full((len(dims),) + chi.shape, fill, dtype=torch.float64, device=DEV)
        launch(g._h, C.c_int(GRADIENT), ptr(d), ptr(out), ptr(mask), None, ptr(ba), None, C.c_int(1),
               C.c_void_p(torch.cuda.current_stream().cuda_stream), None)
        torch.cuda.synchronize()
        return out

    got = gradient(float("nan"))
    assert torch.equal(got, gradient(0.0))
    assert bool((got[:, mask == 0] == 0.0).all())
    # |V^(1/2) B d|^2 = d . K_FULL d, summed over the nodes
    energy = float((torch.from_numpy(vol).to(DEV) * (got * got).sum(0)).sum())
    dm = torch.where(mask > 0, d, 0.0)
    ref = float((dm * g.apply("K_FULL", dm)).sum())
    print(f"  energy {energy:.12e} against {ref:.12e}", flush=True)
    assert abs(energy - ref) <= 1e-11 * ref
