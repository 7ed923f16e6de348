"""Options of a context on the direct kernels: reading one, or setting it and
setting it back, leaves the products of the context as they were."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2403_19854_amd import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda"


def fc():
    from paper_2403_19854_amd import fcrkpm
    return fcrkpm


def options(f):
    return [getattr(f, k) for k in sorted(dir(f)) if k.startswith("OPT_")]


@pytest.mark.parametrize("n,at,degree", [(128, 3.5, 1), (64, 3.5, 2)])
def test_kernels_do_not_depend_on_options_read(n, at, degree):
    """The kernel of a product follows from the geometry alone, also on the
    boxes whose FFT passes hold records of their own (the register path)."""
    print(f"\n[options {n}^3 support {at} degree {degree}]", flush=True)
    f = fc()
    p = W.cube(3, n, at, degree)
    g = f.Problem.from_workload(p, device=DEV)
    x = torch.from_numpy(np.random.default_rng(5).standard_normal(p.shape)).to(DEV)
    x32 = x.float()
    r = torch.from_numpy(p.r).to(DEV)

    def kinds():
        g.profile(True)
        k = g.apply("K", x32)
        g.profile(False)
        return k, sorted(g.profile_read())

    cg = lambda: g.solve(r, mode="f32_refined", tol=1e-14, maxit=12, raise_on_noconv=False)[0]
    k, kd = kinds()
    d = cg()
    assert kd == ["tap_k_f32"]
    k64 = g.apply("K", x)
    assert float((k.double() - k64).abs().max() / k64.abs().max()) <= 2e-5
    for opt in options(f):
        g.get_option(opt)
        again, kd = kinds()
        assert kd == ["tap_k_f32"] and torch.equal(again, k), opt
    for opt in (f.OPT_TAPS, f.OPT_REGPATH, f.OPT_LINECONST):
        g.set_option(opt, 0)
        g.set_option(opt, 1)
        again, kd = kinds()
        assert kd == ["tap_k_f32"] and torch.equal(again, k), opt
    assert torch.equal(cg(), d)
    g.close()
