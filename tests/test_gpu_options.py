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


def test_lines_of_a_box_that_is_not_timed():
    """The stored default is the choice that gives the direct kernels back."""
    f = fc()
    h, chi = (1.0 / 96, 1.0 / 72), np.ones((72, 96), np.uint8)
    chi[-3:], chi[:, -3:] = 0, 0
    g = f.Problem((96, 72), h, (2.5, 2.5), 1, chi, None, None, device=DEV)
    for opt in (f.OPT_SEP_LINES32, f.OPT_SEP_LINES64):
        assert g.get_option(opt) == 4
        g.set_option(opt, 16)
        assert g.get_option(opt) == 16 and g.get_option(f.OPT_TAPS) == 0
        g.set_option(opt, 4)
        assert g.get_option(f.OPT_TAPS) == 1
    g.close()


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


def test_reading_an_option_builds_nothing():
    """What setup stored is returned as it is: no device memory is taken, and
    the values that were read give the choice back when they are set."""
    f = fc()
    p = W.cube(3, 128, 2.5, 1)
    g = f.Problem.from_workload(p, device=DEV)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    stored = [f.OPT_GRAPHS, f.OPT_REGPATH, f.OPT_REGLAYOUT, f.OPT_TUNE_NS0, f.OPT_TUNE_NS1, f.OPT_TUNE_NS2,
              f.OPT_TUNE_NS3, f.OPT_SEP_LINES32, f.OPT_SEP_LINES64, f.OPT_TUNE_CACHED, f.OPT_TAPS]
    value = {opt: g.get_option(opt) for opt in stored}
    assert torch.cuda.mem_get_info()[0] == free
    assert value[f.OPT_TUNE_NS1] == 0 and value[f.OPT_SEP_LINES32] == 16 and value[f.OPT_TAPS] == 1
    for opt, other in ((f.OPT_REGLAYOUT, 1 - value[f.OPT_REGLAYOUT]), (f.OPT_SEP_LINES32, 8), (f.OPT_SEP_LINES64, 4)):
        g.set_option(opt, other)
        assert g.get_option(f.OPT_TAPS) == 0 and g.get_option(opt) == other
        g.set_option(opt, value[opt])
        assert g.get_option(f.OPT_TAPS) == 1 and g.get_option(opt) == value[opt]
    g.close()


def test_options_read_during_a_capture():
    """A capture goes on while options are read, also those whose first read
    builds records."""
    f = fc()
    p = W.cube(3, 64, 2.5, 1)
    g = f.Problem.from_workload(p, device=DEV)
    x = torch.from_numpy(np.random.default_rng(6).standard_normal(p.shape)).to(DEV)
    ref = g.apply("K", x)
    a, b = torch.zeros_like(x), torch.zeros_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.apply("K", x, out=a)
        values = [g.get_option(opt) for opt in options(f)]
        g.apply("K", a, out=b)
    assert values == [g.get_option(opt) for opt in options(f)]
    second = g.apply("K", ref)
    for _ in range(3):
        a.zero_(), b.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(a, ref) and torch.equal(b, second)
        x.add_(0.0)
    g.close()


def test_a_refused_value_builds_nothing():
    """A value out of range is refused before anything is prepared for it."""
    f = fc()
    p = W.cube(3, 128, 2.5, 1)
    g = f.Problem.from_workload(p, device=DEV)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for opt, bad in ((f.OPT_REGLAYOUT, 2), (f.OPT_REGLAYOUT, 7), (f.OPT_REGLAYOUT, -1), (f.OPT_SEP_LINES32, 5),
                     (f.OPT_SEP_LINES64, 0), (f.OPT_TAPS, 2), (f.OPT_REGPATH, -1), (f.OPT_LINECONST, 3),
                     (f.OPT_GRAPHS, 2), (f.OPT_TUNE_NS0, 0), (99, 0)):
        with pytest.raises(f.FcrkpmError):
            g.set_option(opt, bad)
    assert torch.cuda.mem_get_info()[0] == free
    assert g.get_option(f.OPT_TAPS) == 1 and g.get_option(f.OPT_GRAPHS) == 1
    g.close()


def test_a_refused_flux_load_builds_nothing():
    """f^q without boundary areas is refused at once, also by the call that
    allocates nothing."""
    f = fc()
    p = W.cube(3, 64, 2.5, 1)
    g = f.Problem.from_workload(p, device="cuda:0")
    x = torch.ones(p.shape, dtype=torch.float64, device=DEV)
    x32, out = x.float(), torch.empty_like(x)
    out32 = out.float()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for v, o in ((x, out), (x32, out32)):
        for call in (g.apply, g.apply_noalloc):
            with pytest.raises(f.FcrkpmError, match="no boundary areas"):
                call("FQ", v, out=o)
    assert torch.cuda.mem_get_info()[0] == free
    g.close()


def test_direct_contexts_hold_no_workspace():
    """The nonlinear solvers and the lumped mass on the direct kernels leave a
    context with the device memory that setup gave it."""
    f = fc()
    p = W.cube(3, 96, 2.5, 1)
    r = torch.from_numpy(p.r).to(DEV)

    def calls(g):
        yield g.coeffs("lumped")
        for kind in ("cubic", "gradient"):
            yield g.solve_nonlinear_cg(r, 1.0, kind=kind, maxit=2, raise_on_noconv=False)[:2]
        yield g.solve_nonlinear(r, 1.0, maxnewton=1, maxit=8, raise_on_noconv=False)[:2]

    g = f.Problem.from_workload(p, device=DEV)
    kept = list(calls(g))  # the kernels are loaded and torch holds its blocks
    del kept
    g.close()
    g = f.Problem.from_workload(p, device=DEV)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for _ in calls(g):
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free
    g.close()


def fill_memory():
    """Tensors of 16 MB, and a large first one, that hold all device memory (the
    figure that the runtime reports as free is not all that it can still give)."""
    take = lambda nbytes: torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    hold = [take(torch.cuda.mem_get_info()[0] - (4 << 30))]
    try:
        for _ in range(4096):
            hold.append(take(16 << 20))
    except torch.OutOfMemoryError:
        return hold
    raise AssertionError("device memory has no end")


@pytest.mark.parametrize("uniform", [True, False])
def test_preparing_fft_passes_without_memory(uniform):
    """Out of device memory while the FFT passes are prepared: an error, the
    direct products go on, and a later attempt is as good as a first one.  The
    margins let the build stop at the register path's records, at the line
    records and at the workspace (201 MB)."""
    f = fc()
    p = W.cube(3, 128, 2.5, 1)
    vol = p.vol if uniform else p.vol * np.random.default_rng(8).uniform(0.5, 1.5, p.shape)
    make = lambda: f.Problem(p.dims, p.h, p.at, p.degree, p.chi, p.dirichlet, vol, device=DEV)
    x = torch.from_numpy(np.random.default_rng(9).standard_normal(p.shape)).to(DEV)
    x32 = x.float()
    outs = lambda: [torch.zeros_like(x32), torch.zeros_like(x), torch.zeros_like(x), torch.zeros_like(x)]

    def run(g, out):
        for op, v, o in zip(("K", "K", "UH", "FR"), (x32, x, x, x), out):
            g.apply(op, v, out=o)

    fft, direct = outs(), outs()
    g = make()
    g.set_option(f.OPT_TAPS, 0)
    run(g, fft)
    g.close()
    g = make()
    run(g, direct)
    margins = (64, 176) if uniform else (64, 128, 304)
    got = [outs() for _ in margins]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold, freed = fill_memory(), 0
    for margin, out in zip(margins, got):
        print(f"\n[options] {margin} MB free", flush=True)
        del hold[-((margin - freed) // 16):]
        freed = margin
        torch.cuda.empty_cache()
        with pytest.raises(f.FcrkpmError, match="FCRKPM_ERR_OOM"):
            g.set_option(f.OPT_TAPS, 0)
        assert g.get_option(f.OPT_TAPS) == 1
        run(g, out)
    del hold
    torch.cuda.empty_cache()
    for out in got:
        assert all(torch.equal(a, b) for a, b in zip(out, direct))
    g.set_option(f.OPT_TAPS, 0)
    out = outs()
    run(g, out)
    assert all(torch.equal(a, b) for a, b in zip(out, fft))
    assert g.get_option(f.OPT_LINECONST) == g.get_option(f.OPT_KN_REGPATH) == int(uniform)
    g.close()
