"""The register-resident FFT passes (`OPT_TAPS` 0) at every line length they
serve: the direct kernels run these supports by default, so the passes are asked
for here, in both precisions, with every operator and solver that has a form on
them.  Reference: the direct kernels' results, which the oracle pins
(test_gpu_taps.py); bars as between any two paths of the library (FP64 1e-12,
FP32 2e-5 of the largest value, refined solves 1e-8)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2403_19854_amd import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda"


def fc():
    from paper_2403_19854_amd import fcrkpm
    return fcrkpm


def rel(a, b):
    return float((a.double() - b.double()).abs().max() / b.double().abs().max())


@pytest.mark.parametrize("n,at", [(32, 2.5), (48, 1.5), (64, 2.0), (64, 3.5), (80, 2.5), (96, 2.5), (128, 2.5),
                                  (256, 2.5)])
def test_linear_basis(n, at):
    print(f"\n[register path {n}^3 support {at}]", flush=True)
    f = fc()
    p = W.cube(3, n, at, 1)
    g = f.Problem.from_workload(p, device=DEV)
    x = torch.from_numpy(np.random.default_rng(12).standard_normal((2,) + p.shape)).to(DEV)
    kappa = 0.8 * min(p.h) ** 2
    ops = [(op, t) for op in ("K", "K_FULL", "M") for t in (torch.float64, torch.float32)]
    ops += [("UH", torch.float64), ("FR", torch.float64)]
    r = torch.from_numpy(p.r).to(DEV)

    def results():
        g.profile(True)
        out = [g.apply(op, x.to(t)) for op, t in ops]
        out.append(g.gradient_force(x, kappa))
        g.profile(False)
        kinds = set(g.profile_read())
        # (three iterations: rounding has not grown yet)
        sol = [g.solve(r, mode=m, tol=1e-14, maxit=3, raise_on_noconv=False)[0] for m in ("f64", "f32_refined")]
        if n <= 64:
            sol += [g.transient(r, 1.0, 1e-4, 2, r=r, mode=m, tol=1e-14, maxit=3, raise_on_noconv=False)[0]
                    for m in ("f64", "f32_refined")]
        return out, sol, kinds

    direct, dsol, kinds = results()
    assert {"tap_k_f32", "tap_k_f64"} <= kinds and not any(k.startswith("sep_") for k in kinds)
    g.set_option(f.OPT_TAPS, 0)
    # (at support 3.5 more nodes of a line differ from its constant than the
    # line-constant pass corrects: records per element, FP64 on the LDS-tiled passes)
    lines = 1 if at < 3.0 else 0
    assert g.get_option(f.OPT_LINECONST) == lines and g.get_option(f.OPT_KN_REGPATH) == lines
    fft, fsol, kinds = results()
    assert {"sep_mid_k_f32", "sep_mid_k_f64"} <= kinds and not any(k.startswith("tap_") for k in kinds)
    for (op, t), a, b in zip(ops + [("gradient force", torch.float64)], fft, direct):
        e = rel(a, b)
        print(f"  {op} {t}: {e:.2e}", flush=True)
        assert e <= (1e-12 if t == torch.float64 else 2e-5)
    for k, (a, b) in enumerate(zip(fsol, dsol)):
        e = rel(a, b)
        print(f"  solve {k}: {e:.2e}", flush=True)
        assert e <= (1e-10 if k % 2 == 0 else 2e-4)
    g.close()


@pytest.mark.parametrize("n,at", [(64, 3.0), (128, 3.0)])
def test_quadratic_basis(n, at):
    print(f"\n[register path, quadratic ball in {n}^3]", flush=True)
    f = fc()
    p = W.sphere(n, 0.4, at, 2, seed=3)
    g = f.Problem.from_workload(p, device=DEV)
    x = torch.from_numpy(np.random.default_rng(13).standard_normal((2,) + p.shape)).to(DEV).float()
    direct = [g.apply("K", x), g.apply("K_FULL", x)]
    g.set_option(f.OPT_TAPS, 0)
    for a, b in zip([g.apply("K", x), g.apply("K_FULL", x)], direct):
        e = rel(a, b)
        print(f"  K {e:.2e}", flush=True)
        assert e <= 2e-5
    g.close()


def test_refined_solve_on_the_fused_passes():
    """The direction update in the first pass and the dot in the last."""
    f = fc()
    p = W.cube(3, 64, 2.0, 1)
    g = f.Problem.from_workload(p, device=DEV)
    r = torch.from_numpy(p.r).to(DEV)
    d, _, info = g.solve(r, mode="f32_refined", tol=1e-11)
    g.set_option(f.OPT_TAPS, 0)
    for graphs in (True, False):
        g.set_graphs(graphs)
        dr, _, inr = g.solve(r, mode="f32_refined", tol=1e-11)
        e = float((dr - d).norm() / d.norm())
        print(f"\n[register path solve] {e:.2e}; {info['iters']} and {inr['iters']} iterations", flush=True)
        assert e <= 1e-8
    g.close()
