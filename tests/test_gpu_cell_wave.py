"""The one-wave cell kernel (launches wide enough to fill the chip) against
the oracle, element by element on sampled columns.

The mesh is odd in two directions (three colours there) and a block holds an
odd number of columns, wide enough that every launch takes the one-wave
variant at every degree and precision: first and last column tiles, cells
that wrap around in each direction, and both halves of the FP64 planes.
Terms: K + V and the mass (apply_local), the filter's step (cheb_step_local)
and, through a degree-2 filter that forms its own residual, K + V - lambda M;
on the uniform mesh and on a two-level mesh without the GGA term."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NC = 16013   # cell columns per colour with one cell a colour: above every threshold


def _system(p, graded):
    from workloads.configs import custom_system, with_two_level_gga
    n = (3, 2, 3)
    box = tuple(1.6 * v for v in n)
    rng = np.random.Generator(np.random.PCG64(900 + p))
    pos = rng.uniform(0.0, 1.0, size=(2, 3)) * np.asarray(box)
    s = custom_system(n, box, p, p + 2, pos=pos, rcut=0.7, channels="spd8", wells=pos, s_H=0.5, s_S=0.4, seed=40 + p)
    return with_two_level_gga(s, r_fine=0.4, gga=False) if graded else s


def _sample():
    return np.concatenate([np.arange(6), [777, 8000], np.arange(NC - 9, NC)])


def _close(got, want, tol):
    assert np.max(np.abs(got - want).max(axis=0) / np.abs(want).max(axis=0)) <= tol


@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("p", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("prec", [0, 1])
def test_local_terms(p, graded, prec):
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    s = _system(p, graded)
    ref, op = PAWOperator(s), Operator(s)
    dt = torch.float64 if prec == 0 else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(p)
    draw = lambda d: torch.randn(op.ndof, NC, device="cuda", dtype=d, generator=g)  # noqa: E731
    X, Y, Y64 = draw(dt), draw(dt), draw(torch.float64)
    lam = torch.rand(NC, device="cuda", dtype=torch.float64, generator=g)
    j = torch.from_numpy(_sample()).cuda()
    host = lambda t: t[:, j].double().cpu().numpy()  # noqa: E731
    x, y, y64, ln = host(X), host(Y), host(Y64), lam[j].cpu().numpy()
    tol = 1e-12 if prec == 0 else 2e-5
    for which, apply in ((0, ref.loc.apply_H), (1, ref.loc.apply_M)):
        out = op.apply_local(X, Y.clone(), which=which, alpha=0.7, prec=prec)
        _close(host(out), y + 0.7 * apply(x), tol)
    a, ac, zz = 0.37, -0.81, 0.42
    out = op.cheb_step_local(X, Y.clone(), Y64, lam, a, ac, zz, prec=prec)
    _close(host(out), (-ac * x - zz * y) + a * y64 * ln[None, :] + a * ref.loc.apply_H(ref.MDinv[:, None] * x), tol)
    if prec == 0 and not graded:
        b0, bW, bU = -1.0, 2.0, 400.0
        out = op.cheb_filter(X, lam, 2, b0, bW, bU, prec=0)
        from oracle.chfsi import rchfsi_filter
        _close(host(out), rchfsi_filter(ref, x, ln, 2, b0, bW, bU), 1e-9)
    op.close()


@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("p", [2, 3, 6])
@pytest.mark.parametrize("nc", [5, NC])
def test_applies_overwrite(p, graded, nc):
    """H X and S X into a buffer of NaN: the first visit of each DOF writes it
    (few columns: the workgroup variants, many: the one-wave variants)."""
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    s = _system(p, graded)
    ref, op = PAWOperator(s), Operator(s)
    j = np.arange(nc) if nc < 10 else _sample()
    jd = torch.from_numpy(j).cuda()
    X = torch.randn(op.ndof, nc, device="cuda", dtype=torch.float64, generator=torch.Generator(device="cuda").manual_seed(p))
    x = X[:, jd].cpu().numpy()
    for apply, want in ((op.apply_H, ref.apply_H(x)), (op.apply_S, ref.apply_S(x))):
        out = torch.full_like(X, float("nan"))
        _close(apply(X, out=out)[:, jd].cpu().numpy(), want, 1e-12)
        o32 = torch.full(X.shape, float("nan"), device="cuda", dtype=torch.float32)
        _close(apply(X.float(), out=o32, prec="fp32")[:, jd].double().cpu().numpy(), want, 2e-5)
    op.close()


@pytest.mark.parametrize("p", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("prec", [0, 1])
def test_complex_local_terms(p, prec):
    """The complex (k-point) variants: H_loc (k), the step and, in FP64, the
    residual inside a degree-2 filter, on wide blocks of (re, im) pairs."""
    from oracle.chfsi import rchfsi_filter
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system
    n, nc = (3, 2, 3), 15009   # past the thresholds of both precisions
    box = tuple(1.6 * v for v in n)
    pos = [(0.4, 0.5, 0.6), (2.0, 2.2, 3.1)]
    s = custom_system(n, box, p, p + 2, pos=pos, rcut=0.7, channels="spd8", wells=pos, s_H=0.5, s_S=0.4, seed=p,
                      kpoint=(0.3, -0.2, 0.45), is_complex=True)
    ref, op = PAWOperator(s), Operator(s)
    g = torch.Generator(device="cuda").manual_seed(p)
    dt, rdt = (torch.complex128, torch.float64) if prec == 0 else (torch.complex64, torch.float32)
    draw = lambda d: torch.randn(op.ndof, nc, device="cuda", dtype=d, generator=g)  # noqa: E731
    X, Y, Y64 = draw(dt), draw(dt), draw(torch.complex128)
    lam = torch.rand(nc, device="cuda", dtype=torch.float64, generator=g)
    j = torch.from_numpy(np.concatenate([np.arange(5), [4000], np.arange(nc - 6, nc)])).cuda()
    host = lambda t: t[:, j].to(torch.complex128).cpu().numpy()  # noqa: E731
    x, y, y64, ln = host(X), host(Y), host(Y64), lam[j].cpu().numpy()
    tol = 1e-12 if prec == 0 else 2e-5
    _close(host(op.apply_local(X, Y.clone(), which=0, alpha=0.7, prec=prec)), y + 0.7 * ref.loc.apply_H(x), tol)
    a, ac, zz = 0.37, -0.81, 0.42
    real = lambda t: torch.view_as_real(t).reshape(op.ndof, 2 * nc)  # noqa: E731
    RX = real(Y.clone()).contiguous()
    op.cheb_step_local(real(X), RX, real(Y64), lam.repeat_interleave(2), a, ac, zz, prec=prec)
    got = host(torch.view_as_complex(RX.reshape(op.ndof, nc, 2).to(rdt)))
    _close(got, (-ac * x - zz * y) + a * y64 * ln[None, :] + a * ref.loc.apply_H(ref.MDinv[:, None] * x), tol)
    if prec == 0:
        out = op.cheb_filter(X, lam, 2, -1.0, 2.0, 400.0, prec=0)
        _close(host(out), rchfsi_filter(ref, x, ln, 2, -1.0, 2.0, 400.0), 1e-9)
    op.close()
