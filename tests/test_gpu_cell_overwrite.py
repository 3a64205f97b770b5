"""H X and S X into a buffer of NaN in launches per cell colour, where the first
visit of each DOF writes the result and nothing cleared it before.  Widths past
the limit of the gather (4,500 cell columns per colour) and inside one chunk of
512 columns: the workgroup kernel on 120 cells in 12 colours, the one-wave kernel
on 512 cells in 8 colours (two full rounds of waves), with a ragged last column
tile; uniform, complex, graded and GGA operators, both precisions."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,cols", [((6, 4, 5), 463), ((8, 8, 8), 510)])
@pytest.mark.parametrize("p,kind", [(2, "gga"), (3, "uniform"), (4, "graded"), (5, "complex"), (5, "gga"), (6, "uniform"),
                                    (2, "complex"), (6, "complex"), (3, "graded")])
def test_first_visit_overwrites(p, kind, n, cols):
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system, with_two_level_gga
    cplx = kind == "complex"
    kw = dict(kpoint=(0.3, -0.2, 0.45), is_complex=True) if cplx else {}
    pos = np.array([[1.0, 2.0, 3.0], [8.9, 0.2, 4.0]])
    s = custom_system(n, tuple(1.7 * v for v in n), p, p + 2, pos=pos, rcut=1.1, channels="spd8", wells=pos, s_H=0.5,
                      s_S=0.2, seed=3, **kw)
    if kind in ("graded", "gga"):
        s = with_two_level_gga(s, r_fine=0.6, gga=kind == "gga")
    ref, op = PAWOperator(s), Operator(s)
    nc = cols // 2 if cplx else cols
    assert op.ncells * cols > 4500 * op.ncolour
    X = torch.randn(op.ndof, nc, device="cuda", dtype=torch.complex128 if cplx else torch.float64,
                    generator=torch.Generator(device="cuda").manual_seed(p))
    j = torch.tensor([0, 9, nc - 2, nc - 1], device="cuda")
    x = X[:, j].cpu().numpy()
    for name in ("apply_H", "apply_S"):
        want = getattr(ref, name)(x)
        for prec, dt, tol in (("fp64", X.dtype, 1e-12), ("fp32", torch.complex64 if cplx else torch.float32, 2e-5)):
            out = torch.full(X.shape, float("nan"), device="cuda", dtype=dt)
            getattr(op, name)(X.to(dt), out=out, prec=prec)
            assert not torch.isnan(torch.view_as_real(out) if cplx else out).any(), (name, prec)
            got = out[:, j].to(X.dtype).cpu().numpy()
            err = np.max(np.abs(got - want).max(axis=0) / np.abs(want).max(axis=0))
            assert err <= tol, (name, prec, err)
    op.close()
