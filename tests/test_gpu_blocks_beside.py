"""Filters of several blocks on both sides of the width up to which their steps run
all cells in one launch and gather (degrees 5 and 6; 64 cells in 8 colours): the
same bits one block after another and with two in flight, and the same result as
each block filtered by itself, which gathers on both sides."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p,kind,prec,cols", [(6, "uniform", "fp64", 2400), (6, "gga", "fp64", 1800), (6, "graded", "fp32", 3000),
                                              (6, "complex", "fp64", 3000), (5, "graded", "fp64", 2600),
                                              (5, "complex", "fp32", 3400), (4, "uniform", "fp32", 4500)])
def test_several_blocks(p, kind, prec, cols):
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system, with_two_level_gga
    n, cplx = (4, 4, 4), kind == "complex"
    kw = dict(kpoint=(0.3, -0.2, 0.45), is_complex=True) if cplx else {}
    pos = np.array([[1.0, 2.0, 3.0], [3.4, 0.2, 4.0]])
    s = custom_system(n, tuple(1.7 * v for v in n), p, p + 2, pos=pos, rcut=1.1, channels="spd8", wells=pos, s_H=0.5,
                      s_S=0.2, seed=3, **kw)
    if kind in ("graded", "gga"):
        s = with_two_level_gga(s, r_fine=0.6, gga=kind == "gga")
    op = Operator(s)
    lo, hi, beta = op.lanczos_bounds(12)
    args = (5, lo - 0.1, lo + 0.3 * (hi - lo), hi + beta)
    tol = 1e-10 if prec == "fp64" else 1e-5
    lim = cols * op.ncolour // op.ncells // (2 if cplx else 1)
    for B in (lim, lim + 1):
        X = torch.randn(op.ndof, B + 7, device="cuda", dtype=torch.complex128 if cplx else torch.float64,
                        generator=torch.Generator(device="cuda").manual_seed(p))
        lam = torch.linspace(lo, lo + 0.3 * (hi - lo), B + 7, device="cuda", dtype=torch.float64)
        run = lambda x, l, states: op.cheb_filter(x, l, *args, block=B, prec=prec,   # noqa: E731
                                                  ws=op.workspace(states * op.cheb_filter_workspace(B, B, prec)))
        one, two = run(X, lam, 1), run(X, lam, 2)
        assert torch.equal(one, two), B
        for a, b in ((0, B), (B, B + 7)):
            want = run(X[:, a:b].contiguous(), lam[a:b].contiguous(), 1)
            err = ((one[:, a:b] - want).abs().amax(0) / want.abs().amax(0)).max().item()
            assert err <= tol, (B, a, err)
    op.close()
