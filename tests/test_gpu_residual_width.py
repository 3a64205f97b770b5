"""The residual handed from Rayleigh-Ritz to the filter, at sizes where the two
form it in blocks of widths that the applies would run by different kernels:
one-wave, workgroup per colour or one launch of all cells and a gather (by the
cell columns of a colour), and the projector reduction with or without split
rows (by items times column tiles).  The filter given R and the filter that forms
it agree bit for bit, and so does R itself in blocks of any width."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _system(p, n, natoms, kind):
    from workloads.configs import custom_system, with_two_level_gga
    kw = dict(kpoint=(0.3, -0.2, 0.45), is_complex=True) if kind == "complex" else {}
    box = tuple(1.7 * v for v in n)
    pos = np.random.default_rng(p).uniform(0.0, 1.0, (natoms, 3)) * np.asarray(box)
    s = custom_system(n, box, p, p + 2, pos=pos, rcut=1.1, channels="spd8", wells=pos[:2], s_H=0.5, s_S=0.05, seed=3, **kw)
    return with_two_level_gga(s, r_fine=0.6, gga=kind == "gga") if kind in ("graded", "gga") else s


@pytest.mark.parametrize("p,n,natoms,kind,N", [
    (6, (8, 8, 8), 20, "uniform", 256),   # one-wave; items x tiles on both sides of the split
    (6, (6, 6, 6), 2, "uniform", 320),    # workgroup at 256 columns, one-wave past it
    (3, (8, 8, 8), 2, "uniform", 256),
    (2, (6, 5, 6), 2, "graded", 256),
    (4, (8, 8, 6), 2, "graded", 256),
    (4, (8, 7, 6), 2, "gga", 256),
    (4, (6, 6, 6), 2, "complex", 128),
])
def test_residual_is_the_same_in_blocks_of_any_width(p, n, natoms, kind, N):
    from paper_2604_26037_amd import FP32, FP64, Operator
    op = Operator(_system(p, n, natoms, kind))
    lo, hi, beta = op.lanczos_bounds(k=12)
    X = torch.randn(op.ndof, N, device="cuda", dtype=torch.complex128 if kind == "complex" else torch.float64,
                    generator=torch.Generator(device="cuda").manual_seed(p))
    R = torch.empty_like(X)
    lam, _ = op.rayleigh_ritz(X, R=R)
    a = lam.cpu().numpy()
    args = (lam, 3, float(a[0]) - 0.1, float(a[-1]), 1.02 * (hi + beta) + 1.0)
    for prec in (FP64, FP32):
        for block in (N, 96, 64, 17, 5):
            y1 = op.cheb_filter(X, *args, block=block, prec=prec)
            y2 = op.cheb_filter(X, *args, block=block, prec=prec, R=R)
            torch.cuda.synchronize()
            assert torch.equal(y1, y2), (prec, block)
    op.close()
