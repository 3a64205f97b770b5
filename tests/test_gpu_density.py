"""The band-energy density dE/dV against the oracle at every degree: fewer
columns than one tile, ragged tiles over the four waves of a workgroup, with
and without occupations, real, complex and graded operators.  Every value is
a sum of at most 70 positive terms of FP64 interpolations: 1e-12 of the largest."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["real", "complex", "graded"])
@pytest.mark.parametrize("p", [2, 3, 4, 5, 6])
def test_density(p, kind):
    from oracle.grad import grad_veff
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system, with_two_level_gga
    cplx = kind == "complex"
    n = (3, 2, 3)
    box = tuple(1.6 * v for v in n)
    kw = dict(kpoint=(0.3, -0.2, 0.45), is_complex=True) if cplx else {}
    s = custom_system(n, box, p, p + 2, pos=[(0.4, 0.5, 0.6)], rcut=0.7, channels="spd8", wells=[(0.4, 0.5, 0.6)], seed=p, **kw)
    if kind == "graded":
        s = with_two_level_gga(s, r_fine=0.4, gga=True)
    ref, op = PAWOperator(s), Operator(s)
    for nc in (1, 5, 35):
        X = torch.randn(op.ndof, nc, device="cuda", dtype=torch.complex128 if cplx else torch.float64,
                        generator=torch.Generator(device="cuda").manual_seed(nc))
        occ = torch.rand(nc, device="cuda", dtype=torch.float64, generator=torch.Generator(device="cuda").manual_seed(p))
        for o in (None, occ):
            _, dV, _ = op.band_energy_grad(X, o, want_E=False, want_dH=False)
            want = grad_veff(ref, X.cpu().numpy(), None if o is None else o.cpu().numpy())
            assert np.max(np.abs(dV.cpu().numpy().reshape(want.shape) - want)) <= 1e-12 * np.abs(want).max()
    op.close()
