"""Atoms whose radius holds no Gauss point (no support rows) beside ordinary
ones, as the first and as the last atom, against the oracle: the applies, a
filter (its neighbour sums and add-back) and the Delta_H gradient, which is
zero for such an atom."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("empty", [[2], [0], [0, 2]])
def test_empty_support(empty):
    from oracle.chfsi import rchfsi_filter
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system
    n = (3, 2, 3)
    pos = [(0.4, 0.5, 0.6), (2.0, 2.2, 3.1), (3.9, 1.1, 0.7)]
    s = custom_system(n, tuple(1.6 * v for v in n), 4, 6, pos=pos, rcut=1.1, channels="spd8", wells=pos, s_H=0.5,
                      s_S=0.4, seed=7)
    s.rcut[empty] = 1e-6
    ref, op = PAWOperator(s), Operator(s)
    x = np.random.default_rng(3).standard_normal((op.ndof, 7))
    X = torch.from_numpy(x).cuda()
    rel = lambda got, want: np.max(np.abs(got.cpu().numpy() - want).max(axis=0) / np.abs(want).max(axis=0))  # noqa: E731
    assert rel(op.apply_H(X), ref.apply_H(x)) <= 1e-12
    assert rel(op.apply_S(X), ref.apply_S(x)) <= 1e-12
    assert rel(op.apply_Sinv(X), ref.apply_Sinv(x)) <= 1e-12
    lam = np.linspace(0.0, 1.0, 7)
    got = op.cheb_filter(X, torch.from_numpy(lam).cuda(), 6, -1.0, 2.0, 400.0)
    assert rel(got, rchfsi_filter(ref, x, lam, 6, -1.0, 2.0, 400.0)) <= 1e-9
    g = op.band_energy_grad(X, want_E=False, want_dV=False)[2].cpu().numpy().reshape(3, -1)
    assert all((np.abs(g[a]).max() == 0.0) == (a in empty) for a in range(3))
    op.close()
