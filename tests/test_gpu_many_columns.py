"""More columns than a grid's y extent (65,535) of 16-column tiles: the projector
reduction and the atom-block kernels of the gradient, on the smallest mesh."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_a_million_columns():
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system
    n, N = (2, 2, 2), 65535 * 16 + 25
    s = custom_system(n, (3.4, 3.4, 3.4), 2, 4, pos=[(1.0, 1.2, 0.7)], rcut=1.1, channels="spd8", wells=[(1.0, 1.2, 0.7)],
                      s_H=0.5, s_S=0.2, seed=3)
    ref, op = PAWOperator(s), Operator(s)
    # a column of its own size at the end, where a missing tile would show
    X = torch.randn(op.ndof, N, device="cuda", dtype=torch.float64, generator=torch.Generator(device="cuda").manual_seed(1))
    X[:, -25:] *= 300.0
    got = op.band_energy_grad(X, want_E=False, want_dV=False)[2].cpu().numpy().reshape(8, 8)
    # sum_n P_n P_n^T = C^T (X X^T) C, with C from the oracle
    G = (X @ X.T).cpu().numpy()
    C = ref.C.toarray()
    want = C.T @ G @ C
    assert np.abs(got - want).max() <= 1e-11 * np.abs(want).max()
    op.close()
