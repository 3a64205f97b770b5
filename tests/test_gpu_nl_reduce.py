"""The projector reduction on both sides of its row split (the four waves of
a workgroup share an item's rows in small launches, own columns in wide
ones), against the oracle on sampled columns: Sinv_hat, whose result outside
M_D^{-1} X is the reduction's, for 8, 18 and 32 projectors per atom, real and
complex operators, FP64, FP32 and bf16x3, ragged rows and columns."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("channels", ["spd8", "spd18", "max32"])
@pytest.mark.parametrize("cplx", [False, True])
def test_reduce_split(channels, cplx):
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system
    box = (5.4, 6.0, 4.8)
    pos = np.array([[0.2, 0.4, 0.3], [3.1, 3.0, 2.2], [3.9, 3.7, 2.9]])
    kw = dict(kpoint=(0.3, -0.2, 0.45), is_complex=True) if cplx else {}
    s = custom_system((3, 3, 3), box, 3, 5, pos=pos, rcut=1.3, channels=channels, wells=pos, s_H=0.5, s_S=0.4, seed=11, **kw)
    ref, op = PAWOperator(s), Operator(s)
    items = sum(-(-len(n) // 128) for n in ref.supp_nodes)
    wide = 64 * (3000 // items + 2) // (2 if cplx else 1) + 3   # past three waves per SIMD without the split
    for nc in (1, 67, wide):
        X = torch.randn(op.ndof, nc, device="cuda", dtype=torch.complex128 if cplx else torch.float64,
                        generator=torch.Generator(device="cuda").manual_seed(nc))
        j = np.unique(np.concatenate([np.arange(min(nc, 5)), np.arange(max(0, nc - 5), nc)]))
        jd = torch.from_numpy(j).cuda()
        want = ref.apply_Sinv(X[:, jd].cpu().numpy())
        scale = np.abs(want).max(axis=0)
        for prec, tol in (("fp64", 1e-12), ("fp32", 2e-5), ("bf16x3", 1e-3)):
            x = X if prec == "fp64" else X.to(torch.complex64 if cplx else torch.float32)
            got = op.apply_Sinv(x, prec=prec)[:, jd].to(X.dtype).cpu().numpy()
            assert np.max(np.abs(got - want).max(axis=0) / scale) <= tol, (nc, prec)
    op.close()


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("natoms", [1, 2, 5])
def test_add_back_shared_rows(natoms, cplx):
    """The one-launch add-back: support rows of one atom alone and rows that
    up to five overlapping atoms share, H, S and Sinv_hat against the oracle."""
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system
    pos = np.array([[0.3, 0.2, 0.4], [1.0, 0.8, 0.9], [4.9, 0.1, 0.6], [0.5, 5.5, 1.1], [3.0, 3.1, 2.0]])[:natoms]
    kw = dict(kpoint=(0.3, -0.2, 0.45), is_complex=True) if cplx else {}
    s = custom_system((3, 4, 3), (5.4, 6.4, 4.8), 4, 6, pos=pos, rcut=0.9, channels="spd8", wells=pos, s_H=0.5, s_S=0.1,
                      seed=5, **kw)
    ref, op = PAWOperator(s), Operator(s)
    X = torch.randn(op.ndof, 19, device="cuda", dtype=torch.complex128 if cplx else torch.float64,
                    generator=torch.Generator(device="cuda").manual_seed(natoms))
    x = X.cpu().numpy()
    for got, want in ((op.apply_H(X), ref.apply_H(x)), (op.apply_S(X), ref.apply_S(x)), (op.apply_Sinv(X), ref.apply_Sinv(x))):
        assert np.max(np.abs(got.cpu().numpy() - want).max(axis=0) / np.abs(want).max(axis=0)) <= 1e-12
    op.close()
