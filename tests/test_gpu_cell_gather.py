"""One launch of all cells and a gather per DOF (small problems) on both sides
of its limit of 4,500 cell columns per colour, against the oracle; the same
calls with workspaces that leave no room for it; and under capture."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _system(p, cplx=False, n=(6, 4, 5), **kw):   # 120 cells in 12 colours: 450 real columns
    from workloads.configs import custom_system
    if cplx:
        kw.update(kpoint=(0.3, -0.2, 0.45), is_complex=True)
    pos = np.array([[1.0, 2.0, 3.0], [8.9, 0.2, 4.0]])
    return custom_system(n, tuple(1.7 * v for v in n), p, p + 2, pos=pos, rcut=1.1, channels="spd8", wells=pos,
                         s_H=0.5, s_S=0.2, seed=3, **kw)


def _draw(op, n, cplx, seed=0):
    return torch.randn(op.ndof, n, device="cuda", dtype=torch.complex128 if cplx else torch.float64,
                       generator=torch.Generator(device="cuda").manual_seed(seed))


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("p", [2, 3, 4, 5, 6])
def test_apply_at_the_limit(p, cplx):
    from oracle.paw import PAWOperator
    from paper_2604_26037_amd import Operator
    s = _system(p, cplx)
    ref, op = PAWOperator(s), Operator(s)
    lim = 4500 * op.ncolour // op.ncells // (2 if cplx else 1)
    for nc in (1, 37, lim, lim + 1):
        X = _draw(op, nc, cplx, nc)
        j = np.unique([0, nc // 2, nc - 1])
        jd = torch.from_numpy(j).cuda()
        x = X[:, jd].cpu().numpy()
        for name in ("apply_H", "apply_S"):
            want = getattr(ref, name)(x)
            for prec, tol in (("fp64", 1e-12), ("fp32", 2e-5)):
                xin = X if prec == "fp64" else X.to(torch.complex64 if cplx else torch.float32)
                got = getattr(op, name)(xin, prec=prec)[:, jd].to(X.dtype).cpu().numpy()
                err = np.max(np.abs(got - want).max(axis=0) / np.abs(want).max(axis=0))
                assert err <= tol, (name, nc, prec, err)
    op.close()


@pytest.mark.parametrize("p,cplx", [(2, False), (4, True), (6, False)])
def test_workspace_without_room(p, cplx):
    """The smallest workspaces that are accepted leave no room and give the
    same results up to the order of the sums; a workspace for one block always
    stays below two of them (it never makes the filter fork its blocks)."""
    from paper_2604_26037_amd import Operator, PawfeError
    op = Operator(_system(p, cplx, (3, 4, 3)))
    lo, hi, beta = op.lanczos_bounds(12)
    bU, bW, b0 = hi + beta, lo + 0.3 * (hi - lo), lo - 0.1
    X = _draw(op, 24, cplx)
    lam, _ = op.rayleigh_ritz(X)

    def least(call, full):
        lo, hi = 0, full // 256      # sizes are whole multiples of 256
        while hi - lo > 1:
            mid = (lo + hi) // 2
            try:
                call(mid * 256)
                hi = mid
            except PawfeError:
                lo = mid
        return hi * 256

    for prec, tol in (("fp64", 1e-10), ("fp32", 1e-5)):
        for block in (24, 9):
            run = lambda b: op.cheb_filter(X, lam, 6, b0, bW, bU, block=block, prec=prec, ws=op.workspace(b))
            one = op.cheb_filter_workspace(block, block, prec)
            full = op.cheb_filter_workspace(24, block, prec)
            low = least(run, full)
            assert low <= one < 2 * low and full == one * (2 if block < 24 else 1)
            want = run(full)
            scale = want.abs().amax(0)
            for b in (low, one, 2 * low):
                assert ((run(b) - want).abs().amax(0) / scale).max().item() <= tol, (prec, block, b)
    run = lambda b: op.rayleigh_ritz(X.clone(), ws=op.workspace(b))[0]
    full = op.rayleigh_ritz_workspace(24)
    l0, l1 = run(full), run(least(run, full))
    assert (l1 - l0).abs().max().item() <= 1e-10 * l0.abs().max().item()
    op.close()


def test_capture_keeps_its_scratch():
    """A captured apply replays correctly after narrower eager calls of either
    type: none of them may move the scratch that the graph was captured with."""
    from paper_2604_26037_amd import Operator
    op = Operator(_system(4))
    X = _draw(op, 460, False)           # past the limit: launches per colour, narrower calls gather
    Y = torch.zeros_like(X)
    op.apply_H(X, out=Y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        op.apply_H(X, out=Y)
    for k, (n, dt) in enumerate(((40, torch.float64), (450, torch.float32), (450, torch.float64))):
        x = _draw(op, n, False, k + 1).to(dt)
        op.apply_H(x, prec="fp64" if dt == torch.float64 else "fp32")
        X.copy_(_draw(op, 460, False, 10 + k))
        Y.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = Y.clone()
        assert torch.equal(got, op.apply_H(X))
    op.close()
