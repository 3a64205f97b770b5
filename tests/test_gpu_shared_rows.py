"""Rows that several atoms share, in the filter's last add-back of an FP32
filter (FP64 output): the atoms' terms, each an FP32 dot product, are summed in
FP64.  K atoms at one place with the same coefficients give K equal terms t, whose
FP64 sum K t is exact, so six atoms give exactly twice what three give."""

import ctypes as C
import re
import subprocess

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _finalize():
    from paper_2604_26037_amd.pawfe import LIB_PATH, load
    load()
    names = subprocess.run(["nm", "-D", "--defined-only", LIB_PATH], capture_output=True, text=True, check=True).stdout
    name, = re.findall(r"\S*launch_node_finalizeIf\S*", names)
    fn = getattr(C.CDLL(LIB_PATH), name)
    vp, i64 = C.c_void_p, C.c_int64
    # op, RY, ld, d, X, ldx, lamY, Xo, ldo, ncols, stream: Xo = M_D^{-1} (RY - sum_a C^a d_a) + X lamY
    fn.argtypes, fn.restype = [vp, vp, i64, vp, vp, i64, vp, vp, i64, C.c_int, vp], C.c_int
    return fn


@pytest.mark.parametrize("channels,cplx", [("spd8", False), ("spd18", False), ("spd8", True)])
def test_terms_of_shared_rows_are_summed_in_fp64(channels, cplx):
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system
    fn, n, out = _finalize(), (3, 3, 3), {}
    kw = dict(kpoint=(0.2, 0.1, -0.3), is_complex=True) if cplx else {}
    nc = 10
    for k in (3, 6):
        pos = [(2.0, 2.2, 3.1)] * k
        s = custom_system(n, tuple(1.6 * v for v in n), 4, 6, pos=pos, rcut=1.1, channels=channels, wells=pos[:1],
                          s_H=0.5, s_S=0.01, seed=7, **kw)
        op = Operator(s)
        npj = int(s.nproj[0])
        d = np.tile(np.random.default_rng(2).standard_normal((npj, nc)), (k, 1))
        dv = torch.from_numpy(np.ascontiguousarray(d)).cuda()
        RY = torch.zeros(op.ndof, nc, device="cuda", dtype=torch.float32)
        X, lam = torch.zeros(op.ndof, nc, device="cuda", dtype=torch.float64), torch.zeros(nc, device="cuda", dtype=torch.float64)
        out[k] = torch.empty_like(X)
        p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
        assert fn(op._h, p(RY), nc, p(dv), p(X), nc, p(lam), p(out[k]), nc, nc,
                  C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        torch.cuda.synchronize()
        op.close()
    assert (out[3] != 0).sum() > 100
    assert torch.equal(out[6], 2 * out[3])
