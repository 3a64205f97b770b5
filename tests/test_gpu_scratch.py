"""Device memory of the stand-alone calls: the room for per-cell results is an
allocation of its own, taken only by calls that use it, so that it neither
moves the scratch a graph was captured with nor keeps a call from being
captured."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _op(p=4, n=(6, 4, 5), natoms=2, rcut=1.1):   # 120 cells in 12 colours: 450 columns at the limit
    from paper_2604_26037_amd import Operator
    from workloads.configs import custom_system
    pos = np.random.default_rng(5).uniform(0.0, 1.0, (natoms, 3)) * 1.7 * np.asarray(n)
    return Operator(custom_system(n, tuple(1.7 * v for v in n), p, p + 2, pos=pos, rcut=rcut, channels="spd8", wells=pos,
                                  s_H=0.5, s_S=0.02, seed=3))


def _draw(op, n, seed=0, dtype=torch.float64):
    return torch.randn(op.ndof, n, device="cuda", dtype=dtype, generator=torch.Generator(device="cuda").manual_seed(seed))


def _capture(call):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    return g


def test_capture_after_another_call_left_enough_scratch():
    """Lanczos leaves scratch that holds an apply's projector part: the apply is
    captured without a warm call of its own, and gives what it gives eagerly."""
    op, other = _op(), _op()
    X = _draw(op, 8)
    Y = torch.zeros_like(X)
    other.apply_H(X)          # first launches of the process
    op.lanczos_bounds(k=4)
    torch.cuda.synchronize()
    g = _capture(lambda: op.apply_H(X, out=Y))
    for k in range(3):
        X.copy_(_draw(op, 8, k))
        g.replay()
        torch.cuda.synchronize()
        got = Y.clone()
        want = other.apply_H(X)
        assert (got - want).abs().max() <= 1e-12 * want.abs().max()
    op.close()
    other.close()


def test_capture_is_not_moved_by_wider_room():
    """An apply captured at 8 columns replays correctly after a gradient of one
    column, whose scratch fits in the apply's, and after wider and narrower
    applies below the scratch's size."""
    op = _op(natoms=40)
    X = _draw(op, 450)
    op.apply_H(X)             # scratch of 450 columns
    op.apply_H(X[:, :8].contiguous())
    x = X[:, :8].contiguous()
    Y = torch.zeros_like(x)
    torch.cuda.synchronize()
    g = _capture(lambda: op.apply_H(x, out=Y))
    calls = (lambda: op.band_energy_grad(X[:, :1].contiguous()), lambda: op.apply_S(X[:, :200].float(), prec="fp32"),
             lambda: op.apply_S(X), lambda: op.lanczos_bounds(k=4), lambda: op.apply_H(X[:, :1].contiguous()))
    for k, call in enumerate(calls):
        call()
        x.copy_(_draw(op, 8, k))
        Y.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = Y.clone()
        assert torch.equal(got, op.apply_H(x)), k
    op.close()


def test_room_is_taken_only_by_calls_that_use_it():
    """Sinv, bf16x3 and wide blocks take no room (54 MB at 450 columns); an H of
    450 columns does, once."""
    def taken(call):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        before = torch.cuda.mem_get_info()[0]
        call()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return before - torch.cuda.mem_get_info()[0]

    op = _op()
    room = op.ncells * 125 * 450 * 8
    X = _draw(op, 512)
    Y = torch.empty_like(X)
    F, G = X.float(), Y.float()
    op.apply_Sinv(X, out=Y)   # the projector scratch of 512 columns
    assert taken(lambda: op.apply_Sinv(X[:, :450], out=Y[:, :450])) < room // 4
    assert taken(lambda: op.apply_H(F[:, :450], out=G[:, :450], prec="bf16x3")) < room // 4
    assert taken(lambda: op.apply_H(X, out=Y)) < room // 4
    assert taken(lambda: op.apply_H(X[:, :450], out=Y[:, :450])) >= room
    assert taken(lambda: op.apply_S(X[:, :450], out=Y[:, :450])) < room // 4
    op.close()
