"""Iterations of systems with a heavy window, with a group that reads more
units than its list holds (three launches per iteration), with both, and at
the domain counts where the groups grow, against the oracle: eight iterations
to 1e-10 relative and mixed solves to the residual they confirm, as the tests
of the iteration's shapes hold them.  Re-plans between such systems, which
change the groups and the launches, against the host analysis byte for byte."""

import numpy as np
import pytest

import oracle
from group_systems import EDGES, SYSTEMS, line, system
from test_gpu_replan import _compare

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_iterates(name):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2411_06224_amd as mp

    print("[case]", name, flush=True)
    s = system(name)
    P = oracle.MAS(s.row_ptr, s.col_idx, s.val, N=16, gptr=s.gptr, gadj=s.gadj)
    H = mp.BlockMatrix.from_numpy(s.row_ptr, s.col_idx, s.val, device="cuda:0")
    b = torch.as_tensor(s.b, device="cuda:0")
    want = P.pcg(s.b, tol=0.0, max_iter=8)[0]
    for precision in ("f64", "mixed"):
        S = mp.MasPcg(s.row_ptr, s.col_idx, graph=(s.gptr, s.gadj), precision=precision, poison=True)
        S.build(H)
        S.set_kernel_timing(True)
        S.solve(H, b, tol=0.0, max_iter=8)
        kt = S.kernel_timing()
        S.set_kernel_timing(False)
        # one apply for all levels each, the prolongation alone where it is not part of the next product
        assert kt["level0_update"][1] == 8 and kt["apply_coarse"][1] == 0 and kt["update"][1] == 0
        assert kt["apply_level0"][1] == (0 if SYSTEMS[name][2] else 8)
        if precision == "f64":
            for every in (50, 3):
                x, res = S.solve(H, b, tol=0.0, max_iter=8, replace_every=every)
                assert res["iterations"] == 8
                assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-10 * np.linalg.norm(want)
        else:
            x, res = S.solve(H, b, tol=1e-7)
            assert res["status"] == 0
            x = x.cpu().numpy()
            assert np.linalg.norm(s.b - oracle.spmv(s.row_ptr, s.col_idx, s.val, x)) <= 1e-7 * np.linalg.norm(s.b)
        S.close()


@pytest.mark.parametrize("n,domains", EDGES)
def test_group_size_edges(n, domains):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2411_06224_amd as mp

    print("[case]", n, domains, flush=True)
    s = line(n)
    P = oracle.MAS(s.row_ptr, s.col_idx, s.val, N=16, gptr=s.gptr, gadj=s.gadj)
    S = mp.MasPcg(s.row_ptr, s.col_idx, graph=(s.gptr, s.gadj), poison=True)
    H = mp.BlockMatrix.from_numpy(s.row_ptr, s.col_idx, s.val, device="cuda:0")
    S.build(H)
    want = P.pcg(s.b, tol=0.0, max_iter=8)[0]
    x, res = S.solve(H, torch.as_tensor(s.b, device="cuda:0"), tol=0.0, max_iter=8)
    assert res["iterations"] == 8
    assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-10 * np.linalg.norm(want)
    S.close()


@pytest.mark.parametrize("precision", ["f64", "mixed"])
@pytest.mark.parametrize("first,then", [("even", "wide_heavy"), ("heavy", "wide"), ("wide", "even"), ("even", "heavy")])
def test_replan_changes_groups(first, then, precision):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2411_06224_amd as mp

    print("[case]", first, then, precision, flush=True)
    dev = torch.device("cuda:0")
    s, t = system(first), system(then)
    A = mp.MasPcg(s.row_ptr, s.col_idx, graph=(s.gptr, s.gadj), precision=precision, poison=True)
    A.replan(torch.as_tensor(t.row_ptr.astype(np.int32), device=dev), torch.as_tensor(t.col_idx.astype(np.int32), device=dev))
    B = mp.MasPcg(t.row_ptr, t.col_idx, partition=A.ordering()[0] // 16, precision=precision, poison=True)
    _compare(A, B, t.row_ptr, t.col_idx, t.val, dev, tol=1e-6, b=t.b)
    A.close()
    B.close()
