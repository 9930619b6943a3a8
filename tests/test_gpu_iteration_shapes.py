"""The iteration's kernels and the domain inversion at the sizes where their
splits change -- one domain, an odd number (the last pair half empty), a
remainder of a workgroup's four, one and two levels, some hundred to some
thousand domains, far couplings and one row of many blocks -- against the
oracle.  (Where the work groups grow, and groups halved for a heavy window or
reading more units than their lists hold: test_gpu_group_branches.)

Iterates: as the parity tests hold ten iterations to 1e-10 relative, eight
here (rounding of a step, about 1e-15 sqrt(3 n) in the dot products, grows by
at most the conditioning of the preconditioned system, below 1e4).  Inverses:
1e-10 relative in the Frobenius norm, as there.  Mixed solves: the true
residual, which the solver itself confirms in FP64."""

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _chain(n, far=0, hub=0):
    """Nodes in a line with some second neighbours; far: random couplings;
    hub: node 0 coupled with that many nodes."""
    rng = np.random.default_rng(n + far + hub)
    i = np.arange(n)
    e = [np.stack([i[:-1], i[1:]], 1), np.stack([i[:-5:3], i[5::3]], 1) if n > 5 else np.zeros((0, 2), int)]
    if far:
        e.append(rng.integers(0, n, (far, 2)))
    if hub:
        e.append(np.stack([np.zeros(hub, int), 2 + np.arange(hub) * ((n - 2) // hub)], 1))
    e = np.concatenate(e)
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], axis=1), axis=0)
    return synth.bcsr.spd_system_from_edges(n, e, seed=n)


SHAPES = [  # nodes, levels (0: all), domain size, far couplings, hub
    (1, 0, 16, 0, 0), (5, 0, 16, 0, 0), (17, 1, 16, 0, 0), (17, 0, 16, 0, 0), (48, 2, 16, 0, 0), (80, 0, 16, 0, 0),
    (272, 1, 16, 0, 0), (272, 2, 16, 0, 0), (2100, 0, 16, 0, 0), (2100, 0, 5, 0, 0), (2100, 0, 21, 0, 0),
    (3000, 0, 16, 12000, 0), (6000, 0, 16, 0, 3000), (10240, 0, 16, 0, 0), (10256, 0, 16, 0, 0), (20480, 0, 16, 0, 0),
    (20496, 0, 16, 0, 0), (40960, 0, 16, 0, 0), (40976, 0, 16, 0, 0),
]


@pytest.mark.parametrize("n,levels,N,far,hub", SHAPES)
def test_iteration_and_inverses(n, levels, N, far, hub):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2411_06224_amd as mp

    print("[case]", n, levels, N, far, hub, flush=True)
    s = _chain(n, far, hub)
    P = oracle.MAS(s.row_ptr, s.col_idx, s.val, N=N, max_levels=levels, gptr=s.gptr, gadj=s.gadj)
    H = mp.BlockMatrix.from_numpy(s.row_ptr, s.col_idx, s.val, device="cuda:0")
    b = torch.as_tensor(s.b, device="cuda:0")
    for precision in ("f64", "mixed"):
        S = mp.MasPcg(s.row_ptr, s.col_idx, graph=(s.gptr, s.gadj), domain_size=N, max_levels=levels,
                      precision=precision, poison=True)
        S.build(H)
        assert S.info()["levels"] == P.levels
        for l in range(P.levels):
            G = S.inverses(l)
            for d in sorted({0, 1, 2, 3, G.shape[0] // 2, G.shape[0] - 2, G.shape[0] - 1} & set(range(G.shape[0]))):
                R = P.inverse(l, d)
                assert np.linalg.norm(G[d] - R) <= 1e-10 * np.linalg.norm(R), (l, d)
        if precision == "mixed":
            x, res = S.solve(H, b, tol=1e-7)
            x = x.cpu().numpy()
            assert res["status"] == 0
            assert np.linalg.norm(s.b - oracle.spmv(s.row_ptr, s.col_idx, s.val, x)) <= 1e-7 * np.linalg.norm(s.b)
        elif n > 3 * N:  # fewer nodes converge to rounding within the iterations compared
            want = P.pcg(s.b, tol=0.0, max_iter=8)[0]
            for every in (50, 3):
                x, res = S.solve(H, b, tol=0.0, max_iter=8, replace_every=every)
                assert res["iterations"] == 8
                assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-10 * np.linalg.norm(want)
        else:
            want = P.pcg(s.b, tol=1e-11)[0]
            x, res = S.solve(H, b, tol=1e-11)
            assert res["status"] == 0
            assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-8 * np.linalg.norm(want)  # kappa(H) < 1e3
        S.close()
