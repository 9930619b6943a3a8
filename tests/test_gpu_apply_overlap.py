"""mas_apply on vectors that share part of their memory: any overlap but
r == z, which is refused, gives what separate vectors give, bit for bit (the
same kernels read the same values)."""

import pytest

from conftest import cube

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [8, 16])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_overlapping_vectors(N, precision):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2411_06224_amd as mp

    s = cube(8)
    S = mp.MasPcg(s.row_ptr, s.col_idx, graph=(s.gptr, s.gadj), domain_size=N, precision=precision)
    S.build(mp.BlockMatrix.from_numpy(s.row_ptr, s.col_idx, s.val, device="cuda:0"))
    n = 3 * s.n
    want = S.apply(torch.as_tensor(s.b, device="cuda:0"))
    for shift in (-n, 1 - n, -48, -3, -1, 1, 3, 48, n - 1, n):
        buf = torch.empty(3 * n, dtype=torch.float64, device="cuda:0")
        r, z = buf[n : 2 * n], buf[n + shift : 2 * n + shift]
        r.copy_(torch.as_tensor(s.b, device="cuda:0"))
        S.apply(r, out=z)
        assert torch.equal(z, want), shift
    S.close()
