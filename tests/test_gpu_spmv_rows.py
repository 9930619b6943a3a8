"""bcsr_spmv at the edges of its split of the rows: fewer rows than a wave
takes, a last workgroup that is not full, rows of exactly one and more than
one batch of 64 blocks, empty rows at both ends of a workgroup, and a
workgroup whose rows hold more blocks than the waves take one by one (and
whose neighbours do not).  Against scipy's product in FP64, per row within
the rounding of a sum of its products: gamma_n with n = 3 blocks + 2."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = {
    "one_row": [1],
    "three_rows": [3, 0, 2],
    "batch_edges": [64, 63, 65, 1, 128, 127, 129, 0, 0, 64] * 4,
    "ragged_tail": [7] * 45,
    "empty_ends": [0, 5, 5, 0] * 9 + [0],
    "long_block": [6] * 32 + [900, 40, 0, 1500] + [6] * 61,
    "threshold": [512] * 4 + [512, 512, 512, 513] + [256] * 8 + [257] + [256] * 7,
}


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("name", list(CASES))
def test_spmv_row_split(name, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import scipy.sparse as sp
    from paper_2411_06224_amd import BlockMatrix, bcsr_spmv

    print("[case] spmv rows", name, dtype, flush=True)
    length = np.asarray(CASES[name])
    n = max(length.size, int(length.max()))
    length = np.concatenate([length, np.zeros(n - length.size, int)])  # square; the added rows are empty
    rng = np.random.default_rng(11)
    rp = np.concatenate([[0], np.cumsum(length)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in length]).astype(np.int32)
    val = rng.standard_normal((ci.size, 3, 3))
    if dtype == "f32":
        val = val.astype(np.float32)
    x = rng.standard_normal(3 * n)
    H = BlockMatrix.from_numpy(rp, ci, val, dtype=torch.float32 if dtype == "f32" else torch.float64)
    out = torch.full((3 * n,), float("nan"), dtype=torch.float64, device="cuda")
    y = bcsr_spmv(H, torch.as_tensor(x, device="cuda"), out=out).cpu().numpy()
    v64 = val.astype(np.float64)
    A = sp.bsr_matrix((v64, ci, rp), shape=(3 * n, 3 * n))
    B = sp.bsr_matrix((np.abs(v64), ci, rp), shape=(3 * n, 3 * n))
    terms = np.repeat(3 * length + 2, 3)
    bound = 2 * terms * 2.0 ** -53 * (B @ np.abs(x))  # both sides round
    assert np.all(np.abs(y - A @ x) <= bound)
