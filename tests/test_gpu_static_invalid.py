"""spmspv_run_static checks its matrix on the device, in the same call as the
multiply: a matrix that fails a check is EINVAL without a column or row id of
it being followed, and the next call is right.  Sizes on both sides of the
2047 entries up to which a handle takes the expansion."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import compare

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def spv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1610_07902_amd as spv
    spv.load_library()
    oracle.build(force=False)
    return spv


def call(spv, m, n, colptr, rowids, x):
    dev = [torch.as_tensor(np.ascontiguousarray(a)).cuda() for a in (colptr, rowids, np.ones(rowids.size, np.float32), x)]
    xv = torch.ones(x.size, device="cuda")
    yi = torch.full((m,), -1, dtype=torch.int32, device="cuda")
    yv = torch.zeros(m, device="cuda")
    nnz = spv.spmspv_run_static(m, n, rowids.size, dev[0], dev[1], dev[2], 0, spv.SORTED_OUTPUT, x.size, dev[3], xv,
                                yi, yv, m)
    return yi[:nnz], yv[:nnz]


@pytest.mark.parametrize("per", [3, 40])
@pytest.mark.parametrize("fault", ["descending", "past the end", "starts late", "negative row", "row past m"])
def test_invalid_matrix(spv, per, fault):
    m = n = 600
    rng = np.random.default_rng(per)
    lens = rng.integers(1, per + 1, n)
    colptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rowids = np.concatenate([np.sort(rng.choice(m, k, replace=False)) for k in lens]).astype(np.int32)
    assert (rowids.size <= 2047) == (per == 3)
    good = colptr.copy(), rowids.copy()
    if fault == "descending":
        colptr[101] = colptr[100] - 1
    elif fault == "past the end":
        colptr[300] = colptr[n] + 1000000
    elif fault == "starts late":
        colptr[0] = 1
    elif fault == "negative row":
        rowids[colptr[50]] = -5
    else:
        rowids[colptr[50]] = m
    x = rng.permutation(n).astype(np.int32)
    for xs in (x, x[x < 200], np.array([100], np.int32)):
        with pytest.raises(spv.SpmspvError) as e:
            call(spv, m, n, colptr, rowids, xs)
        assert e.value.status == spv.EINVAL
    A = synth.CSC(m, n, good[0], good[1], np.ones(rowids.size, np.float32))
    yi, yv = call(spv, m, n, *good, x)
    compare(0, yi, yv, *oracle.spmspv(A, x, np.ones(n, np.float32), 0, sorted_output=True)[:2], sorted_output=True)
