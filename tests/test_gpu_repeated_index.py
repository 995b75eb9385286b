"""x lists one column over and over, past 2^32 products: the call ends with the
repeated-index error, without a store outside the buckets, and the next
multiply on the handle is right.  (The bound itself: test_reserve_host.py.)"""
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


def matrix(m, n, rows):
    """Column 7 holds rows 0 .. rows - 1, every 1000th other column one entry."""
    lens = np.zeros(n, np.int64)
    lens[::1000] = 1
    lens[7] = rows
    colptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rng = np.random.default_rng(1)
    rowids = rng.integers(0, m, int(lens.sum())).astype(np.int32)
    rowids[colptr[7]:colptr[8]] = np.arange(rows)
    return synth.CSC(m, n, colptr, rowids, np.ones(rowids.size, np.float32))


# one wide bucket of column 7's rows; and more buckets than a 256-thread workgroup reserves for at once
@pytest.mark.parametrize("m,n,rows,tile,shape", [(2500, 4300000, 1024, 11, (256, 4)), (2500, 4300000, 1024, 11, (1024, 8)),
                                                 (70001, 17000000, 256, 8, (256, 4))])
@pytest.mark.parametrize("variant", [0, 1])
def test_past_32_bits(spv, m, n, rows, tile, shape, variant):
    A = matrix(m, n, rows)
    assert n * rows > 1 << 32
    M = spv.Matrix.from_csc(A)
    s = M.schedule
    s.tile_log2, s.merge_variant, s.launch = tile, variant, 1
    s.scatter_block, s.scatter_items = shape
    M.schedule = s
    x = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    xv = torch.ones(n, device="cuda")
    with pytest.raises(spv.SpmspvError) as e:
        M.spmspv(x, xv, 0, True)
    assert e.value.status == spv.EDEVICE
    S = np.arange(0, n, 500, dtype=np.int32)
    S[0] = 7
    yi, yv, _ = M.spmspv(torch.as_tensor(S).cuda(), xv[:S.size], 0, True)
    compare(0, yi, yv, *oracle.spmspv(A, S, np.ones(S.size, np.float32), 0, sorted_output=True)[:2], sorted_output=True)
