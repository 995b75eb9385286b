"""GPU parity of the expansion where it takes a call at any size: even columns,
so that tiles hold one to many chunks and a workgroup takes several tiles, in
every chunk shape, with bounds on both sides of a chunk; and uneven columns
with the heaviest ones listed.  Against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import compare, to_np

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


def matrix(lens, m, seed):
    rng = np.random.default_rng(seed)
    colptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rowids = np.concatenate([rng.choice(m, k, replace=False) for k in lens]).astype(np.int32)
    values = ((rng.integers(0, 1 << 24, rowids.size) + 1) * 2.0 ** -24).astype(np.float32)
    return synth.CSC(m, lens.size, colptr, rowids, values)


def multiply(spv, M, A, S, semiring=0):
    rng = np.random.default_rng(S.size)
    xv = (rng.random(S.size) + 0.1).astype(np.float32) if semiring == 0 else rng.integers(0, 1 << 30, S.size).astype(np.int32)
    yi, yv, _ = M.spmspv(torch.as_tensor(S).cuda(), torch.as_tensor(xv).cuda(), semiring, True)
    oi, ov, W = oracle.spmspv(A, S, xv, semiring, sorted_output=True)
    compare(semiring, yi, yv, oi, ov, True)
    assert M.last_stats()["W"] == W


@pytest.fixture(scope="module", params=[(1, 0), (7, 0), (30, 31), (900, 100)])
def even(spv, request):
    k, more = request.param
    n = 40001 if k < 900 else 3001
    lens = np.random.default_rng(k).integers(k, k + more + 1, n)
    assert lens.max() <= 2 * lens.mean()
    A = matrix(lens, 9973, k)
    return A, spv.Matrix.from_csc(A)


@pytest.mark.parametrize("shape", [(256, 4), (256, 8), (256, 16), (512, 4), (512, 8), (1024, 4), (1024, 8)])
@pytest.mark.parametrize("tile", [8, 13])
def test_even_columns(spv, even, shape, tile):
    A, M = even
    s = M.schedule
    s.scatter_block, s.scatter_items = shape
    s.tile_log2, s.launch = tile, 1
    M.schedule = s
    rng = np.random.default_rng(tile)
    for f in (1, 2500, A.n - 1, A.n):
        multiply(spv, M, A, rng.permutation(A.n)[:f].astype(np.int32), f % 2)


@pytest.mark.parametrize("f", [16, 300, 4100, 20000])
def test_heaviest_columns(spv, f):
    lens = np.minimum(2047, 20000 / (np.arange(30011) + 1) ** 0.8).astype(np.int64)
    A = matrix(lens, 50021, 3)
    M = spv.Matrix.from_csc(A)
    multiply(spv, M, A, np.arange(f, dtype=np.int32))
    multiply(spv, M, A, np.arange(f, dtype=np.int32), 1)


def test_frontiers_of_uneven_columns(spv):
    """Push BFS of a graph whose hubs come first, and of one with even columns."""
    for lens in (np.minimum(2047, 9000 / (np.arange(9001) + 1) ** 0.7).astype(np.int64) + 1,
                 np.random.default_rng(2).integers(5, 9, 60001)):
        A = matrix(lens, lens.size, 4)
        M = spv.Matrix.from_csc(A, pattern=True)
        for semiring in (1, 2):
            lev, par, nl = M.bfs(3, semiring=semiring, parents=semiring == 1)
            olev, opar, onl = oracle.bfs(A, 3)
            assert nl == onl and np.array_equal(to_np(lev), olev)
            if semiring == 1:
                assert np.array_equal(to_np(par), opar)
