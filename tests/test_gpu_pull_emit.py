"""The pull direction's emit at the row counts where its workgroups change from
256 to 512 bitmap words, and where its last workgroup and last word are partial:
multiplies against the oracle and a direction-switching BFS."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import compare, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGE = 512 * 32 * 256


@pytest.fixture(scope="module")
def spv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1610_07902_amd as spv
    spv.load_library()
    oracle.build(force=False)
    synth.build(force=False)
    return spv


@pytest.mark.parametrize("n", [8192, 8193, EDGE - 1, EDGE, EDGE + 1, EDGE + 16384 + 31])
def test_pull(spv, n):
    """Symmetric: a star of the last vertex to every 17th and a path over the last 40."""
    far = np.arange(3, n - 1, 17)
    path = np.arange(n - 41, n - 1)
    a, b = np.concatenate([far, path]), np.concatenate([np.full(far.size, n - 1), path + 1])
    rows, cols = (np.concatenate(p).astype(np.int32) for p in ((a, b), (b, a)))
    key = np.unique(cols.astype(np.int64) * n + rows)
    colptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int32)
    A = synth.CSC(n, n, colptr, (key % n).astype(np.int32), None)
    M = spv.Matrix.from_csc(A, pattern=True, flags=spv.SYMMETRIC)
    s = M.schedule
    s.direction = 1
    M.schedule = s
    rng = np.random.default_rng(n)
    for S in (np.array([n - 1]), np.unique(rng.choice(far, 500)), np.concatenate([far, path])):
        S = np.unique(S).astype(np.int32)
        for semiring, xv in ((0, (rng.random(S.size) + 0.5).astype(np.float32)), (1, S), (2, np.ones(S.size, np.uint8))):
            yi, yv, _ = M.spmspv(torch.as_tensor(S).cuda(), torch.as_tensor(xv).cuda(), semiring, True)
            compare(semiring, yi, yv, *oracle.spmspv(A, S, xv, semiring, sorted_output=True)[:2], sorted_output=True)
    lev, par, nl = M.bfs(n - 41, flags=spv.DIRECTION_OPT)
    olev, opar, onl = oracle.bfs(A, n - 41)
    assert nl == onl and np.array_equal(to_np(lev), olev) and np.array_equal(to_np(par), opar)
