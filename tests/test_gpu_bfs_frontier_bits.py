"""The direction-switching BFS hands each frontier on as a bitmap that the
merges and the pull emit write: levels and parents against the oracle where
bitmap words, merge tiles and emit workgroups end, with both merges, with and
without the captured levels, and a plain pull multiply between searches, which
needs the bitmap zero again."""
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
    synth.build(force=False)
    return spv


def graph(n):
    """Symmetric: random edges (pull levels in the middle) and a path of the
    last vertices (push levels at the end)."""
    rng = np.random.default_rng(n)
    tail = min(n // 8, 12)
    core = n - tail
    a, b = rng.integers(0, core, (2, 4 * n)) if core > 1 else np.zeros((2, 0), np.int64)
    path = np.arange(max(core - 1, 0), n)
    rows, cols = np.concatenate([a, path[:-1]]), np.concatenate([b, path[1:]])
    both = np.concatenate([rows, cols]).astype(np.int32), np.concatenate([cols, rows]).astype(np.int32)
    colptr, rowids = synth.coo_to_csc(n, n, *both)
    return synth.CSC(n, n, colptr, rowids, synth.values(rowids.size, 5))


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 31, 33, 256, 8191, 8193, 16385, 70001])
def test_search_pull_search(spv, n, variant):
    A = graph(n)
    M = spv.Matrix.from_csc(A, flags=spv.SYMMETRIC)
    rng = np.random.default_rng(n)
    for k, root in enumerate([0, n - 1, int(rng.integers(0, n))]):
        s = M.schedule
        s.merge_variant, s.direction = variant, 0
        M.schedule = s
        fl = spv.DIRECTION_OPT | (spv.USE_GRAPH if k % 2 else 0)
        olev, opar, onl = oracle.bfs(A, root)
        lev, par, nl = M.bfs(root, spv.MIN_SELECT2ND_I32, flags=fl)
        assert nl == onl and np.array_equal(to_np(lev), olev) and np.array_equal(to_np(par), opar)
        lev, _, nl = M.bfs(root, spv.OR_AND_BOOL, flags=fl)
        assert nl == onl and np.array_equal(to_np(lev), olev)
        s.direction = 1
        M.schedule = s
        x = rng.choice(n, max(n // 50, 1), replace=False).astype(np.int32)
        yi, yv, _ = M.spmspv(torch.as_tensor(x).cuda(), None, semiring=1, flags=spv.X_VAL_IS_INDEX)
        compare(1, yi, yv, *oracle.spmspv(A, x, x, 1, sorted_output=True)[:2], sorted_output=True)
