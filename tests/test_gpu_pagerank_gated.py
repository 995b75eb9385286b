"""PageRank with the direction taken on the device where push and pull steps mix
in one run, and multiplies on the same handle afterwards: a push step must not
leave x bits behind that a later pull reads.  Against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import compare, to_np
from test_gpu_pagerank import check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PUSH, PULL = 2, 9


@pytest.fixture(scope="module")
def spv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1610_07902_amd as spv
    spv.load_library()
    oracle.build(force=False)
    synth.build(force=False)
    return spv


def network(spv, above, below, f):
    """Class `above` for an x of more than f entries, else `below` (the first
    feature is log2(1 + f), unscaled)."""
    p = np.zeros(spv.MLP_PARAMS, np.float32)
    w1, b1 = p[:64 * 6].reshape(64, 6), p[64 * 6:64 * 7]
    w2 = p[64 * 7:64 * 7 + 64 * 64].reshape(64, 64)
    w3, b3 = p[-10 - 640:-10].reshape(10, 64), p[-10:]
    w1[0, 0], b1[0] = 64.0, -64.0 * np.log2(1.5 + f)
    w2[0, 0] = 1.0
    w3[above, 0] = 1.0e3
    b3[below] = 1.0
    return p, np.zeros(6, np.float32), np.ones(6, np.float32)


def pull_multiply(spv, M, A, rng):
    """One pull multiply per semiring with few x entries."""
    s = M.schedule
    s.direction = 1
    M.schedule = s
    x = np.sort(rng.choice(A.n, 40, replace=False)).astype(np.int32)
    xf = (rng.random(40) + 0.5).astype(np.float32)
    for semiring, xv in ((0, xf), (1, x), (2, np.ones(40, np.uint8))):
        yi, yv, _ = M.spmspv(torch.as_tensor(x).cuda(), torch.as_tensor(xv).cuda(), semiring, True)
        compare(semiring, yi, yv, *oracle.spmspv(A, x, xv, semiring, sorted_output=True)[:2], sorted_output=True)
    s.direction = 0
    M.schedule = s


@pytest.mark.parametrize("above,below", [(PUSH, PULL), (PULL, PUSH)])
def test_directions_mix_in_one_run(spv, above, below):
    A = synth.rmat(13, 16, seed=75, symmetrize=True, with_values=False)
    M = spv.Matrix.from_csc(A, pattern=True, flags=spv.SYMMETRIC)
    _, steps, active = oracle.pagerank(A, 0.85, 1e-6, 100)
    f = int(active[steps - 4] + active[steps - 3]) // 2
    assert active[0] > f > active[steps - 1] > 0   # the last steps are the other class
    M.load_selector(*network(spv, above, below, f))
    r, it = M.pagerank(0.85, 1e-6, 100, flags=spv.USE_SELECTOR)          # read on the host: which classes
    check(A, r, it, 1e-6, 100)
    assert {PUSH, PULL} == set(M.selector_classes())
    r, it = M.pagerank(0.85, 1e-6, 100, flags=spv.USE_SELECTOR | spv.USE_GRAPH)
    check(A, r, it, 1e-6, 100)
    pull_multiply(spv, M, A, np.random.default_rng(1))


@pytest.mark.parametrize("above,below", [(PUSH, PUSH), (PULL, PUSH), (PULL, PULL)])
def test_pull_multiply_afterwards(spv, above, below):
    A = synth.rmat(13, 16, seed=76, symmetrize=True, with_values=False)
    M = spv.Matrix.from_csc(A, pattern=True, flags=spv.SYMMETRIC)
    rng = np.random.default_rng(2)
    for _ in range(2):
        M.load_selector(*network(spv, above, below, 2000))
        r, it = M.pagerank(0.85, 1e-6, 100, flags=spv.USE_SELECTOR | spv.USE_GRAPH)
        check(A, r, it, 1e-6, 100)
        pull_multiply(spv, M, A, rng)
        x = np.sort(rng.choice(A.n, 30, replace=False)).astype(np.int32)
        M.load_selector(*network(spv, PULL, PULL, 1))
        xv = np.ones(30, np.float32)
        yi, yv, _ = M.spmspv(torch.as_tensor(x).cuda(), torch.as_tensor(xv).cuda(), 0, True, flags=spv.USE_SELECTOR)
        compare(0, yi, yv, *oracle.spmspv(A, x, xv, 0, sorted_output=True)[:2], sorted_output=True)
        lev, _, nl = M.bfs(int(x[0]), flags=spv.DIRECTION_OPT)
        olev, _, onl = oracle.bfs(A, int(x[0]))
        assert nl == onl and np.array_equal(to_np(lev), olev)
