"""GPU parity of the multiply at the limits of the expansion kernel, which takes
the place of scan and scatter where no column is longer than 2047 entries:
column lengths on both sides of that line, x lengths around its tiles, chunk
shapes, more buckets than threads, empty columns, a mask, and the frontier
form (BFS, PageRank), each against the oracle."""
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


def matrix(longest, m=70001, n=9001, seed=3):
    """Columns of 0..60 entries, a few of exactly `longest`."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 61, n)
    lens[rng.random(n) < 0.3] = 0
    lens[rng.choice(n, 12, replace=False)] = longest
    colptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rowids = np.concatenate([rng.choice(m, k, replace=False) for k in lens]).astype(np.int32)
    values = ((rng.integers(0, 1 << 24, rowids.size) + 1) * 2.0 ** -24).astype(np.float32)
    return synth.CSC(m, n, colptr, rowids, values)


def x_values(semiring, f, rng):
    if semiring == 0:
        return ((rng.integers(0, 1 << 24, f) + 1) * 2.0 ** -24).astype(np.float32)
    if semiring == 1:
        return rng.integers(-(1 << 30), 1 << 30, f).astype(np.int32)
    return (rng.random(f) < 0.7).astype(np.uint8)


@pytest.fixture(scope="module", params=[2047, 2048])
def at_limit(spv, request):
    A = matrix(request.param)
    assert int(A.degrees().max()) == request.param
    return A, spv.Matrix.from_csc(A)


@pytest.mark.parametrize("f", [0, 1, 15, 16, 17, 255, 256, 257, 4099, 9001])
@pytest.mark.parametrize("semiring", [0, 1, 2])
def test_tiles(spv, at_limit, f, semiring):
    A, M = at_limit
    rng = np.random.default_rng(f + semiring)
    S = rng.permutation(A.n)[:f].astype(np.int32)
    xv = x_values(semiring, f, rng)
    for masked in (False, True):
        member = rng.random(A.m) < 0.4 if masked else np.zeros(A.m, bool)
        words = np.packbits(member, bitorder="little")
        words = np.concatenate([words, np.zeros(-words.size % 4, np.uint8)]).view(np.int32)
        gi, gv, nnz = M.spmspv(torch.as_tensor(S).cuda(), torch.as_tensor(xv).cuda(), semiring, True,
                               mask=torch.as_tensor(words.copy()).cuda() if masked else None)
        oi, ov, W = oracle.spmspv(A, S, xv, semiring, sorted_output=True)
        keep = ~member[oi]
        compare(semiring, gi, gv, oi[keep], ov[keep], True)
        st = M.last_stats()
        assert st["W"] == W and st["err"] == 0 and st["maxlen"] == (int(A.degrees()[S].max()) if f else 0)
        assert st["fnz"] == int((A.degrees()[S] > 0).sum())


@pytest.mark.parametrize("shape", [(256, 4), (256, 8), (256, 16), (512, 4), (512, 8), (1024, 4), (1024, 8)])
@pytest.mark.parametrize("tile", [8, 14])
def test_chunk_shapes(spv, shape, tile):
    """274 buckets (more than a 256-thread workgroup reserves for at once) and five."""
    A = matrix(2047, seed=5)
    M = spv.Matrix.from_csc(A)
    s = M.schedule
    s.scatter_block, s.scatter_items = shape
    s.tile_log2 = tile
    M.schedule = s
    rng = np.random.default_rng(7)
    for f in (3000, A.n):
        S = rng.permutation(A.n)[:f].astype(np.int32)
        xv = x_values(0, f, rng)
        gi, gv, _ = M.spmspv(torch.as_tensor(S).cuda(), torch.as_tensor(xv).cuda(), 0, True)
        oi, ov, _ = oracle.spmspv(A, S, xv, 0, sorted_output=True)
        compare(0, gi, gv, oi, ov, True)


def test_repeated_index_reports_and_recovers(spv):
    """More products than stored entries: an error, and the next call is right."""
    A = matrix(2047, seed=6)
    M = spv.Matrix.from_csc(A)
    S = np.repeat(np.nonzero(A.degrees() == 2047)[0][:2].astype(np.int32), 4000)
    xv = np.ones(S.size, np.float32)
    with pytest.raises(spv.SpmspvError) as e:
        M.spmspv(torch.as_tensor(S).cuda(), torch.as_tensor(xv).cuda(), 0, True)
    assert e.value.status == spv.EDEVICE
    S = np.arange(A.n, dtype=np.int32)
    xv = np.ones(A.n, np.float32)
    gi, gv, _ = M.spmspv(torch.as_tensor(S).cuda(), torch.as_tensor(xv).cuda(), 0, True)
    oi, ov, _ = oracle.spmspv(A, S, xv, 0, sorted_output=True)
    compare(0, gi, gv, oi, ov, True)


@pytest.mark.parametrize("graph", [False, True])
def test_frontiers(spv, graph):
    A = synth.grid(37, 23, 11)
    M = spv.Matrix.from_csc(A, pattern=True)
    for semiring in (1, 2):
        lev, par, nl = M.bfs(5, semiring=semiring, parents=semiring == 1, flags=spv.USE_GRAPH if graph else 0)
        olev, opar, onl = oracle.bfs(A, 5)
        assert nl == onl and np.array_equal(to_np(lev), olev)
        if semiring == 1:
            assert np.array_equal(to_np(par), opar)
