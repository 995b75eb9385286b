"""Merge threads: a default schedule takes them from the call, from what the
heaviest columns could bring too; a schedule that was set, tuned or given
for batches is used and reported as it is.  Results at every choice, with the
heaviest columns in x, against the oracle."""
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


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


def x_values(semiring, f):
    rng = np.random.default_rng(f)
    if semiring == 0:
        return (rng.random(f) + 0.1).astype(np.float32)
    return rng.integers(0, 1 << 30, f).astype(np.int32) if semiring == 1 else (rng.random(f) < 0.7).astype(np.uint8)


def check(spv, M, A, S, semiring, flags=0, T=None):
    xv = x_values(semiring, S.size)
    yi, yv, _ = M.spmspv(dev(S), dev(xv), semiring, True, flags=flags)
    compare(semiring, yi, yv, *oracle.spmspv(A if T is None else T, S, xv, semiring, sorted_output=True)[:2],
            sorted_output=True)


def transpose(A):
    cols = np.repeat(np.arange(A.n, dtype=np.int32), np.diff(A.colptr))
    order = np.lexsort((cols, A.rowids))
    colptr = np.concatenate([[0], np.cumsum(np.bincount(A.rowids, minlength=A.m))]).astype(np.int32)
    return synth.CSC(A.n, A.m, colptr, cols[order], A.values[order])


@pytest.mark.parametrize("semiring", [0, 1, 2])
def test_default_follows_the_call(spv, semiring):
    A = synth.rmat(15, 16, seed=41, symmetrize=True)
    M = spv.Matrix.from_csc(A, flags=spv.WITH_TRANSPOSE)
    T = transpose(A)
    heavy = np.argsort(-A.degrees(), kind="stable").astype(np.int32)
    nb = -(-A.m >> M.schedule.tile_log2)
    seen = set()
    for f in (1, 20, 300, 3000, 20000):
        eff = spv.spmspv_effective_schedule(M.handle, f, 0, semiring)
        most = min(f * int(A.degrees().max()), A.nnz) / nb
        mean = f * A.nnz / A.n / nb
        assert eff.merge_block == (256 if most <= 512 else 512 if mean <= 2048 else 1024), (f, most, mean)
        seen.add(eff.merge_block)
        check(spv, M, A, heavy[:f], semiring)
        check(spv, M, A, heavy[:f], semiring, spv.LEFT, T)
    assert seen == {256, 512, 1024}
    G = synth.grid(20, 20, 20)
    N = spv.Matrix.from_csc(G)
    assert spv.spmspv_effective_schedule(N.handle, 50, 0, semiring).merge_block == 256
    check(spv, N, G, np.arange(50, dtype=np.int32), semiring)


@pytest.mark.parametrize("block", [256, 512, 1024])
def test_given_schedules_are_kept(spv, block):
    A = synth.rmat(12, 16, seed=42, symmetrize=True)
    M = spv.Matrix.from_csc(A)
    M.attach_batch(8, max_f=8 * A.n, max_products=8 * A.nnz)
    assert spv.spmspv_get_batch_schedule(M.handle, 8).merge_block == 512
    heavy = np.argsort(-A.degrees(), kind="stable").astype(np.int32)

    def batch():
        xi = np.concatenate([heavy[k::8][:200] for k in range(8)])
        off = np.arange(9, dtype=np.int64) * 200
        xv = x_values(0, xi.size)
        yo, yi, yv, _ = M.spmspv_batch(dev(off), dev(xi), dev(xv), 0)
        yo = to_np(yo)
        for b in range(8):
            ref = oracle.spmspv(A, xi[off[b]:off[b + 1]], xv[off[b]:off[b + 1]], 0)[:2]
            compare(0, yi[yo[b]:yo[b + 1]], yv[yo[b]:yo[b + 1]], *ref, sorted_output=True)

    batch()
    s = M.schedule
    s.merge_block = block
    M.schedule = s
    for f in (1, 50, 4000):
        assert spv.spmspv_effective_schedule(M.handle, f).merge_block == block
        check(spv, M, A, heavy[:f], 0)
    assert spv.spmspv_get_batch_schedule(M.handle, 8).merge_block == block
    batch()
    M.schedule = None
    s = spv.spmspv_get_batch_schedule(M.handle, 8)
    s.merge_block = block
    spv.spmspv_set_batch_schedule(M.handle, s)
    assert spv.spmspv_get_batch_schedule(M.handle, 8).merge_block == block
    batch()


def test_tuned_schedules_are_kept(spv):
    A = synth.rmat(13, 8, seed=43, symmetrize=True)
    M = spv.Matrix.from_csc(A)
    M.autotune(0, (1e-3, 1e-1), reps=2)
    for f in (8, 800):
        tuned = spv.spmspv_tuned_schedule(M.handle, f)
        assert spv.spmspv_effective_schedule(M.handle, f, spv.AUTO_SCHEDULE).merge_block == tuned.merge_block
