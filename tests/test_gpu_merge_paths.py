"""GPU parity of the LDS merge where it changes its way through a bucket: entry
counts around the registers of one workgroup, a hub row that takes most of a
bucket's entries, more unique rows than the LDS list holds, tiles cut off in the
middle of a bitmap word, and batches that mix such buckets, each against the
oracle."""
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


def matrix(m, n, hub_share, hub_zero=False):
    """n columns of one entry, `hub_share` of them in row 5, the others spread
    evenly over the rows."""
    rng = np.random.default_rng(m + n)
    rows = (np.arange(n, dtype=np.int64) * m // max(n, 1)).astype(np.int32)
    hub = rng.random(n) < hub_share
    rows[hub] = 5
    values = ((rng.integers(0, 1 << 24, n) + 1) * 2.0 ** -24).astype(np.float32)
    if hub_zero:
        values[hub] = -0.0
    return synth.CSC(m, n, np.arange(n + 1, dtype=np.int32), rows, values)


def x_values(semiring, f, rng):
    if semiring == 0:
        return ((rng.integers(0, 1 << 24, f) + 1) * 2.0 ** -24).astype(np.float32)
    if semiring == 1:
        return rng.integers(-(1 << 31), (1 << 31) - 1, f, endpoint=True).astype(np.int32)
    return (rng.random(f) < 0.3).astype(np.uint8)


def run(spv, A, semiring, block):
    M = spv.Matrix.from_csc(A)
    d = spv.spmspv_effective_schedule(M.handle, A.n, 0, semiring).as_dict()
    d.update(tile_log2=14, merge_block=block, merge_variant=0, launch=0)
    M.schedule = spv.Schedule(**d)
    rng = np.random.default_rng(semiring)
    xi = rng.permutation(A.n).astype(np.int32)
    xv = x_values(semiring, A.n, rng)
    yi, yv, nnz = M.spmspv(torch.from_numpy(xi).cuda(), torch.from_numpy(xv).cuda(), semiring, True)
    compare(semiring, yi[:nnz], yv[:nnz], *oracle.spmspv(A, xi, xv, semiring)[:2], sorted_output=True)


@pytest.mark.parametrize("block", [256, 512, 1024])
@pytest.mark.parametrize("over", [-1, 0, 1])
@pytest.mark.parametrize("semiring", [0, 1, 2])
def test_entries_per_workgroup(spv, block, over, semiring):
    run(spv, matrix(9001, 8 * block + over, 0.3), semiring, block)


@pytest.mark.parametrize("hub_share,hub_zero", [(0.0, False), (0.02, False), (0.5, False), (0.5, True), (1.0, False),
                                                (1.0, True)])
@pytest.mark.parametrize("semiring", [0, 1, 2])
def test_hub_row(spv, hub_share, hub_zero, semiring):
    run(spv, matrix(1000, 30011, hub_share, hub_zero), semiring, 1024)


@pytest.mark.parametrize("m", [8191, 8193, 16383, 16384 + 33, 40001])
@pytest.mark.parametrize("semiring", [0, 1, 2])
def test_more_rows_than_the_list(spv, m, semiring):
    run(spv, matrix(m, m + 777, 0.01), semiring, 512)


@pytest.mark.parametrize("semiring", [0, 1, 2])
def test_batch_of_mixed_buckets(spv, semiring):
    A = matrix(8191, 60013, 0.2)
    M = spv.Matrix.from_csc(A)
    d = spv.spmspv_effective_schedule(M.handle, A.n, 0, semiring).as_dict()
    d.update(tile_log2=13, merge_variant=0, launch=0)   # 64 KB of fp64 cells: the shortened list
    M.schedule = spv.Schedule(**d)
    M.attach_batch(8, max_f=8 * A.n, max_products=8 * A.nnz)
    rng = np.random.default_rng(semiring)
    parts = [rng.choice(A.n, f, replace=False).astype(np.int32) for f in (0, 1, 4095, 4097, 60013, 0, 7900, 30000)]
    xi = np.concatenate(parts)
    xv = x_values(semiring, xi.size, rng)
    off = np.concatenate([[0], np.cumsum([p.size for p in parts])]).astype(np.int64)
    yo, yi, yv, _ = M.spmspv_batch(torch.from_numpy(off).cuda(), torch.from_numpy(xi).cuda(),
                                   torch.from_numpy(xv).cuda(), semiring)
    yo = to_np(yo)
    for b, p in enumerate(parts):
        ref = oracle.spmspv(A, p, xv[off[b]:off[b + 1]], semiring)[:2]
        compare(semiring, yi[yo[b]:yo[b + 1]], yv[yo[b]:yo[b + 1]], *ref, sorted_output=True)


@pytest.mark.parametrize("n", [30011, 200003])
@pytest.mark.parametrize("semiring", [0, 1, 2])
def test_long_bucket_among_short_ones(spv, n, semiring):
    """274 buckets of 256 rows: the mean asks for fewer threads, the hub's bucket takes the long way."""
    A = matrix(70001, n, 0.5)
    M = spv.Matrix.from_csc(A)
    s = M.schedule
    s.tile_log2 = 8
    M.schedule = s
    rng = np.random.default_rng(semiring)
    xi = rng.permutation(A.n).astype(np.int32)
    xv = x_values(semiring, A.n, rng)
    yi, yv, nnz = M.spmspv(torch.from_numpy(xi).cuda(), torch.from_numpy(xv).cuda(), semiring, True)
    compare(semiring, yi[:nnz], yv[:nnz], *oracle.spmspv(A, xi, xv, semiring)[:2], sorted_output=True)
