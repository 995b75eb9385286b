"""Schedules at the largest bucket counts that the scatter's LDS holds: with four
items per thread the expansion needs more LDS than the scatter there, so
these calls take scan and scatter.  Each against the oracle."""
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


def lds(block, items, nb):
    """Bytes of (scatter, expansion) as the library computes them."""
    c = block * items
    scatter = (2 * nb + 64 + c // 16) * 4 + max((c + 2) * 2 + (c + 1) * 8, (c + 64) * 8)
    expand = (c + 64) * 8 + (2 * nb + 64) * 4 + (3 * block + 1) * 4 + c // 32 * 8
    return scatter, expand


@pytest.mark.parametrize("block,items,nb", [(1024, 4, 14400), (1024, 4, 14700), (1024, 4, 15060), (512, 4, 17600),
                                            (256, 4, 18970)])
def test_push(spv, block, items, nb):
    scatter, expand = lds(block, items, nb)
    assert scatter + 1024 <= 160 * 1024 and (nb == 14400) == (expand + 1024 <= 160 * 1024)
    m, n = nb * 256 - 7, 5000
    rng = np.random.default_rng(nb)
    lens = rng.integers(0, 30, n)
    colptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rowids = rng.integers(0, m, int(lens.sum())).astype(np.int32)
    A = synth.CSC(m, n, colptr, rowids, (rng.random(rowids.size) + 0.1).astype(np.float32))
    M = spv.Matrix.from_csc(A)
    s = M.schedule
    s.tile_log2, s.scatter_block, s.scatter_items, s.launch = 8, block, items, 1
    M.schedule = s
    S = rng.permutation(n)[:1500].astype(np.int32)
    xv = (rng.random(1500) + 0.1).astype(np.float32)
    yi, yv, _ = M.spmspv(torch.as_tensor(S).cuda(), torch.as_tensor(xv).cuda(), 0, True)
    compare(0, yi, yv, *oracle.spmspv(A, S, xv, 0, sorted_output=True)[:2], sorted_output=True)
