"""Per-response results of the reduce do not depend on what else
is in the batch: a chunk of its groups gives the same bits."""
import numpy as np
import pytest

from gpu_util import down, torch_dev, up

pytestmark = pytest.mark.gpu


def _reduce(torch, dev, a, b, mask, g, ng):
    from paper_2607_24062_amd import acrl
    B, L = a.shape
    out = acrl.acrl_discrepancy_reduce(B, L, ng, up(torch, dev, a.reshape(-1)), up(torch, dev, b.reshape(-1)),
                                       up(torch, dev, mask.reshape(-1)), up(torch, dev, g.astype(np.int32)))
    return {k: down(v) for k, v in out.items()}


# batches above and chunks below 256 responses
@pytest.mark.parametrize("B,L,sizes", [(300, 1028, (5,)), (300, 4097, (12,)), (270, 9000, (8,)), (1100, 40, (11,)),
                                       (1100, 40, (64, 3)), (1500, 9, (1, 33)), (200, 40, (70, 3)), (1000, 9, (300, 7))])
def test_chunk_of_a_batch_reproduces_it(B, L, sizes):
    torch, dev = torch_dev()
    r = np.random.default_rng(B + L)
    g = np.repeat(np.arange(B), np.resize(sizes, B))[:B]
    ng = int(g[-1]) + 1
    mask = (r.random((B, L)) < 0.8).astype(np.uint8)
    a = np.log(r.uniform(1e-5, 1, size=(B, L))).astype(np.float32)
    b = np.minimum(a + r.normal(0, 0.1, size=(B, L)), 0).astype(np.float32)
    whole = _reduce(torch, dev, a, b, mask, g, ng)
    for first, last in ((0, 1), (1, 3), (2, 7)):  # groups
        first, last = min(first, ng - 1), min(last, ng)
        rows = np.flatnonzero((g >= first) & (g < last))
        got = _reduce(torch, dev, a[rows], b[rows], mask[rows], g[rows] - first, last - first)
        for k in ("seq_len", "seq_sum_d", "seq_sum_logratio", "seq_mean_d"):
            assert np.array_equal(got[k], whole[k][rows]), (k, first)
