"""Per-response and per-group results of the reduce do not depend on what else
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


# batches above and chunks below 256 responses and the one-workgroup sums' bounds;
# groups that start anywhere in a wavefront, with 64 responses, and (within the one-workgroup sums) more
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
        for k in ("group_y", "group_nseq"):
            assert np.array_equal(got[k], whole[k][first:last]), (k, first)
    # a batch of one group's responses after empty ones: the batch's statistics are that group's, in all bits
    rows = np.flatnonzero(g == 1)
    one = _reduce(torch, dev, a[rows], b[rows], mask[rows], np.zeros(rows.size), 1)
    for pad in (1, 7, 20):
        z = np.zeros((pad, L), np.uint8)
        got = _reduce(torch, dev, np.concatenate([a[:pad], a[rows]]), np.concatenate([b[:pad], b[rows]]),
                      np.concatenate([z, mask[rows]]), np.repeat([0, 1], [pad, rows.size]), 2)
        assert np.array_equal(got["stats"], one["stats"]), pad


@pytest.mark.parametrize("B", [1, 5, 64, 1023, 1024])
@pytest.mark.parametrize("ids", ["gaps", "outside", "one", "shuffled"])
def test_group_ranges(B, ids):
    """The one-workgroup group sums over empty groups, ids outside [0, n_groups) (INT32_MIN and INT32_MAX among
    them) before, between and after the others, and orders that are none."""
    torch, dev = torch_dev()
    r = np.random.default_rng(B)
    ng, L = 61, 5
    g = np.sort(r.integers(0, 20, size=B) * 3 + 1)
    if ids == "outside":
        g = np.sort(r.choice([-2 ** 31, -7, -1, 0, 2, 30, 60, 61, 99, 2 ** 31 - 1], size=B))
    if ids == "one":
        g = np.full(B, 60)
    if ids == "shuffled":
        g = r.permutation(np.concatenate([g[:-1], [-3]]))
    a = np.log(r.uniform(1e-5, 1, size=(B, L))).astype(np.float32)
    b = np.minimum(a + r.normal(0, 0.1, size=(B, L)), 0).astype(np.float32)
    mask = (r.random((B, L)) < 0.7).astype(np.uint8)
    got = _reduce(torch, dev, a, b, mask, g, ng)
    d = np.abs(np.exp(a.astype(np.float64)) - np.exp(b.astype(np.float64))) * mask
    n = mask.sum(1)
    y, cnt = np.zeros(ng), np.zeros(ng, int)
    for i in range(B):
        if 0 <= g[i] < ng and n[i]:
            y[g[i]] += d[i].sum() / n[i]
            cnt[g[i]] += 1
    y /= np.maximum(cnt, 1)
    assert np.array_equal(got["group_nseq"], cnt)
    np.testing.assert_allclose(got["group_y"], y.astype(np.float32), rtol=1e-6, atol=0)
    assert got["stats"][9] == cnt.sum() and got["stats"][7] == (cnt > 0).sum()
