"""GPU parity of the per-response reductions at the edges of their workgroup
sizes (reduce: 64 threads up to 256 slots, 256 up to 8192, 1024 above;
surrogate: 256 up to 1024 slots or of more than 256 responses, 1024 above; four
slots a thread at a time) and of the one-workgroup group and
batch sums (up to 1024 responses in 64 groups), slots 16-byte aligned and not.

Bounds as in the other tests of these entry points: both sides sum the same
fp32 inputs in fp64, so the sums agree to rounding (1e-12) and the fp32
outputs to one rounding."""
import numpy as np
import pytest

import oracle
from gpu_util import down, torch_dev, up

pytestmark = pytest.mark.gpu

# (B, L, groups)
SHAPES = [(3, 256, 2), (3, 257, 2), (2, 1023, 2), (2, 1024, 1), (3, 1025, 2), (2, 4096, 2), (2, 4097, 1), (2, 8192, 1),
          (2, 8193, 1), (1, 9000, 1),
          (256, 1028, 32), (257, 1028, 32), (1023, 7, 63), (1024, 8, 64), (1024, 8, 65), (1025, 8, 64), (70, 8, 64)]


def _inputs(B, L, ng):
    r = np.random.default_rng(B * 10007 + L * 31 + ng)
    lens = r.integers(0, L + 1, size=B)  # empty responses among them
    lens[0] = L
    mask = (np.arange(L)[None, :] < lens[:, None]).astype(np.uint8)
    a = np.log(r.uniform(1e-5, 1, size=(B, L))).astype(np.float32)
    b = np.minimum(a + r.normal(0, 0.1, size=(B, L)), 0).astype(np.float32)
    g = r.integers(0, ng, size=B).astype(np.int32)
    return r, mask, a, b, g


def _put(torch, dev, x, offset):
    """x on the device, `offset` elements past a 16-byte boundary."""
    x = np.ascontiguousarray(x).reshape(-1)
    buf = torch.zeros(x.size + offset, dtype=up(torch, dev, x[:1]).dtype, device=dev)
    buf[offset:] = up(torch, dev, x)
    return buf[offset:]


@pytest.mark.parametrize("order", ["sorted", "shuffled"])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("B,L,ng", SHAPES)
def test_reduce_at_workgroup_edges(B, L, ng, offset, order):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    r, mask, a, b, g = _inputs(B, L, ng)
    if order == "sorted":
        g = np.sort(g)
    hp, hm = (r.uniform(0, 9, size=(B, L)).astype(np.float32) for _ in range(2))
    t = lambda x: _put(torch, dev, x, offset)  # noqa: E731
    out = acrl.acrl_discrepancy_reduce(B, L, ng, t(a), t(b), t(mask), up(torch, dev, g), entropy_pi=t(hp),
                                       entropy_mu=t(hm))
    got = {k: down(v) for k, v in out.items()}
    ref = oracle.discrepancy_reduce(B, L, a, b, mask, g, ng, hp, hm)
    assert np.array_equal(got["seq_len"], ref["seq_len"])
    assert np.array_equal(got["group_nseq"], ref["group_nseq"])
    np.testing.assert_allclose(got["seq_sum_d"], ref["seq_sum_d"], rtol=1e-12, atol=1e-15)
    np.testing.assert_allclose(got["seq_sum_logratio"], ref["seq_sum_logratio"], rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(got["seq_mean_d"], ref["seq_mean_d"].astype(np.float32), rtol=1e-6, atol=0)
    np.testing.assert_allclose(got["group_y"], ref["group_y"].astype(np.float32), rtol=1e-6, atol=0)
    np.testing.assert_allclose(got["stats"], ref["stats"], rtol=1e-10, atol=1e-15)
    np.testing.assert_allclose(got["d_tok"], ref["d_tok"].astype(np.float32), rtol=1e-6, atol=0)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("B,L,ng", SHAPES)
def test_surrogate_at_workgroup_edges(B, L, ng, offset):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    r, mask, a, b, g = _inputs(B, L, ng)
    adv = r.normal(size=(B, L)).astype(np.float32)
    wt = r.uniform(0, 3, size=(B, L)).astype(np.float32)
    t = lambda x: _put(torch, dev, x, offset)  # noqa: E731
    coef, loss = acrl.acrl_surrogate(B, L, ng, t(mask), up(torch, dev, g), t(a), t(b), t(adv), True, weight=t(wt))
    rc, rl = oracle.surrogate(B, L, mask, g, ng, a, b, adv, adv_per_token=True, weight=wt,
                              eps_low=float(np.float32(0.2)), eps_high=float(np.float32(0.2)))
    np.testing.assert_allclose(down(coef), rc.astype(np.float32), rtol=1e-6, atol=1e-30)
    # the loss is a sum of terms of both signs: relative to the sum of their magnitudes, at most max w r |A|
    np.testing.assert_allclose(down(loss)[0], rl, rtol=1e-10, atol=1e-11)


def test_one_workgroup_skips_foreign_groups():
    """Group ids outside [0, n_groups) enter no group and no batch sum."""
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    B, L, ng = 6, 40, 3
    _, mask, a, b, _ = _inputs(B, L, ng)
    g = np.array([2, -1, 0, 3, 0, 2], np.int32)
    out = acrl.acrl_discrepancy_reduce(B, L, ng, up(torch, dev, a), up(torch, dev, b), up(torch, dev, mask),
                                       up(torch, dev, g))
    keep = np.isin(g, [0, 1, 2])
    ref = oracle.discrepancy_reduce(int(keep.sum()), L, a[keep], b[keep], mask[keep], g[keep], ng)
    np.testing.assert_allclose(down(out["group_y"]), ref["group_y"].astype(np.float32), rtol=1e-6, atol=0)
    np.testing.assert_allclose(down(out["stats"]), ref["stats"], rtol=1e-10, atol=1e-15)
