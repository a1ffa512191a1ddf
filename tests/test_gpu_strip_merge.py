"""The merge of the vocabulary strips' states where a strip holds no
probability at all: every logit of it -inf.  Its own entropy sum is 0 * -inf
there and must not reach the row's."""
import numpy as np
import pytest

from cases import TOL_LOGP, random_bf16, tol_entropy
from gpu_util import down, torch_dev, up, up_bf16

pytestmark = pytest.mark.gpu


# few rows, V = 2100: strips of one vocabulary tile, so whole strips are empty
@pytest.mark.parametrize("T", [1, 70, 200])
@pytest.mark.parametrize("empty", [(0, 1), (3, 5), (8, 9), (1, 8)])
def test_strips_without_probability(T, empty):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    V, d = 2100, 128
    h = up_bf16(torch, dev, random_bf16((T, d), 51))
    w = up_bf16(torch, dev, random_bf16((V, d), 52, std=2.5 / d ** 0.5))
    h[:, 0] = 1.0
    w[:, 0] = 0.0
    lo, hi = 256 * empty[0], min(256 * empty[1], V)
    w[lo:hi, 0] = -float("inf")
    keep = np.r_[0:lo, hi:V]
    ids = np.random.default_rng(53).choice(keep, size=T).astype(np.int32)
    hq = torch.zeros(h.shape, dtype=torch.uint8, device=dev)
    wq = torch.zeros(w.shape, dtype=torch.uint8, device=dev)
    out = acrl.acrl_score_pi_mu(h, w, hq, None, wq, None, acrl.SCALE_PER_TENSOR, up(torch, dev, ids),
                                policies=acrl.POLICY_PI)
    z = down(h.double()) @ down(w.double()[torch.from_numpy(keep).to(dev)]).T
    m = z.max(1, keepdims=True)
    lse = m[:, 0] + np.log(np.exp(z - m).sum(1))
    p = np.exp(z - lse[:, None])
    za = z[np.arange(T), np.searchsorted(keep, ids)]
    assert np.abs(down(out["logp_pi"]) - (za - lse)).max() <= TOL_LOGP
    assert np.abs(down(out["entropy_pi"]) - (lse - (p * z).sum(1))).max() <= tol_entropy(V)
