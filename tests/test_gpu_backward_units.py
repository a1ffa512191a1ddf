"""The LM-head backward at the edges of its transposed operand images (32-row
chunks of W and H, 256-column tiles) and where the dZ pass has more units than
workgroups, so that they claim units from the XCDs' queues.

Bound as in test_gpu_backward: dZ is rounded to bf16, so an element is off by
at most 2^-8 times the sum of its terms' magnitudes."""
import numpy as np
import pytest

import oracle
from gpu_util import down, torch_dev, up, up_bf16
from test_gpu_backward import BOUND, _check_rows
from test_gpu_product_slices import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V,d", [(1, 31, 128), (31, 33, 128), (32, 32, 256), (33, 257, 384), (65, 95, 640)])
def test_transposed_images_at_chunk_edges(T, V, d):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    H, W, ids, coef, lse, rows = _case(T, V, d, T * V + d, T)
    dh, dw = acrl.acrl_lm_head_backward(up_bf16(torch, dev, H), up_bf16(torch, dev, W), up(torch, dev, ids),
                                        up(torch, dev, coef), up(torch, dev, lse))
    rdh, rdw, rdha, rdwa = oracle.lm_head_backward(H[rows], W, ids[rows], coef[rows].astype(np.float64), 1.0,
                                                   want_abs=True)
    _check_rows(down(dh)[rows], rdh, rdha, "dH")
    _check_rows(down(dw), rdw, rdwa, "dW")


# 6 and 5 token tiles over 594 vocabulary tiles; dW of 10 and 14 chunks of K in strips of output tiles, the last
# strip, vocabulary tile and hidden tile partial; with one chunk pair of K
@pytest.mark.parametrize("T,V,d", [(1531, 151936, 128), (1100, 151936, 128), (300, 65801, 896), (420, 33001, 2176),
                                   (20, 100001, 640)])
def test_units_from_queues_and_strips(T, V, d):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    g = torch.Generator(device=dev)
    g.manual_seed(T)
    h = torch.randn((T, d), generator=g, device=dev).bfloat16()
    w = (torch.randn((V, d), generator=g, device=dev) * 2.3 / d ** 0.5).bfloat16()
    ids = torch.randint(0, V, (T,), generator=g, device=dev, dtype=torch.int32)
    coef = torch.randn(T, generator=g, device=dev) / T
    z = h.float() @ w.float().T
    lse = torch.logsumexp(z, 1)
    dz = torch.exp(z - lse[:, None]).neg_()
    dz.scatter_add_(1, ids[:, None].long(), torch.ones(T, 1, device=dev))
    dz *= coef[:, None]
    dh, dw = acrl.acrl_lm_head_backward(h, w, ids, coef, lse)
    for got, a, b in ((dh, dz, w.float()), (dw, dz.T.contiguous(), h.float())):
        ref, mag = a @ b, a.abs() @ b.abs()
        assert bool(((got - ref).abs() <= BOUND * mag + 1e-6 * ref.abs().max()).all())
