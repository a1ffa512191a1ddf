"""The LM-head backward where its products split K into slices: dH of few rows
over a large vocabulary and dW of a small head over many rows, against the
oracle at the bf16 bound; accumulated and unaligned outputs."""
import numpy as np
import pytest

import oracle
from gpu_util import down, torch_dev, up, up_bf16
from test_gpu_backward import _check_rows

pytestmark = pytest.mark.gpu


def _case(T, V, d, seed, live):
    r = np.random.default_rng(seed)
    from cases import random_bf16
    H, W = random_bf16((T, d), seed + 1), random_bf16((V, d), seed + 2, std=2.5 / d ** 0.5)
    ids = r.integers(0, V, size=T).astype(np.int32)
    coef = np.zeros(T, np.float32)
    rows = np.unique(np.concatenate([[0, T - 1], r.choice(T, live, replace=False)]))
    coef[rows] = r.normal(0, 0.02, size=rows.size)
    lse = np.zeros(T, np.float32)
    for t in rows:  # the oracle's own lse (natural units) of the rows that count
        lse[t] = oracle.token_stats(oracle.logits_pi(H[t], W, 1.0), int(ids[t]))[0]
    return H, W, ids, coef, lse, rows


# K of dH in slices (3, 1030 and 260 rows over 20000 / 5000 vocabulary rows: 632 and 160 chunks);
# K of dW in slices (9000 rows: 288 chunks, 2 output tiles)
@pytest.mark.parametrize("T,V,d", [(3, 20000, 128), (1030, 20000, 256), (260, 5000, 384), (9000, 300, 128)])
def test_sliced_products_match_oracle(T, V, d):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    H, W, ids, coef, lse, rows = _case(T, V, d, T + V, min(T, 20))
    args = (up_bf16(torch, dev, H), up_bf16(torch, dev, W), up(torch, dev, ids), up(torch, dev, coef),
            up(torch, dev, lse))
    dh, dw = acrl.acrl_lm_head_backward(*args)
    # accumulated onto a known dW, and dH at an address that is no multiple of 16 bytes
    base = torch.full((V, d), 0.5, dtype=torch.float32, device=dev)
    room = torch.full((T * d + 1,), 7.0, dtype=torch.float32, device=dev)
    dh1, dw1 = acrl.acrl_lm_head_backward(*args, dh=room[1:].view(T, d), dw=base, accumulate_dw=True)
    torch.cuda.synchronize()
    assert np.array_equal(down(dh1), down(dh)) and float(room[0]) == 7.0
    # a sum near 0.5 rounds by up to 2^-25 with each of the T / 16 matrix steps
    # that add to it (2^-24 where it crosses into [0.5, 1))
    np.testing.assert_allclose(down(dw1), down(dw) + 0.5, rtol=0, atol=(T / 16 + 2) * 2.0 ** -24)
    dh, dw = down(dh), down(dw)
    assert np.all(dh[coef == 0] == 0)
    rdh, rdw, rdha, rdwa = oracle.lm_head_backward(H[rows], W, ids[rows], coef[rows].astype(np.float64), 1.0,
                                                   want_abs=True)
    _check_rows(dh[rows], rdh, rdha, "dH")
    _check_rows(dw, rdw, rdwa, "dW")
