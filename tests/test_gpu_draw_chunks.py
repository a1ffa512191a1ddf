"""A draw depends on (seed, token) alone: a call's chunks, whose row counts
select other token tiles and vocabulary strips, draw the same rows.

The head has 9496 blocks of two values of the logit, the larger one in every
sixth vocabulary tile.  About one token in a thousand has two blocks of the
smaller one with the same uniform at the top; which of them is drawn then must
not hang on how each key was rounded, so not on whether a larger logit stood
before the block in its strip (the first of every other strip of three tiles
that a call of 64 rows takes, of all strips in a call of many)."""
import numpy as np
import pytest

import oracle
from gpu_util import down, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scaling", [oracle.PER_TENSOR, oracle.PER_ROW, oracle.MX32])
@pytest.mark.parametrize("small,large", [(0.0151, 0.0263), (0.0297, 0.0371)])
def test_chunked_draws_equal_one_call(scaling, small, large):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    T, V, d = 32768, 151936, 128
    h = torch.ones((T, d), device=dev).bfloat16()
    w = torch.full((V, d), small, device=dev)
    w[(torch.arange(V, device=dev) // 256) % 6 == 0] = large
    w = w.bfloat16()
    hq, hs = acrl.acrl_quantize_fp8(h, scaling)
    wq, ws = acrl.acrl_quantize_fp8(w, scaling)
    packed = acrl.acrl_pack_weights(w, wq, ws, scaling)

    def draw(a, b):
        s = hs if scaling == oracle.PER_TENSOR else hs[a:b].contiguous()
        return acrl.acrl_sample_mu(hq[a:b], s, wq, ws, scaling, seed=77, row_offset=a, packed_weights=packed)[0]

    whole = down(draw(0, T))
    for n in (64, 128, 400, 1100, 3000):
        got = down(torch.cat([draw(a, min(a + n, T)) for a in range(0, T, n)]))
        assert np.array_equal(got, whole), (n, np.flatnonzero(got != whole))
