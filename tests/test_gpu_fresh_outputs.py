"""Outputs that acrl_score_pi_mu allocates itself: every slot of a scored
policy is written or 0, and an unscored policy's outputs are 0, whatever the
memory held before."""
import numpy as np
import pytest

from gpu_util import down, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("policies", [0, 1, 2])
@pytest.mark.parametrize("n_slots,slots,masked", [(None, False, False), (None, False, True), (40, False, False),
                                                  (40, True, False), (33, True, True)])
def test_unwritten_slots_are_zero(n_slots, slots, masked, policies):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    T, V, d = 33, 300, 128
    g = torch.Generator(device=dev)
    g.manual_seed(5)
    h = torch.randn((T, d), generator=g, device=dev).bfloat16()
    w = (torch.randn((V, d), generator=g, device=dev) * 0.2).bfloat16()
    (hq, hs), (wq, ws) = acrl.acrl_quantize_fp8(h, acrl.SCALE_PER_ROW), acrl.acrl_quantize_fp8(w, acrl.SCALE_PER_ROW)
    ids = torch.randint(0, V, (T,), generator=g, device=dev, dtype=torch.int32)
    mask = torch.arange(T, device=dev).remainder(3).ne(0).to(torch.uint8) if masked else None
    where = torch.randperm(n_slots or T, generator=g, device=dev)[:T].to(torch.int32) if slots else None

    def call(fill):
        # memory of the outputs' sizes that held something else
        held = [torch.full((n_slots or T,), fill, device=dev) for _ in range(16)]
        del held
        return {k: down(v) for k, v in acrl.acrl_score_pi_mu(
            h, w, hq, hs, wq, ws, acrl.SCALE_PER_ROW, ids, mask=mask, out_slot=where, n_slots=n_slots,
            policies=policies).items()}

    got, again = call(7.0), call(float("nan"))
    written = np.zeros(n_slots or T, bool)
    rows = np.arange(T) if mask is None else np.nonzero(down(mask))[0]
    written[rows if where is None else down(where)[rows]] = True
    for k, v in got.items():
        assert np.array_equal(v, again[k]), k
        scored = not (policies == 1 and k.endswith("_mu") or policies == 2 and k.endswith("_pi"))
        assert np.all(v[~written] == 0), k
        assert np.all(v[written] != 0) if scored else np.all(v == 0), k
