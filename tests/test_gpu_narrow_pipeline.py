"""The 64- and 128-token tiles where their pipeline runs in its steady state:
more K chunks a tile than stages (16 of FP8 against 6 to 8), one tile a strip
and several, so that stages and weight-row scale slots come round and a tile's
end falls inside the steady loop.  Against float64 of the same operands, and in
all bits against a call whose rows select 256-token tiles."""
import ctypes
import subprocess

import numpy as np
import pytest

from cases import TOL_LOGP, tol_entropy
from gpu_util import down, torch_dev

D = 1024
WIDTHS = {2100: {1: 64, 33: 64, 64: 64, 100: 64, 128: 64},
          151936: {1: 64, 33: 64, 64: 64, 65: 128, 100: 128, 128: 128}}


class _Plan(ctypes.Structure):
    _fields_ = [("tile_t", ctypes.c_int), ("rest", ctypes.c_char * 2044)]  # (the plan's first member, and room)


def _tile_width(acrl, n, V, mx):
    """The token tile that the library plans for a scoring call of n packed rows."""
    out = subprocess.run(["nm", "-D", "--defined-only", acrl.LIB_PATH], capture_output=True, text=True, check=True)
    name, = [w for w in out.stdout.split() if w.startswith("_ZN4acrl10plan_scoreElllblbb")]
    f = getattr(acrl.lib(), name)
    f.restype = _Plan
    f.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_bool, ctypes.c_int64, ctypes.c_bool, ctypes.c_bool]
    return f(n, D, V, mx, 0, True, True).tile_t


@pytest.mark.parametrize("V", sorted(WIDTHS))
def test_rows_select_the_widths_tested(V):
    """Host arithmetic only: a later cost model must not leave a width untested."""
    from paper_2607_24062_amd import acrl
    for mx in (False, True):
        assert {n: _tile_width(acrl, n, V, mx) for n in WIDTHS[V]} == WIDTHS[V]
        assert _tile_width(acrl, 1030, V, mx) == (64 if V == 2100 else 256)
        assert _tile_width(acrl, 16384, V, mx) == 256


def _values(torch, q, s, scaling):
    """float64 of quantized operands."""
    x = q.view(torch.float8_e4m3fn).double()
    if scaling == 2:
        return (x.reshape(q.shape[0], -1, 32) * torch.exp2(s.double() - 127)[..., None]).reshape(q.shape)
    return x * (s.double() if scaling == 0 else s.double()[:, None])


@pytest.mark.gpu
@pytest.mark.parametrize("scaling", [0, 1, 2])
@pytest.mark.parametrize("V", sorted(WIDTHS))
def test_steady_pipeline(scaling, V):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    T = 16384  # rows that select 256-token tiles on both heads
    g = torch.Generator(device=dev)
    g.manual_seed(V + scaling)
    h = torch.randn((T, D), generator=g, device=dev).bfloat16()
    w = (torch.randn((V, D), generator=g, device=dev) * 2.5 / D ** 0.5).bfloat16()
    # (row scales that differ from tile to tile)
    w *= torch.exp2(torch.arange(V, device=dev) // 256 % 3 - 1)[:, None]
    ids = torch.randint(0, V, (T,), generator=g, device=dev, dtype=torch.int32)
    hq, hs = acrl.acrl_quantize_fp8(h, scaling)
    wq, ws = acrl.acrl_quantize_fp8(w, scaling)
    packed = acrl.acrl_pack_weights(w, wq, ws, scaling)

    def rows(n, pw):
        s = hs if scaling == 0 else hs[:n]
        out = acrl.acrl_score_pi_mu(h[:n], w, hq[:n], s, wq, ws, scaling, ids[:n], packed_weights=pw)
        out["draw"], out["draw_logp"] = acrl.acrl_sample_mu(hq[:n], s, wq, ws, scaling, seed=3, packed_weights=pw)
        return {k: down(v) for k, v in out.items()}

    wide = rows(T, packed)
    m = max(WIDTHS[V])
    ref = {}
    hv = _values(torch, hq[:m], hs if scaling == 0 else hs[:m], scaling)
    for tag, a, b in (("pi", h[:m].double(), w.double()), ("mu", hv, _values(torch, wq, ws, scaling))):
        z = a @ b.T
        lse = torch.logsumexp(z, 1)
        ref["logp_" + tag] = down(z.gather(1, ids[:m, None].long())[:, 0] - lse)
        ref["entropy_" + tag] = down(lse - (torch.exp(z - lse[:, None]) * z).sum(1))
        if tag == "mu":
            draw = torch.from_numpy(wide["draw"][:m]).to(dev).long()
            ref["draw_logp"] = down(z.gather(1, draw[:, None])[:, 0] - lse)
        del z
    for n in WIDTHS[V]:
        for pw in (packed, None):
            got = rows(n, pw)
            for k in ("logit_pi", "logit_mu", "draw"):
                assert np.array_equal(got[k], wide[k][:n]), (k, n)
            for k in ref:
                tol = tol_entropy(V) if k.startswith("entropy") else TOL_LOGP
                assert np.abs(got[k] - ref[k][:n]).max() <= tol, (k, n)
