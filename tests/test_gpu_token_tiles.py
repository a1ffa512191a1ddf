"""Token tiles of 64, 128 and 256 rows (calls of few tokens): the logits and
the draws do not depend on the tile width or on the vocabulary strips that a
call's row count selects, and each width matches the oracle at its edges.
Row counts at and beside the tile widths, on a head of many vocabulary tiles
(several per strip) and on one of few."""
import ctypes

import numpy as np
import pytest

import oracle
from cases import TOL_LOGP, random_bf16, tol_entropy
from gpu_util import down, torch_dev, up, up_bf16

D = 128


@pytest.mark.gpu
@pytest.mark.parametrize("scaling", [oracle.PER_TENSOR, oracle.PER_ROW, oracle.MX32])
@pytest.mark.parametrize("V", [2100, 151936])
def test_token_tile_widths(scaling, V):
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    T = 1030
    H = random_bf16((T, D), 21)
    W = random_bf16((V, D), 22, std=2.5 / D ** 0.5)
    ids = np.random.default_rng(23).integers(0, V, size=T).astype(np.int32)
    h, w, idt = up_bf16(torch, dev, H), up_bf16(torch, dev, W), up(torch, dev, ids)
    hq, hs = acrl.acrl_quantize_fp8(h, scaling)
    wq, ws = acrl.acrl_quantize_fp8(w, scaling)
    packed = acrl.acrl_pack_weights(w, wq, ws, scaling)

    def rows(n):  # the first n rows in one call
        s = hs if scaling == oracle.PER_TENSOR else hs[:n]
        out = acrl.acrl_score_pi_mu(h[:n], w, hq[:n], s, wq, ws, scaling, idt[:n], packed_weights=packed)
        draw, lm = acrl.acrl_sample_mu(hq[:n], s, wq, ws, scaling, seed=9, packed_weights=packed)
        out = {k: down(v) for k, v in out.items()}
        out["ids"], out["draw_logp"] = down(draw), down(lm)
        return out

    full = rows(T)
    check = [0, 31, 63, 64, 100, 127, 128, 129, 255, 256]
    hq_o, hs_o = oracle.quantize_fp8(H, scaling)
    wq_o, ws_o = oracle.quantize_fp8(W, scaling)
    sel = np.array(check)
    ref = oracle.score(H[sel], W, hq_o[sel], hs_o if scaling == oracle.PER_TENSOR else hs_o[sel], wq_o, ws_o, scaling,
                       ids[sel])
    for n in (1, 64, 65, 128, 133, 256, 257, 400, 600):
        got = rows(n)
        for k in ("logit_pi", "logit_mu", "ids"):  # whatever the tiles: one order of every sum
            assert np.array_equal(got[k], full[k][:n]), (k, n)
        for k in ("logp_pi", "logp_mu", "entropy_pi", "entropy_mu", "draw_logp"):
            # strips merge in another order: a few fp32 roundings of values up to ~20
            np.testing.assert_allclose(got[k], full[k][:n], rtol=0, atol=1e-5, err_msg="%s %d" % (k, n))
        m = sel < n
        for tag, ent in (("pi", "ent_pi"), ("mu", "ent_mu")):
            assert np.abs(got["logp_" + tag][sel[m]] - ref["logp_" + tag][m]).max() <= TOL_LOGP, (tag, n)
            assert np.abs(got["entropy_" + tag][sel[m]] - ref[ent][m]).max() <= tol_entropy(V), (tag, n)


def test_workspace_grows_with_rows():
    """A workspace sized for many rows serves fewer, whatever tiles and strips
    each row count selects (host arithmetic only)."""
    from paper_2607_24062_amd import acrl
    L = acrl.lib()
    nb = ctypes.c_size_t()
    for d, V in ((128, 100), (2048, 151936), (4096, 32003), (256, 600000)):
        last = 0
        for n in list(range(0, 1100)) + list(range(1100, 40000, 97)):
            desc = acrl.ScoreDesc(n_rows=n, d=d, V=V, mu_scaling=acrl.SCALE_MX32, packed_weights=ctypes.c_void_p(256))
            assert L.acrl_score_workspace_query(ctypes.byref(desc), ctypes.byref(nb)) == 0
            assert nb.value >= last, (d, V, n)
            last = nb.value


@pytest.mark.parametrize("scaling", [oracle.PER_TENSOR, oracle.PER_ROW, oracle.MX32])
def test_unpacked_workspace_grows_with_rows(scaling):
    """The same where the call packs W and Wq itself from some row count on."""
    from paper_2607_24062_amd import acrl
    L = acrl.lib()
    nb = ctypes.c_size_t()
    for d, V in ((128, 100), (2048, 151936), (4096, 32003)):
        last = 0
        for n in sorted(set(list(range(0, 40000, 97)) + [e + k for e in (4096, 8192, 12288, 16384) for k in (-1, 0, 1, 256)])):
            assert L.acrl_score_workspace_size(n, d, V, scaling, ctypes.byref(nb)) == 0
            assert nb.value >= last, (d, V, n)
            last = nb.value


@pytest.mark.parametrize("chunk", [0, 256, 1000, 4096])
@pytest.mark.parametrize("d,V", [(128, 100), (256, 1000), (256, 20000), (1024, 30000), (2048, 151936), (4096, 151936)])
def test_backward_workspace_grows_with_rows(d, V, chunk):
    """The backward's likewise: K slices sized by the rows and (small heads) by the head, W packed above 4 d rows (4096 at least)."""
    from paper_2607_24062_amd import acrl
    L = acrl.lib()
    nb = ctypes.c_size_t()
    last = 0
    lines = [e + k for e in (256, 4096, 4 * d, 12288, 16384, 32768) for k in (-1, 0, 1, 256)]
    for n in sorted(set(list(range(0, 600)) + list(range(600, 40000, 97)) + lines)):
        assert L.acrl_backward_workspace_size(n, d, V, chunk, ctypes.byref(nb)) == 0
        assert nb.value >= last, n
        last = nb.value


@pytest.mark.gpu
@pytest.mark.parametrize("scaling", [oracle.PER_TENSOR, oracle.PER_ROW, oracle.MX32])
@pytest.mark.parametrize("T,V", [(1, 100), (130, 300), (700, 1000), (8192, 300), (8193, 300),
                                 (12288, 300), (12289, 300), (4096, 33000), (4097, 33000)])
def test_weights_read_in_place_equal_packed(scaling, T, V):
    """W and Wq read where they lie (up to 12288 rows, 8192 with the measures, an
    MXFP8 Wq of more than 8 MB up to 4096), packed by the call (above) and packed by the caller:
    the same bits everywhere."""
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    h, w = up_bf16(torch, dev, random_bf16((T, 256), 31)), up_bf16(torch, dev, random_bf16((V, 256), 32, std=0.2))
    idt = up(torch, dev, np.random.default_rng(33).integers(0, V, size=T).astype(np.int32))
    hq, hs = acrl.acrl_quantize_fp8(h, scaling)
    wq, ws = acrl.acrl_quantize_fp8(w, scaling)
    packed = acrl.acrl_pack_weights(w, wq, ws, scaling)
    res = []
    for pw in (None, packed):
        out = acrl.acrl_score_pi_mu(h, w, hq, hs, wq, ws, scaling, idt, packed_weights=pw)
        div = acrl.acrl_score_pi_mu(h, w, hq, hs, wq, ws, scaling, idt, packed_weights=pw, divergence=True)
        draw, lm = acrl.acrl_sample_mu(hq, hs, wq, ws, scaling, seed=5, packed_weights=pw)
        out.update({"div_" + k: v for k, v in div.items()}, draw=draw, lm=lm)
        res.append({k: down(v) for k, v in out.items()})
    for k in res[0]:
        assert np.array_equal(res[0][k], res[1][k], equal_nan=True), k  # (l2 may be NaN: its terms cancel)


@pytest.mark.gpu
def test_backward_weights_read_in_place_equal_packed():
    torch, dev = torch_dev()
    from paper_2607_24062_amd import acrl
    T, V, d = 4097, 1000, 256
    h, w = up_bf16(torch, dev, random_bf16((T, d), 41)), up_bf16(torch, dev, random_bf16((V, d), 42, std=0.2))
    r = np.random.default_rng(43)
    ids = up(torch, dev, r.integers(0, V, size=T).astype(np.int32))
    coef = up(torch, dev, r.normal(0, 1e-2, size=T).astype(np.float32))
    lse = up(torch, dev, np.full(T, 8.0, np.float32))  # any lse: the same recomputed probabilities on both paths
    coef[-1] = 0
    a, aw = acrl.acrl_lm_head_backward(h, w, ids, coef, lse)                          # packs W
    b, bw = acrl.acrl_lm_head_backward(h[:-1], w, ids[:-1], coef[:-1], lse[:-1])  # reads it in place
    torch.cuda.synchronize()
    assert np.array_equal(down(a)[:-1], down(b))
    # one K chunk more moves the slices of dW's sum: fp32 sums of 4096 terms, 2^-24 each, in another order
    assert float((aw - bw).norm() / aw.norm()) <= 1e-5


def test_workspace_holds_the_packed_weights_above_the_lines():
    """An unpacked call's workspace has room for a packed W above 12288 rows, 8192 with the measures, and for a
    packed Wq likewise, of MXFP8 above 4096 where it has more than 8 MB (host arithmetic only)."""
    from paper_2607_24062_amd import acrl
    L = acrl.lib()
    V, d = 4097, 2048
    buf = ctypes.c_void_p(256)

    def extra(n, scaling, div):  # bytes beyond the call's that brings packed weights, in images of Wq (2 of W)
        nb = []
        for pw in (None, buf):
            desc = acrl.ScoreDesc(n_rows=n, d=d, V=V, mu_scaling=scaling, packed_weights=pw, l2=buf if div else None)
            v = ctypes.c_size_t()
            assert L.acrl_score_workspace_query(ctypes.byref(desc), ctypes.byref(v)) == 0
            nb.append(v.value)
        return (nb[0] - nb[1]) // (V * d)

    for scaling in (acrl.SCALE_PER_TENSOR, acrl.SCALE_PER_ROW):
        assert [extra(n, scaling, False) for n in (1, 4096, 12288, 12289)] == [0, 0, 0, 3]
        assert [extra(n, scaling, True) for n in (1, 8192, 8193)] == [0, 0, 3]
    assert [extra(n, acrl.SCALE_MX32, False) for n in (1, 4096, 4097, 12288, 12289)] == [0, 0, 1, 1, 3]
    assert [extra(n, acrl.SCALE_MX32, True) for n in (1, 4096, 4097, 8192, 8193)] == [0, 0, 1, 1, 3]
    V = 4096
    assert [extra(n, acrl.SCALE_MX32, False) for n in (4097, 12288, 12289)] == [0, 0, 3]
