"""Contractions around the length of the ring of LDS stages (three of 64x128 tiles, four of 64x64, two of 128x128): fewer k-tiles
than stages, as many, one more, each ending on a k-tile and inside one.  The old codes of a fold or merge ride behind the
last k-tile, so their place in the ring moves with the number of k-tiles too."""
import numpy as np
import pytest
import torch

from oracle import loqt_oracle as O
from tests.test_gpu_layer import TOL, _merge_policy_check, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [8, 64, 72, 128, 136, 192, 200, 256, 264, 320])
def test_products_over_a_short_contraction(k):
    """y over in = k, Z and dx over out = k, dB over T = k."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    s = 0.5
    for T, out, inp, r in ((70, 136, k, 40), (70, k, 136, 40), (k, 72, 136, 40)):
        r = min(r, out)
        lay, Wq, Pq, d = _setup(T, out, inp, r, seed=k + out, sigma_B=2e-2)
        y = G.bf16_empty(T, out, fill=float("nan"))
        dx = G.bf16_empty(T, inp, fill=float("nan"))
        dB = torch.full((r, inp), float("nan"), dtype=torch.float32, device="cuda")
        L.set_path(L.PATH_FOLDED)
        try:
            L.loqt_linear_fwd(d["x"], d["Wq"], d["Pq"], d["B"], s, y, G.workspace(L.OP_FWD, T, out, inp, r))
            L.loqt_linear_bwd(d["dy"], d["x"], d["Wq"], d["Pq"], d["B"], s, dx, dB, False, G.workspace(L.OP_BWD, T, out, inp, r))
            torch.cuda.synchronize()
        finally:
            L.set_path(L.PATH_AUTO)
        y_ref = O.loqt_linear_fwd(lay.x, Wq, Pq, lay.B, s)
        dx_ref, dB_ref = O.loqt_linear_bwd(lay.dy, lay.x, Wq, Pq, lay.B, s)
        assert G.max_err_over_rms(O.bf16_to_f64(G.bf16_host(y)), y_ref) <= TOL
        assert G.max_err_over_rms(O.bf16_to_f64(G.bf16_host(dx)), dx_ref) <= TOL
        assert G.max_err_over_rms(dB.cpu().numpy().astype(np.float64), dB_ref) <= TOL


@pytest.mark.parametrize("r", [8, 64, 72, 128, 136, 192, 200])
def test_merge_bits_of_every_tile_over_a_short_contraction(r):
    """64x128 (automatic), 128x128, 256x128 and 256x256 tiles hold other numbers of stages and lay the codes out in rows of
    another length; ragged rows and columns.  All sum k in the same order, so the codes are the same bits."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    out, inp = 330, 1100
    lay, Wq, Pq, d = _setup(64, out, inp, r, seed=r)
    got = []
    for tile in (L.TILE_AUTO, L.TILE_128x128, L.TILE_256x128, L.TILE_256x256):
        L.set_tile(tile)
        try:
            q = L.loqt_merge_requant(d["Wq"], d["Pq"], d["B"], 0.5, out=L.NF4Tensor.empty(out, inp))
            torch.cuda.synchronize()
        finally:
            L.set_tile(L.TILE_AUTO)
        got.append(q)
    for q in got[1:]:
        assert torch.equal(q.codes, got[0].codes) and torch.equal(q.absmax, got[0].absmax)
    c, a, _, _ = G.nf4_host(got[0])
    assert _merge_policy_check(c, a, Wq, Pq, lay.B, 0.5) <= 1e-3
