"""Product kernels with waves of their own for the loads: contractions around the number of stages (three, four on 64x64), which
is where the loading waves stop asking for tiles and wait for fewer, ending inside a k-tile and on one; the plan takes 64x64 for these sizes."""
import numpy as np
import pytest
import torch

from oracle import loqt_oracle as O
from tests.test_gpu_layer import TOL, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", ["auto", "128x128", "256x128"])
@pytest.mark.parametrize("K", [24, 64, 128, 136, 192, 256, 264, 320, 456])
def test_contractions_around_the_stages(tile, K):
    """Forward, folded (y: contraction over in) and backward (dx: over out in two segments, dB: over the tokens)."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    T, out, inp, r, s = K + 8, K, K, 24, 0.5
    lay, Wq, Pq, d = _setup(T, out, inp, r, seed=K, sigma_B=2e-2)
    y = G.bf16_empty(T, out, fill=float("nan"))
    dx = G.bf16_empty(T, inp, fill=float("nan"))
    dB = torch.full((r, inp), float("nan"), dtype=torch.float32, device="cuda")
    L.set_tile({"auto": L.TILE_AUTO, "128x128": L.TILE_128x128, "256x128": L.TILE_256x128}[tile])
    try:
        L.set_path(L.PATH_FOLDED)
        L.loqt_linear_fwd(d["x"], d["Wq"], d["Pq"], d["B"], s, y, G.workspace(L.OP_FWD, T, out, inp, r))
        L.set_path(L.PATH_PREPASS)
        L.loqt_linear_bwd(d["dy"], d["x"], d["Wq"], d["Pq"], d["B"], s, dx, dB, False, G.workspace(L.OP_BWD, T, out, inp, r))
        torch.cuda.synchronize()
    finally:
        L.set_path(L.PATH_AUTO)
        L.set_tile(L.TILE_AUTO)
    y_ref = O.loqt_linear_fwd(lay.x, Wq, Pq, lay.B, s)
    dx_ref, dB_ref = O.loqt_linear_bwd(lay.dy, lay.x, Wq, Pq, lay.B, s)
    # (with fewer than 64 tokens the rounding of Z does not average out: 2^-8 of the largest entry, 6 RMS)
    few = 6 * 2.0 ** -8 if T < 64 else 0.0
    assert G.max_err_over_rms(O.bf16_to_f64(G.bf16_host(y)), y_ref) <= TOL
    assert G.max_err_over_rms(O.bf16_to_f64(G.bf16_host(dx)), dx_ref) <= TOL
    assert G.max_err_over_rms(dB.cpu().numpy().astype(np.float64), dB_ref) <= TOL + few
