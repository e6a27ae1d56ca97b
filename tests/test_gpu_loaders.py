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


@pytest.mark.parametrize("T,out,inp,r", [(33, 5100000 // (64 * n - cut) + 1, 64 * n - cut, 24) for n in range(1, 7) for cut in (0, 40) if n > 1 or not cut] +
                         [(64, 13900, 1100, 72), (64, 13824, 1024, 64), (256, 13900, 1720, 136), (128, 13824, 1536, 128)] +
                         [(40, 4200, 1100, 72), (96, 1100, 6400, 40), (192, 10335, 2548, 120)])
def test_fed_by_the_expansion(T, out, inp, r):
    """Products that expand the codes (a few hundred tokens), both directions: slices of one to seven k-tiles, and of ten to
    fourteen, where the feeding waves have a form without branches for k-tiles that are neither cut nor the first of a segment; and
    tiles that are no multiple of eight (33, 9 and 81 forward, 9, 50 and 20 backward), whose slices are dealt to the XCDs together.
    Against the products on expanded weights, which round the same operands: sums in another order, so a bf16 result moves by one step
    at most, and rarely."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    g = torch.Generator(device="cuda")
    g.manual_seed(T + inp)

    def bf16(rows, cols, sigma):
        return (torch.randn((rows, G.rup(cols, 8)), generator=g, device="cuda") * sigma).bfloat16()[:, :cols]
    Wq = L.nf4_quantize(torch.randn((out, G.rup(inp, 4)), generator=g, device="cuda")[:, :inp] * 0.02)
    Pq = L.nf4_quantize(torch.randn((out, G.rup(r, 4)), generator=g, device="cuda")[:, :r] * out ** -0.5)
    x, dy, B = bf16(T, inp, 1.0), bf16(T, out, 1e-2), bf16(r, inp, 2e-2)
    got = []
    try:
        for path in (L.PATH_CODES, L.PATH_PREPASS):
            L.set_path(path)
            assert all(L.expands_codes(op, T, out, inp, r) == (path == L.PATH_CODES) for op in (L.OP_FWD, L.OP_BWD))
            y, dx = G.bf16_empty(T, out, fill=float("nan")), G.bf16_empty(T, inp, fill=float("nan"))
            dB = torch.full((r, inp), float("nan"), device="cuda")
            L.loqt_linear_fwd(x, Wq, Pq, B, 0.5, y, G.workspace(L.OP_FWD, T, out, inp, r))
            L.loqt_linear_bwd(dy, x, Wq, Pq, B, 0.5, dx, dB, False, G.workspace(L.OP_BWD, T, out, inp, r))
            got.append((y.float(), dx.float(), dB))
    finally:
        L.set_path(L.PATH_AUTO)
    # y, dx: a step of the result is up to 2^-7 of it, and U or Z may round to the other side too, which moves a small term of the sum.
    # dB is not rounded, but a step of one entry of Z, 2^-8 of it, times an entry of x goes into it: both up to 4.5 times their
    # rms, and rms(dB) = sqrt(T) rms(Z) rms(x)
    for (a, b), own, rest in zip(zip(*got), (2.0 ** -7, 2.0 ** -7, 0.0), (2.0 ** -9, 2.0 ** -9, 2.0 ** -8 * 4.5 ** 2 / T ** 0.5)):
        assert torch.isfinite(a).all()
        assert ((a - b).abs() <= own * b.abs() + rest * b.pow(2).mean().sqrt()).all()


def test_merges_in_one_launch_on_256x256():
    """A list of large weights of rank 512 and more (1024 tiles of 256x256 and more) is one launch on those tiles; a weight alone takes 128x128
    where they would leave the chip idle.  Same products, same encoder: the same bits."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    layers = []
    for out, inp in [(2048, 2048)] * 15 + [(2041, 2040)]:
        Wq = L.nf4_quantize(torch.randn((out, inp), generator=g, device="cuda") * 0.02)
        Pq = L.nf4_quantize(torch.randn((out, 512), generator=g, device="cuda") * out ** -0.5)
        B = (torch.randn((512, G.rup(inp, 8)), generator=g, device="cuda") * 2e-2).bfloat16()[:, :inp]
        layers.append((Wq, L.NF4Tensor.empty(out, inp), Pq, B, 0.5))
    descs = L.make_merge_descs(layers)
    L.loqt_merge_requant_batched(descs, torch.empty(L.merge_descs_workspace_bytes(descs), dtype=torch.uint8, device="cuda"))
    for Wq, dst, Pq, B, s in layers:
        ref = L.loqt_merge_requant(Wq, Pq, B, s, out=L.NF4Tensor.empty(Wq.rows, Wq.cols))
        assert torch.equal(dst.codes, ref.codes) and torch.equal(dst.absmax, ref.absmax)
