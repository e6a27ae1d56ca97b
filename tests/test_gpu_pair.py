"""Products that share a launch (dx with the gradient, Z with the fold): every pair of tiles, with the gradient straight to its
destination and in slices, Z in one slice and in several, on sizes that end inside tiles.  The gradient has the bits it has
without dx, when every product is a launch of its own."""
import numpy as np
import pytest
import torch

from oracle import loqt_oracle as O
from tests.test_gpu_layer import TOL, _setup

pytestmark = pytest.mark.gpu

CASES = [
    # T, out, in, r, folds          dx / gradient / Z / fold
    (130, 72, 72, 40, True),        # 64x64 / 64x64 in one slice / 64x64 / 64x128
    (520, 72, 72, 40, True),        # 64x64 / 64x64 in slices
    (520, 300, 2600, 264, True),    # 64x128 / 64x64 in one slice
    (1000, 72, 2600, 40, True),     # 64x128 / 64x64 in slices
    (1000, 300, 2600, 264, True),   # 64x128 / 64x128
    (1500, 300, 2600, 40, True),    # 128x128 / 64x64
    (1500, 300, 2600, 264, True),   # 128x128 / 64x128
    (520, 300, 8300, 40, True),     # fold on 128x128
    (3000, 2100, 136, 40, True),    # Z in slices
    (520, 520, 72, 40, False),      # the rank-r term as a second segment of dx
]


@pytest.mark.parametrize("grad", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,out,inp,r,folds", CASES)
def test_shared_launch(T, out, inp, r, folds, grad):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    s = 0.5
    lay, Wq, Pq, d = _setup(T, out, inp, r, seed=T + r, sigma_B=2e-2)
    got = []
    for with_dx in (True, False):
        dx = G.bf16_empty(T, inp, fill=float("nan")) if with_dx else None
        dB = torch.full((r, G.rup(inp, 8)), float("nan"), dtype=grad, device="cuda")[:, :inp]
        L.timing_enable(True)
        L.loqt_linear_bwd(d["dy"], d["x"], d["Wq"], d["Pq"], d["B"], s, dx, dB, False, G.workspace(L.OP_BWD, T, out, inp, r))
        torch.cuda.synchronize()
        L.timing_enable(False)
        n = {k: v[0] for k, v in L.timing_read().items()}
        if with_dx:
            assert n["gemm_dx"] == 1 and n["gemm_db"] == 0
            assert (n["fold_weight"], n["gemm_z"]) == ((1, 0) if folds else (0, 1))
        else:
            assert n["gemm_dx"] == 0 and n["gemm_db"] == 1 and n["gemm_z"] == 1
        got.append((dx, dB))
    assert torch.equal(got[0][1], got[1][1])
    dx_ref, dB_ref = O.loqt_linear_bwd(lay.dy, lay.x, Wq, Pq, lay.B, s)
    assert G.max_err_over_rms(O.bf16_to_f64(G.bf16_host(got[0][0])), dx_ref) <= TOL
    # bf16 output: half a step of the largest entry (6 RMS) on top
    assert G.max_err_over_rms(got[0][1].float().cpu().numpy().astype(np.float64), dB_ref) <= TOL + (6 * 2.0 ** -8 if grad == torch.bfloat16 else 0)


@pytest.mark.parametrize("T,out,inp,r", [(520, 300, 456, 40), (1500, 2600, 300, 72)])
def test_shared_launch_on_the_other_layers(T, out, inp, r):
    """The projection on the input side (V with a fold whose operands are both stored rows x K) and the unquantised layer."""
    from tests import gpu_util as G
    from tests.test_gpu_right import _setup as right_setup
    from paper_2405_16528_amd import binding as L
    s = 0.5
    Wq, Qq, Bp, x, dy, d = right_setup(T, out, inp, r, seed=T)
    dx = G.bf16_empty(T, inp, fill=float("nan"))
    dBp = [torch.full((out, r), float("nan"), device="cuda") for _ in range(2)]
    L.loqt_linear_bwd_right(d["dy"], d["x"], d["Wq"], d["Qq"], d["Bp"], s, dx, dBp[0], False, G.workspace(L.OP_BWD_RIGHT, T, out, inp, r))
    L.loqt_linear_bwd_right(d["dy"], d["x"], d["Wq"], d["Qq"], d["Bp"], s, None, dBp[1], False, G.workspace(L.OP_BWD_RIGHT, T, out, inp, r))
    torch.cuda.synchronize()
    dx_ref, dB_ref = O.loqt_linear_bwd_right(dy, x, Wq, Qq, Bp, s)
    assert torch.equal(dBp[0], dBp[1])
    assert G.max_err_over_rms(O.bf16_to_f64(G.bf16_host(dx)), dx_ref) <= TOL
    assert G.max_err_over_rms(dBp[0].cpu().numpy().astype(np.float64), dB_ref) <= TOL

    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    W, P, B = ((torch.randn(a, G.rup(b, 8), generator=g, device="cuda") * sg).bfloat16()[:, :b] for a, b, sg in ((out, inp, 0.02), (out, r, 0.05), (r, inp, 0.02)))
    dx = G.bf16_empty(T, inp, fill=float("nan"))
    dB = [torch.full((r, inp), float("nan"), device="cuda") for _ in range(2)]
    L.loqt_linear_bwd_nq(d["dy"], d["x"], W, P, B, s, dx, dB[0], False, G.workspace(L.OP_BWD_NQ, T, out, inp, r))
    L.loqt_linear_bwd_nq(d["dy"], d["x"], W, P, B, s, None, dB[1], False, G.workspace(L.OP_BWD_NQ, T, out, inp, r))
    torch.cuda.synchronize()
    assert torch.equal(dB[0], dB[1])
    dy64, x64, P64 = d["dy"].double().cpu(), d["x"].double().cpu(), P.double().cpu()
    dx_ref = dy64 @ (W.double().cpu() + s * P64 @ B.double().cpu())
    assert G.max_err_over_rms(dx.double().cpu().numpy(), dx_ref.numpy()) <= TOL
    assert G.max_err_over_rms(dB[0].double().cpu().numpy(), (s * (dy64 @ P64).t() @ x64).numpy()) <= TOL


def _over(t):
    """A fresh buffer with t's content at its start and room for a gradient of 2000 x 300 in fp32: t's copy, and the buffer."""
    buf = torch.zeros(4 << 20, dtype=torch.uint8, device="cuda")
    whole = torch.as_strided(t, (t.shape[0], t.stride(0)), (t.stride(0), 1))
    n = whole.numel() * 2
    buf[:n].copy_(whole.reshape(-1).view(torch.uint8))
    return buf[:n].view(torch.bfloat16).view(whole.shape)[:, :t.shape[1]], buf


# (the launch that computes dx reads dy and the weight, without a fold B too; the gradient itself reads x, or x and dy)
@pytest.mark.parametrize("grad", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("layer,T,out,inp,r,over", [
    ("left", 130, 72, 72, 40, "dy"), ("left", 130, 72, 72, 40, "x"), ("left", 520, 300, 2600, 264, "dy"),
    ("left", 100, 520, 264, 40, "B"), ("left", 100, 520, 264, 40, "dy"), ("saved", 130, 72, 72, 40, "w_eff"),
    ("nq", 100, 520, 264, 40, "W"), ("nq", 100, 520, 264, 40, "B"), ("right", 130, 72, 72, 40, "dy"), ("right", 130, 72, 72, 40, "x")])
def test_gradient_over_an_input(layer, T, out, inp, r, over, grad):
    """dB in the place of an input: the bits that it and dx have with a buffer of its own."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    g = torch.Generator(device="cuda")
    g.manual_seed(T + r)
    rnd = lambda a, b, sg: (torch.randn(a, G.rup(b, 8), generator=g, device="cuda") * sg).bfloat16()[:, :b]
    nf4 = lambda a, b, sg: L.nf4_quantize(torch.randn(a, G.rup(b, 4), generator=g, device="cuda") * sg, cols=b)
    d = {"x": rnd(T, inp, 1.0), "dy": rnd(T, out, 1.0), "W": rnd(out, inp, 0.02), "w_eff": rnd(out, inp, 0.02), "P": rnd(out, r, 0.05),
         "B": rnd(*((out, r) if layer == "right" else (r, inp)), 0.02)}
    Wq, Pq, Qq = nf4(out, inp, 0.02), nf4(out, r, 0.05), nf4(inp, r, 0.05)
    shape = (out, r) if layer == "right" else (r, inp)
    op = {"left": L.OP_BWD, "saved": L.OP_BWD_SAVED, "nq": L.OP_BWD_NQ, "right": L.OP_BWD_RIGHT}[layer]
    got = []
    for shared in (False, True):
        buf = torch.zeros(4 << 20, dtype=torch.uint8, device="cuda")
        a = dict(d)
        if shared:
            a[over], buf = _over(d[over])
        ld = G.rup(shape[1], 8)
        size = torch.empty(0, dtype=grad).element_size()
        dB = buf[:shape[0] * ld * size].view(grad).view(shape[0], ld)[:, :shape[1]]
        dx, ws = G.bf16_empty(T, inp, fill=float("nan")), G.workspace(op, T, out, inp, r)
        L.timing_enable(True)
        if layer == "left":
            L.loqt_linear_bwd(a["dy"], a["x"], Wq, Pq, a["B"], 0.5, dx, dB, False, ws)
        elif layer == "saved":
            L.loqt_linear_bwd_saved(a["dy"], a["x"], Pq, 0.5, a["w_eff"], dx, dB, False, ws)
        elif layer == "nq":
            L.loqt_linear_bwd_nq(a["dy"], a["x"], a["W"], a["P"], a["B"], 0.5, dx, dB, False, ws)
        else:
            L.loqt_linear_bwd_right(a["dy"], a["x"], Wq, Qq, a["B"], 0.5, dx, dB, False, ws)
        torch.cuda.synchronize()
        L.timing_enable(False)
        n = {k: v[0] for k, v in L.timing_read().items()}
        # one launch without a sum of slices; over an operand of dx two, over one of the gradient a sum of its one slice
        # (on the right side x went into V before)
        own, read = over == ("dy" if layer == "right" else "x"), (layer, over) != ("right", "x")
        assert (n["gemm_dx"], n["gemm_db"], n["reduce_db"]) == ((1, 0, 0) if not (shared and read) else (1, 0, 1) if own else (1, 1, 0))
        got.append((dx.clone(), dB.clone()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("T,out,inp,r", [(70, 130, 136, 40), (100, 1030, 333, 72), (130, 1100, 1000, 264), (65, 24, 2600, 24)])
def test_copies_beside_the_first_product(T, out, inp, r):
    """bf16 copies of W and P in the launch of U: pieces that end inside a work-group's, rows that end inside a piece; U in one
    slice and in several."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    lay, Wq, Pq, d = _setup(T, out, inp, r, seed=T + r, sigma_B=2e-2)
    y = G.bf16_empty(T, out, fill=float("nan"))
    L.set_path(L.PATH_PREPASS)
    try:
        L.timing_enable(True)
        L.loqt_linear_fwd(d["x"], d["Wq"], d["Pq"], d["B"], 0.5, y, G.workspace(L.OP_FWD, T, out, inp, r))
        torch.cuda.synchronize()
        L.timing_enable(False)
    finally:
        L.set_path(L.PATH_AUTO)
    n = {k: v[0] for k, v in L.timing_read().items()}
    assert (n["prepass"], n["gemm_u"], n["gemm_y"]) == (0, 1, 1)
    assert G.max_err_over_rms(O.bf16_to_f64(G.bf16_host(y)), O.loqt_linear_fwd(lay.x, Wq, Pq, lay.B, 0.5)) <= TOL
