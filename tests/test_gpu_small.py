"""Short cuts of small calls: a gradient of one slice that goes straight to its destination, and narrow weights whose merge
takes the pre-pass form when there is a workspace for it.  Both must give the bits of the long way."""
import numpy as np
import pytest
import torch

from oracle import loqt_oracle as O
from paper_2405_16528_amd import synth
from tests.test_gpu_layer import TOL, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grad", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,out,inp,r", [(100, 136, 200, 72), (256, 512, 512, 128), (70, 260, 1000, 256), (256, 1030, 2600, 1024)])
def test_direct_gradient_has_the_bits_of_the_summed_one(T, out, inp, r, grad):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    assert L.plan_tiles(r, inp, T, sliced=True)[1] == 1
    s = 0.5
    lay, Wq, Pq, d = _setup(T, out, inp, r, seed=T + r, sigma_B=2e-2)
    got = []
    for accumulate, pitch in ((False, G.rup(inp, 8)), (True, G.rup(inp, 8)), (False, inp + 3)):  # (odd pitch: summed)
        buf = torch.zeros((r, pitch), dtype=grad, device="cuda") if accumulate else torch.full((r, pitch), float("nan"), dtype=grad, device="cuda")
        dB = buf[:, :inp]
        L.loqt_linear_bwd(d["dy"], d["x"], d["Wq"], d["Pq"], d["B"], s, None, dB, accumulate, G.workspace(L.OP_BWD, T, out, inp, r))
        torch.cuda.synchronize()
        if not accumulate:
            assert bool(torch.isnan(buf[:, inp:]).all())  # nothing past the columns
        got.append(dB.clone())
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    _, ref = O.loqt_linear_bwd(lay.dy, lay.x, Wq, Pq, lay.B, s)
    # bf16 output: half a step of the largest entry (6 RMS) on top
    assert G.max_err_over_rms(got[0].float().cpu().numpy().astype(np.float64), ref) <= TOL + (6 * 2.0 ** -8 if grad == torch.bfloat16 else 0)


@pytest.mark.parametrize("grad", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,out,inp,r", [(100, 136, 129, 72), (256, 512, 333, 128), (70, 260, 1001, 256), (256, 1030, 2606, 1024)])
def test_direct_gradient_keeps_to_its_columns(T, out, inp, r, grad):
    """Columns that end inside the kernel's stores of 4 or 8, in a pitch with room past them."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    assert L.plan_tiles(r, inp, T, sliced=True)[1] == 1
    _, _, _, d = _setup(T, out, inp, r, seed=T + r, sigma_B=2e-2)
    got = []
    for pitch in (G.rup(inp, 8), G.rup(inp, 8) + 8, inp + 3 if (inp + 3) % 4 else inp + 1):  # (the last one: summed)
        buf = torch.full((r + 1, pitch), float("nan"), dtype=grad, device="cuda")
        L.timing_enable(True)
        L.loqt_linear_bwd(d["dy"], d["x"], d["Wq"], d["Pq"], d["B"], 0.5, None, buf[:r, :inp], False, G.workspace(L.OP_BWD, T, out, inp, r))
        torch.cuda.synchronize()
        L.timing_enable(False)
        assert L.timing_read()["reduce_db"][0] == (0 if pitch % 8 == 0 else 1)  # the route the pitch is there for
        assert buf[:, inp:].numel() > 0 and bool(torch.isnan(buf[:, inp:]).all()) and bool(torch.isnan(buf[r]).all())
        got.append(buf[:r, :inp].clone())
    assert not bool(torch.isnan(got[0]).any()) and torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


@pytest.mark.parametrize("out,inp,r", [(512, 512, 128), (300, 456, 64), (1100, 333, 192), (2048, 768, 256), (40, 40, 8)])
def test_narrow_merge_with_and_without_a_workspace(out, inp, r):
    from paper_2405_16528_amd import binding as L
    _, _, _, d = _setup(64, out, inp, r, seed=out + r, sigma_B=2e-2)
    outs = []
    for ws in (torch.empty(256, dtype=torch.uint8, device="cuda"), L.workspace(L.OP_MERGE, 0, out, inp, r)):
        q = L.NF4Tensor.empty(out, inp)
        L.loqt_merge_requant(d["Wq"], d["Pq"], d["B"], 0.5, out=q, ws=ws)
        torch.cuda.synchronize()
        outs.append(q)
    assert torch.equal(outs[0].codes, outs[1].codes) and torch.equal(outs[0].absmax, outs[1].absmax)
    lib = L.lib
    q = L.NF4Tensor.empty(out, inp)
    import ctypes as C
    st = lib.loqt_merge_requant(C.byref(d["Wq"].c()), q.codes.data_ptr(), q.absmax.data_ptr(), C.byref(d["Pq"].c()),
                                d["B"].data_ptr(), d["B"].stride(0), 0.5, None, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st == 0 and torch.equal(q.codes, outs[1].codes) and torch.equal(q.absmax, outs[1].absmax)
