"""Forward and backward calls with a few hundred tokens, whose products expand the codes themselves: sizes that end inside
tiles, k-tiles and blocks, slices of the contraction, padding that holds NaN, against the oracle."""
import contextlib

import numpy as np
import pytest
import torch

from oracle import loqt_oracle as O
from paper_2405_16528_amd import synth
from tests.test_gpu_few import _nan_padded, _nan_scaled
from tests.test_gpu_layer import TOL

pytestmark = pytest.mark.gpu

CASES = [
    # T, out, in, r
    (33, 300, 200, 40),       # tiles of 64 tokens; every contraction ends inside a k-tile
    (64, 512, 576, 128),      # whole k-tiles
    (40, 129, 1000, 72),      # one column past a tile
    (50, 1000, 129, 8),       # rank shorter than a k-tile; the weight's last block almost empty
    (65, 4100, 3500, 72),     # tiles of 128 tokens
    (128, 3456, 4096, 128),
    (129, 3500, 4100, 200),   # tiles of 256 tokens
    (256, 3840, 3712, 192),
]
# sizes that come here by themselves, in both directions
BY_RULE = [
    (40, 3000, 1500, 72),     # tiles of 64 tokens
    (100, 4100, 3500, 72),    # of 128
    (129, 5100, 3500, 200),   # of 256
]


@contextlib.contextmanager
def _path(path):
    from paper_2405_16528_amd import binding as L
    L.set_path(path)
    try:
        yield
    finally:
        L.set_path(L.PATH_AUTO)


@pytest.mark.parametrize("grad", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("path,T,out,inp,r", [("codes", *c) for c in CASES] + [("auto", *c) for c in BY_RULE])
def test_fwd_bwd_parity(path, T, out, inp, r, grad):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    with _path(L.PATH_CODES if path == "codes" else L.PATH_AUTO):
        assert L.expands_codes(L.OP_FWD, T, out, inp, r) and L.expands_codes(L.OP_BWD, T, out, inp, r)
        _parity(T, out, inp, r, grad)


def _parity(T, out, inp, r, grad):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    rng = synth.rng_for(T, "tile", out, inp)
    s = 0.5
    Wq = O.nf4_quantize(synth.normal_f32(rng, (out, inp), 0.02))
    Pq = O.nf4_quantize(synth.normal_f32(rng, (out, r), out ** -0.5))
    B, x = synth.normal_bf16(rng, (r, inp), 2e-2), synth.normal_bf16(rng, (T, inp), 1.0)
    dy = synth.normal_bf16(rng, (T, out), 1e-2)
    y, dx = G.bf16_empty(T, out, fill=float("nan")), G.bf16_empty(T, inp, fill=float("nan"))
    dB = torch.full((r, G.rup(inp, 8)), float("nan"), dtype=grad, device="cuda")[:, :inp]
    q = [_nan_scaled(Wq), _nan_scaled(Pq)]
    ws = G.workspace(L.OP_BWD, T, out, inp, r)
    ws.fill_(0xFF)  # (NaN, whatever the element type)
    L.loqt_linear_fwd(_nan_padded(x, 8), *q, _nan_padded(B, 16), s, y, G.workspace(L.OP_FWD, T, out, inp, r))
    L.loqt_linear_bwd(_nan_padded(dy, 0), _nan_padded(x, 8), *q, _nan_padded(B, 16), s, dx, dB, False, ws)
    torch.cuda.synchronize()
    G.bf16_output_report(G.bf16_host(y), O.loqt_linear_fwd(x, Wq, Pq, B, s))
    dx_ref, dB_ref = O.loqt_linear_bwd(dy, x, Wq, Pq, B, s)
    G.bf16_output_report(G.bf16_host(dx), dx_ref)
    # T below 64: the rounding of Z does not average out (2^-8 of the largest entry, 6 RMS); bf16 output: half a step more
    tol = TOL + (6 * 2.0 ** -8 if T < 64 else 0) + (6 * 2.0 ** -8 if grad == torch.bfloat16 else 0)
    assert G.max_err_over_rms(dB.float().cpu().numpy().astype(np.float64), dB_ref) <= tol
    # the expanded-weight form rounds the same operands: it differs by the order of fp32 sums only, which moves a bf16
    # result by at most one step, and only rarely
    with _path(L.PATH_PREPASS):
        assert not L.expands_codes(L.OP_FWD, T, out, inp, r) and not L.expands_codes(L.OP_BWD, T, out, inp, r)
        y2, dx2 = G.bf16_empty(T, out), G.bf16_empty(T, inp)
        L.loqt_linear_fwd(_nan_padded(x, 8), *q, _nan_padded(B, 16), s, y2, G.workspace(L.OP_FWD, T, out, inp, r))
        L.loqt_linear_bwd(_nan_padded(dy, 0), _nan_padded(x, 8), *q, _nan_padded(B, 16), s, dx2, dB, False, ws)
        torch.cuda.synchronize()
    for a, b in ((y, y2), (dx, dx2)):
        a, b = a.double(), b.double()
        assert float((a != b).double().mean()) < 0.02 and float((a - b).norm() / b.norm()) < 3e-4


@pytest.mark.parametrize("path", ["codes", "auto"])
def test_without_dx_and_with_the_smallest_workspace(path):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    T, out, inp, r, s = 40, 1000, 1500, 72, 0.5
    rng = synth.rng_for(T, "tile small", out, inp)
    Wq = O.nf4_quantize(synth.normal_f32(rng, (out, inp), 0.02))
    Pq = O.nf4_quantize(synth.normal_f32(rng, (out, r), out ** -0.5))
    B, x = synth.normal_bf16(rng, (r, inp), 2e-2), synth.normal_bf16(rng, (T, inp), 1.0)
    dy = synth.normal_bf16(rng, (T, out), 1e-2)
    d = [G.bf16_dev(dy), G.bf16_dev(x), G.nf4_dev(*Wq), G.nf4_dev(*Pq), G.bf16_dev(B), s]

    def region(rows, cols):
        return G.rup(rows * G.rup(cols, 8) * 2, 256)
    # Z, copies of W and P, one slice of dB; or, for the general fused form, Z and one slice
    least = region(T, r) + region(out, inp) + region(out, r) + G.rup(r * inp * 4, 256)
    assert least <= L.loqt_workspace_bytes(L.OP_BWD, T, out, inp, r)
    dx_ref, dB_ref = O.loqt_linear_bwd(dy, x, Wq, Pq, B, s)
    tol = TOL + 6 * 2.0 ** -8
    for with_dx in (True, False):
        dx = G.bf16_empty(T, inp, fill=float("nan")) if with_dx else None
        dB = torch.full((r, inp), float("nan"), dtype=torch.float32, device="cuda")
        with _path(L.PATH_CODES if path == "codes" else L.PATH_AUTO):
            L.timing_enable(True)
            try:
                L.loqt_linear_bwd(*d, dx, dB, False, torch.empty(least, dtype=torch.uint8, device="cuda"))
                torch.cuda.synchronize()
            finally:
                L.timing_enable(False)
        # (the least workspace has room for the slices of Z and dx where the copies of W and P would be, so no copy is made)
        assert (L.timing_read()["prepass"][0] == 0) == (path == "codes")
        assert G.max_err_over_rms(dB.cpu().numpy().astype(np.float64), dB_ref) <= tol
        if with_dx:
            G.bf16_output_report(G.bf16_host(dx), dx_ref)
    with pytest.raises(L.LoqtError), _path(L.PATH_CODES if path == "codes" else L.PATH_AUTO):
        L.loqt_linear_bwd(*d, None, dB, False, torch.empty(least - 1, dtype=torch.uint8, device="cuda"))


def test_timers_cover_the_sum_of_the_slices():
    """What the per-kernel timers leave out is the gaps between launches, in this form as in the one that has a launch per
    product: the sums of the slices belong to their products."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    T, out, inp, r, s, calls = 256, 3840, 3712, 192, 0.5, 10
    rng = synth.rng_for(T, "tile timers")
    Wq = G.nf4_dev(*O.nf4_quantize(synth.normal_f32(rng, (out, inp), 0.02)))
    Pq = G.nf4_dev(*O.nf4_quantize(synth.normal_f32(rng, (out, r), out ** -0.5)))
    B, x = G.bf16_dev(synth.normal_bf16(rng, (r, inp), 2e-2)), G.bf16_dev(synth.normal_bf16(rng, (T, inp), 1.0))
    dy, dx = G.bf16_dev(synth.normal_bf16(rng, (T, out), 1e-2)), G.bf16_empty(T, inp)
    dB, ws = torch.empty((r, inp), dtype=torch.float32, device="cuda"), G.workspace(L.OP_BWD, T, out, inp, r)

    def untimed_per_launch(path):
        with _path(path):
            best = float("inf")
            for _ in range(6):
                begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                L.timing_enable(True)
                for n in range(calls + 3):
                    if n == 3:  # (the first ones fill the queue)
                        torch.cuda.synchronize()
                        L.timing_enable(False)
                        L.timing_enable(True)
                        begin.record()
                    L.loqt_linear_bwd(dy, x, Wq, Pq, B, s, dx, dB, False, ws)
                end.record()
                end.synchronize()
                L.timing_enable(False)
                launches, ms = (sum(v) for v in zip(*L.timing_read().values()))
                best = min(best, (begin.elapsed_time(end) - ms) * 1e3 / launches)
            return best
    tile, plain = untimed_per_launch(L.PATH_CODES), untimed_per_launch(L.PATH_PREPASS)
    print(f"outside of the timers, us per launch: {tile:.1f}, with a launch per product {plain:.1f}")
    assert tile <= plain + 1.0
