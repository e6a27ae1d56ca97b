"""Products that do not fill the chip with 256x256 tiles: the smaller tile shapes and the slices of the contraction that
the launch plan picks for them, on sizes that end inside tiles in every dimension, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import loqt_oracle as O
from tests.test_gpu_layer import TOL, _setup

T64x64, T64x128, T128x128, T256x128, T256x256 = 6, 5, 3, 2, 1


def _ktiles(*ks):
    return 64 * sum(-(-k // 64) for k in ks)


# T, out, in, r, {product: (tile shape, sliced)} -- the plan the case is there for
CASES = [
    (16, 2050, 4100, 72, {"u": (T64x64, True), "y": (T64x128, True), "z": (T64x64, True)}),
    (1, 130, 2100, 40, {"u": (T64x64, True)}),
    (700, 3000, 136, 40, {"z": (T64x64, True), "y": (T64x128, False)}),
    (2100, 2050, 72, 40, {"y": (T128x128, False)}),
    (3000, 2050, 2100, 64, {"y": (T256x128, False)}),
    (3000, 3000, 520, 96, {"y": (T256x256, False)}),
]


@pytest.mark.parametrize("T,out,inp,r,want", CASES)
def test_the_cases_take_the_plans_they_are_there_for(T, out, inp, r, want):
    from paper_2405_16528_amd import binding as L
    fold = T * (inp + out) >= out * inp
    size = {"u": (T, r, inp), "y": (T, out, inp if fold else _ktiles(inp, r)), "z": (T, r, out)}
    for name, (tile, sliced) in want.items():
        got = L.plan_tiles(*size[name])
        assert (got[0], got[1] > 1) == (tile, sliced), (name, got)


def test_plan_has_no_empty_slices_and_keeps_to_its_limit():
    from paper_2405_16528_amd import binding as L
    for M in (1, 16, 300, 4096):
        for N in (40, 1024, 5461):
            for K in (8, 64, 520, 5461, 13824):
                for sliced in (False, True):
                    for most in (1, 3, 32):
                        tile, n = L.plan_tiles(M, N, K, sliced, most)
                        kt = -(-K // 64)
                        assert 1 <= tile <= 6 and 1 <= n <= most and (n - 1) * -(-kt // n) < kt
                        assert not (tile == T256x256 and (sliced or n > 1))


@pytest.mark.parametrize("M,N,K", [(1024, 5120, 13824), (600, 10112, 3520), (1816, 2341, 6546)])
def test_plan_counts_the_unit_that_has_two_tiles(M, N, K):
    """257 to 512 tiles of 128x128 take as long as 512: these sizes are faster on 256x128."""
    from paper_2405_16528_amd import binding as L
    assert 256 < -(-M // 128) * -(-N // 128) < 512
    assert L.plan_tiles(M, N, K, max_splits=1) == (T256x128, 1)


@pytest.mark.parametrize("M,N,K", [(5209, 480, 6160), (4238, 636, 6336), (7080, 267, 4544), (6685, 333, 7496)])
def test_plan_counts_work_groups_by_xcd(M, N, K):
    """81 to 85 tiles of 256x128 in three slices fit 256 compute units, but not the 32 of an XCD."""
    from paper_2405_16528_amd import binding as L
    tile, n = L.plan_tiles(M, N, K)
    tiles = -(-M // 256) * -(-N // 128)
    assert 3 * tiles <= 256 and 3 * -(-tiles // 8) > 32
    assert (tile, n) != (T256x128, 3)


@pytest.mark.parametrize("M,N,K,sliced,want", [
    (746, 3234, 3328, False, (T128x128, 1)), (640, 3970, 4096, False, (T128x128, 1)), (1408, 768, 5248, False, (T128x128, 3)),
    (7808, 384, 7296, False, (T256x128, 2)), (544, 4608, 13760, False, (T256x128, 2)),  # a unit to itself, but slices are ahead
    (768, 3035, 451, True, (T64x128, 1)), (2304, 512, 1878, True, (T64x128, 2)),        # gradients that share the launch of dx
])
def test_plan_prices_128x128_with_a_unit_to_itself(M, N, K, sliced, want):
    from paper_2405_16528_amd import binding as L
    assert L.plan_tiles(M, N, K, sliced) == want


@pytest.mark.gpu
@pytest.mark.parametrize("T,out,inp,r,want", CASES)
def test_fwd_bwd_parity(T, out, inp, r, want):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    s = 0.5
    lay, Wq, Pq, d = _setup(T, out, inp, r, seed=T + out, sigma_B=2e-2)
    y = G.bf16_empty(T, out, fill=float("nan"))
    dx = G.bf16_empty(T, inp, fill=float("nan"))
    dB = torch.full((r, inp), float("nan"), dtype=torch.float32, device="cuda")
    L.loqt_linear_fwd(d["x"], d["Wq"], d["Pq"], d["B"], s, y, G.workspace(L.OP_FWD, T, out, inp, r))
    L.loqt_linear_bwd(d["dy"], d["x"], d["Wq"], d["Pq"], d["B"], s, dx, dB, False, G.workspace(L.OP_BWD, T, out, inp, r))
    torch.cuda.synchronize()
    y_ref = O.loqt_linear_fwd(lay.x, Wq, Pq, lay.B, s)
    dx_ref, dB_ref = O.loqt_linear_bwd(lay.dy, lay.x, Wq, Pq, lay.B, s)
    # y and dx: millions of outputs reach 5 RMS, where bf16 itself is off by up to 2^-8 of that, 2e-2 RMS; so every element
    # has half a bf16 step of its own size plus 1.2e-2 RMS for the bf16 operands (see bf16_output_report)
    ey = G.bf16_output_report(G.bf16_host(y), y_ref)[0]
    ex = G.bf16_output_report(G.bf16_host(dx), dx_ref)[0]
    eb = G.max_err_over_rms(dB.cpu().numpy().astype(np.float64), dB_ref)
    print(f"T={T} out={out} in={inp} r={r}: err/rms y {ey:.2e} dx {ex:.2e} dB {eb:.2e}")
    # dB from a handful of tokens: Z = s dy deq(P) is kept in bf16, off by up to 2^-8 of itself per product, and the
    # products do not average out: 2^-8 of the largest entry (6 RMS) on top of the bound
    assert eb <= (TOL if T >= 64 else TOL + 6 * 2.0 ** -8)


@pytest.mark.gpu
@pytest.mark.parametrize("T,out,inp,r", [(3021, 81, 6892, 21), (1539, 128, 8640, 128), (3060, 241, 5907, 8)])
def test_z_rides_beside_dx_when_its_tiles_are_free(T, out, inp, r):
    """Short contractions: Z adds no round of 128x128 tiles to those of dx, so it has no launch of its own."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    rounds = [-(-(-(-T // 128) * (-(-inp // 128) + extra)) // 512) for extra in (0, -(-r // 128))]
    assert rounds[0] == rounds[1]
    s = 0.5
    lay, Wq, Pq, d = _setup(T, out, inp, r, seed=T + out, sigma_B=2e-2)
    dx, ws = G.bf16_empty(T, inp, fill=float("nan")), G.workspace(L.OP_BWD, T, out, inp, r)
    dB = torch.full((r, inp), float("nan"), dtype=torch.float32, device="cuda")
    L.loqt_linear_bwd(d["dy"], d["x"], d["Wq"], d["Pq"], d["B"], s, dx, dB, False, ws)
    L.timing_enable(True)
    L.loqt_linear_bwd(d["dy"], d["x"], d["Wq"], d["Pq"], d["B"], s, dx, dB, False, ws)
    torch.cuda.synchronize()
    L.timing_enable(False)
    launches = {name: n for name, (n, _) in L.timing_read().items()}
    assert launches["gemm_z"] == 0 and launches["gemm_dx"] == 1
    dx_ref, dB_ref = O.loqt_linear_bwd(lay.dy, lay.x, Wq, Pq, lay.B, s)
    G.bf16_output_report(G.bf16_host(dx), dx_ref)
    assert G.max_err_over_rms(dB.cpu().numpy().astype(np.float64), dB_ref) <= TOL


@pytest.mark.gpu
def test_smaller_workspace_means_fewer_slices():
    """A workspace with no room for the slices of U and y is still accepted, down to the operands' own copies."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    T, out, inp, r, s = 16, 2050, 4100, 72, 0.5

    def region(rows, cols):
        return G.rup(rows * G.rup(cols, 8) * 2, 256)
    least = region(T, r) + region(out, inp) + region(out, r)
    assert least < L.loqt_workspace_bytes(L.OP_FWD, T, out, inp, r)
    lay, Wq, Pq, d = _setup(T, out, inp, r, seed=3, sigma_B=2e-2)
    y_ref = O.loqt_linear_fwd(lay.x, Wq, Pq, lay.B, s)
    for extra in (0, 256, 2 * T * 72 * 4):
        y = G.bf16_empty(T, out, fill=float("nan"))
        L.loqt_linear_fwd(d["x"], d["Wq"], d["Pq"], d["B"], s, y,
                          torch.empty(least + extra, dtype=torch.uint8, device="cuda"))
        assert G.max_err_over_rms(O.bf16_to_f64(G.bf16_host(y)), y_ref) <= TOL
    with pytest.raises(L.LoqtError):
        L.loqt_linear_fwd(d["x"], d["Wq"], d["Pq"], d["B"], s, y,
                          torch.empty(least - 1, dtype=torch.uint8, device="cuda"))
