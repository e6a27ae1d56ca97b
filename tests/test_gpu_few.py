"""Forward calls with a handful of tokens (the codes are expanded in registers, no copy of the weight): sizes that end
inside chunks, row tiles and token tiles, padding that holds NaN, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import loqt_oracle as O
from paper_2405_16528_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # T, out, in, r
    (1, 130, 40, 8),          # contractions shorter than a chunk of 128
    (16, 512, 512, 128),      # whole chunks only
    (17, 300, 1000, 72),      # second token tile with one token; chunk tails of both segments
    (32, 100, 2176, 200),     # 17 whole chunks: one wave has two
    (3, 4200, 136, 40),       # two row tiles per work-group
    (31, 8300, 200, 64),      # three
    (16, 12300, 328, 24),     # four, one token tile
    (32, 12300, 72, 24),      # four, two token tiles
    (9, 72, 8300, 40),        # U in slices of its contraction
    (16, 12200, 2200, 24),    # three, whole chunks (one in flight in bf16), one wave has two
    (32, 16500, 392, 16),     # three in two rounds; bf16 rows leave the kernel
]


def _nan_padded(bits, extra):
    """bf16 bits (rows, cols) in a device buffer whose pitch padding is NaN."""
    rows, cols = bits.shape
    buf = np.full((rows, (cols + 7) // 8 * 8 + extra), 0x7FC0, dtype=np.uint16)
    buf[:, :cols] = bits
    return torch.from_numpy(buf.view(np.int16)).cuda().view(torch.bfloat16)[:, :cols]


def _nan_scaled(q):
    """NF4 on the device with 64 columns of padding, its codes arbitrary and its scales NaN."""
    from tests import gpu_util as G
    codes, absmax = q
    t = G.nf4_dev(codes, absmax, G.rup(codes.shape[1], 64) + 64)
    t.codes[:, -32:] = 0xF3
    t.absmax[:, -1] = float("nan")
    return t


@pytest.mark.parametrize("T,out,inp,r", CASES)
def test_forward_parity(T, out, inp, r):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    assert L.resolved_path(L.OP_FWD, T, out, inp) == L.PATH_FUSED
    rng = synth.rng_for(T, "few", out, inp)
    s = 0.5
    Wq = O.nf4_quantize(synth.normal_f32(rng, (out, inp), 0.02))
    Pq = O.nf4_quantize(synth.normal_f32(rng, (out, r), out ** -0.5))
    B, x = synth.normal_bf16(rng, (r, inp), 2e-2), synth.normal_bf16(rng, (T, inp), 1.0)
    y = G.bf16_empty(T, out, fill=float("nan"))
    L.loqt_linear_fwd(_nan_padded(x, 8), _nan_scaled(Wq), _nan_scaled(Pq), _nan_padded(B, 16), s, y,
                      G.workspace(L.OP_FWD, T, out, inp, r))
    torch.cuda.synchronize()
    ref = O.loqt_linear_fwd(x, Wq, Pq, B, s)
    # operands: the levels in bf16 instead of the scaled weights (each off by at most 2^-8), output in bf16
    err = G.bf16_output_report(G.bf16_host(y), ref)[0]
    print(f"few T={T} out={out} in={inp} r={r}: err/rms y {err:.2e}")
    # and not less exact than the expanded weight
    L.set_path(L.PATH_PREPASS)
    try:
        y2 = G.bf16_empty(T, out)
        L.loqt_linear_fwd(_nan_padded(x, 8), _nan_scaled(Wq), _nan_scaled(Pq), _nan_padded(B, 16), s, y2,
                          G.workspace(L.OP_FWD, T, out, inp, r))
    finally:
        L.set_path(L.PATH_AUTO)
    rel = [np.linalg.norm(O.bf16_to_f64(G.bf16_host(t)) - ref) / np.linalg.norm(ref) for t in (y, y2)]
    assert rel[0] <= rel[1] * 1.1 + 2e-4, rel  # (a few outputs of one token scatter by a tenth)


@pytest.mark.parametrize("T,out,inp,r", CASES)
def test_forward_nq_parity(T, out, inp, r):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    rng = synth.rng_for(T, "few nq", out, inp)
    s = 0.5
    W, P = synth.normal_bf16(rng, (out, inp), 0.02), synth.normal_bf16(rng, (out, r), out ** -0.5)
    B, x = synth.normal_bf16(rng, (r, inp), 2e-2), synth.normal_bf16(rng, (T, inp), 1.0)
    y = G.bf16_empty(T, out, fill=float("nan"))
    L.loqt_linear_fwd_nq(_nan_padded(x, 8), _nan_padded(W, 8), _nan_padded(P, 0), _nan_padded(B, 16), s, y,
                         G.workspace(L.OP_FWD_NQ, T, out, inp, r))
    torch.cuda.synchronize()
    G.bf16_output_report(G.bf16_host(y), O.loqt_linear_fwd_nq(x, W, P, B, s))


@pytest.mark.parametrize("T", [5, 20])
@pytest.mark.parametrize("mag", [3e38, 1e-30])
def test_inputs_at_the_ends_of_the_range(T, mag):
    """A block's products are summed before they meet its scale: that must not leave fp32's range where y is inside it."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    out, inp, r, s = 520, 1100, 72, 1.0
    rng = synth.rng_for(T, "few range")
    Wq = O.nf4_quantize(synth.normal_f32(rng, (out, inp), 1e-3))
    Pq = O.nf4_quantize(synth.normal_f32(rng, (out, r), 1e-3))
    B = synth.normal_bf16(rng, (r, inp), 1e-3)
    x = O.f32_to_bf16_rne((np.sign(rng.standard_normal((T, inp))) * mag * rng.uniform(0.5, 1.0, (T, inp))).astype(np.float32))
    y = G.bf16_empty(T, out, fill=float("nan"))
    L.loqt_linear_fwd(G.bf16_dev(x), G.nf4_dev(*Wq), G.nf4_dev(*Pq), G.bf16_dev(B), s, y, G.workspace(L.OP_FWD, T, out, inp, r))
    torch.cuda.synchronize()
    G.bf16_output_report(G.bf16_host(y), O.loqt_linear_fwd(x, Wq, Pq, B, s))


def test_the_line_between_the_forms():
    """32 tokens are a handful, 33 are not; the backward pass and the pair that keeps the weight never are."""
    from paper_2405_16528_amd import binding as L
    assert L.resolved_path(L.OP_FWD, 32, 512, 512) == L.PATH_FUSED
    assert L.resolved_path(L.OP_FWD, 33, 512, 512) == L.PATH_PREPASS
    assert L.resolved_path(L.OP_BWD, 16, 512, 512) == L.PATH_PREPASS


def _us_per_call(forms, calls=20, runs=9):
    """The fastest of several replays of each form (recorded, so that the host is not what is measured), taken in turn."""
    graphs = []
    for form in forms:
        form()
        torch.cuda.synchronize()
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            for _ in range(calls):
                form()
    best = [float("inf")] * len(forms)
    for _ in range(runs):
        for j, graph in enumerate(graphs):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            graph.replay()
            end.record()
            end.synchronize()
            best[j] = min(best[j], begin.elapsed_time(end) * 1e3 / calls)
    return best


@pytest.mark.parametrize("T,out,inp,r", [
    (32, 7232, 128, 24),      # one chunk per product: fifteen of sixteen waves have none
    (16, 2112, 128, 112),
    (32, 512, 512, 128),      # four
    (32, 11904, 128, 8),      # three row tiles per work-group
    (32, 17216, 192, 192),    # more rows than the kernel takes
])
def test_unquantised_forward_is_not_behind_the_plain_products(T, out, inp, r):
    """With as good as no weight to stream the kernel has to cost no more than the products it stands in for."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    rng = synth.rng_for(T, "few time", out, inp)
    W, P = G.bf16_dev(synth.normal_bf16(rng, (out, inp), 0.02)), G.bf16_dev(synth.normal_bf16(rng, (out, r), out ** -0.5))
    B, x = G.bf16_dev(synth.normal_bf16(rng, (r, inp), 2e-2)), G.bf16_dev(synth.normal_bf16(rng, (T, inp), 1.0))
    y, ws = G.bf16_empty(T, out), G.workspace(L.OP_FWD_NQ, T, out, inp, r)

    def plain():
        L.loqt_linear_fwd_nq(x, W, P, B, 0.5, y, ws)

    def other():
        L.set_path(L.PATH_PREPASS)
        try:
            plain()
        finally:
            L.set_path(L.PATH_AUTO)
    few_us, other_us = _us_per_call([plain, other])
    print(f"few T={T} out={out} in={inp} r={r}: {few_us:.1f} us, plain products {other_us:.1f}")
    assert few_us <= 1.15 * other_us


@pytest.mark.parametrize("T,inp", [(16, 8320), (3, 5760), (32, 4097)])
def test_unquantised_forward_with_no_room_for_slices(T, inp):
    """U over a long contraction goes out in slices where the workspace has room for them; one that holds U and nothing else
    is accepted as well."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    out, r, s = 96, 40, 0.5
    rng = synth.rng_for(T, "few room", inp)
    W, P = synth.normal_bf16(rng, (out, inp), 0.02), synth.normal_bf16(rng, (out, r), out ** -0.5)
    B, x = synth.normal_bf16(rng, (r, inp), 2e-2), synth.normal_bf16(rng, (T, inp), 1.0)
    least = G.rup(T * G.rup(r, 8) * 2, 256)
    assert least < L.loqt_workspace_bytes(L.OP_FWD_NQ, T, out, inp, r)
    ref = O.loqt_linear_fwd_nq(x, W, P, B, s)
    for size in (least, L.loqt_workspace_bytes(L.OP_FWD_NQ, T, out, inp, r)):
        ws = torch.full((size + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        y = G.bf16_empty(T, out, fill=float("nan"))
        L.loqt_linear_fwd_nq(G.bf16_dev(x), G.bf16_dev(W), G.bf16_dev(P), G.bf16_dev(B), s, y, ws[:size])
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0xFF).all())
        G.bf16_output_report(G.bf16_host(y), ref)


@pytest.mark.parametrize("T,out,inp,r,beside", [
    # (contractions from 1300, 1800 and 2300 on, by rows: the lines from which U goes beside the weight; shorter ones come last)
    (4, 3600, 1304, 40, True),      # rows of W and U per work-group (16 each): 1 and 1
    (17, 3601, 1336, 520, True),    # 2 and 1
    (32, 8201, 2312, 72, True),     # 3 and 1
    (3, 11001, 2312, 440, True),    # 3 and 2
    (11, 11001, 2312, 900, True),   # 4 and 1
    (16, 13001, 2312, 900, True),   # 4 and 2
    (8, 11001, 2312, 900, False),   # as many work-groups as the chip holds only with slower tiles
    (18, 13001, 2312, 40, False),
    (31, 2000, 8, 8, False),        # no room for the sums
    (4, 3600, 1296, 40, False),     # U first
    (17, 4112, 1792, 72, False),
    (3, 8208, 2288, 40, False),
])
def test_u_beside_the_weight(T, out, inp, r, beside):
    """U and the sums of x deq(W)^T in one launch, the rank-r term in the next: against the oracle, and nothing past the workspace."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    rng = synth.rng_for(T, "few beside", out, inp)
    s = 0.5
    Wq = O.nf4_quantize(synth.normal_f32(rng, (out, inp), 0.02))
    Pq = O.nf4_quantize(synth.normal_f32(rng, (out, r), out ** -0.5))
    B, x = synth.normal_bf16(rng, (r, inp), 2e-2), synth.normal_bf16(rng, (T, inp), 1.0)
    size = L.loqt_workspace_bytes(L.OP_FWD, T, out, inp, r)
    if inp == 8:  # U and the copies of W and P, the least that a call accepts
        size = sum(G.rup(n * G.rup(k, 8) * 2, 256) for n, k in ((T, r), (out, inp), (out, r)))
        assert size < 4 * T * out
    ws = torch.full((size + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    y = G.bf16_empty(T, out, fill=float("nan"))
    L.timing_enable(True)
    L.loqt_linear_fwd(_nan_padded(x, 8), _nan_scaled(Wq), _nan_scaled(Pq), _nan_padded(B, 16), s, y, ws[:size])
    torch.cuda.synchronize()
    L.timing_enable(False)
    n = {k: v[0] for k, v in L.timing_read().items()}
    assert (n["gemm_u"], n["gemm_y"]) == (1, 1)
    assert bool((ws[size:] == 0xFF).all())
    # the sums of the weight lie behind U
    u_end = G.rup(T * G.rup(r, 8) * 2, 256)
    assert bool((ws[u_end:u_end + 16 * out] != 0xFF).any()) == beside
    G.bf16_output_report(G.bf16_host(y), O.loqt_linear_fwd(x, Wq, Pq, B, s))
