"""The fold and the merge of a small weight of low rank read P as its codes: the same bits as with P expanded by a launch of its
own, on ranks that end anywhere inside a k-tile, with rows and columns that end inside tiles, up to the largest that they take."""
import numpy as np
import pytest
import torch

from oracle import loqt_oracle as O

pytestmark = pytest.mark.gpu


def _launches(L, f):
    L.timing_enable(True)
    f()
    torch.cuda.synchronize()
    L.timing_enable(False)
    return {k: v[0] for k, v in L.timing_read().items()}


@pytest.mark.parametrize("out,inp,r,codes", [
    (1, 8, 1, True), (64, 128, 64, True), (65, 136, 63, True), (130, 72, 65, True), (129, 130, 129, True), (300, 264, 128, True),
    (63, 1030, 192, True), (1000, 333, 200, True), (190, 520, 255, True), (512, 512, 256, True), (64, 128, 257, False), (2000, 130, 40, True),
    (2048, 2048, 64, True), (2049, 2048, 64, False)])
def test_same_bits_as_expanded(out, inp, r, codes):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    s, T = 0.5, 64
    g = np.random.default_rng(out + r)
    Wq, Pq = (G.nf4_dev(*O.nf4_quantize((g.standard_normal(n) * 0.02).astype(np.float32))) for n in ((out, inp), (out, r)))
    x, B = ((torch.from_numpy(g.standard_normal((n, G.rup(inp, 8)))) * 0.02).bfloat16().cuda()[:, :inp] for n in (T, r))
    got = []
    for path in (L.PATH_AUTO, L.PATH_FOLDED):
        w_eff = G.bf16_empty(out, inp, fill=float("nan"))
        y = G.bf16_empty(T, out, fill=float("nan"))
        L.set_path(path)
        try:
            n = _launches(L, lambda: L.loqt_linear_fwd_save(x, Wq, Pq, B, s, y, w_eff, G.workspace(L.OP_FWD, T, out, inp, r)))
            merged = []
            m = _launches(L, lambda: merged.append(L.loqt_merge_requant(Wq, Pq, B, s, out=L.NF4Tensor.empty(out, inp),
                                                                                ws=G.workspace(L.OP_MERGE, 0, out, inp, r))))
        finally:
            L.set_path(L.PATH_AUTO)
        expanded = not (codes and path == L.PATH_AUTO)
        assert (n["prepass"], m["prepass"]) == (expanded, expanded)
        got.append((w_eff, y, merged[0].codes, merged[0].absmax))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("layers,codes", [
    ([(65, 136, 63), (130, 72, 65), (300, 264, 256), (1, 8, 1)], True),
    ([(1000, 333, 128), (63, 1030, 40), (2048, 2048, 64)], True),      # up to 900 tiles with ranks of 128 at most
    ([(2048, 2048, 64), (64, 128, 129)], False),                       # 64x128, 513 tiles
    ([(64, 128, 300), (190, 520, 255)], False),
    ([(3000, 2048, 200), (512, 1030, 64)], False),                     # between: 128x128
    ([(4096, 4096, 64), (64, 128, 64)], False),
    ([(2048, 2048, 520), (2048, 4224, 512)], False),                   # a little over two rounds of 64x128, high ranks: 128x128
])
def test_group_same_bits_as_one_by_one(layers, codes):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    g = np.random.default_rng(len(layers))
    sets = []
    for out, inp, r in layers:
        Wq, Pq = (G.nf4_dev(*O.nf4_quantize((g.standard_normal(n) * 0.02).astype(np.float32))) for n in ((out, inp), (out, r)))
        B = (torch.from_numpy(g.standard_normal((r, G.rup(inp, 8)))) * 0.02).bfloat16().cuda()[:, :inp]
        sets.append((Wq, L.NF4Tensor.empty(out, inp), Pq, B, 0.5))
    descs = L.make_merge_descs(sets)
    n = _launches(L, lambda: L.loqt_merge_requant_batched(descs, torch.empty(L.merge_descs_workspace_bytes(descs), dtype=torch.uint8, device="cuda")))
    assert (n["prepass"], n["merge_requant"]) == (0 if codes else 1, 1)
    L.set_path(L.PATH_FOLDED)
    try:
        for Wq, got, Pq, B, s in sets:
            ref = L.loqt_merge_requant(Wq, Pq, B, s, out=L.NF4Tensor.empty(Wq.rows, Wq.cols))
            assert torch.equal(ref.codes, got.codes) and torch.equal(ref.absmax, got.absmax)
    finally:
        L.set_path(L.PATH_AUTO)


def test_output_over_the_codes_of_P():
    """A merge that writes where P is reads all of P first."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    g = np.random.default_rng(3)
    out, inp, r = 512, 512, 256
    Wq, Pq = (G.nf4_dev(*O.nf4_quantize((g.standard_normal(n) * 0.02).astype(np.float32))) for n in ((out, inp), (out, r)))
    B = (torch.from_numpy(g.standard_normal((r, inp))) * 0.02).bfloat16().cuda()
    ref = L.loqt_merge_requant(Wq, Pq, B, 0.5, out=L.NF4Tensor.empty(out, inp))
    got = L.NF4Tensor.empty(out, inp)
    over = got.codes.view(-1)[:Pq.codes.numel()].view(Pq.codes.shape)
    over.copy_(Pq.codes)
    Pq.codes = over
    n = _launches(L, lambda: L.loqt_merge_requant(Wq, Pq, B, 0.5, out=got))
    assert n["prepass"] == 1
    assert torch.equal(ref.codes, got.codes) and torch.equal(ref.absmax, got.absmax)


def _in_place_of(t, buf):
    """t's content at the start of the buffer `buf`, as a view of it."""
    over = buf.view(torch.uint8).reshape(-1)[:t.numel() * t.element_size()].view(t.dtype).view(t.shape)
    over.copy_(t)
    return over


@pytest.mark.parametrize("part", ["codes", "absmax"])
def test_saved_weight_over_P(part):
    """A forward call that leaves W_eff where P is reads all of P first."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    g = np.random.default_rng(4)
    T, out, inp, r = 64, 512, 512, 256
    Wq, Pq = (G.nf4_dev(*O.nf4_quantize((g.standard_normal(n) * 0.02).astype(np.float32))) for n in ((out, inp), (out, r)))
    x, B = ((torch.from_numpy(g.standard_normal((n, inp))) * 0.02).bfloat16().cuda() for n in (T, r))
    got = []
    for over in (False, True):
        w_eff = torch.zeros((out, inp), dtype=torch.bfloat16, device="cuda")
        y = G.bf16_empty(T, out, fill=float("nan"))
        if over:
            setattr(Pq, part, _in_place_of(getattr(Pq, part), w_eff))
        n = _launches(L, lambda: L.loqt_linear_fwd_save(x, Wq, Pq, B, 0.5, y, w_eff, G.workspace(L.OP_FWD_SAVE, T, out, inp, r)))
        assert n["prepass"] == over
        got.append((w_eff, y))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("target,part", [("codes", "codes"), ("codes", "absmax"), ("absmax", "absmax")])
def test_group_that_writes_over_another_layers_P(target, part):
    """The merges of a group share a launch: an output of one in the place of another's P, and every P is read first."""
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    g = np.random.default_rng(5)
    sets = []
    for out, inp, r in ((512, 512, 128), (300, 264, 64)):
        Wq, Pq = (G.nf4_dev(*O.nf4_quantize((g.standard_normal(n) * 0.02).astype(np.float32))) for n in ((out, inp), (out, r)))
        B = (torch.from_numpy(g.standard_normal((r, inp))) * 0.02).bfloat16().cuda()
        sets.append((Wq, L.NF4Tensor.empty(out, inp), Pq, B, 0.5))
    refs = [L.loqt_merge_requant(Wq, Pq, B, s, out=L.NF4Tensor.empty(Wq.rows, Wq.cols)) for Wq, _, Pq, B, s in sets]
    torch.cuda.synchronize()
    setattr(sets[1][2], part, _in_place_of(getattr(sets[1][2], part), getattr(sets[0][1], target)))
    descs = L.make_merge_descs(sets)
    n = _launches(L, lambda: L.loqt_merge_requant_batched(descs, torch.empty(L.merge_descs_workspace_bytes(descs), dtype=torch.uint8, device="cuda")))
    assert (n["prepass"], n["merge_requant"]) == (1, 1)
    for ref, (_, got, *_) in zip(refs, sets):
        assert torch.equal(ref.codes, got.codes) and torch.equal(ref.absmax, got.absmax)
