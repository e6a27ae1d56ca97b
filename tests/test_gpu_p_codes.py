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
