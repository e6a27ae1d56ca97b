"""The last rows and columns of bf16 results: stores at the edges of a tile are bounded by segments of eight, four, two and one
elements.  A result is the corner of that of a larger matrix (every tile sums in the same order: the same bits), and nothing is
written beside it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

GUARD = 7.0


def _guarded(rows, cols, like=None):
    """rows x cols inside a larger buffer of GUARD"""
    buf = torch.full((rows + 3, (cols + 7) // 8 * 8 + 16), GUARD, dtype=torch.bfloat16, device="cuda")
    if like is not None:
        buf[:rows, :cols] = like[:rows, :cols]
    return buf, buf[:rows, :cols]


def _untouched(buf, rows, cols):
    return bool((buf[rows:] == GUARD).all()) and bool((buf[:, cols:] == GUARD).all())


@pytest.mark.parametrize("rows", [129, 256, 300])
@pytest.mark.parametrize("cols", [257, 258, 259, 260, 261, 262, 263, 384, 391, 449])
@pytest.mark.parametrize("tile", ["256x256", "256x128", "128x128", "auto"])
def test_rows_and_columns_past_the_last_full_segment(tile, rows, cols):
    from tests import gpu_util as G
    from paper_2405_16528_amd import binding as L
    g = torch.Generator(device="cuda").manual_seed(rows * 1000 + cols)
    M, N, K, r = 512, 512, 200, 72
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((N, K), generator=g, device="cuda").to(torch.bfloat16)
    P = torch.randn((N, r), generator=g, device="cuda").to(torch.bfloat16)
    B = torch.randn((r, K), generator=g, device="cuda").to(torch.bfloat16)
    # the transposed problem of the fold and the unquantised merge: their columns are those of B
    Wq, Pq = L.nf4_quantize(torch.randn((M, N), generator=g, device="cuda")), L.nf4_quantize(torch.randn((M, r), generator=g, device="cuda"))
    Wn = torch.randn((M, N), generator=g, device="cuda").to(torch.bfloat16)
    Pn = torch.randn((M, r), generator=g, device="cuda").to(torch.bfloat16)
    Bn = torch.randn((r, N), generator=g, device="cuda").to(torch.bfloat16)
    xs = torch.randn((256, N), generator=g, device="cuda").to(torch.bfloat16)

    def rows_of(q, n):
        return L.NF4Tensor(q.codes[:n], q.absmax[:n], n, q.cols, q.ld)

    def results(m, n):
        y_buf, y = _guarded(m, n)
        L.loqt_linear_fwd_nq(x[:m], W[:n], P[:n], B, 0.5, y, G.workspace(L.OP_FWD_NQ, m, n, K, r))
        w_buf, w_eff = _guarded(m, n)
        Wm = rows_of(Wq, m)
        Wm.cols = n
        L.loqt_linear_fwd_save(xs[:, :n], Wm, rows_of(Pq, m), Bn[:, :n], 0.5, G.bf16_empty(256, m), w_eff,
                               G.workspace(L.OP_FWD_SAVE, 256, m, n, r))
        a_buf, acc = _guarded(m, n, Wn)
        L.loqt_merge_nq(acc, Pn[:m], Bn[:, :n], 0.5)
        torch.cuda.synchronize()
        for buf in (y_buf, w_buf, a_buf):
            assert _untouched(buf, m, n)
        return y.clone(), w_eff.clone(), acc.clone()
    try:
        L.set_path(L.PATH_FOLDED)  # (whatever the rows)
        L.set_tile({"256x256": L.TILE_256x256, "256x128": L.TILE_256x128, "128x128": L.TILE_128x128, "auto": L.TILE_AUTO}[tile])
        for small, large in zip(results(rows, cols), results(M, N)):
            assert torch.equal(small, large[:rows, :cols])
    finally:
        L.set_tile(L.TILE_AUTO)
        L.set_path(L.PATH_AUTO)
