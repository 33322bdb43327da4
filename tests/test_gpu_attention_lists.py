"""Attention backward collected by source rows: the lane layout's edges, the sizes where the route changes, and
inputs with more entries than the lists hold (the kernels with float atomics take those), against the oracle
at the bounds of the general test."""
import pytest
import torch

import test_gpu_layer_bwd as general
from test_gpu_layer_bwd import hb  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SHAPES = [  # n_src, n_dst, d_in, d_out, longest segment, heads
    (700, 511, 20, 24, 5, 6), (700, 512, 20, 24, 5, 6),       # one word a head; either side of the row threshold
    (900, 600, 16, 320, 7, 16),                               # five words on eight lanes, two groups of heads
    (800, 520, 12, 260, 9, 1), (800, 520, 12, 512, 9, 1),     # two words a lane: 65 and 128 words a head
    (900, 530, 8, 30, 6, 3),                                  # ten columns a head: no whole words
    (300, 520, 16, 32, 150, 2)]                               # 75 entries a row on average: past the lists


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", SHAPES)
def test_attention_backward_by_source_rows(hb, orc, dt, shape):  # noqa: F811
    general.test_attention_backward_vs_oracle(hb, orc, dt, shape)


def test_the_lists_are_rebuilt_on_every_call(hb):  # noqa: F811
    """The same workspace, three calls, gradients that differ by summation order only."""
    import numpy as np
    rng = np.random.default_rng(4)
    n_src, n_dst, d_in, d_out, heads = 900, 640, 24, 64, 4
    H, W, _, dOut, indptr, idx, self_idx = general._inputs(rng, torch.float32, (n_src, n_dst, d_in, d_out, 8))
    t, dev = general._t, general.DEV
    a_s, a_d = torch.randn(d_out, device=dev), torch.randn(d_out, device=dev)
    fwd_ws = torch.empty(hb.hopgnn_gat_fwd_ws_bytes(torch.float32, n_src, d_in, d_out, heads), dtype=torch.uint8, device=dev)
    out = torch.empty((n_dst, d_out), device=dev)
    hb.hopgnn_gat_fwd(H, n_src, t(self_idx), t(indptr), t(idx), n_dst, W, a_s, a_d, None, heads, True, out, fwd_ws)
    ws = torch.empty(hb.hopgnn_gat_bwd_ws_bytes(torch.float32, n_src, n_dst, d_in, d_out, heads), dtype=torch.uint8, device=dev)
    ws.fill_(0x5A)
    first = None
    for _ in range(3):
        g = [torch.zeros((d_in, d_out), device=dev), torch.zeros(d_out, device=dev), torch.zeros(d_out, device=dev)]
        dH = torch.empty((n_src, d_in), device=dev)
        hb.hopgnn_gat_bwd(H, n_src, t(self_idx), t(indptr), t(idx), n_dst, W, a_s, a_d, out, fwd_ws, True, t(dOut), heads,
                          g[0], g[1], g[2], None, dH, ws)
        torch.cuda.synchronize()
        got = g + [dH]
        first = first or [x.clone() for x in got]
        for x, y in zip(got, first):       # fp32 sums in another order (the bound of the general test)
            assert float((x - y).abs().max() / y.pow(2).mean().sqrt()) <= 1e-4


@pytest.mark.parametrize("heads,d_out", [(4, 64), (3, 30)])      # by source rows; the kernels with float atomics
def test_entries_past_the_device_count_stay_inside_the_lists(hb, heads, d_out):  # noqa: F811
    """Entries (and the rows' own terms, without self_idx) that name rows between the device's count and the
    capacity, with z and scores of zero there: the result is that of the whole capacity with zero rows, and
    nothing past the count or outside the workspace is written."""
    import numpy as np
    rng = np.random.default_rng(7)
    n_src, n_dst, live, d_in = 1200, 900, 600, 24
    H, W, _, dOut, indptr, idx, _ = general._inputs(rng, torch.float32, (n_src, n_dst, d_in, d_out, 8))
    assert int((idx >= live).sum()) > 1000
    H[live:] = 0
    t, dev = general._t, general.DEV
    a_s, a_d = torch.randn(d_out, device=dev), torch.randn(d_out, device=dev)
    ws_bytes = hb.hopgnn_gat_bwd_ws_bytes(torch.float32, n_src, n_dst, d_in, d_out, heads)
    res = []
    for count in (None, torch.tensor([live], dtype=torch.int64, device=dev)):
        fwd_ws = torch.zeros(hb.hopgnn_gat_fwd_ws_bytes(torch.float32, n_src, d_in, d_out, heads), dtype=torch.uint8, device=dev)
        out = torch.empty((n_dst, d_out), device=dev)
        hb.hopgnn_gat_fwd(H, n_src, None, t(indptr), t(idx), n_dst, W, a_s, a_d, None, heads, True, out, fwd_ws, count)
        room = torch.full((ws_bytes + (1 << 20),), 0x5A, dtype=torch.uint8, device=dev)      # positions of 0x5A5A5A5A if left alone
        g = [torch.zeros((d_in, d_out), device=dev), torch.zeros(d_out, device=dev), torch.zeros(d_out, device=dev)]
        dH = torch.full((n_src, d_in), 7.0, device=dev)
        hb.hopgnn_gat_bwd(H, n_src, None, t(indptr), t(idx), n_dst, W, a_s, a_d, out, fwd_ws, True, t(dOut), heads,
                          g[0], g[1], g[2], None, dH, room[:ws_bytes], n_src_dev=count)
        torch.cuda.synchronize()
        assert bool((room[ws_bytes:] == 0x5A).all())
        res.append([out] + g + [dH])
    assert bool((res[1][4][live:] == 7.0).all())
    for x, y in zip(res[1][:4] + [res[1][4][:live]], res[0][:4] + [res[0][4][:live]]):     # the bound of the test above
        assert float((x - y).abs().max() / y.pow(2).mean().sqrt()) <= 1e-4


HUBS = [  # as SHAPES
    (700, 2400, 20, 24, 14, 6), (900, 3200, 16, 320, 9, 16), (800, 3000, 12, 260, 10, 1),
    (3, 3000, 16, 64, 6, 4)]            # fewer source rows than a workgroup has wavefronts, all with long lists


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", HUBS)
def test_long_lists_are_cut_into_pieces(hb, orc, monkeypatch, dt, shape):  # noqa: F811
    """A third of the entries name one row, and rows 1..16 are named by 500..515 entries each (their own terms
    come on top): lists on both sides of a piece's length and of many pieces."""
    plain = general._rand_csr

    def hubs(rng, n_dst, n_src, max_len, p_invalid=0.15):
        indptr, idx = plain(rng, n_dst, n_src, max_len, p_invalid)
        order = rng.permutation(len(idx))
        cut = len(idx) // 3
        idx[order[:cut]] = 0
        for row in range(1, min(17, n_src)):
            idx[order[cut:cut + 499 + row]] = row
            cut += 499 + row
        return indptr, idx

    monkeypatch.setattr(general, "_rand_csr", hubs)
    general.test_attention_backward_vs_oracle(hb, orc, dt, shape)
