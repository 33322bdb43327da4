"""Slot-tree passes that take their layers' deepest rows once per distinct vertex of a micrograph, against the same call
without the tree's shape (plan.fuse_tree = 0): the same bits in the last layer and in every row the layers store."""
import ctypes

import pytest
import torch

from helpers import to_bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # graph, fanouts, seeds, group, merge, dtype, dim, hidden, layers that take distinct rows
    ("rmat", [10, 10], 2100, 1, False, torch.float32, 256, 512, 1),            # 42 % of the vertices have no neighbours
    ("rmat", [9, 11, 3], 1200, 1, False, torch.float32, 100, 260, 2),          # widths off the tile, fewer than 2048 micrographs
    ("rmat", [9, 11, 3], 700, 1, False, torch.float32, 100, 260, 1),           # the second layer too small for it
    ("ring", [4, 3, 3, 2], 2200, 1, False, torch.float32, 64, 256, 3),         # four layers; levels of 2, 3, 4 distinct vertices
    ("rmat", [16, 32, 2], 300, 1, False, torch.float32, 64, 256, 1),           # 512 slots a micrograph on the widest level
    ("rmat", [64, 2], 700, 1, False, torch.bfloat16, 256, 512, 1),             # the widest group of siblings, exchanged operands
    ("rmat", [10, 10, 10], 300, 3, True, torch.float16, 128, 512, 2),          # a merged group, three keys
    ("rmat", [10, 10], 6000, 2, False, torch.float16, 256, 512, 1),            # batches of a group run one after the other
    ("rmat", [12, 10, 2], 1500, 2, True, torch.bfloat16, 128, 520, 2),         # workgroups that walk over 256-row tiles
]


def _graph(kind):
    from paper_2409_00657_amd import synth
    if kind == "rmat":
        return synth.rmat_graph(13, 9.0, seed=11, device=DEV)
    n = 4096                                       # a vertex and the next
    off = torch.arange(n + 1, dtype=torch.int64, device=DEV) * 2
    idx = torch.stack([torch.arange(n), (torch.arange(n) + 1) % n], 1).view(-1).to(torch.int32).to(DEV)
    return synth.Graph(n, off, idx)


@pytest.mark.parametrize("kind,fan,B,G,merge,dt,d,hidden,layers", CASES)
def test_distinct_rows_give_the_plain_bits(kind, fan, B, G, merge, dt, d, hidden, layers):
    from paper_2409_00657_amd import synth
    from paper_2409_00657_amd.pipeline import HotPath
    g = _graph(kind)
    n, L = g.n_vertices, len(fan)
    X = synth.features(n, d, dt, device=DEV)
    W = synth.sage_weights(d, hidden, L, dt, device=DEV, bias=True)
    tree = HotPath(g.offsets, g.indices, X, W, B, fan, group=G, merge=merge, fuse_tree=True)
    plain = HotPath(g.offsets, g.indices, X, W, B, fan, group=G, merge=merge, fuse_tree=False)
    # the plan asks for the distinct rows' scratch: the same plan over a graph too dense for repeats asks for less
    ws = int(tree._lib.hopgnn_batch_tree_ws_bytes(ctypes.byref(tree.plan)))
    edges, tree.plan.graph.n_edges = tree.plan.graph.n_edges, 1 << 40
    without = int(tree._lib.hopgnn_batch_tree_ws_bytes(ctypes.byref(tree.plan)))
    tree.plan.graph.n_edges = edges
    sh, es = tree.shape, X.element_size()
    rows = [max((sh.levels[L - k] * hidden * es for k in range(1, layers + 1) if k % 2 == par), default=0) for par in (0, 1)]
    lists = sum(sh.levels[L - k] * (G if not merge else 1) * 8 for k in range(1, layers + 1))
    assert 0 <= ws - without - sum(rows) - lists - sh.n_dst(1) * 4 < 4096 * (layers + 3) + 8 * B * G * layers
    for it, n_batches in enumerate((G, G, max(G - 1, 1))):      # the last call fills a part of the plan
        seeds = synth.seeds(n, B * n_batches, 300 + it, device=DEV)
        keys = [17 * it + b for b in range(n_batches)]
        out_t = torch.full((n_batches * B, hidden), float("nan"), dtype=dt, device=DEV)
        out_p = torch.full((n_batches * B, hidden), float("nan"), dtype=dt, device=DEV)
        for h in tree.H:
            h.fill_(float("nan"))
        tree.forward(seeds, keys, out_t)
        plain.forward(seeds, keys, out_p)
        torch.cuda.synchronize()
        assert not torch.isnan(out_t.float()).any()
        assert to_bits(out_t).tobytes() == to_bits(out_p).tobytes()
        if n_batches != G:
            continue
        assert torch.equal(tree.ids, plain.ids) and torch.equal(tree.remap, plain.remap)
        for k in range(1, L):
            keep = sh.n_dst(k + 1)
            assert to_bits(tree.H[k - 1][:keep]).tobytes() == to_bits(plain.H[k - 1][:keep]).tobytes(), k
            assert torch.isnan(tree.H[k - 1][keep:].float()).all()
