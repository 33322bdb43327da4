"""hopgnn_sample around the sizes where it changes its way: levels held in LDS with every distinct vertex drawn once
(from 2048 micrographs and 2 M slots, up to 512 slots on the widest non-leaf level and 4096 leaves), levels walked in memory
otherwise; bit for bit the oracle."""
import numpy as np
import pytest
import torch

from paper_2409_00657_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("fan", [[1], [1, 1, 1], [64], [65, 1], [256, 2], [257, 3], [512, 8], [512, 9], [513, 2], [8, 64, 8],
                                 [4096], [4097], [2, 2, 2, 2, 2, 2, 2, 2], [16, 16, 16], [3, 170, 1]])
@pytest.mark.parametrize("graph,B", [("few", 2048), ("rmat", 2049), ("rmat", 9)])
def test_levels_at_the_edges(orc, fan, graph, B):
    from paper_2409_00657_amd import binding as hb
    if graph == "few":      # 5 vertices, one without neighbours: nearly every slot repeats another
        off = torch.tensor([0, 4, 5, 5, 9, 11], dtype=torch.int64, device=DEV)
        idx = torch.tensor([1, 3, 4, 2, 3, 0, 0, 1, 4, 3, 2], dtype=torch.int32, device=DEV)
    else:                   # as many different vertices as draws, degrees from 0 to thousands
        g = synth.rmat_graph(14, 14.0, seed=5, device=DEV, offsets_i64=False)
        off, idx = g.offsets, g.indices
    n, L = off.numel() - 1, len(fan)
    seeds = synth.seeds(n, B, 2, device=DEV)
    seeds[3] = seeds[1]
    T = B * hb.hopgnn_slots_per_seed(fan)
    S = T - B * int(np.prod(fan))
    ids = torch.full((T,), -7, dtype=torch.int32, device=DEV)
    indptr = torch.full((S + 1,), -7, dtype=torch.int32, device=DEV)
    slot_idx = torch.full((max(S - B, 1),), -7, dtype=torch.int32, device=DEV)
    hb.hopgnn_sample(off, idx, seeds, fan, 2 ** 63 + 17, ids, indptr, slot_idx if L > 1 else None)
    torch.cuda.synchronize()
    ref_ids, ref_indptr = orc.sample(off.cpu().numpy(), idx.cpu().numpy(), seeds.cpu().numpy(), fan, 2 ** 63 + 17)
    np.testing.assert_array_equal(ids.cpu().numpy(), ref_ids)
    np.testing.assert_array_equal(indptr.cpu().numpy(), ref_indptr)
    if L > 1:
        ref = np.where(ref_ids[B:S] >= 0, B + np.arange(S - B), -1)
        np.testing.assert_array_equal(slot_idx.cpu().numpy()[:S - B], ref)
