"""hopgnn_pregather from the sizes where marks go through the per-workgroup table and slots are placed four at a time
(2 000 000 and 4 194 304 slots): the sorted set and the positions, on aligned and misaligned arrays and remainders."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_ids", [1_999_999, 2_000_000, 2_000_003, 4_194_303, 4_194_304, 4_194_307, 16_777_217 + 8192])
@pytest.mark.parametrize("shift", [0, 1])
def test_set_and_positions(n_ids, shift):
    from paper_2409_00657_amd import binding as hb
    n = 300_007
    g = torch.Generator(device=DEV).manual_seed(n_ids)
    ids = torch.full((n_ids + shift,), -1, dtype=torch.int32, device=DEV)
    ids[shift:] = (torch.rand(n_ids, generator=g, device=DEV) ** 4 * n).to(torch.int32)      # the low ids over and over
    ids[shift::7] = -1
    ids[-1], ids[shift + 5] = n - 1, 0
    remap = torch.full((n_ids + shift,), -9, dtype=torch.int32, device=DEV)
    uniq = torch.empty(min(n_ids, n), dtype=torch.int32, device=DEV)
    n_uniq = torch.zeros(1, dtype=torch.int64, device=DEV)
    ws = torch.empty(hb.hopgnn_pregather_ws_bytes(n_ids, n, hb.PG_BITMAP), dtype=torch.uint8, device=DEV)
    v = ids[shift:]
    for _ in range(2):
        hb.hopgnn_pregather(v, n, uniq, n_uniq, remap[shift:], ws, algo=hb.PG_BITMAP)
        ref = torch.unique(v[v >= 0])
        U = int(n_uniq)
        assert U == ref.numel() and torch.equal(uniq[:U], ref)
        r = remap[shift:]
        assert bool((r[v < 0] == -1).all()) and torch.equal(uniq[r[v >= 0].long()], v[v >= 0])
    assert shift == 0 or int(remap[0]) == -9
