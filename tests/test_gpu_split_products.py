"""The fp32 contractions (projection, weight gradient, input gradient) as eight bf16 products of split operands, against
64-bit products: tile edges, magnitudes at both ends of the type, infinities, single products, sums of one sign, and
the bits of a row beside different neighbours."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# A sum of K products in fp32: rounding errors of 2^-24 each, their square root over K of it; a factor of 4 for
# the worst of a tensor's elements over the tensor's scale.  The partial product left out stays below 2^-33.
BOUND = lambda K: 4 * max(K, 16) ** 0.5 * 2.0 ** -24

# (rows, d_in, d_out): one row and word, remainders of the 64-row tile, widths off the 16-byte grid, the first
# sizes of the 128-row tile (512 tiles and more) with remainders in every direction, on and off that grid
SHAPES = [(1, 4, 4), (63, 20, 12), (65, 7, 5), (129, 100, 256), (64, 16, 64), (33000, 36, 132), (65537, 12, 68),
          (33000, 37, 133), (65537, 13, 70), (33000, 67, 130)]


@pytest.fixture(scope="module")
def hb():
    from paper_2409_00657_amd import binding
    binding.load_library()
    return binding


def _inputs(n, d_in, d_out, seed=0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    r = lambda *s: torch.randn(s, generator=g, device=DEV)
    H, Ws, Wn, G = r(n, d_in), r(d_in, d_out) / d_in ** 0.5, r(d_in, d_out) / d_in ** 0.5, r(n, d_out)
    idx = torch.randperm(n, generator=g, device=DEV).to(torch.int32)      # one neighbour each: the mean is its row
    return H, Ws, Wn, G, torch.arange(n + 1, device=DEV, dtype=torch.int32), idx


def _forward(H, Ws, Wn, idx):
    """Every vertex has one neighbour and is a root: the single-call pass is the plain layer over all rows."""
    from paper_2409_00657_amd.pipeline import HotPath
    n, out = H.shape[0], torch.empty((H.shape[0], Ws.shape[1]), device=DEV)
    hp = HotPath(torch.arange(n + 1, device=DEV, dtype=torch.int64), idx, H, [(Ws, Wn, None)], n, [1])
    hp.forward(torch.arange(n, device=DEV, dtype=torch.int32), [3], out)
    return out


def _backward(hb, H, Ws, Wn, G, indptr, idx):
    n, (d_in, d_out) = H.shape[0], Ws.shape
    gWs, gWn, gb = torch.zeros_like(Ws), torch.zeros_like(Wn), torch.zeros(d_out, device=DEV)
    dH = torch.empty_like(H)
    ws = torch.empty(hb.hopgnn_sage_bwd_ws_bytes(H.dtype, n, d_in, d_out, True), dtype=torch.uint8, device=DEV)
    hb.hopgnn_sage_bwd(H, n, None, indptr, idx, n, Ws, Wn, None, False, G, gWs, gWn, gb, dH, ws)
    return gWs, gWn, gb, dH


def _err(a, ref):
    return float(((a.double() - ref).abs().max() / ref.pow(2).mean().sqrt()).item())


def _ref(H, Ws, Wn, G, idx):
    H, Ws, Wn, G, i = H.double(), Ws.double(), Wn.double(), G.double(), idx.long()
    dH = G @ Ws.t().contiguous()
    dH.index_add_(0, i, G @ Wn.t().contiguous())
    return H @ Ws + H[i] @ Wn, (H.t().contiguous() @ G, H[i].t().contiguous() @ G, G.sum(0), dH)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("scale", [1.0, 1e-30])
def test_products_of_split_operands(hb, shape, scale):
    n, d_in, d_out = shape
    H, Ws, Wn, G, indptr, idx = _inputs(*shape)
    H, G = H * scale, G * scale
    out_ref, bwd_ref = _ref(H, Ws, Wn, G, idx)
    out = _forward(H, Ws, Wn, idx)
    assert _err(out, out_ref) <= BOUND(2 * d_in)
    if scale != 1.0:
        G = G / scale          # their product with H stays a normal number
        bwd_ref = _ref(H, Ws, Wn, G, idx)[1]
    grads = _backward(hb, H, Ws, Wn, G, indptr, idx)
    for a, ref, K in zip(grads, bwd_ref, (n, n, n, 2 * d_out)):
        assert _err(a, ref) <= BOUND(K)


@pytest.mark.parametrize("shape", [(65, 20, 12), (65, 7, 5), (33000, 36, 132)])
def test_infinities_and_the_largest_floats(hb, shape):
    """An infinite operand gives the infinities and NaNs of the plain products, and only in its own row (column)."""
    n, d_in, d_out = shape
    H, Ws, Wn, G, indptr, idx = _inputs(*shape, seed=1)
    big = torch.finfo(torch.float32).max      # rounds to infinity as bf16
    H[3, 1], H[5, 2], H[n - 1, d_in - 1], H[7, 0] = float("inf"), -float("inf"), float("nan"), big
    Ws[0], Wn[0] = 0.25, -0.125
    out_ref, _ = _ref(H, Ws, Wn, G, idx)
    out = _forward(H, Ws, Wn, idx)
    ref32 = out_ref.float()
    assert torch.equal(torch.isnan(out), torch.isnan(ref32)) and torch.equal(torch.isposinf(out), torch.isposinf(ref32))
    assert torch.equal(torch.isneginf(out), torch.isneginf(ref32))
    rows = torch.isfinite(ref32).all(1) & (ref32.abs().amax(1) < 1e30)
    assert _err(out[rows], out_ref[rows]) <= BOUND(2 * d_in)
    huge = torch.isfinite(ref32).all(1) & ~rows
    assert int(huge.sum()) == 2 and torch.allclose(out[huge].double(), out_ref[huge], rtol=BOUND(2 * d_in))

    H, Ws, Wn, G, indptr, idx = _inputs(*shape, seed=2)
    G[4, 2], G[n - 1, 0] = float("inf"), -float("inf")
    _, ref = _ref(H, Ws, Wn, G, idx)
    for a, r in zip(_backward(hb, H, Ws, Wn, G, indptr, idx), ref):
        r32 = r.float()
        for kind in (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(kind(a), kind(r32))
        ok = torch.isfinite(r32)
        assert float(((a[ok].double() - r[ok]).abs().max() / r[ok].pow(2).mean().sqrt()).item()) <= BOUND(max(n, 2 * d_out))


def _two_layers(fuse, big):
    """Forward pass of two layers over 33 000 first-layer rows of 256 columns (520 large tiles), the outputs of
    every stored row; `big`: an infinity, a NaN and the largest float among the features."""
    from paper_2409_00657_amd import synth
    from paper_2409_00657_amd.pipeline import HotPath
    g = synth.rmat_graph(13, 9.0, seed=11, device=DEV)
    X = synth.features(g.n_vertices, 100, torch.float32, device=DEV)
    W = synth.sage_weights(100, 256, 2, torch.float32, device=DEV, bias=True)
    seeds = synth.seeds(g.n_vertices, 3000, 300, device=DEV)
    if big:
        v = seeds[:4].long().unique()[:3]
        X[v[0], 5], X[v[1], 7], X[v[2], 0] = float("inf"), float("nan"), torch.finfo(torch.float32).max
    hp = HotPath(g.offsets, g.indices, X, W, 3000, [10, 3], fuse_tree=fuse)
    out = torch.empty((3000, 256), device=DEV)
    hp.forward(seeds, [17], out)
    torch.cuda.synchronize()
    return out, hp.H[0][:3000].clone()


def _same_bits(a, b):
    return torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.nan_to_num(a, nan=0.0), torch.nan_to_num(b, nan=0.0))


def test_fused_and_plain_tiles_give_the_same_bits_beside_infinities():
    """The two cut the rows into tiles at different places."""
    fused, plain = _two_layers(True, True), _two_layers(False, True)
    assert not bool(torch.isfinite(plain[1]).all()) and bool(torch.isfinite(plain[0]).all(1).any())
    for a, b in zip(fused, plain):
        assert _same_bits(a, b)
    clean = _two_layers(True, False)
    top = plain[1].abs().amax(1)            # a row reached by one of the three holds infinities, huge values or, where the
    rows = torch.isfinite(plain[1]).all(1) & (top < 1e30) & (top > 0)      # ReLU has met its NaNs, nothing but zeros
    assert int(rows.sum()) > 2500 and torch.equal(fused[1][rows], clean[1][rows])


@pytest.mark.parametrize("shape", [(129, 100, 256), (33000, 36, 132)])
def test_an_infinity_leaves_the_other_rows_and_columns_their_bits(hb, shape):
    n, d_in, d_out = shape
    H, Ws, Wn, G, indptr, idx = _inputs(*shape, seed=3)
    idx = torch.arange(n, device=DEV, dtype=torch.int32)
    H2, G2 = H.clone(), G.clone()
    H2[5, 2], G2[9, 3] = float("inf"), float("-inf")
    a, b = _forward(H, Ws, Wn, idx), _forward(H2, Ws, Wn, idx)
    keep = torch.arange(n, device=DEV) != 5
    assert torch.equal(a[keep], b[keep]) and not bool(torch.isfinite(b[5]).any())
    g1, g2 = _backward(hb, H, Ws, Wn, G, indptr, idx), _backward(hb, H, Ws, Wn, G2, indptr, idx)
    cols, rows = torch.arange(d_out, device=DEV) != 3, torch.arange(n, device=DEV) != 9
    assert torch.equal(g1[0][:, cols], g2[0][:, cols]) and torch.equal(g1[1][:, cols], g2[1][:, cols])
    assert torch.equal(g1[3][rows], g2[3][rows]) and not bool(torch.isfinite(g2[3][9]).any())


def _slots_backward(hb, H, Ws, Wn, G):
    """n destination rows with one child row each: the input gradients of a row and of its child, no atomics."""
    n, (d_in, d_out) = G.shape[0], Ws.shape
    gWs, gWn, gb = torch.zeros_like(Ws), torch.zeros_like(Wn), torch.zeros(d_out, device=DEV)
    dH = torch.empty((2 * n, d_in), device=DEV)
    indptr = torch.arange(n + 1, device=DEV, dtype=torch.int32)
    idx = torch.arange(n, 2 * n, device=DEV, dtype=torch.int32)
    ws = torch.empty(hb.hopgnn_sage_bwd_ws_bytes(torch.float32, n, d_in, d_out, True), dtype=torch.uint8, device=DEV)
    hb.hopgnn_sage_bwd_slots(H, 2 * n, indptr, idx, n, n, Ws, Wn, None, False, G, gWs, gWn, gb, dH, ws)
    return gWs, gWn, dH[:n], dH[n:]


@pytest.mark.parametrize("shape", [(65, 20, 12), (777, 7, 5), (129, 100, 256), (33000, 36, 132)])
@pytest.mark.parametrize("scale", [1e-34, 1e-36, 2e-38])
def test_the_smallest_magnitudes(hb, shape, scale):
    """Down to and among the subnormal floats: the bound of ordinary magnitudes, for each operand in turn."""
    n, d_in, d_out = shape
    H, Ws, Wn, G, _, idx = _inputs(*shape, seed=4)
    small = H * scale
    assert _err(_forward(small, Ws, Wn, idx), _ref(small, Ws, Wn, G, idx)[0]) <= BOUND(2 * d_in)
    Wss, Wns = Ws * scale, Wn * scale
    assert _err(_forward(H, Wss, Wns, idx), _ref(H, Wss, Wns, G, idx)[0]) <= BOUND(2 * d_in)
    H = torch.cat([H, H[idx.long()]])
    for h, g in ((H, G * scale), (H * scale, G)):
        gWs, gWn, dSelf, dNeigh = _slots_backward(hb, h, Ws, Wn, g)
        hd, gd = h.double(), g.double()
        for got, ref, K in ((gWs, hd[:n].t().contiguous() @ gd, n), (gWn, hd[n:].t().contiguous() @ gd, n),
                            (dSelf, gd @ Ws.double().t().contiguous(), d_out), (dNeigh, gd @ Wn.double().t().contiguous(), d_out)):
            assert _err(got, ref) <= BOUND(K)


@pytest.mark.parametrize("shape", [(65, 20, 12), (33000, 36, 132)])
def test_operands_beyond_the_scaled_range(hb, shape):
    """Finite values past 2^103, and sums past 2^79 of smaller ones, come out as the fp32 instruction forms them."""
    n, d_in, d_out = shape
    H, Ws, Wn, G, indptr, idx = _inputs(*shape, seed=6)
    H[3] *= 1e33
    H[5] *= 1e25
    G[7] *= 1e33
    G[9] *= 1e25
    out_ref, ref = _ref(H, Ws, Wn, G, idx)
    out = _forward(H, Ws, Wn, idx)
    assert bool(torch.isfinite(out).all())
    row_err = (out.double() - out_ref).abs().amax(1) / out_ref.pow(2).mean(1).sqrt()
    mixed = torch.isin(torch.arange(n, device=DEV), torch.tensor([3, 5], device=DEV)) | torch.isin(idx, torch.tensor([3, 5], device=DEV, dtype=torch.int32))
    assert float(row_err[~mixed].max()) <= BOUND(2 * d_in) and float(row_err.max()) <= BOUND(2 * d_in)
    G2 = torch.cat([H, H[idx.long()]]).clamp(-9, 9)
    gWs, gWn, dSelf, dNeigh = _slots_backward(hb, G2, Ws, Wn, G)
    for got, r in ((dSelf, G.double() @ Ws.double().t().contiguous()), (dNeigh, G.double() @ Wn.double().t().contiguous())):
        assert float(((got.double() - r).abs().amax(1) / r.pow(2).mean(1).sqrt()).max()) <= BOUND(d_out)
    for got, h in ((gWs, G2[:n]), (gWn, G2[n:])):
        assert _err(got, h.double().t().contiguous() @ G.double()) <= BOUND(n)


@pytest.mark.parametrize("shape", [(65, 20, 12), (777, 76, 48), (33000, 36, 132)])
def test_a_single_product_rounds_once(hb, shape):
    """Rows with one non-zero element: every result is one product of two floats, so it carries
    one rounding (and what the split adds to it)."""
    n, d_in, d_out = shape
    H, Ws, Wn, G, indptr, idx = _inputs(*shape, seed=8)
    r = torch.arange(n, device=DEV)
    one_h = torch.zeros_like(H)
    one_h[r, r % d_in] = H[r, r % d_in]
    # one rounding of the product, half a last place; the seven small partial products, together below 2^-7 of it, are
    # summed with a rounding of 2^-24 of their sum each: 7 x 2^-31, less than 1/16 of 2^-24
    once = lambda got, ref: bool(((got.double() - ref).abs() <= ref.abs() * 2.0 ** -24 * (1 + 1 / 16)).all())
    assert once(_forward(one_h, Ws, torch.zeros_like(Wn), idx), one_h.double() @ Ws.double())
    one_h[d_in:] = 0          # one row per column: one product per weight gradient element
    one_g = torch.zeros_like(G)
    one_g[r, r % d_out] = G[r, r % d_out]
    gWs, _, _, _ = _slots_backward(hb, torch.cat([one_h, one_h]), Ws, Wn, G)
    assert once(gWs, one_h.double().t().contiguous() @ G.double())
    _, _, dSelf, dNeigh = _slots_backward(hb, torch.cat([one_h, one_h]), Ws, Wn, one_g)
    assert once(dSelf, one_g.double() @ Ws.double().t().contiguous()) and once(dNeigh, one_g.double() @ Wn.double().t().contiguous())


@pytest.mark.parametrize("shape", [(513, 600, 520), (33000, 600, 136), (20000, 16, 16)])
def test_sums_of_one_sign(hb, shape):
    """Terms that cannot cancel: roundings that lean one way would add up over K."""
    n, d_in, d_out = shape
    H, Ws, Wn, G, indptr, idx = (t.abs() for t in _inputs(*shape, seed=9))
    out_ref, ref = _ref(H, Ws, Wn, G, idx)
    got = _backward(hb, H, Ws, Wn, G, indptr, idx)
    # relative 2-norm error of a sum whose K roundings lean no way: sqrt(K) 2^-24 of the sum's middle, at most half that
    rel = lambda a, r: float((a.double() - r).norm() / r.norm())
    assert rel(_forward(H, Ws, Wn, idx), out_ref) <= 0.5 * (2 * d_in) ** 0.5 * 2.0 ** -24
    for a, r, K in zip(got, ref, (n, n, n, 2 * d_out)):
        assert rel(a, r) <= 0.5 * max(K, 16) ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("shape", [(33000, 36, 132), (33000, 37, 133), (5000, 12, 68)])
def test_a_rows_bits_do_not_depend_on_the_rows_beside_it(hb, shape):
    """The whole input, a tenth of it and a few rows (large tiles, small tiles) give a row the same bits, through
    hopgnn_sage_fwd, hopgnn_sage_fwd_agg's mean and the single-call pass."""
    n, d_in, d_out = shape
    H, Ws, Wn, _, indptr, idx = _inputs(*shape, seed=10)
    b = torch.randn(d_out, device=DEV)
    ws = torch.empty(hb.hopgnn_sage_fwd_ws_bytes(torch.float32, n, d_in, d_out), dtype=torch.uint8, device=DEV)
    outs = []
    for rows in (n, n // 10, 33):
        out, out_agg = torch.empty((rows, d_out), device=DEV), torch.empty((rows, d_out), device=DEV)
        hb.hopgnn_sage_fwd(H, n, None, indptr, idx, rows, Ws, Wn, b, True, out, ws)
        hb.hopgnn_sage_fwd_agg(H, n, None, indptr, idx, rows, Ws, Wn, b, hb.AGG_MEAN, True, out_agg, ws)
        assert torch.equal(out, out_agg)
        outs.append(out)
    assert torch.equal(outs[1], outs[0][:n // 10]) and torch.equal(outs[2], outs[0][:33])
    plain = torch.empty((n, d_out), device=DEV)
    hb.hopgnn_sage_fwd(H, n, None, indptr, idx, n, Ws, Wn, None, False, plain, ws)
    assert torch.equal(plain, _forward(H, Ws, Wn, idx))


def test_merged_batches_keep_their_bits():
    """Two batches in one call (520 large tiles) and one after the other (260 tiles' worth of small ones)."""
    from paper_2409_00657_amd import synth
    from paper_2409_00657_amd.pipeline import HotPath
    g = synth.rmat_graph(13, 9.0, seed=11, device=DEV)
    X = synth.features(g.n_vertices, 100, torch.float32, device=DEV)
    W = synth.sage_weights(100, 256, 2, torch.float32, device=DEV, bias=True)
    seeds = synth.seeds(g.n_vertices, 3000, 300, device=DEV)
    outs = []
    for merge in (True, False):
        hp = HotPath(g.offsets, g.indices, X, W, 1500, [10, 3], group=2, merge=merge)
        outs.append(torch.empty((3000, 256), device=DEV))
        hp.forward(seeds, [17, 18], outs[-1])
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])


def test_the_training_forward_and_the_single_call_agree_to_rounding():
    from paper_2409_00657_amd import synth
    from paper_2409_00657_amd.pipeline import HotPath
    g = synth.rmat_graph(13, 9.0, seed=11, device=DEV)
    X = synth.features(g.n_vertices, 100, torch.float32, device=DEV)
    W = synth.sage_weights(100, 256, 2, torch.float32, device=DEV, bias=True)
    seeds = synth.seeds(g.n_vertices, 3000, 300, device=DEV)
    hp = HotPath(g.offsets, g.indices, X, W, 3000, [10, 3])
    out = torch.empty((3000, 256), device=DEV)
    hp.forward(seeds, [17], out)
    assert torch.equal(hp.run_batch(seeds, 17), out)
    hp.enable_backward()
    train = hp.run_batch(seeds, 17)
    assert _err(train, out.double()) <= 2 * (BOUND(200) + BOUND(512))      # two layers, a rounding error on either side
