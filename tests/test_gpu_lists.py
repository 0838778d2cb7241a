"""Neighbour lists: what they hold, and layers over them against the oracle and against whole tiles."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

from oracle import qgnn
from test_gpu_stack import block_graph

pytestmark = pytest.mark.gpu

q = pytest.importorskip("paper_2111_09547_amd")
import paper_2111_09547_amd.binding as B  # noqa: E402
from paper_2111_09547_amd.model import BatchNorm, QuantGNN  # noqa: E402
from gpu_util import dev, as_u32  # noqa: E402


def with_degrees(rng, n, k, degrees):
    """uint8 [n, k]: row i has degrees[i % len] bits."""
    a = np.zeros((n, k), np.uint8)
    for i in range(n):
        d = min(degrees[i % len(degrees)], k)
        a[i, rng.choice(k, d, replace=False)] = 1
    return a


@pytest.mark.parametrize("n,k,block", [(100, 100, 0), (700, 700, 0), (3 * 96 - 5, 96, 96), (2 * 1056 - 500, 1056, 1056)])
@pytest.mark.parametrize("kbits", [32, 64, 128])
def test_lists_and_the_map_of_one_pass(n, k, block, kbits):
    rng = np.random.default_rng(n)
    a = with_degrees(rng, n, k, [0, 1, 16, 17, 32, 64, 65, 255, 256, 257, 5, 700])
    if block:
        a[n // block * block:, n % block:] = 0
    A = q.qgtc_pack_bits(dev(a), 1, q.LEFT, block_rows=block)
    tmap = B._alloc_tile_map(A, 16, kbits)
    nb = B.qgtc_build_neighbours(A, tmap=tmap)
    ref = q.qgtc_build_tile_map(A, 16, kbits)
    deg = a.sum(1).astype(np.int64)
    assert (nb.deg.cpu().numpy() == deg).all() and torch.equal(tmap.deg, ref.deg) and torch.equal(tmap.row_cnt, ref.row_cnt)
    assert torch.equal(tmap.nnz_tiles, ref.nnz_tiles)
    kept = torch.arange(ref.c.n_tile_cols, device="cuda")[None] < ref.row_cnt[:, None]
    assert torch.equal(torch.where(kept, tmap.col_idx, 0), torch.where(kept, ref.col_idx, 0))
    host = nb.buffer.cpu().numpy().view(np.uint16)
    at = lambda ptr: (ptr - nb.buffer.data_ptr()) // 2
    first, rest, cap = at(nb.c.first), at(nb.c.rest), nb.c.rest_cap
    for i in range(n):
        got = np.concatenate([host[first + 16 * i:first + 16 * i + 16], host[rest + cap * i:rest + cap * (i + 1)]])
        have = min(deg[i], 256)
        got = got[:max(-(-have // 16), 1) * 16]      # whole blocks
        entries = np.sort(got[got != 0xffff])
        assert len(entries) == have and (np.isin(entries, np.nonzero(a[i])[0])).all() and len(np.unique(entries)) == have
        e = np.arange(len(got))                      # entry e at 4 (e % 4) + e / 4 of its block
        order = got[e // 16 * 16 + 4 * (e % 4) + e // 4 % 4]
        assert (order[:have] != 0xffff).all() and (order[have:] == 0xffff).all()


@pytest.mark.parametrize("blocks,block,short,dims,s,t,gin", [
    (3, 64, 5, "1-2", 1, 1, True),                   # a piece of one column
    (5, 96, 31, "17-33-16", 5, 3, False),            # two pieces, of which one column
    (3, 160, 33, "64-65-47", 8, 8, True),            # whole groups of columns and one more
    (2, 1024, 1, "130-129-7", 8, 4, False),          # sixteen pieces, seven of them empty
    (2, 512, 0, "256-200-64", 7, 8, True),
    (2, 288, 3, "300-101-5", 8, 8, False),  # two parts of 256 columns, the second of few pieces
    (3, 288, 7, "370-40-2", 8, 5, True),            # ... of up to eight
    (130, 256, 0, "384-16", 8, 8, True),
    (1, 640, 40, "1024-256-16", 8, 8, True),         # four parts, more weights than LDS keeps
    (130, 256, 77, "64-64-12", 8, 8, True),          # a tile per wave: one, four and more output tiles
    (130, 256, 0, "300-16-100", 8, 8, False),
    (33, 1024, 9, "513-64", 6, 6, True),
    (40, 1024, 0, "16-16-32", 8, 8, True),
])
@pytest.mark.parametrize("degree", [2.0, 20.0])
def test_layers_over_lists_equal_the_oracle(blocks, block, short, dims, s, t, gin, degree):
    rng = np.random.default_rng(blocks + block + s)
    d = [int(v) for v in dims.split("-")]
    a, csr = block_graph(rng, blocks, block, short, degree)
    n = a.shape[0]
    hubs = [0, n // 2, n - 1]                        # more neighbours than a tile's waves take, and than a list holds
    csr = csr.tolil()
    for r, want in zip(hubs, (65, 256, 700)):
        r0 = r // block * block
        cols = rng.choice(min(block, n - r0), min(want, block, n - r0), replace=False)
        a[r, cols] = 1
        csr[r, r0 + cols] = 1
    csr = csr.tocsr()
    X = rng.standard_normal((n, d[0])).astype(np.float32)
    Ws = [rng.uniform(-0.5, 0.5, dh).astype(np.float32) for dh in zip(d[:-1], d[1:])]
    make = lambda lists: QuantGNN(dev(a), [dev(W) for W in Ws], s, t, gin, block_rows=block, lists=lists)
    net, tiles = make(True), make(False)
    assert net.lists is not None and tiles.lists is None
    xr, x = (float(X.min()), float(X.max())), dev(X)
    ranges = tiles.calibrate(x, xr)
    assert net.calibrate(x, xr) == ranges
    rqs = [((0, qgnn.inv_scale(0.0, float(r.agg_hi), s)),
            None if r.out_hi is None else (0, qgnn.inv_scale(0.0, float(r.out_hi), s))) for r in ranges]
    wr = [(float(W.min()), float(W.max())) for W in Ws]
    _, trace, _ = qgnn.forward_dequantized(csr, X, xr, Ws, wr, s, t, gin, rqs=rqs)
    assert (as_u32(net.forward(x, xr, ranges, want_int=True)) == trace[-1]["Z"]).all()
    out = tiles.forward(x, xr, ranges)
    assert torch.equal(net.forward(x, xr, ranges), out)
    planes = q.qgtc_pack_bits(x, s, q.RIGHT, quant=xr)
    assert torch.equal(net.forward(None, xr, ranges, x_bits=planes), out)
    net.pack_static(x, xr)
    assert torch.equal(net.forward(x, xr, ranges, x_packed=True), out)


def test_rows_that_are_all_hubs():
    """Every row has more neighbours than a list holds, without blocks."""
    rng = np.random.default_rng(3)
    n, dims = 900, [40, 48, 9]
    a = (rng.random((n, n), dtype=np.float32) < 0.4).astype(np.uint8)
    x = dev(rng.standard_normal((n, dims[0])).astype(np.float32))
    Ws = [dev(rng.uniform(-0.5, 0.5, dh).astype(np.float32)) for dh in zip(dims[:-1], dims[1:])]
    nets = [QuantGNN(dev(a), Ws, 8, 8, True, lists=lists) for lists in (True, False)]
    ranges = nets[1].calibrate(x, (-3.0, 3.0))
    outs = [net.forward(x, (-3.0, 3.0), ranges) for net in nets]
    assert torch.equal(outs[0], outs[1])
    graph = nets[0].capture(x, (-3.0, 3.0), ranges, outs[0], with_static=True)
    for _ in range(3):
        outs[0].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("form,s,t", [("stack", 8, 8), ("stack", 5, 3), ("two bytes", 16, 16), ("two bytes", 11, 7),
                                      ("update first", 8, 8), ("update first", 4, 6)])
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("below", [False, True])
@pytest.mark.parametrize("dims", ["70-20-33-9", "300-130-70"])
def test_lower_bounds_of_requantization(form, s, t, relu, below, dims):
    """Epilogues with a lower bound under (below) or in the middle of the results, behind affine maps of the columns too:
    every code against the oracle, in rows of a ragged last tile and of 65, 256 and more neighbours."""
    rng = np.random.default_rng(s + t)
    d, block, short = [int(v) for v in dims.split("-")], 320, 41
    a, csr = block_graph(rng, 3, block, short, 7.0)
    n = a.shape[0]
    csr = csr.tolil()
    for r, many in ((0, 65), (n // 2, 256), (n - 1, 279), (1, 300)):
        r0 = r // block * block
        cols = rng.choice(min(block, n - r0), min(many, min(block, n - r0)), replace=False)
        a[r, cols] = 1
        csr[r, r0 + cols] = 1
    csr = csr.tocsr()
    X = rng.standard_normal((n, d[0])).astype(np.float32)
    codes = qgnn.quantize(X, -3.0, 3.0, s)
    A = q.qgtc_pack_bits(dev(a), 1, q.LEFT, block_rows=block)
    lists = B.qgtc_build_neighbours(A)

    def bits(c, affine=None):
        """An epilogue that requantizes such results, and what it makes of them."""
        v = qgnn.as_signed(c).astype(np.float64) if affine is None else qgnn.as_signed(c) * affine[0][None].astype(np.float64) + affine[1][None]
        v = np.maximum(v, 0) if relu else v
        # (rq_lo is 32 bits; sums modulo 2^32 span all of them)
        lo = max(int(v.min() - (v.max() - v.min()) / 3 - 2 if below else np.quantile(v, 0.4)) + 1, -1 << 31)
        inv = qgnn.inv_scale(float(lo), float(max(v.max(), lo + 1)), s)
        ep = q.Epilogue(mode=q.OUT_BITS, relu=relu, rq_nbits=s, rq_lo=lo, rq_inv_scale=float(inv))
        if affine is None:
            return ep, qgnn.requantize(c, lo, inv, s, relu)
        ep.col_scale, ep.col_shift = dev(affine[0]), dev(affine[1])
        return ep, qgnn.requantize_affine(c, *affine, lo, inv, s, relu)

    for affine in (False, True)[:1 if form == "update first" else 2]:
        layers, x = [], codes
        for l, (di, h) in enumerate(zip(d[:-1], d[1:])):
            last = l == len(d) - 2
            w = rng.integers(0, 1 << t, (di, h)).astype(np.uint32)
            product = lambda v: qgnn.update(v, w)
            around = lambda v: qgnn.aggregate(csr, v, True)
            steps = [product, around] if form == "update first" else [around, product]
            first, y = bits(steps[0](x))
            z = steps[1](y)
            if last:
                second = q.Epilogue(mode=q.OUT_I32, relu=relu)
            else:
                maps = (rng.uniform(0.5, 1.5, h).astype(np.float32), rng.uniform(-9.0, 9.0, h).astype(np.float32)) if affine else None
                second, x = bits(z, maps)
            (second if form == "update first" else first).self_term = True
            part = lambda v, k: q.qgtc_pack_bits(dev(v.astype(np.int32)), k, q.RIGHT_BYTES)
            W = part(w & 255, min(t, 8))
            layers.append(((W, part(w >> 8, t - 8) if t > 8 else None) if form == "two bytes" else W, first, second))
        buffers = [torch.zeros(int(B.lib().qgtc_stack_buffer_bytes(n, max(d))) // (2 if s > 8 else 4) + 4, dtype=torch.int32, device="cuda")
                   for _ in range(2)]
        out = torch.zeros((n, d[-1]), dtype=torch.int32, device="cuda")
        if form == "two bytes":
            B.qgtc_wide_forward(B.WideStack(A, layers, s, buffers, lists), out, src=dev(X), quant=(-3.0, 3.0))
        elif form == "update first":
            B.qgtc_stack_forward_update_first(B.Stack(A, None, layers, s, buffers, lists), out, dev(X), (-3.0, 3.0))
        else:
            B.qgtc_stack_forward(B.Stack(A, None, layers, s, buffers, lists), out, src=dev(X), quant=(-3.0, 3.0))
        assert (out.cpu().numpy() == qgnn.int_output(z, relu)).all()
        assert len(np.unique(x)) > 2 and len(torch.unique(out)) > 2


def test_lists_follow_the_adjacency():
    """pack_static() of another adjacency, and one that was replaced without it."""
    rng = np.random.default_rng(5)
    graphs = [block_graph(rng, 3, 96, 0, deg)[0] for deg in (4.0, 30.0)]
    W = dev(rng.uniform(-1, 1, (20, 9)).astype(np.float32))
    x = dev(rng.standard_normal((288, 20)).astype(np.float32))
    net, other = (QuantGNN(dev(g), [W], 4, 4, False, block_rows=96, lists=True) for g in graphs)
    ranges = other.calibrate(x, (-3.0, 3.0))
    want = QuantGNN(dev(graphs[1]), [W], 4, 4, False, block_rows=96, lists=False).forward(x, (-3.0, 3.0), ranges, want_int=True)
    net.forward(x, (-3.0, 3.0), ranges, want_int=True)
    first = net.A
    net.A_src.copy_(dev(graphs[1]))
    net.pack_static()
    assert torch.equal(net.forward(x, (-3.0, 3.0), ranges, want_int=True), want)
    net.A_src.copy_(dev(graphs[0]))
    net.pack_static()
    net.A = other.A
    assert net.A is not first and torch.equal(net.forward(x, (-3.0, 3.0), ranges, want_int=True), want)


@pytest.mark.parametrize("s,update_first", [(4, False), (16, False), (8, True)])
@pytest.mark.parametrize("tmap", ["built again", "replaced", "none"])
def test_passes_follow_an_adjacency_that_is_packed_in_place(s, update_first, tmap):
    """Other bits in A, and their map built where the old one was, or in place of it: passes are over the new adjacency.
    Without a map A is all there is to follow: lists are then used on request only."""
    rng = np.random.default_rng(7)
    graphs = [dev(block_graph(rng, 5, 96, 0, deg)[0]) for deg in (4.0, 30.0, 6.0)]
    W, xr = dev(rng.uniform(-1, 1, (20, 9)).astype(np.float32)), (-3.0, 3.0)
    x = dev(rng.standard_normal((480, 20)).astype(np.float32))
    net = QuantGNN(graphs[0], [W], s, s, False, block_rows=96, use_map=tmap != "none", update_first=update_first,
                   lists=None if tmap == "none" else True)
    assert (net.lists is None) == (tmap == "none")
    for g in graphs[1:] + graphs[:1]:
        plain = QuantGNN(g, [W], s, s, False, block_rows=96, lists=False, update_first=update_first)
        ranges = plain.calibrate(x, xr)
        q.qgtc_pack_bits(g, 1, q.LEFT, out=net.A)
        if tmap == "built again":
            q.qgtc_build_tile_map(net.A, 16, net.tile_kbits, out=net.map)
        elif tmap == "replaced":
            net.map = q.qgtc_build_tile_map(net.A, 16, net.tile_kbits)
            net.deg = net.map.deg
        want = plain.forward(x, xr, ranges, want_int=True)
        assert torch.equal(net.forward(x, xr, ranges, want_int=True), want)
        assert net.calibrate(x, xr) == ranges
        if tmap != "none":                           # (the degrees are the map's)
            want = plain.forward(x, xr, ranges)
            assert torch.equal(net.forward(x, xr, ranges), want)
            out = torch.empty_like(want)
            graph = net.capture(x, xr, ranges, out)
            for _ in range(3):
                out.zero_()
                graph.replay()
                assert torch.equal(net.forward(x, xr, ranges), want)
                assert torch.equal(out, want)


@pytest.mark.parametrize("s", [4, 16])
@pytest.mark.parametrize("use_map", [True, False])
@pytest.mark.parametrize("replaced", ["A", "A and its map and degrees", "A of fewer subgraphs"])
def test_fp32_output_follows_a_replaced_adjacency(s, use_map, replaced):
    """The degrees, which only the fp32 output reads (times the range's lower end), belong to the new adjacency,
    also in runs on planes and in calibrate()."""
    rng = np.random.default_rng(6)
    small, large = block_graph(rng, 5, 96, 0, 4.0)[0], block_graph(rng, 5, 96, 0, 30.0)[0]
    if replaced == "A of fewer subgraphs":          
        small, large = large, small[:288].copy()
    W, xr = dev(rng.uniform(-1, 1, (20, 9)).astype(np.float32)), (-3.0, 3.0)
    net, other = (QuantGNN(dev(g), [W], s, s, False, block_rows=96, lists=True, use_map=use_map) for g in (small, large))
    x = dev(rng.standard_normal((large.shape[0], 20)).astype(np.float32))
    plain = QuantGNN(dev(large), [W], s, s, False, block_rows=96, lists=False, use_map=use_map)
    ranges = plain.calibrate(x, xr)
    want = plain.forward(x, xr, ranges)
    net.forward(dev(rng.standard_normal((small.shape[0], 20)).astype(np.float32)), xr, ranges)
    net.A = other.A
    if replaced == "A and its map and degrees":
        net.map, net.deg = other.map, other.deg
    mine = (net.map, net.deg)
    assert torch.equal(net.forward(x, xr, ranges), want)
    if replaced == "A and its map and degrees":
        assert net.map is mine[0] and net.deg is mine[1]
    assert torch.equal(net.forward(x, xr, ranges, streams=2), want)
    assert net.calibrate(x, xr) == ranges
    out = torch.empty_like(want)
    graph = net.capture(x, xr, ranges, out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        assert torch.equal(net.forward(x, xr, ranges), want)
        assert torch.equal(out, want)


@pytest.mark.parametrize("blocks,block,short,dims,s,t,gin", [
    (3, 96, 5, "12-16-5", 8, 8, True),               # a quarter of a wave per row, one output tile
    (3, 96, 5, "13-40-70", 3, 5, False),             # rows that are no multiple of 16 bytes, several tiles, two groups of them
    (2, 288, 31, "128-64-16", 8, 4, True),           # half a wave per row
    (2, 288, 0, "129-16-200", 5, 8, False),
    (140, 256, 77, "260-16-16", 8, 8, True),         # two parts of 256 columns, a tile per wave in every kernel
    (1, 672, 0, "1024-200-3", 7, 8, False),   # four parts, more output tiles than one group
])
def test_update_first_over_lists(blocks, block, short, dims, s, t, gin):
    rng = np.random.default_rng(blocks + block + s)
    d = [int(v) for v in dims.split("-")]
    a, _ = block_graph(rng, blocks, block, short, 6.0)
    a[:: max(1, a.shape[0] // 5), : min(block, 70)] = 1   # some heavy rows
    n = a.shape[0]
    if short:
        a[(blocks - 1) * block:, block - short:] = 0
    Ws = [dev(rng.uniform(-0.5, 0.5, dh).astype(np.float32)) for dh in zip(d[:-1], d[1:])]
    x = dev(rng.standard_normal((n, d[0])).astype(np.float32))
    x[0, 0], x[1, 1], x[n - 1, d[0] - 1] = float("nan"), float("inf"), -float("inf")
    nets = [QuantGNN(dev(a), Ws, s, t, gin, block_rows=block, update_first=True, lists=lists) for lists in (True, False)]
    assert nets[0].lists is not None and nets[1].lists is None
    xr = (-3.0, 3.0)
    ranges = nets[1].calibrate(x, xr)
    assert nets[0].calibrate(x, xr) == ranges
    wide = torch.full((n, d[0] + 3), float("nan"), device="cuda")
    wide[:, 1:1 + d[0]] = x
    for ints in (True, False):
        want = nets[1].forward(x, xr, ranges, want_int=ints)
        assert int((want != 0).sum()) > 0
        assert torch.equal(nets[0].forward(x, xr, ranges, want_int=ints), want)
        assert torch.equal(nets[0].forward(wide[:, 1:1 + d[0]], xr, ranges, want_int=ints), want)


@pytest.mark.parametrize("blocks,block,short,dims,s,t,gin", [
    (3, 64, 5, "1-2-3", 9, 1, True),                 # a piece of one column, one byte of weights
    (5, 96, 31, "17-33-16", 12, 9, False),           # two pieces, of which one column; a bit of the weights' second byte
    (3, 160, 33, "64-65-47", 16, 8, True),           # four waves per tile
    (2, 1024, 1, "130-129-7", 16, 16, False),
    (2, 288, 3, "300-101-5", 16, 12, False),         # two parts of 256 columns
    (1, 640, 40, "512-256-16", 16, 16, True),        # more weights than LDS keeps
    (130, 256, 77, "64-64-12", 16, 16, True),        # a tile per wave
    (130, 256, 0, "300-16-100", 10, 15, False),
    (40, 1024, 0, "16-16-32", 16, 16, True),
])
def test_codes_of_two_bytes_over_lists(blocks, block, short, dims, s, t, gin):
    """9 to 16 bits: the oracle's integers (modulo 2^32), and the planes' results, also with batch normalization."""
    rng = np.random.default_rng(blocks + block + s)
    d = [int(v) for v in dims.split("-")]
    a, _ = block_graph(rng, blocks, block, short, 20.0)
    n = a.shape[0]
    for r, want in zip([0, n // 2, n - 1], (65, 256, 700)):
        r0 = r // block * block
        a[r, rng.choice(min(block, n - r0), min(want, block, n - r0), replace=False)] = 1
    r, c = np.nonzero(a)
    csr = sp.csr_matrix((np.ones(len(r), np.int64), (r, c + r // block * block)), shape=(n, n))
    X = rng.standard_normal((n, d[0])).astype(np.float32)
    Ws = [rng.uniform(-0.5, 0.5, dh).astype(np.float32) for dh in zip(d[:-1], d[1:])]
    xr, x = (-3.0, 3.0), dev(X)
    wr = [(float(W.min()), float(W.max())) for W in Ws]
    norms = [BatchNorm(*(rng.uniform(0.5, 1.5, h).tolist() for _ in range(4))) for h in d[1:-1]] + [None]
    for bn in (None, norms):
        net, tiles = (QuantGNN(dev(a), [dev(W) for W in Ws], s, t, gin, block_rows=block, lists=lists, batchnorm=bn) for lists in (True, False))
        assert net.lists is not None and tiles.lists is None
        ranges = tiles.calibrate(x, xr)
        assert net.calibrate(x, xr) == ranges
        out, ints = tiles.forward(x, xr, ranges), tiles.forward(x, xr, ranges, want_int=True)
        assert torch.equal(net.forward(x, xr, ranges, x_packed=True), out)     # as calibrate() left them: planes
        assert torch.equal(net.forward(x, xr, ranges), out)
        assert torch.equal(net.forward(x, xr, ranges, want_int=True), ints)
        if bn is None:
            rqs = [((0, qgnn.inv_scale(0.0, float(r.agg_hi), s)),
                    None if r.out_hi is None else (0, qgnn.inv_scale(0.0, float(r.out_hi), s))) for r in ranges]
            _, trace, _ = qgnn.forward_dequantized(csr, X, xr, Ws, wr, s, t, gin, rqs=rqs)
            assert (as_u32(ints) == trace[-1]["Z"]).all()
    planes = q.qgtc_pack_bits(x, s, q.RIGHT, quant=xr)
    assert torch.equal(net.forward(None, xr, ranges, x_bits=planes), out)
    codes = dev(np.clip(np.floor((X.astype(np.float64) + 3.0) / 6.0 * 2 ** s), 0, 2 ** s - 1).astype(np.int32))
    assert torch.equal(net.forward(codes, xr, ranges), tiles.forward(codes, xr, ranges))
    for old, new in zip(net.Ws, Ws):                 # other weights in place, as a recorded step meets them
        old.copy_(dev(new[::-1].copy()))
    net.pack_static(x, xr)
    for old in tiles.Ws:
        old.copy_(old.flip(0))
    tiles.pack_static()
    want = tiles.forward(x, xr, ranges)
    graph = net.capture(x, xr, ranges, out, with_static=True)
    for _ in range(3):
        out.zero_()
        graph.replay()
        assert torch.equal(net.forward(x, xr, ranges), want)
        assert torch.equal(out, want)


@pytest.mark.parametrize("t", [7, 16])
def test_planes_of_weights_are_packed_by_pack_static(monkeypatch, t):
    """Two-byte codes over lists, run by run on planes: no pass packs the weights, eager and recorded ones have
    those of the last pack_static()."""
    rng = np.random.default_rng(t)
    a, _ = block_graph(rng, 5, 96, 31, 6.0)
    Ws = [rng.uniform(-1, 1, dh).astype(np.float32) for dh in ((20, 24), (24, 9))]
    net, plain = (QuantGNN(dev(a), [dev(W) for W in Ws], 16, t, False, block_rows=96, lists=lists) for lists in (True, False))
    x, xr = dev(rng.standard_normal((a.shape[0], 20)).astype(np.float32)), (-3.0, 3.0)
    ranges = plain.calibrate(x, xr)
    want = plain.forward(x, xr, ranges)
    net.Ws[0].neg_()                                 # not packed yet
    assert torch.equal(net.forward(x, xr, ranges, streams=2), want)
    out = torch.empty_like(want)
    graph = net.capture(x, xr, ranges, out, streams=2)
    packed, real = [], B.qgtc_pack_bits
    monkeypatch.setattr(B, "qgtc_pack_bits", lambda src, *args, **k: packed.append(tuple(src.shape)) or real(src, *args, **k))
    assert torch.equal(net.forward(x, xr, ranges, streams=2), want)
    assert packed == [tuple(x.shape)]
    plain.Ws[0].neg_()
    for pack in (False, True):
        if pack:
            net.pack_static()
            plain.pack_static()
            want = plain.forward(x, xr, ranges)
        for _ in range(2):
            out.zero_()
            graph.replay()
            assert torch.equal(net.forward(x, xr, ranges), want)
            assert torch.equal(net.forward(x, xr, ranges, streams=2), want)
            assert torch.equal(out, want)


@pytest.mark.parametrize("t", [3, 8])
def test_update_first_over_lists_packs_the_weights_once(monkeypatch, t):
    """All of them in one launch; planes, which other features than fp32 and calibrate() take, from when those first need
    them on, eager and recorded."""
    rng = np.random.default_rng(t)
    a, _ = block_graph(rng, 5, 96, 31, 6.0)
    Ws = [rng.uniform(-1, 1, dh).astype(np.float32) for dh in ((20, 24), (24, 9))]
    calls, real_bits, real_weights = [], B.qgtc_pack_bits, B.qgtc_pack_weights
    monkeypatch.setattr(B, "qgtc_pack_bits", lambda src, *args, **k: calls.append(tuple(src.shape)) or real_bits(src, *args, **k))
    monkeypatch.setattr(B, "qgtc_pack_weights", lambda *args, **k: calls.append("weights") or real_weights(*args, **k))
    net, plain = (QuantGNN(dev(a), [dev(W) for W in Ws], 8, t, False, block_rows=96, lists=lists, update_first=True) for lists in (True, False))
    x, xr = dev(rng.standard_normal((a.shape[0], 20)).astype(np.float32)), (-3.0, 3.0)
    codes = dev(rng.integers(0, 256, (a.shape[0], 20)).astype(np.int32))
    ranges = plain.calibrate(x, xr)
    packed = lambda: [c for c in calls if c in ("weights", (20, 24), (24, 9))]
    calls.clear()
    net.pack_static()
    assert packed() == ["weights"]
    assert torch.equal(net.forward(x, xr, ranges), plain.forward(x, xr, ranges))
    assert net.calibrate(x, xr) == ranges
    out = torch.empty((a.shape[0], 9), device="cuda")
    graph = net.capture(codes, xr, ranges, out)
    for changed in (False, True):
        if changed:
            for one in (net, plain):
                one.Ws[0].neg_()
                calls.clear()
                one.pack_static()
            calls.clear()
        want = plain.forward(codes, xr, ranges)
        for _ in range(2):
            out.zero_()
            graph.replay()
            assert torch.equal(net.forward(codes, xr, ranges), want) and torch.equal(out, want)
        assert torch.equal(net.forward(x, xr, ranges), plain.forward(x, xr, ranges))
    assert not packed()


@pytest.mark.parametrize("s,t,update_first", [(4, 4, False), (8, 7, True), (16, 7, False), (12, 16, False)])
def test_weights_of_another_kind_are_packed(s, t, update_first):
    """pack_static() of weights that were replaced by integers, by rows of a wider matrix, or where the old ones were."""
    rng = np.random.default_rng(s + t)
    a, _ = block_graph(rng, 5, 96, 31, 6.0)
    shapes = ((20, 24), (24, 9))
    Ws = [dev(rng.uniform(-1, 1, dh).astype(np.float32)) for dh in shapes]
    nets = [QuantGNN(dev(a), Ws, s, t, False, block_rows=96, lists=lists, update_first=update_first) for lists in (True, False)]
    assert nets[0].lists is not None and nets[1].lists is None
    x, xr = dev(rng.standard_normal((a.shape[0], 20)).astype(np.float32)), (-3.0, 3.0)
    ranges = nets[1].calibrate(x, xr)
    outs = []
    for W in (dev(rng.integers(0, 1 << t, shapes[0]).astype(np.int32)), dev(rng.uniform(-1, 1, (20, 31)).astype(np.float32))[:, 3:27],
              dev(rng.integers(0, 1 << min(t, 8), shapes[0]).astype(np.uint8)), Ws[0].clone()):
        for net in nets:
            net.Ws[0] = W
            net.pack_static()
        want = nets[1].forward(x, xr, ranges)
        assert not any(torch.equal(want, o) for o in outs)
        assert torch.equal(nets[0].forward(x, xr, ranges), want)
        assert torch.equal(nets[0].forward(x, xr, ranges, want_int=True), nets[1].forward(x, xr, ranges, want_int=True))
        if not update_first:
            assert torch.equal(nets[0].forward(x, xr, ranges, streams=2), want)
        outs.append(want)
    for net in nets:
        net.Ws[0] = net.Ws[0].view(24, 20)
        with pytest.raises((q.QgtcError, AssertionError)):
            net.pack_static()


@pytest.mark.parametrize("s,t,update_first", [(4, 4, False), (8, 8, True), (4, 3, True), (16, 7, False), (12, 16, False)])
def test_passes_follow_replaced_weights(s, t, update_first):
    """W[l] replaced, all of W replaced, and other weights packed into an operand: what a network without lists computes
    from the same operands, eager and recorded."""
    rng = np.random.default_rng(s + t)
    a, _ = block_graph(rng, 5, 96, 31, 6.0)
    shapes = ((20, 24), (24, 9))
    sets = [[dev(rng.uniform(-1, 1, dh).astype(np.float32)) for dh in shapes] for _ in range(4)]
    nets = [QuantGNN(dev(a), sets[0], s, t, False, block_rows=96, lists=lists, update_first=update_first) for lists in (True, False)]
    assert nets[0].lists is not None and nets[1].lists is None
    x, xr = dev(rng.standard_normal((a.shape[0], 20)).astype(np.float32)), (-3.0, 3.0)
    ranges = nets[1].calibrate(x, xr)

    def operand(W, layout):
        return q.qgtc_pack_bits(W, t, layout, quant=(-1.0, 1.0))

    outs = []
    for step in ("first", "one", "one of them in place", "all", "none"):
        for net in nets:
            if step == "one":
                net.W[1] = operand(sets[1][1], net.w_layout[1])
            elif step == "one of them in place":
                q.qgtc_pack_bits(sets[2][0], t, net.w_layout[0], quant=(-1.0, 1.0), out=net.W[0])
            elif step == "all":
                net.W = [operand(W, lay) for W, lay in zip(sets[3], net.w_layout)]
            elif step == "none":
                net.pack_static()
        want = nets[1].forward(x, xr, ranges, want_int=True)
        assert torch.equal(want, outs[0]) if step == "none" else not any(torch.equal(want, o) for o in outs)
        assert torch.equal(nets[0].forward(x, xr, ranges, want_int=True), want)
        if not update_first:
            assert torch.equal(nets[0].forward(x, xr, ranges, want_int=True, streams=2), want)
        assert torch.equal(nets[0].forward(x, xr, ranges), nets[1].forward(x, xr, ranges))
        out = torch.empty_like(want)
        graph = nets[0].capture(x, xr, ranges, out, want_int=True)
        for _ in range(2):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
        outs.append(want)


@pytest.mark.parametrize("n", [1, 17, 31, 33, 64 + 15])
@pytest.mark.parametrize("dims", ["3-2", "70-20", "130-64", "300-9", "512-16"])
@pytest.mark.parametrize("s", [8, 16])
def test_last_tile_of_few_rows_with_a_self_term(n, dims, s):
    """Units behind the last row, for every split of a tile: the layers of whole tiles' results."""
    rng = np.random.default_rng(n + s)
    block = 64
    blocks = -(-n // block)
    a, _ = block_graph(rng, blocks, block, blocks * block - n, 6.0)
    d = [int(v) for v in dims.split("-")]
    W, xr = dev(rng.uniform(-1, 1, d).astype(np.float32)), (-3.0, 3.0)
    x = dev(rng.standard_normal((n, d[0])).astype(np.float32))
    nets = [QuantGNN(dev(a), [W], s, s, True, block_rows=block, lists=lists) for lists in (True, False)]
    ranges = nets[1].calibrate(x, xr)
    for ints in (True, False):
        assert torch.equal(*[net.forward(x, xr, ranges, want_int=ints) for net in nets])


def test_features_of_more_words_than_a_launch_has_threads():
    """2^24 rows of 1009 columns (64 GiB), read element by element: the codes are those of the same rows by themselves."""
    n, d, xr = (1 << 24) + 50, 1009, (-1.0, 1.0)
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GiB")
    x = torch.empty((n, d), device="cuda")
    buf = torch.zeros(int(B.lib().qgtc_stack_buffer_bytes(n, d)) // 4, dtype=torch.int32, device="cuda")
    cut = ((1 << 31) - 1) // 256                     # rows of the first launch
    at = [(0, 40), (cut - 20, cut + 20), (2 * cut - 20, 2 * cut + 20), (n - 40, n)]
    for r0, r1 in at:
        x[r0:r1] = torch.rand((r1 - r0, d), device="cuda") * 2 - 1
    B.qgtc_stack_input(x, 8, xr, buf, rows_form=True)
    part = torch.zeros(1 << 20, dtype=torch.int32, device="cuda")
    for r0, r1 in at:
        B.qgtc_stack_input(x[r0:r1].clone(), 8, xr, part, rows_form=True)
        assert torch.equal(buf[r0 * 256:r1 * 256], part[:(r1 - r0) * 256]) and len(part[:(r1 - r0) * 256].unique()) > 1000
    del x, buf
    torch.cuda.empty_cache()


@pytest.mark.parametrize("rows,cols,block,extra,d", [
    (1, 32, 32, 0, 4),
    (65, 64, 64, 0, 12),           # a wave with one row, one word of a row
    (1000, 416, 416, 16, 100),     # pieces that are no whole words, a stride
    (130, 2048, 2048, 0, 64),      # the longest rows of one launch, lists of 256 entries and more
    (2000, 2000, 0, 0, 8),         # one block
    (300, 2080, 2080, 0, 8),       # too long: a launch each
    (100, 100, 0, 1, 8),           # no whole pieces
    (128, 128, 128, 0, 7),         # features of a width that is not
])
@pytest.mark.parametrize("with_map,with_x", [(True, True), (False, True), (True, False)])
def test_a_batch_is_packed_like_its_parts(rows, cols, block, extra, d, with_map, with_x):
    import paper_2111_09547_amd.binding as B
    cols = min(cols, block) if block else cols
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    wide = (torch.rand((rows, cols + extra), generator=gen, device="cuda") < torch.rand((rows, 1), generator=gen, device="cuda") ** 4).to(torch.uint8)
    wide += 2 * torch.randint(0, 2, wide.shape, generator=gen, device="cuda", dtype=torch.uint8)    # (bit 0 counts)
    src = wide[:, :cols]
    x = torch.randn((rows, d), generator=gen, device="cuda")
    Ws = [torch.rand(s, generator=gen, device="cuda") for s in ((d, 64), (64, 17))]
    ranges = [(float(W.min()), float(W.max())) for W in Ws]
    got = []
    for together in (False, True):
        A = B.alloc_bits(rows, cols, 1, B.LEFT, block)
        lists = B.qgtc_build_neighbours(B.qgtc_pack_bits(torch.zeros_like(src), 1, B.LEFT, out=A))
        lists.buffer.fill_(-1)                                     # (what is not an entry of a list is not read)
        tmap = B._alloc_tile_map(A, 16, 32) if with_map else None
        A.words.fill_(-1)
        ops = [B.alloc_bits(*W.shape, t, B.RIGHT_BYTES) for W, t in zip(Ws, (8, 3))]
        for op in ops:
            op.words.zero_()
        sums = torch.zeros(17, dtype=torch.int32, device="cuda")
        codes = torch.zeros(B.lib().qgtc_stack_buffer_bytes(rows, d) // 4 + 4, dtype=torch.int32, device="cuda")
        weights = (B.WeightSources(Ws, ranges, ops), 1, sums)
        if together:
            B.qgtc_pack_batch(src, A, lists, tmap, weights, x if with_x else None, 8, (-2.0, 2.0), codes)
        else:
            B.qgtc_pack_weights(*weights)
            if with_x:
                B.qgtc_stack_input(x, 8, (-2.0, 2.0), codes, rows_form=True)
            B.qgtc_pack_bits(src, 1, B.LEFT, out=A)
            B.qgtc_build_neighbours(A, lists, tmap)
        got.append([A.words, lists.buffer, sums, codes, *[op.words for op in ops]] + ([tmap.row_cnt, tmap.deg] if with_map else []))
        if with_map:
            cnt = tmap.row_cnt
            used = torch.arange(tmap.c.n_tile_cols, device="cuda")[None, :] < cnt[:, None]
            got[-1].append(torch.where(used, tmap.col_idx, -1))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("rows,cols,d", [(130, 2048, 20), (700, 1056, 8), (100, 1024, 4), (200, 1536, 128)])
@pytest.mark.parametrize("with_map", [True, False])
def test_a_recorded_batch_is_packed_like_one_that_is_not(rows, cols, d, with_map):
    """Few long rows go in launches of their own where they are recorded: every replay, on new inputs, against the call itself."""
    gen = torch.Generator(device="cuda").manual_seed(rows + cols)
    src, x = torch.zeros((rows, cols), dtype=torch.uint8, device="cuda"), torch.zeros((rows, d), device="cuda")
    W = torch.rand((d, 17), generator=gen, device="cuda")
    made = []
    for _ in range(2):
        A = B.alloc_bits(rows, cols, 1, B.LEFT, cols)
        lists = B.qgtc_build_neighbours(B.qgtc_pack_bits(src, 1, B.LEFT, out=A))
        lists.buffer.fill_(-1)
        tmap = B._alloc_tile_map(A, 16, 32) if with_map else None
        op = B.alloc_bits(d, 17, 8, B.RIGHT_BYTES)
        sums = torch.zeros(17, dtype=torch.int32, device="cuda")
        codes = torch.zeros(B.lib().qgtc_stack_buffer_bytes(rows, d) // 4 + 4, dtype=torch.int32, device="cuda")
        weights = (B.WeightSources([W], [(0.0, 1.0)], [op]), 0, sums)
        made.append(((src, A, lists, tmap, weights, x, 8, (-2.0, 2.0), codes),
                     [A.words, lists.deg, lists.buffer, op.words, sums, codes] + ([tmap.row_cnt, tmap.deg] if with_map else [])))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        B.qgtc_pack_batch(*made[0][0])
    for _ in range(3):
        src.copy_(torch.rand((rows, cols), generator=gen, device="cuda") < torch.rand((rows, 1), generator=gen, device="cuda") ** 4)
        x.normal_(generator=gen)
        for _, outs in made:
            for out in outs:
                out.zero_()
        graph.replay()
        B.qgtc_pack_batch(*made[1][0])
        for got, want in zip(made[0][1], made[1][1]):
            assert torch.equal(got, want)
        assert len(made[0][1][0].unique()) > 20


def test_heavy_rows_of_a_large_graph_in_narrow_layers():
    """262144 rows and more, of which more than the workgroups that take heavy rows have more neighbours than a tile's waves take."""
    gen = torch.Generator(device="cuda").manual_seed(5)
    n, block = 262144 + 70, 128
    a = (torch.rand((n, block), generator=gen, device="cuda") < 0.02).to(torch.uint8)
    a[::41] = 1
    a[n // block * block:, n % block:] = 0
    x = torch.randn((n, 20), generator=gen, device="cuda")
    Ws = [torch.rand((d, h), generator=gen, device="cuda") - 0.5 for d, h in ((20, 16), (16, 5))]
    nets = [QuantGNN(a, Ws, 8, 8, True, block_rows=block, lists=lists) for lists in (True, False)]
    ranges = nets[1].calibrate(x, (-3.0, 3.0))
    assert torch.equal(*[net.forward(x, (-3.0, 3.0), ranges) for net in nets])


@pytest.mark.parametrize("n,block,dims,bn,update_first", [
    # 49 to 64 columns, a wave per tile, more than four workgroups per compute unit
    (65536 + 70, 128, "64-50-64-12", False, False),  # codes and fp32 from four output tiles, and from one
    (65536 + 70, 128, "49-64-16-48-3", True, False), # behind an affine map
    (65536 + 70, 128, "70-64-49", False, True),      # sums of 49 and 64 columns
    # 129 to 256 columns, four waves per tile, more than three
    (12288 + 35, 512, "129-200-256-70", False, False),
    (12288 + 35, 512, "256-130-160-5", True, False),
])
@pytest.mark.parametrize("degree", [2.0, 12.0])
def test_layers_of_more_workgroups_have_kernels_of_fewer_registers(n, block, dims, bn, update_first, degree):
    """Against layers of whole tiles."""
    gen = torch.Generator(device="cuda").manual_seed(7)
    a = (torch.rand((n, block), generator=gen, device="cuda") < degree / block).to(torch.uint8)
    a[::301] = 1
    a[n // block * block:, n % block:] = 0
    d = [int(v) for v in dims.split("-")]
    x = torch.randn((n, d[0]), generator=gen, device="cuda")
    Ws = [torch.rand(dh, generator=gen, device="cuda") - 0.5 for dh in zip(d[:-1], d[1:])]
    rng = np.random.default_rng(2)
    norms = [BatchNorm(*(rng.uniform(lo, hi, h).tolist() for lo, hi in ((0.5, 1.5), (-0.3, 0.6), (-0.02, 0.04), (0.01, 0.04)))) for h in d[1:-1]] + [None]
    nets = [QuantGNN(a, Ws, 8, 8, True, block_rows=block, lists=lists, update_first=update_first, batchnorm=norms if bn else None)
            for lists in (True, False)]
    assert nets[0].lists is not None and nets[1].lists is None
    ranges = nets[1].calibrate(x, (-3.0, 3.0))
    for ints in (True, False):
        got, want = [net.forward(x, (-3.0, 3.0), ranges, want_int=ints) for net in nets]
        assert torch.equal(got, want) and len(want.unique()) > 100     # (sums of two 8-bit codes alone take more)
