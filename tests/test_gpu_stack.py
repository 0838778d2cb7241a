"""The fused stack (activations kept as codes) and the aggregation's splits, at the edges of
their tiles: every column split, several passes, rows that end inside a unit, small diagonal
blocks side by side, waves that share K.  Integers are compared exactly."""
import numpy as np
import pytest
import torch
import scipy.sparse as sp

from oracle import qgnn

pytestmark = pytest.mark.gpu

q = pytest.importorskip("paper_2111_09547_amd")
import paper_2111_09547_amd.binding as B  # noqa: E402
from paper_2111_09547_amd.model import BatchNorm, LayerRanges, QuantGNN  # noqa: E402
from gpu_util import dev, as_u32, assert_fp32_close  # noqa: E402


def block_graph(rng, blocks, block, short, degree):
    """(compact uint8 [n, block], the same as a csr matrix) of Bernoulli subgraphs."""
    n = blocks * block - short
    a = (rng.random((n, block), dtype=np.float32) < min(0.6, degree / block)).astype(np.uint8)
    if short:
        a[(blocks - 1) * block:, block - short:] = 0
    r, c = np.nonzero(a)
    csr = sp.csr_matrix((np.ones(len(r), np.int64), (r, c + r // block * block)), shape=(n, n))
    return a, csr


@pytest.mark.parametrize("blocks,block,short,dims,s,t,gin", [
    (3, 64, 5, "1-2", 1, 1, False),
    (7, 32, 9, "16-17-5", 8, 8, True),             # several small blocks per workgroup
    (5, 96, 31, "17-33-16", 5, 3, True),
    (3, 416, 171, "32-48-64-7", 8, 4, False),      # 7 units of 64 rows: the last one half empty
    (2, 1024, 1, "64-65-2", 8, 8, True),
    (4, 128, 0, "128-129-40", 4, 8, False),        # two passes, output tiles kept
    (3, 160, 33, "300-101-47", 7, 7, True),
    (1, 2048, 40, "513-16-200", 8, 8, False),      # more weights than the LDS keeps, then thirteen output tiles
    (110, 320, 77, "40-64-20", 3, 8, True),        # an empty unit in every second workgroup
    (66, 1024, 100, "130-70-33-64", 8, 8, False),  # enough rows for four units side by side
])
@pytest.mark.parametrize("kbits", [None, 128, 32])
def test_stack_equals_oracle(blocks, block, short, dims, s, t, gin, kbits):
    rng = np.random.default_rng(blocks * 1000 + block + s)
    d = [int(v) for v in dims.split("-")]
    a, csr = block_graph(rng, blocks, block, short, 6.0)
    n = a.shape[0]
    X = rng.standard_normal((n, d[0])).astype(np.float32)
    Ws = [rng.uniform(-0.5, 0.5, dh).astype(np.float32) for dh in zip(d[:-1], d[1:])]
    net = QuantGNN(dev(a), [dev(W) for W in Ws], s, t, gin, tile_kbits=kbits or 128, use_map=kbits is not None,
                   block_rows=block)
    assert net._fused
    xr = (float(X.min()), float(X.max()))
    x = dev(X)
    ranges = net.calibrate(x, xr)
    rqs = [((0, qgnn.inv_scale(0.0, float(r.agg_hi), s)),
            None if r.out_hi is None else (0, qgnn.inv_scale(0.0, float(r.out_hi), s))) for r in ranges]
    wr = [(float(W.min()), float(W.max())) for W in Ws]
    ref, trace, _ = qgnn.forward_dequantized(csr, X, xr, Ws, wr, s, t, gin, rqs=rqs)
    z = net.forward(x, xr, ranges, want_int=True)
    assert (as_u32(z) == trace[-1]["Z"]).all()
    out = net.forward(x, xr, ranges)
    assert_fp32_close(out.cpu().numpy(), ref, f"{dims} s={s}")
    # features that arrive as planes, with an odd row stride, and already packed: the same bits
    planes = q.qgtc_pack_bits(x, s, q.RIGHT, quant=xr)
    assert torch.equal(net.forward(None, xr, ranges, x_bits=planes), out)
    wide = torch.full((n, d[0] + 3), float("nan"), device="cuda")
    wide[:, 1:1 + d[0]] = x
    assert torch.equal(net.forward(wide[:, 1:1 + d[0]], xr, ranges), out)
    net.pack_static(x, xr)
    assert torch.equal(net.forward(x, xr, ranges, x_packed=True), out)


def test_stack_refuses_what_the_layers_refuse():
    rng = np.random.default_rng(1)
    a, _ = block_graph(rng, 2, 64, 0, 6.0)
    W = rng.uniform(-1, 1, (20, 9)).astype(np.float32)
    net = QuantGNN(dev(a), [dev(W)], 4, 4, False, block_rows=64)
    x = dev(rng.standard_normal((128, 20)).astype(np.float32))
    ranges = net.calibrate(x, (-3.0, 3.0))
    with pytest.raises(AssertionError):
        net.pack_static(x[:, :19].contiguous(), (-3.0, 3.0))
    with pytest.raises(AssertionError):
        net.forward(x[:127], (-3.0, 3.0), ranges)
    with pytest.raises(AssertionError):
        net.forward(x, (-3.0, 3.0), ranges, streams=[1])
    with pytest.raises(q.QgtcError):
        net.forward(x, (3.0, -3.0), ranges)
    with pytest.raises(q.QgtcError):                 # rows of the output closer than its columns
        net.forward(x, (-3.0, 3.0), ranges, out=torch.empty((128, 8), device="cuda"))


@pytest.mark.parametrize("s", [1, 8, 11])
@pytest.mark.parametrize("rows,k,cols,density", [
    (70, 2500, 20, 0.3), (200, 1100, 16, 0.002),     # four waves share the stages of a unit
    (130, 257, 20, 0.2), (500, 640, 16, 0.01), (70, 1024, 65, 0.3),   # ... all of K one stage, in part and whole
    (33000, 130, 32, 0.2), (33000, 260, 17, 0.01),   # two waves of 16 columns
    (6700, 200, 300, 0.2), (6700, 1300, 290, 0.001),  # two waves of 32 columns, several workgroups along the columns
])
def test_aggregate_splits(s, rows, k, cols, density):
    rng = np.random.default_rng(rows + k + s)
    a = (rng.random((rows, k), dtype=np.float32) < density).astype(np.uint8)
    a[rows // 2:rows // 2 + 40] = 0                  # empty rows, and a whole unit without a tile
    a[:, -1] |= (np.arange(rows) % 97 == 0).astype(np.uint8)
    x = rng.integers(0, 1 << s, (k, cols)).astype(np.int32)
    ref = qgnn.aggregate(sp.csr_matrix(a.astype(np.int64)), x.astype(np.uint32))
    A = q.qgtc_pack_bits(dev(a), 1, q.LEFT)
    X = q.qgtc_pack_bits(dev(x), s, q.RIGHT)
    for tmap in (None, q.qgtc_build_tile_map(A, 16, 128), q.qgtc_build_tile_map(A, 16, 32)):
        y = q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32))
        assert (as_u32(y) == ref).all()


@pytest.mark.parametrize("s", [3, 8, 11])
@pytest.mark.parametrize("blocks,block,short,cols", [(5, 288, 31, 16), (3, 512, 0, 40), (2, 1024, 77, 130), (3, 1056, 1, 20)])
def test_aggregate_blocks_as_one_stage(s, blocks, block, short, cols):
    """Diagonal blocks whose K is one stage of the four waves of a unit (up to 1024 columns; 1056
    are more), with the rows themselves added."""
    rng = np.random.default_rng(block + s)
    a, csr = block_graph(rng, blocks, block, short, 9.0)
    x = rng.integers(0, 1 << s, (a.shape[0], cols)).astype(np.int32)
    ref = qgnn.aggregate(csr, x.astype(np.uint32), True)
    A, X = q.qgtc_pack_bits(dev(a), 1, q.LEFT, block_rows=block), q.qgtc_pack_bits(dev(x), s, q.RIGHT)
    for tmap in (None, q.qgtc_build_tile_map(A, 16, 64)):
        y = q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32, self_term=True))
        assert (as_u32(y) == ref).all()


@pytest.mark.parametrize("cols", [16, 32])
@pytest.mark.parametrize("s", [3, 8])
def test_four_units_side_by_side_on_planes(cols, s):
    """Rows for four units per workgroup, narrow column groups: half of the waves have no piece
    of a staged X to store, and multiply with words of A that were requested two stages before."""
    rows, k, h = 66000, 1300, 20
    rng = np.random.default_rng(cols + s)
    a = sp.random(rows, k, density=0.03, format="csr", random_state=rng, dtype=np.float32)
    a.data[:] = 1
    some = np.ones(rows, np.float32)
    some[rows // 2:rows // 2 + 130] = 0              # a unit without a bit
    a = sp.csr_matrix(sp.diags(some) @ a)
    a.eliminate_zeros()
    x = rng.integers(0, 1 << s, (k, cols)).astype(np.int32)
    w = rng.integers(0, 1 << s, (cols, h)).astype(np.int32)
    y, _, z, (lo, inv) = qgnn.layer(a.astype(np.int64), x.astype(np.uint32), w.astype(np.uint32), s)
    A = q.qgtc_pack_bits(dev(a.astype(np.uint8).toarray()), 1, q.LEFT)
    X, W = q.qgtc_pack_bits(dev(x), s, q.RIGHT), q.qgtc_pack_bits(dev(w), s, q.RIGHT)
    first = q.Epilogue(mode=q.OUT_BITS, rq_nbits=s, rq_lo=lo, rq_inv_scale=float(inv))
    for tmap in (None, q.qgtc_build_tile_map(A, 16, 64)):
        assert (as_u32(q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32))) == y).all()
        assert (as_u32(q.qgtc_layer(A, tmap, X, W, first, q.Epilogue(mode=q.OUT_I32))) == z).all()


def small_net(rng, blocks=3, block=96, dims=(20, 24, 9), s=4, bn=False):
    a, _ = block_graph(rng, blocks, block, 0, 6.0)
    Ws = [dev(rng.uniform(-1, 1, dh).astype(np.float32)) for dh in zip(dims[:-1], dims[1:])]
    norms = [BatchNorm(*(rng.uniform(0.5, 1.5, h).tolist() for _ in range(4))) for h in dims[1:-1]] + [None]
    net = QuantGNN(dev(a), Ws, s, s, False, block_rows=block, batchnorm=norms if bn else None)
    return net, dev(rng.standard_normal((blocks * block, dims[0])).astype(np.float32))


@pytest.mark.parametrize("ints", [False, True])
def test_buffers_are_made_on_the_callers_stream(monkeypatch, ints):
    """Memory that a network keeps belongs to the caller's stream: what is made on one of the
    network's own streams is given back in the order of that one alone."""
    net, x = small_net(np.random.default_rng(5), bn=True)
    xr = (-3.0, 3.0)
    if ints:
        x = torch.randint(0, 16, x.shape, dtype=torch.int32, device="cuda")
    ranges = [LayerRanges(300, 2.0), LayerRanges(400, None)]
    caller, made = torch.cuda.current_stream(), []
    real_alloc, real_fold = B.alloc_bits, B.qgtc_fold_batchnorm
    monkeypatch.setattr(B, "alloc_bits", lambda *a, **k: made.append(torch.cuda.current_stream()) or real_alloc(*a, **k))
    monkeypatch.setattr(B, "qgtc_fold_batchnorm", lambda *a: made.append(torch.cuda.current_stream()) or real_fold(*a))
    net.pack_static(x, xr)
    graph = net.capture(x, xr, ranges, torch.empty((x.shape[0], 9), device="cuda"), with_static=True)
    assert made and all(m == caller for m in made)
    assert (net._x_bufs is not None) == ints         # planes only where the features need them
    del graph


def test_calibration_leaves_the_features_packed():
    net, x = small_net(np.random.default_rng(6))
    xr = (-3.0, 3.0)
    ranges = net.calibrate(x, xr)
    out = net.forward(x, xr, ranges)
    net.calibrate(x, xr)
    assert torch.equal(net.forward(x, xr, ranges, x_packed=True), out)
    assert net._x_bufs is None


@pytest.mark.parametrize("s", [1, 8])
def test_calibration_makes_no_buffers_of_planes(monkeypatch, s):
    """... and stays inside those of the codes, also with a hidden layer wider than the others."""
    net, x = small_net(np.random.default_rng(16), blocks=3, block=32, dims=(3, 50, 17, 9), s=s)
    for i, c in enumerate(net._codes):               # the same buffers with a margin behind them
        wide = torch.full((c.numel() + 64,), 0x5a5a5a5a, dtype=torch.int32, device="cuda")
        net._codes[i] = wide[:c.numel()]
        net._codes[i].margin = wide
    packed = net._W_planes = [q.qgtc_pack_bits(W, net.t, q.RIGHT, quant=r) for W, r in zip(net.Ws, net.w_ranges)]
    made, real = [], B.alloc_bits
    monkeypatch.setattr(B, "alloc_bits", lambda *a, **k: made.append(a[3]) or real(*a, **k))
    net.calibrate(x, (-3.0, 3.0))
    assert B.RIGHT not in made and net._W_planes is packed
    for c in net._codes:
        assert (c.margin[c.numel():] == 0x5a5a5a5a).all()


def test_prepared_pass_follows_the_operands():
    """Adjacency, weights and self term replaced between passes with the same ranges."""
    rng = np.random.default_rng(7)
    net, x = small_net(rng)
    other, _ = small_net(rng)
    xr, ranges = (-3.0, 3.0), [LayerRanges(300, 900.0), LayerRanges(400, None)]
    net.w_ranges = other.w_ranges                    # (the same key but for the operands)
    first = net.forward(x, xr, ranges).clone()
    want = other.forward(x, xr, ranges)
    assert not torch.equal(first, want)
    net.A, net.A_src, net.Ws = other.A, other.A_src, other.Ws
    net.pack_static()                                # into the same map and weights
    assert torch.equal(net.forward(x, xr, ranges), want)
    net.self_term = other.self_term = True
    with_self = net.forward(x, xr, ranges)
    assert not torch.equal(with_self, want) and torch.equal(with_self, other.forward(x, xr, ranges))


def test_prepared_pass_follows_the_batch_normalization():
    """A hidden layer's batch normalization replaced, and taken away, between passes with the same ranges."""
    net, x = small_net(np.random.default_rng(8), bn=True)
    xr, ranges = (-3.0, 3.0), [LayerRanges(300, 2.0), LayerRanges(400, None)]

    def fresh(bn):
        other = QuantGNN(net.A, net.Ws, net.s, net.t, False, block_rows=96, batchnorm=bn)
        return other.forward(x, xr, ranges)

    bn = net.batchnorm[0]
    outs = [net.forward(x, xr, ranges)]
    for new in (BatchNorm([0.5 * v for v in bn.gamma], bn.beta, bn.mean, bn.var), None, bn):
        net.batchnorm[0] = new
        outs.append(net.forward(x, xr, ranges))
        assert torch.equal(outs[-1], fresh(list(net.batchnorm)))
    assert torch.equal(outs[0], outs[3]) and not torch.equal(outs[0], outs[1]) and not torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("width", [2, 8])
def test_planes_of_another_width_than_the_networks(width):
    """forward(x_bits=...) takes planes of any width up to 8 bits, as qgtc_layer does."""
    net, _ = small_net(np.random.default_rng(9), dims=(20, 24, 9))
    n, ranges = net.A.rows, [LayerRanges(6 << width, 2000.0), LayerRanges(100, None)]
    X = q.qgtc_pack_bits(torch.randint(0, 1 << width, (n, 20), dtype=torch.int32, device="cuda"), width, q.RIGHT)
    got = net.forward(None, (0.0, 1.0), ranges, x_bits=X, want_int=True)
    (f0, s0), (f1, s1) = net._epilogues((0.0, 1.0), ranges, True)
    hidden = q.qgtc_layer(net.A, net.map, X, net.W[0], f0, s0)
    assert torch.equal(got, q.qgtc_layer(net.A, net.map, hidden, net.W[1], f1, s1))
    assert int(got.abs().sum()) > 0


@pytest.mark.parametrize("cols", [20, 21, 3])        # 16-byte loads, element by element, narrower than four columns
@pytest.mark.parametrize("s", [1, 5, 8])
def test_features_that_are_no_ordinary_numbers(cols, s):
    """NaN, infinities, zeros of both signs and the largest values through the quantizer of a
    stack: the codes of Eq. (2) with its clamp, a NaN as code 0."""
    rng = np.random.default_rng(cols + s)
    net, _ = small_net(rng, dims=(cols, 9), s=s)
    n, xr, ranges = net.A.rows, (-1.5, 2.0), [LayerRanges(8 << s, None)]
    x = rng.standard_normal((n, cols)).astype(np.float32)
    some = np.array([np.nan, np.inf, -np.inf, 3.4e38, -3.4e38, 0.0, -0.0, 1e-40, -1.5, 2.0], np.float32)
    x.flat[rng.permutation(x.size)[:x.size // 2]] = np.resize(some, x.size // 2)
    with np.errstate(over="ignore", invalid="ignore"):
        codes = qgnn.quantize(np.where(np.isnan(x), np.float32(xr[0]), x), *xr, s)
    X = q.qgtc_pack_bits(dev(codes.astype(np.int32)), s, q.RIGHT)
    want = net.forward(None, xr, ranges, x_bits=X, want_int=True)
    assert torch.equal(net.forward(dev(x), xr, ranges, want_int=True), want)
    assert (as_u32(q.qgtc_unpack_bits(q.qgtc_pack_bits(dev(x), s, q.RIGHT, quant=xr))) == codes).all()


@pytest.mark.parametrize("dims", ["200-40-9", "300-150-200-7"])
@pytest.mark.parametrize("s,t", [(8, 8), (4, 7)])
def test_batchnorm_behind_several_passes(dims, s, t):
    """Column maps of hidden layers whose output tiles are kept over several passes (up to 4 and up to 16)."""
    rng = np.random.default_rng(s)
    d = [int(v) for v in dims.split("-")]
    a, csr = block_graph(rng, 3, 160, 33, 6.0)
    X = rng.standard_normal((a.shape[0], d[0])).astype(np.float32)
    Ws = [rng.uniform(-0.5, 0.5, dh).astype(np.float32) for dh in zip(d[:-1], d[1:])]
    params = [dict(gamma=rng.uniform(0.5, 1.5, h), beta=rng.uniform(-0.3, 0.6, h), mean=rng.uniform(-0.2, 0.4, h),
                   var=rng.uniform(0.5, 2.0, h), eps=1e-5) for h in d[1:-1]] + [None]
    net = QuantGNN(dev(a), [dev(W) for W in Ws], s, t, False, block_rows=160,
                   batchnorm=[p and BatchNorm(**p) for p in params])
    assert net._fused
    xr, x = (float(X.min()), float(X.max())), dev(X)
    ranges = net.calibrate(x, xr)
    rqs = [((0, qgnn.inv_scale(0.0, float(r.agg_hi), s)),
            None if r.out_hi is None else (0, qgnn.inv_scale(0.0, float(r.out_hi), s))) for r in ranges]
    wr = [(float(W.min()), float(W.max())) for W in Ws]
    ref, trace, _ = qgnn.forward_dequantized(csr, X, xr, Ws, wr, s, t, False, rqs=rqs, batchnorms=params)
    assert (as_u32(net.forward(x, xr, ranges, want_int=True)) == trace[-1]["Z"]).all()
    assert_fp32_close(net.forward(x, xr, ranges).cpu().numpy(), ref, f"{dims} s={s}")


@pytest.mark.parametrize("kind", ["11 bits", "two kernels", "integer features", "batch normalization"])
def test_independent_runs_of_subgraphs(monkeypatch, kind):
    """What is not one native call - more than 8 bits, the two-kernel path, features that are not
    fp32 - runs layer by layer, and as several runs of whole subgraphs on streams of their own
    where asked to: the same bytes as one run, eager and recorded."""
    rng = np.random.default_rng(13)
    s = 11 if kind in ("11 bits", "batch normalization") else 8
    a, _ = block_graph(rng, 5, 96, 31, 6.0)
    Ws = [dev(rng.uniform(-1, 1, dh).astype(np.float32)) for dh in ((20, 24), (24, 9))]
    norm = BatchNorm(*(rng.uniform(0.5, 1.5, 24).tolist() for _ in range(4)))
    net = QuantGNN(dev(a), Ws, s, s, False, block_rows=96,
                   batchnorm=[norm, None] if kind == "batch normalization" else None,
                   tuning=q.Tuning(layer_path=q.LAYER_TWO_KERNELS) if kind == "two kernels" else None)
    assert net._fused == (kind == "integer features")
    x, xr = dev(rng.standard_normal((a.shape[0], 20)).astype(np.float32)), (-3.0, 3.0)
    if kind == "integer features":
        x = torch.randint(0, 1 << s, x.shape, dtype=torch.int32, device="cuda")
    ranges = net.calibrate(x, xr)
    firsts, real = [], net._run_layers
    monkeypatch.setattr(net, "_run_layers", lambda r0, *args: firsts.append(r0) or real(r0, *args))
    want, want_z = net.forward(x, xr, ranges).clone(), net.forward(x, xr, ranges, want_int=True).clone()
    assert firsts == [0, 0] and int(want_z.abs().sum()) > 0
    for streams, rows in ((2, [0, 288]), (3, [0, 192, 384]), ([4, 1], [0, 384]), ([1, 4], [0, 96])):
        for want_int, ref in ((False, want), (True, want_z)):
            firsts.clear()
            got = net.forward(x, xr, ranges, want_int=want_int, streams=streams)
            torch.cuda.synchronize()
            assert firsts == rows and torch.equal(got, ref), streams
    out = torch.empty_like(want)
    graph = net.capture(x, xr, ranges, out, streams=[1, 4], with_static=True)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(net.forward(x, xr, ranges), want)
    del graph


def test_adjacency_rows_of_64_MiB_and_more():
    """Rows that lie so far apart that only 32 of them are within 4 GiB: the same integers as
    from the same rows side by side, narrow and wide, alone and in a layer."""
    rng = np.random.default_rng(12)
    rows, k, pitch, s = 70, 300, 1 << 24, 3
    a = (rng.random((rows, k)) < 0.1).astype(np.uint8)
    near = q.qgtc_pack_bits(dev(a), 1, q.LEFT)
    c = B._BitsC.from_buffer_copy(near.c)
    words = torch.zeros(rows * pitch, dtype=torch.int32, device="cuda")
    c.ld_words, c.plane_stride_words, c.data = pitch, rows * pitch, words.data_ptr()
    words.view(rows, pitch)[:, :near.c.ld_words] = near.words.view(rows, near.c.ld_words)
    far = q.Bits(words, c)
    for cols in (5, 40, 200):
        x = rng.integers(0, 1 << s, (k, cols)).astype(np.int32)
        w = rng.integers(0, 1 << s, (cols, 7)).astype(np.int32)
        X, W = q.qgtc_pack_bits(dev(x), s, q.RIGHT), q.qgtc_pack_bits(dev(w), s, q.RIGHT_BYTES)
        y, _, z, (lo, inv) = qgnn.layer(a, x.astype(np.uint32), w.astype(np.uint32), s)
        first = q.Epilogue(mode=q.OUT_BITS, rq_nbits=s, rq_lo=lo, rq_inv_scale=float(inv))
        for A in (near, far):
            for tmap in (None, q.qgtc_build_tile_map(A, 16, 32)):
                assert (as_u32(q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32))) == y).all()
                assert (as_u32(q.qgtc_layer(A, tmap, X, W, first, q.Epilogue(mode=q.OUT_I32))) == z).all()
