"""GPU parity: each entry point of the C ABI against the CPU oracle, element by
element, on seeded inputs that span several tiles and ragged tails."""
import numpy as np
import pytest
import torch

from oracle import qgnn, bitplane as bp
from workloads import make_workload

pytestmark = pytest.mark.gpu

q = pytest.importorskip("paper_2111_09547_amd")
from gpu_util import assert_fp32_close, dev, as_u32, pack_adjacency, words_np, sync  # noqa: E402


def rand_graph(rng, n, k, p):
    return (rng.random((n, k)) < p).astype(np.uint8)


# ------------------------------------------------------------------ pack / unpack
@pytest.mark.parametrize("bits", [1, 5, 8])
@pytest.mark.parametrize("shape", [(1, 1), (45, 77), (130, 64), (64, 300), (512, 16)])
def test_pack_bytes_layout(bits, shape):
    """Codes as bytes in matrix-core operand order: position of every byte as the
    header states it, 7 + 1 split for 8 bits, zero fill, from fp32 and from integers."""
    rows, cols = shape
    rng = np.random.default_rng([3, bits, rows, cols])
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    lo, hi = float(x.min()), float(x.max()) + 1e-3
    codes = qgnn.quantize(x, lo, hi, bits)
    for src, kw in ((dev(x), dict(quant=(lo, hi))), (dev(codes.view(np.int32)), {})):
        b = q.alloc_bits(rows, cols, bits, q.RIGHT_BYTES)
        b.words.fill_(-1)
        q.qgtc_pack_bits(src, bits, q.RIGHT_BYTES, out=b, **kw)
        assert (as_u32(q.qgtc_unpack_bits(b)) == codes).all()
        raw = b.words.cpu().numpy().view(np.uint8)
        n_nt, n_ks = -(-cols // 16), -(-rows // 64)
        parts = 2 if bits == 8 else 1
        want = np.zeros((parts, n_nt, n_ks, 64, 16), dtype=np.uint8)
        for k in range(rows):
            for c in range(cols):
                lane = c % 16 + 16 * ((k % 64) // 16)
                v = int(codes[k, c])
                want[0, c // 16, k // 64, lane, k % 16] = v & 0x7f if bits == 8 else v
                if bits == 8:
                    want[1, c // 16, k // 64, lane, k % 16] = v >> 7
        assert b.c.ld_words == 256 * n_ks and b.c.plane_stride_words == n_nt * n_ks * 256
        assert (raw[:want.size] == want.ravel()).all()


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("bits", [1, 2, 3, 8, 13, 32])
@pytest.mark.parametrize("shape", [(1, 1), (45, 77), (130, 64), (64, 2100)])
def test_pack_integers_roundtrip(layout, bits, shape):
    rng = np.random.default_rng([1, layout, bits, shape[0]])
    v = rng.integers(0, 2 ** bits, size=shape, dtype=np.uint64).astype(np.uint32)
    b = q.qgtc_pack_bits(dev(v.view(np.int32)), bits, layout)
    sync()
    want = bp.pack(v, bits, layout)
    assert (words_np(b) == want).all()
    if layout == q.LEFT:                      # padding words up to ld are zero
        w = b.words.cpu().numpy().view(np.uint32)[:b.c.plane_stride_words * bits]
        w = w.reshape(bits, shape[0], b.c.ld_words)
        assert (w[:, :, want.shape[2]:] == 0).all()
    assert (as_u32(q.qgtc_unpack_bits(b)) == v).all()


def test_pack_u8_masks_high_bits():
    rng = np.random.default_rng(2)
    v = rng.integers(0, 256, size=(70, 40)).astype(np.uint8)
    b = q.qgtc_pack_bits(dev(v), 3, q.RIGHT)
    assert (as_u32(q.qgtc_unpack_bits(b)) == (v & 7)).all()


@pytest.mark.parametrize("bits", [1, 2, 4, 8, 16, 24, 32])
def test_pack_quantizes_like_eq2(bits):
    rng = np.random.default_rng([3, bits])
    x = rng.standard_normal((333, 50)).astype(np.float32)
    x[0, 0], x[1, 1] = 1e30, -1e30            # far outside the range: clamped
    lo, hi = -2.5, 3.25
    b = q.qgtc_pack_bits(dev(x), bits, q.RIGHT, quant=(lo, hi))
    want = qgnn.quantize(x, lo, hi, bits)
    assert (as_u32(q.qgtc_unpack_bits(b)) == want).all()
    # min-max range of the data itself
    lo, hi = float(x[2:].min()), float(x[2:].max())
    b = q.qgtc_pack_bits(dev(x[2:]), bits, q.LEFT, quant=(lo, hi))
    assert (as_u32(q.qgtc_unpack_bits(b)) == qgnn.quantize(x[2:], lo, hi, bits)).all()


def test_row_and_col_sums():
    rng = np.random.default_rng(4)
    v = rng.integers(0, 64, size=(150, 90)).astype(np.uint32)
    bl = q.qgtc_pack_bits(dev(v.view(np.int32)), 6, q.LEFT)
    br = q.qgtc_pack_bits(dev(v.view(np.int32)), 6, q.RIGHT)
    assert (q.qgtc_row_sums(bl).cpu().numpy() == v.sum(axis=1)).all()
    assert (q.qgtc_col_sums(br).cpu().numpy() == v.sum(axis=0)).all()


# ----------------------------------------------------------------------- tile map
@pytest.mark.parametrize("tile", [(8, 128), (16, 128), (16, 64), (16, 32), (32, 256), (64, 512)])
def test_tile_map_matches_brute_force(tile):
    rng = np.random.default_rng([5, tile[0], tile[1]])
    n, k = 203, 1000
    A = rand_graph(rng, n, k, 0.0008)
    A[40:60] = 0                                 # some all-zero rows of tiles
    Ab = pack_adjacency(A)
    m = q.qgtc_build_tile_map(Ab, tile[0], tile[1])
    sync()
    lists, deg = qgnn.tile_map(A, tile[0], tile[1])
    cnt = m.row_cnt.cpu().numpy()
    idx = m.col_idx.cpu().numpy()
    assert cnt.tolist() == [len(l) for l in lists]
    for tr, l in enumerate(lists):
        assert idx[tr, :len(l)].tolist() == l
    assert int(m.nnz_tiles.cpu()[0]) == sum(len(l) for l in lists)
    assert (m.deg.cpu().numpy() == deg).all()



def test_device_is_what_the_kernels_are_written_for():
    """The launch shapes read the compute-unit count from the device; the workgroup dealing
    is written for 8 XCDs of 32 compute units: check both on the device the tests run on."""
    d = q.qgtc_device_info()
    assert d["is_gfx950"]
    assert d["compute_units"] == torch.cuda.get_device_properties(0).multi_processor_count
    assert d["xcds"] == d["xcds_assumed"] == 8 and d["compute_units"] == 256


@pytest.mark.parametrize("shape", [(1, 1), (100, 300), (257, 257), (1000, 2100), (4100, 640)])
def test_tile_stats_match_the_oracle_at_three_widths(shape):
    """qgtc_tile_stats: non-zero tiles at 16 x 32 / 64 / 128 in one pass, against the brute-force
    tile map of the oracle and against the three maps built one by one."""
    n, k = shape
    rng = np.random.default_rng([5, n, k])
    A = rand_graph(rng, n, k, 0.004)
    if n > 64:
        A[40:90, :] = 0                             # rows of tiles without any edge
    Ab = pack_adjacency(A)
    got = q.qgtc_tile_stats(Ab).cpu().numpy().tolist()
    want = [sum(len(l) for l in qgnn.tile_map(A, 16, kb)[0]) for kb in (32, 64, 128)]
    # (row, 32-bit word) pairs that hold a bit: brute force on the dense matrix
    pad = np.zeros((n, -(-k // 32) * 32), dtype=np.uint8)
    pad[:, :k] = A
    row_words = int(pad.reshape(n, -1, 32).any(axis=2).sum())
    assert got == want + [-(-n // 16), row_words, 0, 0, 0]
    assert q.tile_stats_numbers(q.qgtc_tile_stats(Ab)) == dict(nnz_tiles=want, n_tile_rows=-(-n // 16),
                                                               nnz_row_words=row_words)
    for i, kb in enumerate((32, 64, 128)):
        assert int(q.qgtc_build_tile_map(Ab, 16, kb).nnz_tiles.cpu()[0]) == want[i]
    # a second call into the same buffer starts from zero again
    buf = q.qgtc_tile_stats(Ab)
    assert q.qgtc_tile_stats(Ab, out=buf).cpu().numpy().tolist() == got


def test_tile_stats_on_block_diagonal_storage():
    w = make_workload(5, n_blocks=2)
    g = w.graph
    Ab = pack_adjacency(g, "compact")
    got = q.qgtc_tile_stats(Ab).cpu().numpy().tolist()
    compact = g.dense_compact()
    want = [sum(len(l) for l in qgnn.tile_map(compact, 16, kb)[0]) for kb in (32, 64, 128)]
    row_words = int(compact.reshape(g.n_nodes, -1, 32).any(axis=2).sum())
    assert got == want + [g.n_nodes // 16, row_words, 0, 0, 0]
    assert want[0] > want[1] > want[2]


def expected_run_log2(cnt):
    """The rule stated for nnz_tiles[1] in qgtc.h, on the host."""
    w = np.asarray(cnt, dtype=np.int64) + 1
    for sh in (6, 5, 4):
        load = np.zeros(8, dtype=np.int64)
        np.add.at(load, (np.arange(len(w)) >> sh) & 7, w)
        if load.max() * 8 * 50 <= w.sum() * 51:
            return sh
    return 3


@pytest.mark.parametrize("case", ["uniform", "hubs_first", "mild_skew", "small", "ragged"])
def test_tile_map_run_hint(case):
    """nnz_tiles[1]: long runs for evenly spread tiles, short ones when a few tile rows
    hold most tiles or when there are too few tile rows for eight long runs."""
    rng = np.random.default_rng(17)
    n = {"small": 100 * 16, "ragged": 1000 * 16 + 5}.get(case, 1024 * 16)
    k = 2048
    A = np.zeros((n, k), dtype=np.uint8)
    rows = np.arange(n)
    A[rows, rows % k] = 1                                     # one tile per tile row at least
    if case == "hubs_first":
        A[:64 * 16:16, ::128] = 1                             # the first 64 tile rows hold every tile
    if case == "mild_skew":
        for tr in range(0, 1024, 4):
            A[tr * 16, rng.integers(0, k, size=3)] = 1
    Ab = pack_adjacency(A)
    m = q.qgtc_build_tile_map(Ab, 16, 128)
    sync()
    cnt = m.row_cnt.cpu().numpy()
    total, run = m.nnz_tiles.cpu().numpy().tolist()
    assert total == cnt.sum()
    assert run == expected_run_log2(cnt)
    if case == "uniform":
        assert run == 6
    if case in ("hubs_first", "small"):
        assert run == 3


# ---------------------------------------------------------------------- aggregate
def run_aggregate(A, X, s, tile_kbits=None, block=0, ep=None):
    if block:
        n = A.shape[0]
        compact = np.zeros((n, block), dtype=np.uint8)
        for r in range(n):
            b0 = (r // block) * block
            seg = A[r, b0:b0 + block]
            compact[r, :seg.size] = seg
        Ab = q.qgtc_pack_bits(dev(compact), 1, q.LEFT, block_rows=block)
    else:
        Ab = pack_adjacency(A)
    Xb = q.qgtc_pack_bits(dev(X.view(np.int32)), s, q.RIGHT)
    m = q.qgtc_build_tile_map(Ab, 16, tile_kbits) if tile_kbits else None
    return q.qgtc_aggregate(Ab, m, Xb, ep or q.Epilogue(mode=q.OUT_I32)), m


def test_config1_tiny_aggregation():
    w = make_workload(1)
    A = w.graph.dense()
    want = qgnn.aggregate(A, w.X)
    for kb in (None, 128, 64, 32):
        got, _ = run_aggregate(A, w.X, w.s, kb)
        assert (as_u32(got) == want).all(), kb
    # 1-bit all-ones features give the node degrees
    ones = np.ones((A.shape[0], 16), dtype=np.uint32)
    got, m = run_aggregate(A, ones, 1, 128)
    assert (as_u32(got) == w.graph.degrees()[:, None]).all()
    assert (m.deg.cpu().numpy() == w.graph.degrees()).all()


@pytest.mark.parametrize("s", [1, 2, 3, 4, 5, 6, 7, 8, 11, 16, 32])
@pytest.mark.parametrize("shape", [(100, 100, 70), (257, 257, 16), (96, 300, 33), (40, 40, 130)])
def test_aggregate_int32_ragged(s, shape):
    n, k, d = shape
    rng = np.random.default_rng([6, s, n, d])
    A = rand_graph(rng, n, k, 0.05)
    X = rng.integers(0, 2 ** s, size=(k, d), dtype=np.uint64).astype(np.uint32)
    want = qgnn.aggregate(A, X)
    for kb in (None, 128, 32):
        got, _ = run_aggregate(A, X, s, kb)
        assert (as_u32(got) == want).all(), kb


@pytest.mark.parametrize("d", [16, 70, 200])
def test_aggregate_does_not_depend_on_xcd_run(d):
    """The way workgroups are dealt to the XCDs is a scheduling choice only."""
    rng = np.random.default_rng([8, d])
    n, s = 2100, 3                       # 132 tile rows: several runs per XCD and a ragged tail
    A = rand_graph(rng, n, n, 0.01)
    X = rng.integers(0, 2 ** s, size=(n, d)).astype(np.uint32)
    want = qgnn.aggregate(A, X)
    for run in (-1, 0, 1, 3, 64, 4096):
        ep = q.Epilogue(mode=q.OUT_I32, tuning=q.Tuning(agg_xcd_run=run))
        got, _ = run_aggregate(A, X, s, 128, ep=ep)
        assert (as_u32(got) == want).all(), run
    with pytest.raises(q.QgtcError) as e:                  # out of range: refused, nothing launched
        run_aggregate(A, X, s, 128, ep=q.Epilogue(mode=q.OUT_I32, tuning=q.Tuning(agg_xcd_run=5000)))
    assert e.value.status == 7


@pytest.mark.parametrize("d", [16, 32, 64, 200])
def test_aggregate_block_diagonal_compact_and_self_term(d):
    rng = np.random.default_rng([7, d])
    n, block, s = 330, 96, 5
    A = np.zeros((n, n), dtype=np.uint8)
    for b0 in range(0, n, block):
        b1 = min(n, b0 + block)
        A[b0:b1, b0:b1] = rand_graph(rng, b1 - b0, b1 - b0, 0.08)
    X = rng.integers(0, 2 ** s, size=(n, d)).astype(np.uint32)
    for self_term in (False, True):
        want = qgnn.aggregate(A, X, self_term)
        ep = q.Epilogue(mode=q.OUT_I32, self_term=self_term)
        for kb in (None, 128, 64):
            got, _ = run_aggregate(A, X, s, kb, block=block, ep=ep)
            assert (as_u32(got) == want).all(), (self_term, kb)
        got, _ = run_aggregate(A, X, s, 128, ep=ep)          # same graph, dense storage
        assert (as_u32(got) == want).all()


@pytest.mark.parametrize("d", [16, 24, 64, 100])
@pytest.mark.parametrize("rq_bits", [1, 3, 8, 12])
def test_aggregate_bits_and_f32_epilogues(d, rq_bits):
    rng = np.random.default_rng([8, d, rq_bits])
    n, s = 150, 4
    A = rand_graph(rng, n, n, 0.1)
    X = rng.integers(0, 2 ** s, size=(n, d)).astype(np.uint32)
    Y = qgnn.aggregate(A, X)
    rq_lo, inv = 3, qgnn.inv_scale(3.0, float(Y.max()), rq_bits)
    ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=rq_bits, rq_lo=rq_lo, rq_inv_scale=float(inv))
    got, _ = run_aggregate(A, X, s, 128, ep=ep)
    want = qgnn.requantize(Y, rq_lo, inv, rq_bits)
    assert (words_np(got) == bp.pack(want, rq_bits, bp.LEFT)).all()
    assert (as_u32(q.qgtc_unpack_bits(got)) == want).all()
    # a destination with the default LEFT strides (rows padded to 128 bits), poisoned: the
    # zero padding is part of what the epilogue writes, so the result can serve as the left
    # operand of a kernel that reads whole 128-bit rows
    dst = q.alloc_bits(n, d, rq_bits, q.LEFT)
    assert dst.c.ld_words % 4 == 0 and dst.c.ld_words >= -(-d // 32)
    dst.words.fill_(-1)
    Ab = pack_adjacency(A)
    q.qgtc_aggregate(Ab, q.qgtc_build_tile_map(Ab, 16, 128), q.qgtc_pack_bits(dev(X.view(np.int32)), s, q.RIGHT),
                     ep, out=dst)
    raw = dst.words.cpu().numpy().view(np.uint32)[:rq_bits * n * dst.c.ld_words].reshape(rq_bits, n, -1)
    kw = -(-d // 32)
    assert (raw[:, :, :kw] == bp.pack(want, rq_bits, bp.LEFT)).all()
    assert (raw[:, :, kw:] == 0).all()
    # fp32: sx * Y + lo_x * deg
    deg = A.sum(axis=1).astype(np.int32)
    ep = q.Epilogue(mode=q.OUT_F32, cc=0.37, rs=-1.25, row_i=dev(deg))
    got, _ = run_aggregate(A, X, s, 128, ep=ep)
    ref = qgnn.dequantize(Y, cc=0.37, rs=-1.25, row_i=deg)
    assert_fp32_close(got.cpu().numpy(), ref, '')
    # int32 with ReLU on the signed accumulator (wrapped values count as negative)
    Xbig = np.full((n, d), 2 ** 31 - 1, dtype=np.uint32)
    ep = q.Epilogue(mode=q.OUT_I32, relu=True)
    got, _ = run_aggregate(A, Xbig, 32, 128, ep=ep)
    assert (got.cpu().numpy() == qgnn.int_output(qgnn.aggregate(A, Xbig), relu=True)).all()


# ------------------------------------------------------------------------- update
@pytest.mark.parametrize("st", [(1, 1), (2, 3), (4, 4), (8, 8), (8, 2), (3, 7), (16, 16), (32, 32), (12, 5)])
@pytest.mark.parametrize("shape", [(100, 64, 64), (257, 128, 16), (70, 40, 5), (1000, 512, 16), (64, 300, 70)])
def test_update_int32(st, shape):
    s, t = st
    n, d, h = shape
    rng = np.random.default_rng([9, s, t, n])
    Yq = rng.integers(0, 2 ** s, size=(n, d), dtype=np.uint64).astype(np.uint32)
    Wq = rng.integers(0, 2 ** t, size=(d, h), dtype=np.uint64).astype(np.uint32)
    Yb = q.qgtc_pack_bits(dev(Yq.view(np.int32)), s, q.LEFT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    got = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_I32))
    assert (as_u32(got) == qgnn.update(Yq, Wq)).all()


@pytest.mark.parametrize("rq_bits", [1, 4, 8, 10])
def test_update_bits_and_f32_epilogues(rq_bits):
    rng = np.random.default_rng([10, rq_bits])
    n, d, h, s, t = 300, 64, 24, 4, 3
    Yq = rng.integers(0, 2 ** s, size=(n, d)).astype(np.uint32)
    Wq = rng.integers(0, 2 ** t, size=(d, h)).astype(np.uint32)
    Yb = q.qgtc_pack_bits(dev(Yq.view(np.int32)), s, q.LEFT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    Z = qgnn.update(Yq, Wq)
    inv = qgnn.inv_scale(0.0, float(Z.max()), rq_bits)
    ep = q.Epilogue(mode=q.OUT_BITS, relu=True, rq_nbits=rq_bits, rq_lo=0, rq_inv_scale=float(inv))
    got = q.qgtc_update(Yb, Wb, ep)
    want = qgnn.requantize(Z, 0, inv, rq_bits, relu=True)
    assert (words_np(got) == bp.pack(want, rq_bits, bp.RIGHT)).all()
    rs = Yq.sum(axis=1).astype(np.int32)
    cs = Wq.sum(axis=0).astype(np.int32)
    rl = rng.integers(1, 30, size=n).astype(np.int32)
    kw = dict(cc=1.7e-3, rs=-0.031, l0a=0.4, l0b=-0.9, ck=-6.4, cs=0.0125)
    for relu in (False, True):
        ep = q.Epilogue(mode=q.OUT_F32, relu=relu, row_i=dev(rs), row_l=dev(rl), col_i=dev(cs), **kw)
        got = q.qgtc_update(Yb, Wb, ep).cpu().numpy()
        ref = qgnn.dequantize(Z, row_i=rs, row_l=rl, col_i=cs, relu=relu, **kw)
        assert_fp32_close(got, ref, '')


# -------------------------------------------------------------------------- layer
@pytest.mark.parametrize("cfg,bits,nb", [(2, 4, None), (3, 1, 2), (3, 3, 2), (3, 8, 2), (3, 16, 1), (3, 32, 1)])
def test_layer_matches_oracle(cfg, bits, nb):
    w = make_workload(cfg, bits=bits, n_blocks=nb)
    A = w.graph.dense()
    xr = (float(w.X.min()), float(w.X.max()))
    wr = (float(w.W[0].min()), float(w.W[0].max()))
    Xq = qgnn.quantize(w.X, xr[0], xr[1], w.s)
    Wq = qgnn.quantize(w.W[0], wr[0], wr[1], w.t)
    Y, Yq, Z, (rq_lo, rq_inv) = qgnn.layer(A, Xq, Wq, w.s)
    Ab = pack_adjacency(A)
    m = q.qgtc_build_tile_map(Ab)
    Xb = q.qgtc_pack_bits(dev(w.X), w.s, q.RIGHT, quant=xr)
    Wb = q.qgtc_pack_bits(dev(w.W[0]), w.t, q.RIGHT, quant=wr)
    assert (as_u32(q.qgtc_unpack_bits(Xb)) == Xq).all()
    assert (as_u32(q.qgtc_unpack_bits(Wb)) == Wq).all()
    agg_ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=w.s, rq_lo=rq_lo, rq_inv_scale=float(rq_inv))
    got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, q.Epilogue(mode=q.OUT_I32))
    assert (as_u32(got) == Z).all()
    # the two halves on their own
    y32 = q.qgtc_aggregate(Ab, m, Xb, q.Epilogue(mode=q.OUT_I32))
    assert (as_u32(y32) == Y).all()
    yb = q.qgtc_aggregate(Ab, m, Xb, agg_ep)
    assert (as_u32(q.qgtc_unpack_bits(yb)) == Yq).all()
    # running twice gives the same bytes (no races)
    again = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, q.Epilogue(mode=q.OUT_I32))
    assert torch.equal(got, again)


# ------------------------------------------------- update on the matrix cores
def test_popcount_probe_runs_and_leaves_its_sink_alone():
    sink = torch.zeros(4, dtype=torch.int32, device="cuda")
    q.qgtc_probe_popcount(64, 4, 10, sink)
    sync()
    assert int(sink.abs().sum()) == 0


@pytest.mark.parametrize("d", [16, 64, 130])
def test_degenerate_graphs(d):
    """Empty tile lists: an adjacency without any edge, one with edges in a single tile
    row only, and isolated nodes with the GIN self term; aggregation and fused layer."""
    rng = np.random.default_rng([13, d])
    n, s, t, h = 200, 4, 3, 24
    Xq = rng.integers(0, 2 ** s, size=(n, d)).astype(np.uint32)
    Wq = rng.integers(0, 2 ** t, size=(d, h)).astype(np.uint32)
    Xb = q.qgtc_pack_bits(dev(Xq.view(np.int32)), s, q.RIGHT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT_BYTES)
    one_row = np.zeros((n, n), dtype=np.uint8)
    one_row[37, [3, 150, 199]] = 1
    for A in (np.zeros((n, n), dtype=np.uint8), one_row):
        for self_term in (False, True):
            Ab = pack_adjacency(A)
            for kb in (128, 32):
                m = q.qgtc_build_tile_map(Ab, 16, kb)
                assert int(m.nnz_tiles.cpu()[0]) == (0 if A.sum() == 0 else len({c // kb for c in (3, 150, 199)}))
                want = qgnn.aggregate(A, Xq, self_term)
                got = q.qgtc_aggregate(Ab, m, Xb, q.Epilogue(mode=q.OUT_I32, self_term=self_term))
                assert (as_u32(got) == want).all(), (self_term, kb)
                Yq = qgnn.requantize(want, 0, np.float32(0.5), s)
                agg_ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=s, rq_lo=0, rq_inv_scale=0.5, self_term=self_term)
                got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, q.Epilogue(mode=q.OUT_I32))
                assert (as_u32(got) == qgnn.update(Yq, Wq)).all(), (self_term, kb)


def test_empty_operands_launch_nothing():
    Ab = q.alloc_bits(0, 64, 1, q.LEFT)
    Xb = q.alloc_bits(64, 16, 2, q.RIGHT)
    out = q.qgtc_aggregate(Ab, None, Xb, q.Epilogue(mode=q.OUT_I32))
    sync()
    assert tuple(out.shape) == (0, 16)
    Yb = q.alloc_bits(0, 64, 2, q.LEFT)
    Wb = q.alloc_bits(64, 8, 2, q.RIGHT)
    out = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_I32))
    sync()
    assert tuple(out.shape) == (0, 8)


@pytest.mark.parametrize("st", [(8, 8), (8, 3), (5, 8), (1, 1)])
@pytest.mark.parametrize("shape", [(100, 64, 64), (257, 130, 16), (70, 40, 5), (1000, 512, 16), (33, 7, 70)])
def test_update_from_bytes(st, shape):
    """Left operand as one byte per code (QGTC_LEFT_BYTES): layout as the header states
    it, zero fill, and the update on it against the oracle in all three output modes."""
    n, d, h = shape
    s, t = st
    rng = np.random.default_rng([12, n, d, h, s, t])
    x = rng.standard_normal((n, d)).astype(np.float32)
    lo, hi = float(x.min()), float(x.max()) + 1e-3
    Yq = qgnn.quantize(x, lo, hi, s)
    Wq = rng.integers(0, 2 ** t, size=(d, h)).astype(np.uint32)
    Yb = q.alloc_bits(n, d, s, q.LEFT_BYTES)
    Yb.words.fill_(-1)
    q.qgtc_pack_bits(dev(x), s, q.LEFT_BYTES, quant=(lo, hi), out=Yb)
    ld = Yb.c.ld_words * 4
    assert ld % 16 == 0 and ld >= d
    raw = Yb.words.cpu().numpy().view(np.uint8)[:n * ld].reshape(n, ld)
    assert (raw[:, :d] == Yq).all() and (raw[:, d:] == 0).all()
    assert (as_u32(q.qgtc_unpack_bits(Yb)) == Yq).all()
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    Z = qgnn.update(Yq, Wq)
    assert (as_u32(q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_I32))) == Z).all()
    inv = qgnn.inv_scale(0.0, float(max(1, Z.max())), 4)
    got = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_BITS, relu=True, rq_nbits=4, rq_lo=1, rq_inv_scale=float(inv)))
    assert (words_np(got) == bp.pack(qgnn.requantize(Z, 1, inv, 4, relu=True), 4, bp.RIGHT)).all()
    got = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_F32, cc=0.37)).cpu().numpy()
    ref = qgnn.dequantize(Z, cc=0.37)
    assert_fp32_close(got, ref, '')


@pytest.mark.parametrize("src", ["f32", "i32", "u8"])
@pytest.mark.parametrize("n,d,pad,skip", [
    (1, 4, 0, 0), (3, 12, 0, 0), (257, 20, 4, 0), (70, 516, 0, 0), (1025, 1040, 8, 0), (4099, 8, 0, 0),   # 16-byte loads
    (257, 20, 3, 0), (70, 21, 0, 0), (33, 64, 0, 1), (1, 3, 0, 0),                       # element by element
])
def test_left_bytes_in_quads_and_element_by_element(src, n, d, pad, skip):
    """Codes as bytes from rows of every alignment: `pad` elements behind each row, `skip` in
    front of the first; padding bytes are zeros."""
    rng = np.random.default_rng([31, n, d, pad, skip])
    flat = rng.standard_normal(skip + n * (d + pad)).astype(np.float32)
    if src == "f32":
        flat[skip] = np.nan
        flat[skip + 1:skip + 3] = [np.inf, -np.inf]
    else:
        flat = rng.integers(0, 256, flat.shape).astype(np.int32 if src == "i32" else np.uint8)
    x = flat[skip:].reshape(n, d + pad)[:, :d]
    t = dev(flat)[skip:].view(n, d + pad)[:, :d]
    if src == "f32":
        ref = qgnn.quantize(np.nan_to_num(x, nan=-9.0, posinf=9.0, neginf=-9.0), -1.5, 2.0, 5)   # NaN: code 0
    else:
        ref = x.astype(np.uint32) & 31
    Yb = q.alloc_bits(n, d, 5, q.LEFT_BYTES)
    Yb.words.fill_(-1)
    q.qgtc_pack_bits(t, 5, q.LEFT_BYTES, quant=(-1.5, 2.0) if src == "f32" else None, out=Yb)
    ld = Yb.c.ld_words * 4
    raw = Yb.words.cpu().numpy().view(np.uint8)[:n * ld].reshape(n, ld)
    assert (raw[:, :d] == ref).all() and (raw[:, d:] == 0).all()


# ------------------------------------------------------------------- fused layer
def _compact_rows(A, block):
    """Block-diagonal storage: row r keeps the columns of its own diagonal block."""
    n = A.shape[0]
    out = np.zeros((n, block), dtype=np.uint8)
    for r in range(n):
        b0 = (r // block) * block
        seg = A[r, b0:b0 + block]
        out[r, :seg.size] = seg
    return out


def _layer_case(rng, n, d, h, s, t, block, self_term, p_edge=0.06):
    A = np.zeros((n, n), dtype=np.uint8)
    if block:
        for b0 in range(0, n, block):
            b1 = min(n, b0 + block)
            A[b0:b1, b0:b1] = rand_graph(rng, b1 - b0, b1 - b0, p_edge)
    else:
        A = rand_graph(rng, n, n, p_edge)
    if self_term:
        A[np.arange(n), np.arange(n)] = 0
    Xq = rng.integers(0, 2 ** s, size=(n, d)).astype(np.uint32)
    Wq = rng.integers(0, 2 ** t, size=(d, h)).astype(np.uint32)
    return A, Xq, Wq


@pytest.mark.parametrize("shape", [(200, 5, 3), (300, 16, 16), (100, 24, 40), (64, 32, 8),
                                   (40, 33, 5), (100, 64, 64), (330, 70, 16), (257, 128, 100),
                                   (530, 200, 256), (96, 512, 16), (200, 600, 40), (64, 1024, 24)])
@pytest.mark.parametrize("st", [(8, 8), (8, 3), (4, 8), (7, 7), (1, 1), (2, 5)])
def test_fused_layer_all_outputs(shape, st):
    """qgtc_layer as one kernel: int32, packed low-bit and fp32 outputs against the
    oracle, and against the same call run as two kernels, for every way of
    splitting the tile lists between waves."""
    n, d, h = shape
    s, t = st
    rng = np.random.default_rng([11, n, d, h, s, t])
    block = 96 if n % 2 == 0 else 0
    self_term = (n + s) % 2 == 0
    A, Xq, Wq = _layer_case(rng, n, d, h, s, t, block, self_term)
    Y = qgnn.aggregate(A, Xq, self_term)
    rq_inv = qgnn.inv_scale(0.0, float(max(1, qgnn.as_signed(Y).max())), s)
    Yq = qgnn.requantize(Y, 0, rq_inv, s)
    Z = qgnn.update(Yq, Wq)

    Xb = q.qgtc_pack_bits(dev(Xq.view(np.int32)), s, q.RIGHT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    Wbytes = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT_BYTES)
    assert (as_u32(q.qgtc_unpack_bits(Wbytes)) == Wq).all()
    assert (as_u32(q.qgtc_col_sums(Wbytes)) == Wq.sum(axis=0, dtype=np.uint64).astype(np.uint32)).all()
    agg_ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=s, rq_lo=0, rq_inv_scale=float(rq_inv),
                        self_term=self_term)
    out_bits = min(s, 6)
    z_inv = qgnn.inv_scale(0.0, float(max(1, qgnn.as_signed(Z).max())), out_bits)
    want_bits = bp.pack(qgnn.requantize(Z, 3, z_inv, out_bits, relu=True), out_bits, bp.RIGHT)
    rl = rng.integers(1, 30, size=n).astype(np.int32)
    cs = Wq.sum(axis=0).astype(np.int32)
    kw = dict(cc=1.7e-3, rs=-0.031, l0a=0.4, l0b=-0.9, ck=-6.4, cs=0.0125)
    want_f32 = qgnn.dequantize(Z, row_i=Yq.sum(axis=1, dtype=np.int64), row_l=rl, col_i=cs, **kw)

    storages = [(pack_adjacency(A), 128), (pack_adjacency(A), None)]
    if block:
        compact = np.zeros((n, block), dtype=np.uint8)
        for r in range(n):
            b0 = (r // block) * block
            seg = A[r, b0:b0 + block]
            compact[r, :seg.size] = seg
        storages.append((q.qgtc_pack_bits(dev(compact), 1, q.LEFT, block_rows=block), 32))
    for Ab, kb in storages:
        m = q.qgtc_build_tile_map(Ab, 16, kb) if kb else None
        for path in (q.LAYER_FUSED, q.LAYER_TWO_KERNELS):
            tn = q.Tuning(layer_path=path)
            tag = (kb, path)
            q.qgtc_prof_enable(True)
            q.qgtc_prof_reset()
            got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, q.Epilogue(mode=q.OUT_I32, tuning=tn))
            fused_launches = q.qgtc_prof_read(q.KERNEL_LAYER)[1]
            q.qgtc_prof_enable(False)
            q.qgtc_prof_reset()
            assert fused_launches == (1 if path == q.LAYER_FUSED else 0), tag
            assert (as_u32(got) == Z).all(), tag
            # weights cached as bytes in operand order: always the fused kernel
            got = q.qgtc_layer(Ab, m, Xb, Wbytes, agg_ep, q.Epilogue(mode=q.OUT_I32, tuning=tn))
            assert (as_u32(got) == Z).all(), tag
            ep = q.Epilogue(mode=q.OUT_BITS, relu=True, rq_nbits=out_bits, rq_lo=3,
                            rq_inv_scale=float(z_inv), tuning=tn)
            # poison the destination: every word, padding included, must be written
            dst = q.alloc_bits(n, h, out_bits, q.RIGHT)
            dst.words.fill_(-1)
            got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, ep, out=dst)
            assert (words_np(got) == want_bits).all(), tag
            ep = q.Epilogue(mode=q.OUT_F32, row_i=None, row_l=dev(rl), col_i=dev(cs), tuning=tn, **kw)
            got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, ep).cpu().numpy()
            assert_fp32_close(got, want_f32, str(tag))


# ------------------------------------------------- folded batch normalization
@pytest.mark.parametrize("shape", [(200, 24, 40), (330, 70, 16), (257, 128, 100), (96, 512, 16), (64, 64, 64)])
@pytest.mark.parametrize("st", [(8, 8), (4, 4), (3, 5), (11, 11)])
def test_column_affine_epilogue(shape, st):
    """A per-column affine map in front of the activation (a batch normalization folded
    into the kernel): low-bit and fp32 outputs of qgtc_aggregate, of both update kernels
    and of qgtc_layer as one and as two kernels, against the oracle."""
    n, d, h = shape
    s, t = st
    rng = np.random.default_rng([29, n, d, h, s, t])
    block = 96 if n % 2 == 0 else 0
    A, Xq, Wq = _layer_case(rng, n, d, h, s, t, block, False)
    Y = qgnn.aggregate(A, Xq)
    rq_bits = min(s, 8)
    y_inv = qgnn.inv_scale(0.0, float(max(1, qgnn.as_signed(Y).max())), rq_bits)
    Yq = qgnn.requantize(Y, 0, y_inv, rq_bits)
    Z = qgnn.update(Yq, Wq)
    out_bits = min(s, 8)

    def bn_params(C, cols, value_scale):
        x = value_scale * qgnn.as_signed(C).astype(np.float64)
        gamma = rng.uniform(0.5, 2.0, size=cols)
        beta = rng.uniform(-1.0, 1.0, size=cols)
        return qgnn.fold_batchnorm(gamma, beta, x.mean(axis=0), x.var(axis=0) + 1e-3, 1e-5, value_scale), \
            qgnn.fold_batchnorm(gamma, beta, x.mean(axis=0), x.var(axis=0) + 1e-3, 1e-5, 1.0)

    Ab = pack_adjacency(A)
    m = q.qgtc_build_tile_map(Ab, 16, 128)
    Xb = q.qgtc_pack_bits(dev(Xq.view(np.int32)), s, q.RIGHT)

    # aggregation: codes along the columns (LEFT) and fp32
    (a, b), (a1, b1) = bn_params(Y, d, 2.0e-3)
    v = qgnn.as_signed(Y) * a[None, :].astype(np.float64) + b[None, :]
    inv = qgnn.inv_scale(0.0, float(max(1e-3, v.max())), out_bits)
    want = qgnn.requantize_affine(Y, a, b, 0, inv, out_bits, relu=True)
    ep = q.Epilogue(mode=q.OUT_BITS, relu=True, rq_nbits=out_bits, rq_lo=0, rq_inv_scale=float(inv),
                    col_scale=dev(a), col_shift=dev(b))
    got = q.qgtc_aggregate(Ab, m, Xb, ep)
    assert (words_np(got) == bp.pack(want, out_bits, bp.LEFT)).all()
    ep = q.Epilogue(mode=q.OUT_F32, cc=2.0e-3, relu=True, col_scale=dev(a1), col_shift=dev(b1))
    got = q.qgtc_aggregate(Ab, m, Xb, ep).cpu().numpy()
    ref = qgnn.dequantize(Y, cc=2.0e-3, relu=True, col_a=a1, col_b=b1)
    assert_fp32_close(got, ref, '')

    # update and layer: codes along the rows (RIGHT) and fp32; the shift may be absent
    (a, b), (a1, b1) = bn_params(Z, h, 1.0e-4)
    v = qgnn.as_signed(Z) * a[None, :].astype(np.float64) + b[None, :]
    inv = qgnn.inv_scale(0.0, float(max(1e-3, v.max())), out_bits)
    want_bits = bp.pack(qgnn.requantize_affine(Z, a, b, 0, inv, out_bits, relu=True), out_bits, bp.RIGHT)
    want_noshift = bp.pack(qgnn.requantize_affine(Z, a, None, 0, inv, out_bits, relu=False), out_bits, bp.RIGHT)
    rs = Yq.sum(axis=1, dtype=np.int64)
    kw = dict(cc=1.0e-4, rs=-2.0e-3)
    want_f32 = qgnn.dequantize(Z, row_i=rs, relu=True, col_a=a1, col_b=b1, **kw)
    ep_bits = q.Epilogue(mode=q.OUT_BITS, relu=True, rq_nbits=out_bits, rq_lo=0, rq_inv_scale=float(inv),
                         col_scale=dev(a), col_shift=dev(b))
    ep_noshift = q.Epilogue(mode=q.OUT_BITS, rq_nbits=out_bits, rq_lo=0, rq_inv_scale=float(inv),
                            col_scale=dev(a))
    Yb = q.qgtc_pack_bits(dev(Yq.view(np.int32)), rq_bits, q.LEFT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    for path in (q.UPDATE_POPCOUNT, q.UPDATE_MATRIX_CORES):
        ep_bits.tuning = ep_noshift.tuning = q.Tuning(update_path=path)
        assert (words_np(q.qgtc_update(Yb, Wb, ep_bits)) == want_bits).all(), path
        assert (words_np(q.qgtc_update(Yb, Wb, ep_noshift)) == want_noshift).all(), path
        ep = q.Epilogue(mode=q.OUT_F32, row_i=dev(rs.astype(np.int32)), relu=True,
                        col_scale=dev(a1), col_shift=dev(b1), tuning=q.Tuning(update_path=path), **kw)
        got = q.qgtc_update(Yb, Wb, ep).cpu().numpy()
        assert_fp32_close(got, want_f32, str(path))
    agg_ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=rq_bits, rq_lo=0, rq_inv_scale=float(y_inv))
    for path in (q.LAYER_FUSED, q.LAYER_TWO_KERNELS):
        ep_bits.tuning = ep_noshift.tuning = q.Tuning(layer_path=path)
        dst = q.alloc_bits(n, h, out_bits, q.RIGHT)
        dst.words.fill_(-1)
        assert (words_np(q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, ep_bits, out=dst)) == want_bits).all(), path
        assert (words_np(q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, ep_noshift)) == want_noshift).all(), path
        ep = q.Epilogue(mode=q.OUT_F32, row_i=None, relu=True, col_scale=dev(a1), col_shift=dev(b1),
                        tuning=q.Tuning(layer_path=path), **kw)
        got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, ep).cpu().numpy()
        assert_fp32_close(got, want_f32, str(path))


@pytest.mark.parametrize("st", [(1, 1), (2, 3), (4, 4), (7, 7), (8, 8), (8, 2), (3, 8), (8, 7)])
@pytest.mark.parametrize("shape", [(100, 64, 64), (257, 128, 16), (70, 40, 5), (1000, 512, 16), (64, 300, 70),
                                   (4096, 64, 64), (33, 16, 130)])
def test_update_matrix_core_path_equals_popcount_and_oracle(st, shape):
    s, t = st
    n, d, h = shape
    rng = np.random.default_rng([11, s, t, n])
    Yq = rng.integers(0, 2 ** s, size=(n, d), dtype=np.uint64).astype(np.uint32)
    Wq = rng.integers(0, 2 ** t, size=(d, h), dtype=np.uint64).astype(np.uint32)
    Yq[0, :] = 2 ** s - 1                      # extreme codes (top bit set at 8 bits)
    Wq[:, 0] = 2 ** t - 1
    Yb = q.qgtc_pack_bits(dev(Yq.view(np.int32)), s, q.LEFT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    Z = qgnn.update(Yq, Wq)
    inv = qgnn.inv_scale(0.0, float(Z.max()), 5)
    rs = Yq.sum(axis=1).astype(np.int32)
    cs = Wq.sum(axis=0).astype(np.int32)
    kw = dict(cc=1.7e-3, rs=-0.031, l0a=0.4, l0b=-0.9, ck=-6.4, cs=0.0125)
    outs = {}
    for path in (q.UPDATE_POPCOUNT, q.UPDATE_MATRIX_CORES):
        tn = q.Tuning(update_path=path)
        z = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_I32, tuning=tn))
        bits = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_BITS, relu=True, rq_nbits=5, rq_lo=0,
                                                rq_inv_scale=float(inv), tuning=tn))
        f = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_F32, row_i=dev(rs), row_l=dev(rs),
                                             col_i=dev(cs), tuning=tn, **kw))
        outs[path] = (as_u32(z), words_np(bits), f.cpu().numpy())
    for path, (z, bits, f) in outs.items():
        assert (z == Z).all(), path
        assert (bits == bp.pack(qgnn.requantize(Z, 0, inv, 5, relu=True), 5, bp.RIGHT)).all(), path
        ref = qgnn.dequantize(Z, row_i=rs, row_l=rs, col_i=cs, **kw)
        assert_fp32_close(f, ref, str(path))


@pytest.mark.parametrize("st", [(4, 4), (8, 8), (3, 8)])
@pytest.mark.parametrize("shape", [(33, 129, 17), (31, 256, 64), (500, 160, 130), (32800, 200, 64), (32768, 256, 33),
                                   (131201, 150, 50), (131073, 256, 64),   # four workgroups per compute unit and more
                                   (30000, 70, 40), (27000, 500, 33), (17000, 300, 64)])   # 16 columns each, and too many of them
def test_update_of_five_to_eight_words_in_slices_of_16_and_64_columns(st, shape):
    """Rows of 5 to 8 words are one super-step, up to a number of rows that depends on the bits; few rows have a workgroup
    per 16 columns, many one per 64."""
    s, t = st
    n, d, h = shape
    rng = np.random.default_rng([12, s, t, n, h])
    Yq = rng.integers(0, 2 ** s, size=(n, d), dtype=np.uint64).astype(np.uint32)
    Wq = rng.integers(0, 2 ** t, size=(d, h), dtype=np.uint64).astype(np.uint32)
    Yb = q.qgtc_pack_bits(dev(Yq.view(np.int32)), s, q.LEFT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    Z = qgnn.update(Yq, Wq)
    tn = q.Tuning(update_path=q.UPDATE_MATRIX_CORES)
    assert (as_u32(q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_I32, tuning=tn))) == Z).all()
    inv = qgnn.inv_scale(0.0, float(Z.max()), 4)
    bits = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_BITS, rq_nbits=4, rq_lo=0, rq_inv_scale=float(inv), tuning=tn))
    assert (words_np(bits) == bp.pack(qgnn.requantize(Z, 0, inv, 4), 4, bp.RIGHT)).all()


# ------------------------------------------------------------ zero-word jumping
@pytest.mark.parametrize("s", [3, 4, 8, 11])
@pytest.mark.parametrize("shape,p_edge", [((300, 64), 0.01), ((300, 64), 0.6), ((130, 20), 0.03), ((257, 130), 0.002),
                                          ((64, 16), 1.0), ((515, 300), 0.0)])
def test_zero_word_jumping_gives_the_same_integers(s, shape, p_edge):
    """Rows and columns of tiles without a bit, every chunk of K taken (no map) and those of the
    list alone (a map of each tile width), stand-alone and inside the fused layer, where stages of
    zeros are left out: the same integers as the oracle.  The hints of qgtc_tuning that describe
    the walk of a tile list change nothing."""
    n, d = shape
    rng = np.random.default_rng([83, s, n, d, int(p_edge * 1000)])
    A = rand_graph(rng, n, n, p_edge)
    if n > 100:
        A[33:70, :] = 0                                     # rows of tiles without a bit
        A[:, 64:160] = 0                                    # whole word columns without a bit
    Xq = rng.integers(0, 2 ** s, size=(n, d), dtype=np.uint64).astype(np.uint32)
    Y = qgnn.aggregate(A, Xq, True)
    Ab = pack_adjacency(A)
    Xb = q.qgtc_pack_bits(dev(Xq.view(np.int32)), s, q.RIGHT)
    h, t = 24, 5
    Wq = rng.integers(0, 2 ** t, size=(d, h)).astype(np.uint32)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    rq_bits = min(s, 8)
    inv = qgnn.inv_scale(0.0, float(max(1, qgnn.as_signed(Y).max())), rq_bits)
    Z = qgnn.update(qgnn.requantize(Y, 0, inv, rq_bits), Wq)
    for kb in (None, 32, 64, 128):
        m = q.qgtc_build_tile_map(Ab, 16, kb) if kb else None
        for tn in (None, q.Tuning(zero_words=q.ZERO_WORDS_SKIP, even_progress=2, layer_ksplit=4)):
            got = q.qgtc_aggregate(Ab, m, Xb, q.Epilogue(mode=q.OUT_I32, self_term=True, tuning=tn))
            assert (as_u32(got) == Y).all(), (kb, tn)
            agg_ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=rq_bits, rq_inv_scale=float(inv), self_term=True)
            got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, q.Epilogue(mode=q.OUT_I32, tuning=tn))
            assert (as_u32(got) == Z).all(), (kb, tn)


@pytest.mark.parametrize("s", [5, 6, 8])
@pytest.mark.parametrize("k_words", [2047, 2048, 2049])
def test_largest_sums_of_long_rows(s, k_words):
    """Rows of ones against columns of the largest code, beside sparse rows, over 65504 to 65568
    positions of K: the sums of codes less 128 (8 bits) and 128 x the bits of the row that is added
    back are at their largest, with the last chunk whole and in part, and with all chunks taken
    and those of the list."""
    k = 32 * k_words
    n, d, h, t = 40, 20, 24, 4
    rng = np.random.default_rng([97, s, k_words])
    A = (rng.random((n, k)) < 0.002).astype(np.uint8)
    A[3, :] = 1
    A[12, :] = 1
    A[27, :] = 1
    A[21, : k // 2] = 1
    A[16:20, :] = 0
    Xq = rng.integers(0, 2 ** s, size=(k, d), dtype=np.uint64).astype(np.uint32)
    Xq[:, 0] = 2 ** s - 1                                   # every plane: a count of k
    Xq[:, 7] = 2 ** (s - 1)
    Y = qgnn.aggregate(A, Xq, False)
    assert Y[12, 0] == k * (2 ** s - 1)
    Wq = rng.integers(0, 2 ** t, size=(d, h)).astype(np.uint32)
    inv = qgnn.inv_scale(0.0, float(Y.max()), s)
    Z = qgnn.update(qgnn.requantize(Y, 0, inv, s), Wq)
    Ab = pack_adjacency(A)
    Xb = q.qgtc_pack_bits(dev(Xq.view(np.int32)), s, q.RIGHT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    for kb in (None, 32, 64, 128):
        m = q.qgtc_build_tile_map(Ab, 16, kb) if kb else None
        got = q.qgtc_aggregate(Ab, m, Xb, q.Epilogue(mode=q.OUT_I32))
        assert (as_u32(got) == Y).all(), kb
        agg_ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=s, rq_inv_scale=float(inv))
        got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, q.Epilogue(mode=q.OUT_I32))
        assert (as_u32(got) == Z).all(), kb


# ------------------------------------------------------------ seeded random shapes
@pytest.mark.parametrize("seed", range(48))
def test_layer_on_random_shapes(seed):
    """qgtc_layer on shapes and bit widths drawn from a seeded generator (single rows and
    columns, ragged tails, widths above 8 bits that leave the fused kernel, every storage
    and tile width), int32 and low-bit outputs against the oracle."""
    rng = np.random.default_rng([61, seed])
    n = int(rng.choice([1, 2, 15, 16, 17, 31, 33, 64, 100, 129, 255, 400]))
    d = int(rng.choice([1, 2, 7, 16, 17, 32, 33, 63, 64, 65, 130, 260]))
    h = int(rng.choice([1, 3, 15, 16, 17, 40, 64, 100, 256, 260]))
    s = int(rng.choice([1, 2, 3, 5, 8, 8, 8, 9, 12]))
    t = int(rng.choice([1, 2, 4, 7, 8, 8, 10]))
    block = int(rng.choice([0, 0, 32, 64, 96]))
    kb = [None, 32, 64, 128][int(rng.integers(0, 4))]
    self_term = bool(rng.integers(0, 2))
    A, Xq, Wq = _layer_case(rng, n, d, h, s, t, block, self_term, p_edge=float(rng.choice([0.0, 0.02, 0.3])))
    Y = qgnn.aggregate(A, Xq, self_term)
    rq_bits = min(s, int(rng.choice([s, 8, 4])))
    rq_inv = qgnn.inv_scale(0.0, float(max(1, qgnn.as_signed(Y).max())), rq_bits)
    Yq = qgnn.requantize(Y, 0, rq_inv, rq_bits)
    Z = qgnn.update(Yq, Wq)
    out_bits = int(rng.choice([1, 3, 8, min(s, 8)]))
    z_inv = qgnn.inv_scale(0.0, float(max(1, qgnn.as_signed(Z).max())), out_bits)
    want_bits = bp.pack(qgnn.requantize(Z, 1, z_inv, out_bits, relu=True), out_bits, bp.RIGHT)

    if block:
        Ab = q.qgtc_pack_bits(dev(_compact_rows(A, block)), 1, q.LEFT, block_rows=block)
    else:
        Ab = pack_adjacency(A)
    m = q.qgtc_build_tile_map(Ab, 16, kb) if kb else None
    Xb = q.qgtc_pack_bits(dev(Xq.view(np.int32)), s, q.RIGHT)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    agg_ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=rq_bits, rq_lo=0, rq_inv_scale=float(rq_inv),
                        self_term=self_term)
    tag = dict(n=n, d=d, h=h, s=s, t=t, block=block, kb=kb, self_term=self_term, rq_bits=rq_bits, out_bits=out_bits)
    got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, q.Epilogue(mode=q.OUT_I32))
    assert (as_u32(got) == Z).all(), tag
    ep = q.Epilogue(mode=q.OUT_BITS, relu=True, rq_nbits=out_bits, rq_lo=1, rq_inv_scale=float(z_inv))
    dst = q.alloc_bits(n, h, out_bits, q.RIGHT)
    dst.words.fill_(-1)
    got = q.qgtc_layer(Ab, m, Xb, Wb, agg_ep, ep, out=dst)
    assert (words_np(got) == want_bits).all(), tag
    if s <= 8 and t <= 8 and d <= 1024 and h <= 256:            # weights as bytes: the fused kernel only
        Wby = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT_BYTES)
        got = q.qgtc_layer(Ab, m, Xb, Wby, agg_ep, q.Epilogue(mode=q.OUT_I32))
        assert (as_u32(got) == Z).all(), tag


@pytest.mark.parametrize("seed", range(40))
def test_aggregate_and_update_on_random_shapes(seed):
    """qgtc_aggregate and qgtc_update by themselves on seeded random shapes and bit widths
    up to 32 (results modulo 2^32), every output mode, against the oracle."""
    rng = np.random.default_rng([67, seed])
    n = int(rng.choice([1, 5, 16, 31, 48, 65, 128, 200, 333]))
    k = n
    d = int(rng.choice([1, 3, 16, 20, 32, 50, 64, 70, 129, 300]))
    h = int(rng.choice([1, 2, 15, 16, 33, 64, 90]))
    s = int(rng.choice([1, 2, 4, 7, 8, 9, 13, 16, 24, 32]))
    t = int(rng.choice([1, 3, 8, 8, 11, 16, 32]))
    self_term = bool(rng.integers(0, 2))
    kb = [None, 32, 64, 128][int(rng.integers(0, 4))]
    A = rand_graph(rng, n, k, float(rng.choice([0.0, 0.05, 0.5])))
    Xq = rng.integers(0, 2 ** s, size=(k, d), dtype=np.uint64).astype(np.uint32)
    tag = dict(n=n, d=d, h=h, s=s, t=t, self_term=self_term, kb=kb)
    Y = qgnn.aggregate(A, Xq, self_term)
    Ab = pack_adjacency(A)
    m = q.qgtc_build_tile_map(Ab, 16, kb) if kb else None
    Xb = q.qgtc_pack_bits(dev(Xq.view(np.int32)), s, q.RIGHT)
    got = q.qgtc_aggregate(Ab, m, Xb, q.Epilogue(mode=q.OUT_I32, self_term=self_term))
    assert (as_u32(got) == Y).all(), tag
    rq_bits = int(rng.choice([1, 4, 8, 12]))
    hi = float(max(1, qgnn.as_signed(Y).max()))
    inv = qgnn.inv_scale(0.0, hi, rq_bits)
    Yq = qgnn.requantize(Y, 0, inv, rq_bits, relu=True)
    ep = q.Epilogue(mode=q.OUT_BITS, relu=True, rq_nbits=rq_bits, rq_lo=0, rq_inv_scale=float(inv),
                    self_term=self_term)
    Yb = q.qgtc_aggregate(Ab, m, Xb, ep)
    assert (words_np(Yb) == bp.pack(Yq, rq_bits, bp.LEFT)).all(), tag
    got = q.qgtc_aggregate(Ab, m, Xb, q.Epilogue(mode=q.OUT_F32, cc=0.013, self_term=self_term)).cpu().numpy()
    ref = qgnn.dequantize(Y, cc=0.013)
    assert_fp32_close(got, ref, str(tag))

    Wq = rng.integers(0, 2 ** t, size=(d, h), dtype=np.uint64).astype(np.uint32)
    Z = qgnn.update(Yq, Wq)
    Wb = q.qgtc_pack_bits(dev(Wq.view(np.int32)), t, q.RIGHT)
    got = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_I32, relu=True))
    assert (as_u32(got) == qgnn.int_output(Z, relu=True).view(np.uint32)).all(), tag
    out_bits = int(rng.choice([1, 5, 8, 16]))
    z_inv = qgnn.inv_scale(0.0, float(max(1, qgnn.as_signed(Z).max())), out_bits)
    got = q.qgtc_update(Yb, Wb, q.Epilogue(mode=q.OUT_BITS, rq_nbits=out_bits, rq_lo=0, rq_inv_scale=float(z_inv)))
    assert (words_np(got) == bp.pack(qgnn.requantize(Z, 0, z_inv, out_bits), out_bits, bp.RIGHT)).all(), tag


# ------------------------------------------------------------------ long rows: features as codes
@pytest.mark.parametrize("n,k,d,s,block,density,codes", [
    (8200, 2049, 257, 8, 0, 0.3, True),        # floats: 17 chunks of K, the last one of a column; odd rows
    (8200, 2048, 257, 8, 0, 0.3, False),
    (16400, 2500, 33, 3, 0, 0.01, True),       # floats
    (8200, 2561, 70, 8, 0, 0.01, True),        # floats
    (700, 8193, 17, 8, 0, 0.3, True),          # bytes: four waves share a stage
    (65, 8192, 1, 1, 0, 0.5, False),
    (65, 11000, 1, 1, 0, 0.5, True),           # floats
    (4 * 2560 + 100, 2560, 100, 8, 2560, 0.002, True),   # floats
    (700, 8193, 16, 8, 0, 0.3, 257 * 512),     # bytes (their room): four waves share a stage
    (65, 11000, 5, 5, 0, 0.5, 344 * 512),
    (33000, 2561, 16, 8, 0, 0.05, 81 * 512),   # one wave of 16 columns
    (6600, 65900, 150, 8, 0, 0.01, 2060 * 512 * 10),     # two of them; sums of 2^24 and more
    (8200, 2500, 256, 8, 0, 0.01, True),       # two of 32; more than a round of workgroups of floats
])
@pytest.mark.parametrize("with_map", [False, True])
def test_aggregation_of_long_rows(n, k, d, s, block, density, codes, with_map):
    """Against int64 products of the same integers (below 2^31), and planes against codes for packed results."""
    import ctypes as C
    import paper_2111_09547_amd.binding as B
    gen = torch.Generator(device="cuda").manual_seed(n + k)
    a = (torch.rand((n, k), generator=gen, device="cuda") < density).to(torch.uint8)
    a[:, k // 3:k // 3 + 700] = 0                                  # chunks without a bit
    if block:
        a[n // block * block:, n % block:] = 0
    x = torch.randint(0, 1 << s, (n if block else k, d), generator=gen, device="cuda", dtype=torch.int32)
    A, X = q.qgtc_pack_bits(a, 1, q.LEFT, block_rows=block), q.qgtc_pack_bits(x, s, q.RIGHT)
    tmap = q.qgtc_build_tile_map(A, 16, 128) if with_map else None
    nbytes = B.lib().qgtc_aggregate_workspace_bytes(C.byref(A.c), C.byref(X.c))
    assert (nbytes > 0) == codes if isinstance(codes, bool) else nbytes == codes
    parts = [slice(r, min(r + block, n)) for r in range(0, n, block)] if block else [slice(0, n)]
    want = torch.cat([a[p, :p.stop - p.start if block else k].double() @ (x[p] if block else x).double() for p in parts]).to(torch.int32)
    square = block > 0
    if square:
        self_ep = q.Epilogue(mode=q.OUT_I32, self_term=True)
        assert torch.equal(q.qgtc_aggregate(A, tmap, X, self_ep), want + x)
    assert torch.equal(q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32)), want)
    ep = q.Epilogue(mode=q.OUT_BITS, rq_nbits=s, rq_lo=0, rq_inv_scale=qgnn.inv_scale(0.0, float(want.max()) + 1, s))
    got, planes = q.qgtc_aggregate(A, tmap, X, ep), B.alloc_bits(n, d, s, q.LEFT)
    e = ep.to_c()
    B._check(B.lib().qgtc_aggregate(C.byref(A.c), C.byref(tmap.c) if tmap else None, C.byref(X.c), C.byref(e), C.byref(planes.c), 0,
                                    B._stream()), "qgtc_aggregate")
    assert torch.equal(q.qgtc_unpack_bits(got), q.qgtc_unpack_bits(planes))
    if with_map:                                                   # the room is the graph's
        out = torch.empty_like(want)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32), out=out)
        for _ in range(3):
            out.zero_()
            graph.replay()
            assert torch.equal(q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32)), want)
            assert torch.equal(out, want)


@pytest.mark.parametrize("n,k,d,block,forms", [
    # forms of X at 1 and 2, 3 and 4, 5 to 8 bits: floats, bytes, planes
    (1030, 8193, 65, 0, "fbb"),    # 65 chunks, the last one of a column; three column groups, the last one of a column
    (1024, 4609, 64, 0, "ppp"),    # few workgroups
    (1024, 7169, 20, 0, "ffp"),    # 32 rows per workgroup
    (1024, 65664, 33, 0, "fbf"),
    (1025, 65792, 17, 0, "fff"),
    (2065, 65792, 500, 0, "fff"),  # sums up to the last exact ones at 8 bits
    (40 * 256 + 1, 8300, 250, 0, "fff"),
    (20 * 256 - 31, 8300, 130, 0, "fff"),
    (20 * 256 - 31, 8300, 40, 0, "fff"),
    (8300, 8300, 40, 0, "fff"),    # 128 rows per workgroup at 5 to 8 bits
    # up to 32 columns: 64, 128 and 256 rows per workgroup
    (8300, 7200, 20, 0, "ffp"),
    (16500, 2100, 20, 0, "fff"),
    (33000, 2100, 30, 0, "fff"),
    # more: 32, 64, 128 and 256 rows (5 to 8 bits: 256 at 16500 rows)
    (7000, 4700, 40, 0, "ffp"),
    (8300, 4700, 40, 0, "ffp"),
    (16500, 4700, 40, 0, "fff"),
    (33000, 2100, 40, 0, "fff"),
    (2 * 8224 + 33, 8224, 70, 8224, "fff"),   # diagonal blocks, the last one of two words of rows
])
@pytest.mark.parametrize("s", [1, 2, 3, 4, 5, 8])
def test_aggregation_on_small_floats_is_exact(n, k, d, block, forms, s):
    """Products of 4- and 6-bit floats against float64: whole tiles of ones and of the largest code, rows and chunks of
    zeros, the self term, with and without a map that leaves chunks out."""
    import ctypes as C
    import paper_2111_09547_amd.binding as B
    gen = torch.Generator(device="cuda").manual_seed(n + s)
    a = (torch.rand((n, k), generator=gen, device="cuda") < 0.4).to(torch.uint8)
    a[:40] = 1
    a[100:140] = 0
    a[64:, k // 2:k // 2 + 1100] = 0
    if block:
        a[n // block * block:, n % block:] = 0
    x = torch.randint(0, 1 << s, (n if block else k, d), generator=gen, device="cuda", dtype=torch.int32)
    x[:, :9] = (1 << s) - 1
    A, X = q.qgtc_pack_bits(a, 1, q.LEFT, block_rows=block), q.qgtc_pack_bits(x, s, q.RIGHT)
    words, form = -(-x.shape[0] // 32), forms[0 if s <= 2 else 1 if s <= 4 else 2]
    room = {"f": words * -(-d // 32) * 32 * (16 if s <= 2 else (24 if s <= 4 else 48)), "b": words * -(-d // 16) * 512, "p": 0}[form]
    assert B.lib().qgtc_aggregate_workspace_bytes(C.byref(A.c), C.byref(X.c)) == room
    parts = [slice(r, min(r + block, n)) for r in range(0, n, block)] if block else [slice(0, n)]
    want = torch.cat([a[p, :p.stop - p.start if block else k].double() @ (x[p] if block else x).double() for p in parts]).to(torch.int32)
    for tmap in (None, q.qgtc_build_tile_map(A, 16, 128)):
        assert torch.equal(q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32)), want)
        if block:
            assert torch.equal(q.qgtc_aggregate(A, tmap, X, q.Epilogue(mode=q.OUT_I32, self_term=True)), want + x)


@pytest.mark.parametrize("n,k,d,s,block", [
    (1030, 8193, 65, 2, 0),        # 4-bit floats, the last columns alone, a row of workgroups of six rows
    (8300, 4700, 42, 4, 0),        # 6-bit floats
    (16500, 2100, 30, 8, 0),       # two parts of 6 bits
    (8210, 8210, 44, 3, 0),        # square, no multiple of 32, with the self term
    (4 * 2304 + 40, 2304, 72, 1, 2304),
])
def test_outputs_of_long_rows(n, k, d, s, block):
    """Every output of the products of floats against the same call without room, which takes planes: int32, fp32 with all
    row and column terms, into whole and into odd strides, and codes of 12 bits with padding to be cleared.  Both form the
    same expression of the same integers, so that the results are the same bits."""
    import ctypes as C
    import paper_2111_09547_amd.binding as B
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    a = (torch.rand((n, k), generator=gen, device="cuda") < 0.1).to(torch.uint8)
    a[:, k // 3:k // 3 + 900] = 0
    if block:
        a[n // block * block:, n % block:] = 0
    x = torch.randint(0, 1 << s, (n if block else k, d), generator=gen, device="cuda", dtype=torch.int32)
    A, X = q.qgtc_pack_bits(a, 1, q.LEFT, block_rows=block), q.qgtc_pack_bits(x, s, q.RIGHT)
    nbytes = B.lib().qgtc_aggregate_workspace_bytes(C.byref(A.c), C.byref(X.c))
    assert nbytes == -(-x.shape[0] // 32) * -(-d // 32) * 32 * (16 if s <= 2 else (24 if s <= 4 else 48))
    room = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    tmap = q.qgtc_build_tile_map(A, 16, 128)

    def both(ep, made):
        """made: a fresh output, as (what to compare, pointer, leading dimension)"""
        out = []
        for ws, size in ((None, 0), (room.data_ptr(), nbytes)):
            res, ptr, ld = made()
            B._check(B.lib().qgtc_aggregate_ws(C.byref(A.c), C.byref(tmap.c), C.byref(X.c), C.byref(ep.to_c()), ws, size, ptr, ld, B._stream()),
                     "qgtc_aggregate_ws")
            out.append(res)
        assert torch.equal(*out)
        return out[1]

    def strided(ld, first):
        def made():
            res = torch.full((n, ld), -7, dtype=torch.int32, device="cuda")
            return res, res.data_ptr() + 4 * first, ld
        return made

    ints = lambda m: torch.randint(0, 1000, (m,), generator=gen, device="cuda", dtype=torch.int32)
    reals = lambda m: torch.randn(m, generator=gen, device="cuda")
    square = block > 0 or n == k
    whole = -(-d // 4) * 4 + 4
    for self_term in (False, True) if square else (False,):
        got = both(q.Epilogue(mode=q.OUT_I32, self_term=self_term), strided(d + 3, 1))
        want = torch.cat([a[r:r + (block or n), :min(block, n - r) if block else k].double() @ (x[r:r + block] if block else x).double()
                          for r in range(0, n, block or n)])
        assert torch.equal(got[:, 1:1 + d], want.to(torch.int32) + (x if self_term else 0)) and bool((got[:, 0] == -7).all())
        both(q.Epilogue(mode=q.OUT_I32, relu=True, self_term=self_term), strided(whole, 0))
        terms = dict(cc=0.013, rs=-0.7, l0a=0.25, l0b=0.5, ck=3.0, cs=0.125, row_i=ints(n), row_l=ints(n), col_i=ints(d))
        affine = dict(col_scale=reals(d), col_shift=reals(d))
        for extra in ({}, terms, {**terms, **affine, "relu": True}):
            for made in (strided(whole, 0), strided(d + 1 + (d & 1), 0), strided(whole, 3)):
                got = both(q.Epilogue(mode=q.OUT_F32, self_term=self_term, **{"cc": 0.013, **extra}), made)
                assert len(got.unique()) > 20
        words = -(-d // 32)

        def planes(nbits, ld):
            def made():
                res = B.alloc_bits(n, d, nbits, q.LEFT, ld_words=ld)
                res.words.fill_(-1)
                made.keep = res                                     # (its descriptor is read by the call)
                return res.words, C.cast(C.pointer(res.c), C.c_void_p), 0
            return made
        inv = qgnn.inv_scale(0.0, float(want.max()) + (1 << s), 12)
        for nbits, ld in ((12, words + 3), (16, words), (8, words + 1)):
            both(q.Epilogue(mode=q.OUT_BITS, self_term=self_term, relu=True, rq_nbits=nbits, rq_lo=2, rq_inv_scale=inv, **affine), planes(nbits, ld))


def test_aggregation_with_less_room_than_it_asks_for():
    """Room for X as bytes is enough where floats would be taken, and room that nothing fits in is not used where the
    product goes without; too little for bytes, or misaligned, stays refused where bytes are what room is for."""
    import ctypes as C
    import paper_2111_09547_amd.binding as B
    OK, ALIGN, WORKSPACE = 0, 4, 6
    room = torch.empty((1 << 21) + 16, dtype=torch.uint8, device="cuda")
    as_bytes = 260 * 512 * 9                                       # (5089, 8300, 130) in groups of 16 columns
    for n, k, d, s, calls in [
        (5089, 8300, 130, 8, [(as_bytes, 0, OK), (as_bytes - 1, 0, WORKSPACE), (1 << 21, 4, ALIGN)]),
        (7000, 4700, 40, 2, [(16, 0, OK), (1 << 20, 4, OK)]),
        (1024, 7169, 20, 4, [(1 << 15, 0, OK)]),
    ]:
        gen = torch.Generator(device="cuda").manual_seed(n + k)
        a = (torch.rand((n, k), generator=gen, device="cuda") < 0.4).to(torch.uint8)
        x = torch.randint(0, 1 << s, (k, d), generator=gen, device="cuda", dtype=torch.int32)
        A, X = q.qgtc_pack_bits(a, 1, q.LEFT), q.qgtc_pack_bits(x, s, q.RIGHT)
        want = (a.double() @ x.double()).to(torch.int32)
        ep = q.Epilogue(mode=q.OUT_I32).to_c()
        assert B.lib().qgtc_aggregate_workspace_bytes(C.byref(A.c), C.byref(X.c)) > calls[0][0]
        for nbytes, offset, status in calls:
            out = torch.full((n, d), -1, dtype=torch.int32, device="cuda")
            got = B.lib().qgtc_aggregate_ws(C.byref(A.c), None, C.byref(X.c), C.byref(ep), room.data_ptr() + offset, nbytes, out.data_ptr(), d, B._stream())
            assert got == status, (n, k, d, s, nbytes, offset)
            assert status != OK or torch.equal(out, want)


@pytest.mark.parametrize("s", [1, 3, 4, 5, 8])
@pytest.mark.parametrize("n,d", [(1, 1), (3, 33), (300, 64), (70000, 31), (33000, 132)])
def test_left_planes_are_decoded_four_columns_at_a_time(n, d, s):
    """Into rows of whole and of odd widths, one and four items per thread."""
    import ctypes as C
    import paper_2111_09547_amd.binding as B
    v = torch.randint(0, 1 << s, (n, d), device="cuda", dtype=torch.int32)
    bits = q.qgtc_pack_bits(v, s, q.LEFT)
    assert torch.equal(q.qgtc_unpack_bits(bits), v)
    ld = -(-d // 4) * 4 + 4
    wide = torch.full((n, ld), -1, device="cuda", dtype=torch.int32)
    B._check(B.lib().qgtc_unpack_bits(C.byref(bits.c), C.c_void_p(wide.data_ptr()), ld, B._stream()), "qgtc_unpack_bits")
    assert torch.equal(wide[:, :d], v) and bool((wide[:, d:] == -1).all())
