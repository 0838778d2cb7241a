"""The paper's PyTorch-level names (Section 5) against the oracle: to_bit / to_val round
trip and Eq. (2), bitMM2Int and bitMM2Bit for a binary and for a multi-bit left operand."""
import numpy as np
import pytest
import torch

from oracle import qgnn, bitplane as bp

pytestmark = pytest.mark.gpu

q = pytest.importorskip("paper_2111_09547_amd")
import paper_2111_09547_amd.binding as B  # noqa: E402
from paper_2111_09547_amd.bit_tensor import (BitTensor, to_bit, to_val, bitMM2Int, bitMM2Bit,  # noqa: E402
                                             calibrate_inv_scale, enable_tensor_methods)
from gpu_util import dev, as_u32, words_np  # noqa: E402


@pytest.mark.parametrize("bits", [1, 3, 8, 13])
def test_to_bit_and_back(bits):
    rng = np.random.default_rng([71, bits])
    v = rng.integers(0, 2 ** bits, size=(77, 45)).astype(np.int32)
    for side in ("left", "right"):
        assert (to_val(to_bit(dev(v), bits, side=side)).cpu().numpy() == v).all()
    x = rng.normal(size=(60, 33)).astype(np.float32)
    got = to_val(to_bit(dev(x), bits)).cpu().numpy()                 # min-max by default
    assert (got.view(np.uint32) == qgnn.quantize(x, float(x.min()), float(x.max()), bits)).all()
    got = to_val(to_bit(dev(x), bits, quant=(-1.0, 2.5))).cpu().numpy()
    assert (got.view(np.uint32) == qgnn.quantize(x, -1.0, 2.5, bits)).all()


@pytest.mark.parametrize("sa,sb", [(1, 4), (1, 8), (3, 5), (8, 8), (2, 11)])
def test_bit_products(sa, sb):
    rng = np.random.default_rng([72, sa, sb])
    m, k, n = 150, 96, 40
    L = rng.integers(0, 2 ** sa, size=(m, k)).astype(np.uint32)
    R = rng.integers(0, 2 ** sb, size=(k, n)).astype(np.uint32)
    Lb = to_bit(dev(L.view(np.int32)), sa, side="left")
    Rb = to_bit(dev(R.view(np.int32)), sb, side="right")
    C = qgnn.matmul_mod32(L, R)
    assert (as_u32(bitMM2Int(Lb, Rb)) == C).all()
    bit_c = 5
    inv = qgnn.inv_scale(0.0, float(max(1, qgnn.as_signed(C).max())), bit_c)
    want = qgnn.requantize(C, 0, inv, bit_c)
    layout = bp.LEFT if sa == 1 else bp.RIGHT        # next left operand after an aggregation, next X after an update
    assert calibrate_inv_scale(Lb, Rb, bit_c) == float(inv)          # the range found from the data
    got = bitMM2Bit(Lb, Rb, bit_c, inv_scale=float(inv))
    assert isinstance(got, BitTensor) and got.nbits == bit_c and got.shape == (m, n)
    assert got.side == ("left" if sa == 1 else "right") and got.storage.dtype == torch.int32
    assert (words_np(got.bits) == bp.pack(want, bit_c, layout)).all()
    assert (got.to_val().cpu().numpy().view(np.uint32) == want).all()


def test_tensor_methods_as_the_paper_writes_them():
    """Section 5: Tensor.to_bit(nbits) gives a bit-Tensor, .to_val() decodes it."""
    enable_tensor_methods()
    rng = np.random.default_rng(73)
    x = rng.normal(size=(50, 20)).astype(np.float32)
    xb = dev(x).to_bit(3)
    assert isinstance(xb, BitTensor) and xb.nbits == 3 and xb.side == "right"
    assert (xb.to_val().cpu().numpy().view(np.uint32) == qgnn.quantize(x, float(x.min()), float(x.max()), 3)).all()
    a = (rng.random((50, 50)) < 0.1).astype(np.uint8)
    ab = dev(a).to_bit(1, side="left")
    assert ab.is_adjacency()
    assert (as_u32(bitMM2Int(ab, xb)) == qgnn.aggregate(a, qgnn.quantize(x, float(x.min()), float(x.max()), 3))).all()


@pytest.mark.parametrize("d", [64, 100, 128])
def test_one_bit_layer_chained_through_the_products(d):
    """Aggregate, requantize to ONE bit, update: the 1-bit result of bitMM2Bit is a left
    operand without the 128-bit row padding of an adjacency (d = 64: two words per row), so
    the second product must run as an update, not as an aggregation."""
    rng = np.random.default_rng([74, d])
    n, h, t = 130, 24, 3
    A = (rng.random((n, n)) < 0.08).astype(np.uint8)
    Xq = rng.integers(0, 2, size=(n, d)).astype(np.uint32)
    Wq = rng.integers(0, 2 ** t, size=(d, h)).astype(np.uint32)
    Y = qgnn.aggregate(A, Xq)
    inv = qgnn.inv_scale(0.0, float(max(1, Y.max())), 1)
    Yq = qgnn.requantize(Y, 0, inv, 1)
    Z = qgnn.update(Yq, Wq)
    Ab = to_bit(dev(A), 1, side="left")
    Xb = to_bit(dev(Xq.view(np.int32)), 1, side="right")
    Wb = to_bit(dev(Wq.view(np.int32)), t, side="right")
    Yb = bitMM2Bit(Ab, Xb, 1, inv_scale=float(inv))
    assert Yb.nbits == 1 and Yb.side == "left" and (Yb.to_val().cpu().numpy().view(np.uint32) == Yq).all()
    assert Yb.is_adjacency() == (Yb.bits.c.ld_words % 4 == 0 and Yb.bits.c.data % 16 == 0)
    assert (as_u32(bitMM2Int(Yb, Wb)) == Z).all()
    # the same 1-bit result written into a padded destination is a valid adjacency operand
    dst = q.alloc_bits(n, d, 1, q.LEFT)
    dst.words.fill_(-1)
    q.qgtc_aggregate(Ab.bits, None, Xb.bits, q.Epilogue(mode=q.OUT_BITS, rq_nbits=1, rq_inv_scale=float(inv)), out=dst)
    padded = BitTensor(dst)
    assert padded.is_adjacency()
    assert (as_u32(bitMM2Int(padded, Wb)) == Z).all()


def test_product_builds_no_map_that_nobody_reads(monkeypatch):
    """Operands whose rows are one stage of the aggregation: two launches and an allocation less;
    longer rows still get a map, and the integers are the product's either way."""
    import paper_2111_09547_amd.bit_tensor as bt
    built = []
    real = bt.B.qgtc_build_tile_map
    monkeypatch.setattr(bt.B, "qgtc_build_tile_map", lambda *a, **k: built.append(a) or real(*a, **k))
    rng = np.random.default_rng(11)
    for n, d, want in ((256, 16, False), (100, 3, False), (257, 16, False), (1024, 16, False), (1025, 16, True), (3000, 16, True), (2100, 300, True)):
        a = (rng.random((n, n)) < 0.03).astype(np.uint8)
        x = rng.integers(0, 4, (n, d)).astype(np.int32)
        A, X = to_bit(dev(a), 1, side="left"), to_bit(dev(x), 2)
        built.clear()
        y = bitMM2Int(A, X)
        assert bool(built) == want == bt.B.qgtc_aggregate_reads_map(A.bits, d), (n, d)
        assert (as_u32(y) == qgnn.aggregate(a, x.astype(np.uint32))).all()


@pytest.mark.parametrize("t", [1, 5, 8])
@pytest.mark.parametrize("shapes", [[(1, 1)], [(64, 16), (65, 17), (300, 101), (512, 16)], [(16 + i, 70 - i) for i in range(19)]])
def test_weights_of_a_stack_in_one_launch(t, shapes):
    """As qgtc_pack_bits of each, also more than one launch takes; the column sums of any one of them."""
    rng = np.random.default_rng(t + len(shapes))
    Ws = [torch.from_numpy(rng.uniform(-0.5, 0.5, s).astype(np.float32)).cuda() for s in shapes]
    ranges = [(-0.4, 0.45 + 0.01 * i) for i in range(len(Ws))]
    want = [q.qgtc_pack_bits(W, t, q.RIGHT_BYTES, quant=r) for W, r in zip(Ws, ranges)]
    outs = [B.alloc_bits(*s, t, q.RIGHT_BYTES) for s in shapes]
    sources = B.WeightSources(Ws, ranges, outs)
    for k in {0, len(Ws) // 2, len(Ws) - 1}:
        sums = torch.full((shapes[k][1] + 3,), -7, dtype=torch.int32, device="cuda")
        B.qgtc_pack_weights(sources, k, sums)
        assert torch.equal(sums[:-3], q.qgtc_col_sums(want[k])) and (sums[-3:] == -7).all()
    for got, ref in zip(outs, want):
        assert torch.equal(got.words, ref.words)
    B.qgtc_pack_weights(sources)
    with pytest.raises(q.QgtcError):
        B.qgtc_pack_weights(sources, len(Ws), sums)


@pytest.mark.parametrize("n,d,pitch,layers", [(1, 4, 4, 1), (129, 64, 64, 3), (1000, 128, 132, 16), (77, 100, 101, 2), (77, 101, 101, 2), (300, 64, 64, 17)])
@pytest.mark.parametrize("t", [3, 8])
def test_features_and_weights_in_one_launch(n, d, pitch, layers, t):
    """As the two calls, where one launch takes both and where it does not (odd columns or pitch, many weights)."""
    rng = np.random.default_rng(n + d)
    x = torch.from_numpy(rng.uniform(-1, 1, (n, pitch)).astype(np.float32)).cuda()[:, :d]
    Ws = [torch.from_numpy(rng.uniform(-0.5, 0.5, (d + i, 16 + i)).astype(np.float32)).cuda() for i in range(layers)]
    ranges = [(-0.4, 0.45 + 0.01 * i) for i in range(layers)]
    outs = [[B.alloc_bits(*W.shape, t, q.RIGHT_BYTES) for W in Ws] for _ in range(2)]
    buffers = [torch.full((B.lib().qgtc_stack_buffer_bytes(n, d) // 4,), 5, dtype=torch.int32, device="cuda") for _ in range(2)]
    sums = [torch.full((Ws[-1].shape[1] + 3,), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
    B.qgtc_pack_weights(B.WeightSources(Ws, ranges, outs[0]), layers - 1, sums[0])
    B.qgtc_stack_input(x, t, (-0.9, 0.8), buffers[0], rows_form=True)
    B.qgtc_stack_input(x, t, (-0.9, 0.8), buffers[1], rows_form=True, weights=(B.WeightSources(Ws, ranges, outs[1]), layers - 1, sums[1]))
    assert torch.equal(*buffers) and torch.equal(*sums)
    for a, b in zip(*outs):
        assert torch.equal(a.words, b.words)
