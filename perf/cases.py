"""The workloads this framework's speed is judged by, each as a user's program runs it.

A case says what is run, on which graph, with which layer widths, bit widths and options.
The sizes are those of the benchmark configurations (workloads/configs.py), of the sweeps
and of the tests; draw() spreads further cases over the same ranges.  Kinds of work:

  net      a stack of quantized layers (QuantGNN) on one batch of subgraphs.  `mode`:
             graph   features in, fp32 out, recorded once as a HIP graph and replayed (a server
                     whose adjacency and weights stay)
             step    the same with everything in front of it - packing the adjacency, its
                     zero-tile map, packing the weights - inside the graph (bench.py's step)
             eager   forward() as a script calls it, launch by launch
             batch   mini-batch inference without a graph: each batch brings a new adjacency
                     and new features (pack_static, then forward)
             packet  the same with the batch in host memory: packed to bit planes on the CPU,
                     one copy to the device, then map and layers (SubgraphPacket)
  product  the paper's bit-Tensor calls on plain tensors: to_bit twice, bitMM2Int
  held     bitMM2Int of operands and tile map that are kept packed
  chain    bitMM2Bit, its codes decoded (to_val), and bitMM2Int of them with weights
"""
import math

import numpy as np
import torch

import paper_2111_09547_amd as q
from paper_2111_09547_amd.bit_tensor import bitMM2Bit, bitMM2Int, calibrate_inv_scale, to_bit
from paper_2111_09547_amd.model import BatchNorm, QuantGNN
from paper_2111_09547_amd.packing import SubgraphPacket

PACK_THREADS = 16


def _net(mode, graph, blocks, block, dims, bits, wbits=None, degree=8.0, short=0, dense=False, gin=False, bn=False,
         update_first=False):
    """blocks x block nodes (the last subgraph short by `short`), `degree` neighbours per
    node on average, dims "in-hidden-..-out", bits per feature and weight; dense: one N x N
    adjacency instead of one row of diagonal blocks."""
    return {"do": "net", "mode": mode, "graph": graph, "blocks": blocks, "block": block, "short": short,
            "degree": degree, "dims": dims, "s": bits, "t": wbits or bits, "dense": dense, "gin": gin, "bn": bn,
            "update_first": update_first}


def listed():
    def named(name, case):
        return dict(case, name=name)
    return [
        # one product of small matrices, straight from plain tensors: host work and launches
        named("product 256x16 2bit", {"do": "product", "n": 256, "d": 16, "s": 2, "density": 0.03}),
        # a single GCN layer on a small batch, called from a script (4-bit embeddings)
        named("gcn1 4096 eager 4bit", _net("eager", "uniform", 16, 256, "128-16", 4, degree=6.1, dense=True)),
        # one layer on 8 subgraphs of 1024 in a serving loop, at the common width ...
        named("gcn1 8192 graph 8bit", _net("graph", "uniform", 8, 1024, "64-64", 8, degree=10.2, dense=True)),
        # ... and at 16 bits, for accuracy (two products, wider than the int8 matrix cores)
        named("gcn1 8192 graph 16bit", _net("graph", "uniform", 8, 1024, "64-64", 16, degree=10.2, dense=True)),
        # the benchmark's step: 5-layer GIN on 64 communities of 1024, all packing included
        named("gin5 65536 step 8bit", _net("step", "uniform", 64, 1024, "128-64-64-64-64-64", 8, degree=8.2, gin=True)),
        # the same network on mini-batches of 8 communities, each batch new, no graph recorded
        named("gin5 8192 batch 8bit", _net("batch", "uniform", 8, 1024, "128-64-64-64-64-64", 8, degree=8.2, gin=True)),
        # a large power-law graph cut into subgraphs, wide input features, both product orders
        named("gcn2 262144 graph 8bit", _net("graph", "powerlaw", 128, 2048, "512-16-16", 8)),
        named("gcn2 262144 update-first 4bit", _net("graph", "powerlaw", 128, 2048, "512-16-16", 4, update_first=True)),
        # nothing a multiple of anything: odd widths, mixed bit widths, a short last subgraph,
        # batch normalization folded into the hidden layers
        named("gcn3 ragged bn graph", _net("graph", "uniform", 37, 416, "300-101-47-7", 5, 3, degree=14.0, short=171, bn=True)),
        # a loader that packs on the host and ships low-bit planes
        named("gin2 16384 packet 8bit", _net("packet", "uniform", 16, 1024, "128-64-16", 8, degree=8.2, gin=True)),
        # the aggregation alone, every tile of the adjacency occupied
        named("held 8192x64 2bit", {"do": "held", "n": 8192, "d": 64, "s": 2, "density": 0.5}),
        # a large layer spelled as the paper's two products, with the codes read back
        named("chain 16384x256 4bit", {"do": "chain", "n": 16384, "d": 256, "h": 64, "s": 4, "t": 4, "density": 0.05}),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    do = rng.choice(["net"] * 7 + ["product", "held", "chain"])
    bits = rng.choice([1, 2, 3, 4, 4, 5, 6, 7, 8, 8, 8])
    if do == "product":
        return {"do": do, "n": _log_int(rng, 100, 4096), "d": _log_int(rng, 3, 512), "s": bits,
                "density": round(rng.uniform(0.01, 0.5), 3)}
    if do == "held":
        return {"do": do, "n": _log_int(rng, 500, 12000), "d": _log_int(rng, 8, 512), "s": rng.choice([bits, bits, 16]),
                "density": round(rng.uniform(0.05, 0.5), 3)}
    if do == "chain":
        return {"do": do, "n": _log_int(rng, 500, 12000), "d": _log_int(rng, 16, 256), "h": _log_int(rng, 5, 128), "s": bits,
                "t": rng.choice([bits, 4, 8]), "density": round(rng.uniform(0.02, 0.3), 3)}
    mode = rng.choice(["graph", "graph", "step", "eager", "batch", "packet"])
    graph = rng.choice(["uniform", "uniform", "powerlaw"])
    nodes = _log_int(rng, 500, 32768 if mode in ("packet", "batch") else 131072)
    dense = graph == "uniform" and nodes <= 8192 and rng.random() < 0.4
    block = 32 * (_log_int(rng, 16, 64) if graph == "powerlaw" else _log_int(rng, 2, 48))
    blocks = max(1, nodes // block)
    layers = rng.choice([1, 2, 2, 3, 5])
    wide = 512 if nodes <= 65536 else 256
    width = [_log_int(rng, 8, wide)] + [rng.choice([16, 32, 64, 128, _log_int(rng, 9, 200)]) for _ in range(layers - 1)]
    dims = "-".join(str(v) for v in width + [_log_int(rng, 2, 64)])
    update_first = mode in ("graph", "eager") and rng.random() < 0.2
    bn = not update_first and layers > 1 and rng.random() < 0.25
    if rng.random() < 0.1 and not bn and not update_first:
        bits = 16
    return _net(mode, graph, blocks, block, dims, bits, rng.choice([bits, bits, min(bits, 4)]),
                degree=round(rng.uniform(4.0, 24.0), 1), short=rng.choice([0, rng.randrange(block // 2)]), dense=dense,
                gin=rng.random() < 0.5, bn=bn, update_first=update_first)


# ------------------------------------------------------------------------------- inputs
def _dims(case):
    d = [int(v) for v in case["dims"].split("-")]
    return list(zip(d[:-1], d[1:]))


def _nodes(case):
    return case["blocks"] * case["block"] - case["short"]


def _uniform(case, gen):
    """Undirected Bernoulli subgraphs, self-loops unless the network adds its own self term:
    uint8 [n, block], one row of diagonal blocks."""
    nb, b, n = case["blocks"], case["block"], _nodes(case)
    p = min(0.5, case["degree"] / b)
    a = torch.zeros((nb * b, b), dtype=torch.uint8, device="cuda")
    view = a.view(nb, b, b)
    per = max(1, (1 << 25) // (b * b))
    for i in range(0, nb, per):
        part = view[i:i + per]
        up = torch.triu(torch.rand(part.shape, generator=gen, device="cuda") < p, diagonal=1)
        part.copy_(up | up.transpose(1, 2))
        if not case["gin"]:
            part.diagonal(dim1=1, dim2=2).fill_(1)
    if case["short"]:
        a = a[:n]
        a[(nb - 1) * b:, b - case["short"]:] = 0
    return a.contiguous()


def _powerlaw(case, gen, seed):
    """A power-law graph (expected degrees w_i ~ (i + 1)^(-1/1.1), mean 12) relabelled in
    breadth-first order from its largest hub and cut into subgraphs of `block` consecutive
    nodes, edges across the cut dropped: hubs and most edges sit in the first subgraphs."""
    b, n = case["block"], _nodes(case)
    w = (np.arange(n, dtype=np.float64) + 1.0) ** (-1.0 / 1.1)
    cum = torch.from_numpy(np.cumsum(w / w.sum())).cuda()
    ends = torch.searchsorted(cum, torch.rand((2, 6 * n), generator=gen, device="cuda", dtype=torch.float64))
    u, v = ends.clamp_(max=n - 1)
    src, dst = torch.cat([u, v]), torch.cat([v, u])
    unseen = 2 * n
    place = torch.full((n,), unseen, dtype=torch.int64, device="cuda")     # position in the new order
    place[0], done = 0, 1
    while True:
        best = torch.full((n,), unseen, dtype=torch.int64, device="cuda")  # earliest neighbour already placed
        best.scatter_reduce_(0, dst, place[src], "amin")
        found = torch.nonzero((place == unseen) & (best < unseen)).flatten()
        if found.numel() == 0:
            break
        found = found[torch.argsort(best[found], stable=True)]
        place[found] = done + torch.arange(found.numel(), device="cuda")
        done += found.numel()
    rest = torch.nonzero(place == unseen).flatten()
    place[rest] = done + torch.arange(rest.numel(), device="cuda")
    r, c = place[src], place[dst]
    keep = (r // b == c // b) & (r != c)
    a = torch.zeros((n, b), dtype=torch.uint8, device="cuda")
    a[r[keep], c[keep] % b] = 1
    if not case["gin"]:
        i = torch.arange(n, device="cuda")
        a[i, i % b] = 1
    return a


def _adjacency(case, gen, seed):
    a = _powerlaw(case, gen, seed) if case["graph"] == "powerlaw" else _uniform(case, gen)
    if not case["dense"]:
        return a
    n, b = _nodes(case), case["block"]
    full = torch.zeros((n, n), dtype=torch.uint8, device="cuda")
    for i in range(case["blocks"]):
        r1 = min(n, (i + 1) * b)
        full[i * b:r1, i * b:r1] = a[i * b:r1, :r1 - i * b]
    return full


def _batchnorms(case, rng):
    """Statistics of a trained network's size for every hidden layer."""
    out = []
    for i, (_, h) in enumerate(_dims(case)):
        last = i == len(_dims(case)) - 1
        out.append(None if last else BatchNorm(rng.uniform(0.5, 1.5, h).tolist(), rng.uniform(-0.3, 0.6, h).tolist(),
                                               (rng.uniform(-0.2, 0.4, h) * 0.1).tolist(),
                                               (rng.uniform(0.5, 2.0, h) * 0.02).tolist()))
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    st = {"case": case}
    s = case["s"]
    if case["do"] != "net":
        n, d = case["n"], case["d"]
        a = (torch.rand((n, n), generator=gen, device="cuda") < case["density"]).to(torch.uint8)
        x = torch.randint(0, 1 << s, (n, d), generator=gen, device="cuda", dtype=torch.int32)
        if case["do"] == "product":
            st.update(a=a, x=x)
            return st
        st["A"], st["X"] = to_bit(a, 1, side="left"), to_bit(x, s)
        st["map"] = q.qgtc_build_tile_map(st["A"].bits, 16, 128)
        if case["do"] == "chain":
            w = torch.randint(0, 1 << case["t"], (d, case["h"]), generator=gen, device="cuda", dtype=torch.int32)
            st["W"] = to_bit(w, case["t"])
            st["inv"] = calibrate_inv_scale(st["A"], st["X"], s, tile_map=st["map"])
        return st

    rng = np.random.default_rng([seed, 7])
    dims, n = _dims(case), _nodes(case)
    a = _adjacency(case, gen, seed)
    x = torch.randn((n, dims[0][0]), generator=gen, device="cuda")
    ws = [torch.rand(dh, generator=gen, device="cuda") * 0.2 - 0.1 for dh in dims]
    xr = (float(x.min()), float(x.max()))
    block_rows = 0 if case["dense"] else case["block"]
    mode = case["mode"]
    kw = dict(tile_kbits="auto", block_rows=block_rows, update_first=case["update_first"],
              batchnorm=_batchnorms(case, rng) if case["bn"] else None)
    if mode == "packet":
        pk = SubgraphPacket(n, a.shape[1], dims[0][0], s, block_rows=block_rows)
        st.update(packet=pk, a_host=a.cpu(), x_host=x.cpu())
        pk.pack(st["a_host"], st["x_host"], xr, threads=PACK_THREADS)
        a, _ = pk.upload()
    net = QuantGNN(a, ws, s, case["t"], case["gin"], **kw)
    ranges = net.calibrate(x, xr)
    st.update(net=net, x=x, xr=xr, ranges=ranges)
    if mode in ("graph", "step"):
        st["out"] = torch.empty((n, dims[-1][1]), dtype=torch.float32, device="cuda")
        st["replay"] = net.capture(x, xr, ranges, st["out"], streams=net.auto_runs(), with_static=mode == "step")
    return st


# --------------------------------------------------------------------------------- a pass
def run(st):
    case = st["case"]
    do = case["do"]
    if do == "product":
        return bitMM2Int(to_bit(st["a"], 1, side="left"), to_bit(st["x"], case["s"]))
    if do == "held":
        return bitMM2Int(st["A"], st["X"], tile_map=st["map"])
    if do == "chain":
        y = bitMM2Bit(st["A"], st["X"], case["s"], st["inv"], tile_map=st["map"])
        return {"codes": y.to_val(), "z": bitMM2Int(y, st["W"])}
    mode, net = case["mode"], st["net"]
    if mode in ("graph", "step"):
        st["replay"].replay()
        return st["out"]
    if mode == "eager":
        return net.forward(st["x"], st["xr"], st["ranges"])
    if mode == "batch":
        net.pack_static(st["x"], st["xr"])
        return net.forward(st["x"], st["xr"], st["ranges"], x_packed=True)
    pk = st["packet"]
    if "copied" in st:
        st["copied"].synchronize()          # the pinned buffer is free again once its last copy is through
    pk.pack(st["a_host"], st["x_host"], st["xr"], threads=PACK_THREADS)
    _, x_bits = pk.upload()
    st["copied"] = torch.cuda.Event()
    st["copied"].record()
    net.pack_static()
    return net.forward(None, st["xr"], st["ranges"], x_bits=x_bits)


def work(case):
    """Inputs read once, outputs written once; two operations per edge and feature in the
    aggregation, per product in the update."""
    s = case["s"]
    if case["do"] != "net":
        n, d = case["n"], case["d"]
        edges = case["density"] * n * n
        bits = n * n / 8 + n * d * s / 8
        if case["do"] == "product":
            return {"bytes": n * n + 4 * n * d + 4 * n * d, "flops": 2 * edges * d}
        if case["do"] == "held":
            return {"bytes": bits + 4 * n * d, "flops": 2 * edges * d}
        h = case["h"]
        return {"bytes": bits + d * h * case["t"] / 8 + 4 * n * d + 4 * n * h, "flops": 2 * edges * d + 2 * n * d * h}
    n, dims, t = _nodes(case), _dims(case), case["t"]
    entries = n * (n if case["dense"] else case["block"])
    edges = n * (2.3 if case["graph"] == "powerlaw" else case["degree"])
    data = 4 * n * dims[0][0] + sum(d * h for d, h in dims) * t / 8 + 4 * n * dims[-1][1] + entries / 8
    if case["mode"] in ("step", "batch"):
        data += entries + sum(d * h for d, h in dims) * 4
    elif case["mode"] == "packet":
        data += entries + n * dims[0][0] * s / 8 + entries / 8
    return {"bytes": data, "flops": sum(2 * edges * d + 2 * n * d * h for d, h in dims)}


def tolerance(case):
    # integers and codes are exact; the network's fp32 output is one fp64 expression of exact
    # integers, rounded once
    return {"rel": 1e-6} if case["do"] == "net" else "exact"
