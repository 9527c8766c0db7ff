"""The work that a user of this framework has it do, as cases that can be timed.

Two kinds of case, all through the package's public entry points:

* ``layer``: one sparse 1x1 convolution, ``Plan(...).run(x, y)``: fp32 or
  fp16 storage, unstructured or 1 x 4 output-channel-blocked weights, uniform
  or heavy-tailed rows, from one small image plane to the widest batches;
* ``network``: one MobileNet v1 forward pass by ``MobileNetV1Engine`` (stem,
  13 blocks of depthwise 3x3 and sparse 1x1, pooling, classifier), launched
  eagerly or replayed as one graph.

Weights: mask positions drawn without replacement at an exact count (whole
1 x 4 blocks for blocked layers; Beta(1.5, 8.5) row densities for the
heavy-tailed ones), values ~ N(0, 2 / (0.1 cin)), bias ~ N(0, 0.01).  Inputs:
X = max(0, N(0, 1)), images uniform in [-1, 1].  Everything follows from the
seed alone.
"""

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1911_09723_amd import Plan
from paper_1911_09723_amd.mobilenet import MobileNetV1Engine

DEVICE = "cuda:0"

# (cin, cout, depthwise stride) of MobileNet v1's blocks at width 1.0.
BLOCKS = ((32, 64, 1), (64, 128, 2), (128, 128, 1), (128, 256, 2), (256, 256, 1), (256, 512, 2), (512, 512, 1),
          (512, 512, 1), (512, 512, 1), (512, 512, 1), (512, 512, 1), (512, 1024, 2), (1024, 1024, 1))
CLASSES = 1000


def _layer(name, cin, cout, side, batch, sparsity=0.9, block_rows=1, rows="uniform", storage="f32", act="relu6"):
    case = dict(kind="layer", cin=cin, cout=cout, h=side, w=side, batch=batch, sparsity=sparsity,
                block_rows=block_rows, rows=rows, storage=storage, act=act)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest call: one early layer on a single image (latency, one launch)
        _layer("c32_64_56_b1", 32, 64, 56, 1, act="relu"),
        # a middle layer of MobileNet v1 on a single image: the interactive use
        _layer("c512_512_14_b1", 512, 512, 14, 1),
        # MobileNet v1's first pointwise layer, a serving batch: few channels, large planes
        _layer("c32_64_112_b64", 32, 64, 112, 64),
        # an early layer of middling width at the same batch
        _layer("c128_128_56_b64", 128, 128, 56, 64),
        # the layer shape that most of MobileNet v1 consists of, at a large batch
        _layer("c512_512_14_b256", 512, 512, 14, 256, act="relu"),
        # the same with 1 x 4 blocked weights
        _layer("c512_512_14_b256_1x4", 512, 512, 14, 256, block_rows=4, act="relu"),
        # MobileNet v2 contraction (linear bottleneck): few outputs, heavy-tailed rows
        _layer("c144_24_56_b128_beta", 144, 24, 56, 128, sparsity=0.85, rows="beta", act="none"),
        # MobileNet v2 late expansion on the 7 x 7 plane: odd plane size, heavy-tailed rows
        _layer("c160_960_7_b128_beta", 160, 960, 7, 128, sparsity=0.85, rows="beta"),
        # EfficientNet-B0-sized fp16 expansions, 1 x 4 blocked: even and odd planes
        _layer("c112_672_14_b512_f16_1x4", 112, 672, 14, 512, block_rows=4, storage="f16"),
        _layer("c320_1280_7_b512_f16_1x4", 320, 1280, 7, 512, block_rows=4, storage="f16"),
        # a whole network: single-image graph replay, and an eager serving batch
        dict(name="mobilenet_v1_b1_graph", kind="network", side=224, batch=1, graph=True),
        dict(name="mobilenet_v1_b64", kind="network", side=224, batch=64, graph=False),
    ]


def _log(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    """A layer of the listed ranges: any channel counts from 16 to 1280 and
    planes from 5 x 5 to 112 x 113, batches from one image to 512 or what the
    largest listed layers read and write (300 MB) and multiply."""
    storage, block_rows, rows = rng.choice((("f32", 1, "uniform"), ("f32", 1, "uniform"), ("f32", 1, "beta"),
                                            ("f32", 4, "uniform"), ("f16", 4, "uniform"), ("f16", 1, "uniform")))
    cin, cout = _log(rng, 16, 1280), _log(rng, 16, 1280)
    if rng.random() < 0.7:  # channel counts in use are mostly multiples of 8
        cin, cout = cin // 8 * 8, cout // 8 * 8
    cout = cout // block_rows * block_rows
    side = _log(rng, 5, 112) if rng.random() < 0.4 else rng.choice((7, 14, 28, 56))
    sparsity = rng.choice((0.7, 0.8, 0.85, 0.9, 0.9, 0.95))
    size = 2 if storage == "f16" else 4
    most = min(300e6 / (size * (cin + cout) * side * side),
               1.3e9 / ((1 - sparsity) * cin * cout * side * side), 512)
    batch = 1 if rng.random() < 0.2 or most < 2 else _log(rng, 1, most)
    case = _layer(None, cin, cout, side, batch, sparsity, block_rows, rows, storage,
                  rng.choice(("relu", "relu6", "none")))
    return dict(case, w=side + rng.choice((0, 0, 0, 1)))


def _beta_counts(rng, rows, cin, total):
    """Heavy-tailed row lengths with an exact total."""
    p = rng.beta(1.5, 8.5, size=rows)
    exact = np.minimum(p * (total / p.sum()), cin)
    counts = np.floor(exact).astype(np.int64)
    for r in np.argsort(counts - exact, kind="stable").tolist() * cin:
        if counts.sum() >= total:
            break
        counts[r] = min(counts[r] + 1, cin)
    return counts


def _weights(cin, cout, sparsity, block_rows, rows, storage, rng):
    """Block-CSR arrays and a bias."""
    nrows = cout // block_rows
    total = int(round((1 - sparsity) * nrows * cin))
    if rows == "beta":
        counts = _beta_counts(rng, nrows, cin, total)
        col = np.concatenate([np.sort(rng.choice(cin, size=int(k), replace=False)) for k in counts])
    else:
        pos = np.sort(rng.choice(nrows * cin, size=total, replace=False))
        counts = np.bincount(pos // cin, minlength=nrows)
        col = pos % cin
    row_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    values = (rng.standard_normal(len(col) * block_rows) * math.sqrt(2 / (0.1 * cin))).astype(np.float32)
    if storage == "f16":
        values = values.astype(np.float16).astype(np.float32)
    bias = (rng.standard_normal(cout) * 0.1).astype(np.float32)
    return SimpleNamespace(cin=cin, cout=cout, block_rows=block_rows, row_ptr=row_ptr, col_idx=col.astype(np.int32),
                           values=values, bias=bias)


def _network(seed):
    rng = np.random.default_rng(seed)

    def normal(shape, variance):
        return (rng.standard_normal(shape) * math.sqrt(variance)).astype(np.float32)

    blocks = [SimpleNamespace(cin=ci, cout=co, stride=s, dw_k=normal((ci, 3, 3), 2 / 9), dw_b=normal(ci, 0.01),
                              pw=_weights(ci, co, 0.9, 1, "uniform", "f32", rng)) for ci, co, s in BLOCKS]
    return SimpleNamespace(stem_w=normal((32, 3, 3, 3), 2 / 27), stem_b=normal(32, 0.01), blocks=blocks,
                           fc_w=normal((CLASSES, 1024), 1 / 1024), fc_b=normal(CLASSES, 0.01))


def _layer_parts(case, seed):
    wt = _weights(case["cin"], case["cout"], case["sparsity"], case["block_rows"], case["rows"], case["storage"],
                  np.random.default_rng(seed))
    dtype = torch.float16 if case["storage"] == "f16" else torch.float32
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    x = torch.randn((case["batch"], case["cin"], case["h"], case["w"]), generator=gen, device=DEVICE).relu_()
    return wt, x.to(dtype)


def _network_parts(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    image = torch.rand((case["batch"], case["side"], case["side"], 3), generator=gen, device=DEVICE) * 2 - 1
    return _network(seed), image


def prepare(case, seed):
    if case["kind"] == "layer":
        wt, x = _layer_parts(case, seed)
        plan = Plan(wt.cout, wt.cin, wt.block_rows, wt.row_ptr, wt.col_idx, wt.values, wt.bias, case["act"],
                    case["storage"])
        y = torch.empty((x.shape[0], wt.cout) + x.shape[2:], dtype=x.dtype, device=DEVICE)
        return SimpleNamespace(case=case, plan=plan, x=x, y=y)
    net, image = _network_parts(case, seed)
    engine = MobileNetV1Engine(net, case["batch"], case["side"], case["side"])
    if case["graph"]:
        engine.capture()
    return SimpleNamespace(case=case, engine=engine, image=image)


def run(state):
    if state.case["kind"] == "layer":
        return state.plan.run(state.x, state.y)
    if state.case["graph"]:
        state.engine.x.copy_(state.image)
        return state.engine.replay()
    return state.engine.forward(state.image)


def _layer_work(cin, cout, columns, nnz, blocks, rows, size):
    weights = size * nnz + 4 * blocks + 4 * (rows + 1) + 4 * cout
    return size * columns * (cin + cout) + weights, 2 * nnz * columns


def work(case):
    """X (or the image) read once, Y (every intermediate tensor of a network
    written once and read once), and the weights; two operations a stored
    weight and column."""
    if case["kind"] == "layer":
        rows = case["cout"] // case["block_rows"]
        blocks = int(round((1 - case["sparsity"]) * rows * case["cin"]))
        total, flops = _layer_work(case["cin"], case["cout"], case["batch"] * case["h"] * case["w"],
                                   blocks * case["block_rows"], blocks, rows, 2 if case["storage"] == "f16" else 4)
        return {"bytes": total, "flops": flops}
    n, side = case["batch"], case["side"]
    h = (side - 1) // 2 + 1
    total = 4 * n * (3 * side * side + 32 * h * h) + 4 * 28 * 32
    flops = 2 * n * h * h * 27 * 32
    for cin, cout, stride in BLOCKS:
        ho = (h - 1) // stride + 1
        blocks = int(round(0.1 * cin * cout))
        b, f = _layer_work(cin, cout, n * ho * ho, blocks, blocks, cout, 4)
        # the block's input read and its output written once: what lies between can stay on chip
        total += b + 4 * n * cin * (h * h - ho * ho) + 40 * cin
        flops += f + 18 * n * cin * ho * ho
        h = ho
    total += 4 * n * (1024 * h * h + CLASSES) + 4 * CLASSES * 1025
    return {"bytes": total, "flops": flops + 2 * n * 1024 * CLASSES}


def tolerance(case):
    if case["kind"] == "network":
        # fp32 rounding through 28 layers
        return {"rel": 2e-6, "max": 2e-5}
    if case["storage"] == "f16":
        # fp32 sums rounded once to fp16 (unit roundoff 2^-11; a sum in another
        # order moves a few values by one last place)
        return {"rel": 1e-3, "max": 4e-3}
    return {"rel": 1e-6, "max": 1e-5}


_CLAMP = {"none": (None, None), "relu": (0.0, None), "relu6": (0.0, 6.0)}


def _clamp(v, act):
    low, high = _CLAMP[act]
    return v if low is None else v.clamp_(min=low, max=high)


def _dense(wt):
    d = np.zeros((wt.cout, wt.cin))
    k = wt.block_rows
    row = np.repeat(np.arange(wt.cout // k), np.diff(wt.row_ptr))
    for i in range(k):
        d[row * k + i, wt.col_idx] = wt.values[i::k]
    return torch.from_numpy(d).to(DEVICE)


def _pointwise(wt, x, act):
    n, c, h, w = x.shape
    y = torch.empty((n, wt.cout, h, w), dtype=torch.float64, device=DEVICE)
    d, b = _dense(wt), torch.from_numpy(wt.bias).to(DEVICE).double()[:, None]
    for i in range(n):
        y[i] = _clamp(d @ x[i].reshape(c, h * w).double() + b, act).view(wt.cout, h, w)
    return y


def _taps(x, stride):
    """The nine zero-padded 3 x 3 neighbours of NCHW x, in row order."""
    n, c, h, w = x.shape
    p = torch.zeros((n, c, h + 2, w + 2), dtype=x.dtype, device=x.device)
    p[:, :, 1:-1, 1:-1] = x
    for dy in range(3):
        for dx in range(3):
            yield dy, dx, p[:, :, dy:dy + h:stride, dx:dx + w:stride]


def exact(case, seed):
    if case["kind"] == "layer":
        wt, x = _layer_parts(case, seed)
        return _pointwise(wt, x, case["act"])
    net, image = _network_parts(case, seed)

    def put(a):
        return torch.from_numpy(a).to(DEVICE).double()

    x, stem = image.permute(0, 3, 1, 2).double(), put(net.stem_w)
    y = 0
    for dy, dx, tap in _taps(x, 2):
        n, c, h, w = tap.shape
        y = y + torch.matmul(stem[:, dy, dx], tap.reshape(n, c, h * w)).view(n, -1, h, w)
    y = _clamp(y + put(net.stem_b)[:, None, None], "relu6")
    for blk in net.blocks:
        k, d = put(blk.dw_k), 0
        for dy, dx, tap in _taps(y, blk.stride):
            d = d + k[:, dy, dx][:, None, None] * tap
        d = _clamp(d + put(blk.dw_b)[:, None, None], "relu6")
        y = _pointwise(blk.pw, d, "relu6")
    return y.mean(dim=(2, 3)) @ put(net.fc_w).T + put(net.fc_b)
