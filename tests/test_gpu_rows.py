"""GPU parity of the row kernels (fp32, the automatic choice: one for runs of
few columns, one over LDS tiles for longer runs of up to 160 input channels).

Each case is compared with the oracle to the fp32 tolerance and bit for bit
with the direct-load kernel (kernel option 2): both sum each output in
ascending input channel from zero.  The sizes sit at the kernels' edges: rows
of no weight and around batches of 8 and groups of 4, planes of 4 columns, not
a multiple of 4 (the last unit repeats columns of the one before) and below 4
(other kernels), partial blocks of 64 units, tiles that span images and end
inside one, runs of less than a round of tiles, of whole rounds and with tiles
shared by parts of the rows, the input widths where the tile changes, and the
widest input.
"""

import zlib

import numpy as np
import pytest

from synth import make_layer, densify
from gpu_util import gpu_run, assert_parity, assert_runs, note, to_gpu, device

pytestmark = pytest.mark.gpu

# (cin, cout, h, w, n, sparsity, k, act)
FEW = [
    (16, 16, 2, 2, 1, 0.0, 1, "relu"),       # one unit; rows of two whole batches
    (5, 3, 1, 1, 1, 0.0, 1, "relu6"),        # H*W below 4
    (33, 20, 1, 5, 1, 0.7, 1, "none"),       # the second unit repeats 3 columns
    (72, 96, 7, 7, 5, 0.85, 2, "relu"),      # 65 units: a block of one unit
    (64, 130, 5, 5, 7, 0.9, 1, "relu6"),
    (512, 64, 14, 14, 1, 0.9, 1, "relu6"),
    (1300, 40, 6, 6, 2, 0.95, 1, "none"),    # wider than every staged kernel
    (128, 256, 8, 8, 2, 0.9, 4, "relu"),
]
STRIP = [
    (16, 20, 64, 64, 9, 0.8, 1, "relu"),       # 9216 units of 64: less than a round, shared by parts
    (17, 17, 13, 13, 250, 0.5, 1, "none"),     # odd planes, tiles span images, a ragged last tile
    (79, 48, 32, 32, 130, 0.85, 1, "relu6"),   # the widest 64-unit tile
    (80, 40, 32, 32, 40, 0.85, 4, "relu"),     # 32-unit tiles, 2 columns a lane
    (80, 140, 21, 21, 90, 0.8, 1, "none"),     # one workgroup of 16 wavefronts a compute unit
    (128, 256, 28, 28, 168, 0.9, 1, "relu"),   # the same: two rounds and shared tiles
    (159, 300, 28, 28, 42, 0.9, 2, "relu6"),   # the widest input there
    (160, 260, 7, 7, 90, 0.85, 1, "relu"),     # the widest input, 31-unit tiles
    (161, 260, 7, 7, 90, 0.85, 1, "relu"),     # past it
    (24, 144, 2, 2, 4200, 0.85, 1, "none"),    # planes of one unit
    (159, 300, 21, 21, 42, 0.9, 1, "relu6"),   # the widest input of the 16 wavefronts, odd planes
    (96, 576, 14, 14, 128, 0.85, 1, "relu6"),  # 98 tiles of 16 wavefronts, shared by 2 parts
    (112, 400, 9, 9, 200, 0.9, 1, "none"),     # 66 of them by 2, odd planes
    (80, 256, 14, 14, 30, 0.95, 1, "relu"),    # 23 tiles by 4 parts
]
OTHER = [(159, 300, 28, 28, 42, 0.9, 2, "relu6"), (161, 260, 7, 7, 90, 0.85, 1, "relu")]  # of these, not by the LDS kernel


def _check(spec, what):
    cin, cout, h, w, n, s, k, act = spec
    layer = make_layer(cin, cout, h, w, n, s, block_rows=k, act=act, seed=zlib.crc32(repr(spec).encode()) % 1000)
    note("%s %s" % (what, spec))
    assert_runs(layer, "strip" if h * w < 4 or spec in OTHER else what)
    y = gpu_run(layer)
    assert_parity(layer, y, what=str(spec))
    assert np.array_equal(y.view(np.uint32), gpu_run(layer, kernel=2).view(np.uint32))


@pytest.mark.parametrize("spec", FEW, ids=lambda s: "%d-%d-%dx%d-n%d-s%g-k%d-%s" % s)
def test_few_columns_match_oracle_and_direct_kernel(spec):
    _check(spec, "rows")


@pytest.mark.parametrize("spec", STRIP, ids=lambda s: "%d-%d-%dx%d-n%d-s%g-k%d-%s" % s)
def test_lds_rows_match_oracle_and_direct_kernel(spec):
    _check(spec, "lds rows")


@pytest.mark.parametrize("n", [3, 260])
def test_rows_without_weights_and_a_long_row(n):
    """Rows and channels without a stored weight, and one long row (of fewer
    than the 32 weights from which the direct-load kernel splits rows)."""
    layer = make_layer(48, 56, 12, 12, n, 0.8, act="none", seed=4)
    rng = np.random.default_rng(4)
    rp, ci = [0], []
    for r in range(layer.cout):
        s, e = layer.row_ptr[r], layer.row_ptr[r + 1]
        cols = list(range(31)) if r == 17 else [] if r % 5 == 0 else [c for c in layer.col_idx[s:e] if c % 3]
        ci += [int(c) for c in cols]
        rp.append(len(ci))
    layer.row_ptr, layer.col_idx = np.array(rp, np.int32), np.array(ci, np.int32)
    layer.values = rng.standard_normal(len(ci)).astype(np.float32)
    note("rows empty n=%d" % n)
    assert_runs(layer, "rows" if n == 3 else "lds rows")
    y = gpu_run(layer)
    assert_parity(layer, y, what="empty rows")
    assert np.array_equal(y.view(np.uint32), gpu_run(layer, kernel=2).view(np.uint32))


@pytest.mark.parametrize("hw,n", [((8, 8), 5), ((7, 7), 5), ((1, 2), 5), ((8, 8), 600), ((7, 7), 800)])
def test_rows_unaligned_pointers(hw, n):
    """x and y one element off a 16-byte boundary: the same bits, nothing
    written outside y."""
    import torch
    from paper_1911_09723_amd import Plan
    layer = make_layer(40, 50, hw[0], hw[1], n, 0.8, act="relu", seed=5)
    note("rows unaligned %s n=%d" % (hw, n))
    assert_runs(layer, "strip" if hw == (1, 2) else "rows" if n == 5 else "lds rows")
    ref = gpu_run(layer)
    plan = Plan.from_layer(layer)
    try:
        flat = to_gpu(np.concatenate([np.zeros(1, np.float32), layer.x.ravel()]))
        ybuf = torch.full((1 + ref.size + 8,), 7.0, device=device())
        y = ybuf[1:1 + ref.size].view(ref.shape)
        plan.run(flat[1:].view(layer.x.shape), y)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy().view(np.uint32), ref.view(np.uint32))
        assert float(ybuf[0]) == 7.0 and torch.all(ybuf[1 + ref.size:] == 7.0)
    finally:
        plan.close()


@pytest.mark.parametrize("hw,n", [((8, 8), 4), ((7, 7), 4), ((1, 1), 4), ((8, 8), 600), ((7, 7), 800)])
@pytest.mark.parametrize("act", ["relu6", "none"])
def test_rows_infinities_and_nans_stay_on_their_rows(hw, n, act):
    """Non-finite inputs reach the rows that store a weight at their channel
    and no other (padding reads a row of zeros)."""
    layer = make_layer(70, 45, hw[0], hw[1], n, 0.8, act=act, seed=17)
    x = layer.x.copy()
    x[0, 3, 0, 0] = np.inf
    x[1, 40, -1, -1] = -np.inf
    x[n - 1, 69, -1, -1] = np.nan
    x[n - 1, 12, 0, 0] = np.inf
    note("rows non-finite %s n=%d %s" % (hw, n, act))
    assert_runs(layer, "strip" if hw == (1, 1) else "rows" if n == 4 else "lds rows")
    y = gpu_run(layer, x=x).astype(np.float64)
    wd = densify(45, 70, 1, layer.row_ptr, layer.col_idx, layer.values)
    stored = densify(45, 70, 1, layer.row_ptr, layer.col_idx, np.ones_like(layer.values)) > 0
    finite = np.where(np.isfinite(x), x, 0).astype(np.float64)
    s = np.einsum("rc,nchw->nrhw", wd, finite) + layer.bias[None, :, None, None]
    for i, c, r0, c0 in np.argwhere(~np.isfinite(x)):
        for r in np.flatnonzero(stored[:, c]):
            s[i, r, r0, c0] += wd[r, c] * float(x[i, c, r0, c0])
    if act == "relu6":
        s = np.where(np.isnan(s), 0.0, np.clip(s, 0, 6))  # a NaN clamps to the lower bound
    else:
        s = np.where(np.isnan(s), -np.inf, s)
    assert np.array_equal(np.isfinite(y), np.isfinite(s))
    ok = np.isfinite(s)
    assert np.array_equal(y[~ok], s[~ok])
    # fp32 sums of at most 70 terms, each of size 1
    assert np.all(np.abs(y[ok] - s[ok]) <= 1e-4)


# heavy-tailed layers whose strip plan packs rows as two pieces (cin, cout, h, w, n, sparsity, act)
SPLIT = [
    (128, 64, 14, 14, 1, 0.85, "none"),     # few columns
    (144, 200, 7, 7, 1, 0.85, "relu"),
    (100, 100, 13, 13, 1, 0.85, "none"),
    (600, 64, 14, 14, 1, 0.97, "relu6"),
    (144, 24, 56, 56, 12, 0.85, "none"),    # LDS tiles, 2 columns a lane
    (96, 64, 28, 28, 48, 0.85, "relu"),
    (120, 32, 21, 21, 60, 0.85, "none"),    # odd planes
]


@pytest.mark.parametrize("spec", SPLIT, ids=lambda s: "%d-%d-%dx%d-n%d-s%g-%s" % s)
def test_split_rows_keep_the_strip_kernels_sums(spec):
    """The even and the odd weights of a split row are summed apart, as in the
    strip kernel (option 1): the same bits, so no more rounding error."""
    from paper_1911_09723_amd import Plan
    cin, cout, h, w, n, s, act = spec
    layer = make_layer(cin, cout, h, w, n, s, pattern="beta", act=act, seed=cin * 7 + cout)
    plan = Plan.from_layer(layer)
    try:
        assert plan.info()["split_rows"] > 0, "the case must split at least one row"
    finally:
        plan.close()
    note("rows split %s" % (spec,))
    assert_runs(layer, "rows" if n == 1 else "lds rows")
    y = gpu_run(layer)
    assert_parity(layer, y, what=str(spec))
    assert np.array_equal(y.view(np.uint32), gpu_run(layer, kernel=1).view(np.uint32))


@pytest.mark.parametrize("cin,cout,s,n,name", [(640, 96, 0.95, 256, "outer"), (1264, 40, 0.95, 512, "outer"),
                                               (1400, 96, 0.98, 512, "passes")])
def test_wide_heavy_tailed_rows_do_not_depend_on_the_batch(cin, cout, s, n, name):
    """Heavy-tailed layers too wide for an LDS strip: a short run takes the row
    kernel, a long one a kernel that sums every row in one chain.  An image
    alone gives the bits that it gives among others."""
    layer = make_layer(cin, cout, 7, 7, n, s, pattern="beta", act="none", seed=cin)
    note("rows wide %d -> %d" % (cin, cout))
    assert_runs(layer, name)
    y = gpu_run(layer)
    assert_parity(layer, y, what="%d -> %d" % (cin, cout))
    layer.x, layer.n = layer.x[:2], 2
    assert_runs(layer, "rows")
    assert np.array_equal(gpu_run(layer).view(np.uint32), y[:2].view(np.uint32))
