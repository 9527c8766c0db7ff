"""GPU parity of the half kernel (fp16 storage, the automatic choice): dense
fragments of W on the matrix cores.

Each case is compared with the oracle to the fp16 tolerance.  A tile is whole
image planes or an even piece of one, in parts of 16 units of 4 neighbouring
columns of a plane.  The sizes sit at the kernel's edges: input channels around
blocks of 32 and 8, output channels around groups of 32, 16 and 4 rows, planes
whose last unit is short (H*W not a multiple of 4) or only (H*W below 4), one,
two and four parts at a time, wavefronts that share a row tile (large planes of
up to 64 channels), short runs whose tiles are shared by workgroups of 4 and 8
wavefronts, and the widest input of its range and one past it.
"""

import zlib

import numpy as np
import pytest

from synth import make_layer, densify
from gpu_util import gpu_run, assert_parity, assert_runs, note, to_gpu, device

pytestmark = pytest.mark.gpu

# (cin, cout, h, w, n, sparsity, k, act)
SHAPES = [
    (32, 32, 8, 8, 1, 0.5, 1, "relu"),        # one part, one block, two row tiles
    (33, 36, 8, 8, 1, 0.8, 4, "none"),        # a block with one channel, a row tile with 4 rows
    (31, 30, 4, 15, 1, 0.8, 2, "relu6"),      # ragged block and row tile, 15 units
    (7, 4, 1, 4, 1, 0.0, 4, "none"),          # the smallest vector case
    (9, 1, 1, 1, 1, 0.0, 1, "relu"),          # one column
    (40, 65, 1, 3, 7, 0.7, 1, "relu"),        # H*W below 4: element loads and stores
    (72, 100, 1, 2, 45, 0.8, 4, "none"),
    (24, 40, 1, 1, 130, 0.5, 1, "relu6"),     # units of one column
    (48, 33, 5, 5, 6, 0.8, 1, "relu"),        # 7 units a plane, the last of one column
    (64, 48, 3, 3, 29, 0.8, 2, "none"),       # 3 units a plane
    (320, 128, 7, 7, 700, 0.9, 4, "relu6"),   # two parts of two odd planes, the most blocks held in registers
    (321, 128, 14, 14, 90, 0.9, 1, "relu"),   # one block more: two row tiles a group
    (128, 672, 14, 14, 96, 0.9, 4, "relu6"),  # two parts, 42 row tiles for 16 wavefronts
    (96, 160, 13, 13, 400, 0.9, 1, "none"),   # four parts of an odd plane
    (288, 96, 12, 12, 400, 0.9, 2, "relu"),   # four parts, 9 blocks
    (40, 240, 18, 18, 300, 0.9, 4, "relu6"),  # two wavefronts share a row tile
    (40, 240, 17, 17, 300, 0.9, 1, "relu"),   # the same, odd planes
    (40, 240, 28, 28, 90, 0.9, 4, "none"),    # four wavefronts
    (33, 100, 23, 23, 120, 0.8, 1, "none"),   # the same, odd planes
    (64, 300, 7, 7, 6, 0.8, 1, "relu"),       # a short run: workgroups of 4 wavefronts
    (155, 1540, 1, 1, 1931, 0.95, 4, "none"), # of 8
    (1216, 40, 7, 7, 3, 0.9, 1, "relu"),      # the widest input
    (1217, 40, 7, 7, 3, 0.9, 1, "relu"),      # past it
]


@pytest.mark.parametrize("spec", SHAPES, ids=lambda s: "%d-%d-%dx%d-n%d-s%g-k%d-%s" % s)
def test_half_matches_oracle(spec):
    cin, cout, h, w, n, s, k, act = spec
    layer = make_layer(cin, cout, h, w, n, s, block_rows=k, storage="f16", act=act,
                       seed=zlib.crc32(repr(spec).encode()) % 1000)
    note("half %s" % (spec,))
    assert_runs(layer, "half" if cin <= 1216 else "direct")
    assert_parity(layer, gpu_run(layer), what=str(spec))


@pytest.mark.parametrize("hw", [(8, 8), (7, 7), (1, 2)])
def test_half_alignment_and_batch_do_not_change_bits(hw):
    """x and y one and two elements off an 8-byte boundary, and each image on
    its own: the same bits (the order of summation is the plan's)."""
    import torch
    from paper_1911_09723_amd import Plan
    layer = make_layer(72, 100, hw[0], hw[1], 5, 0.8, storage="f16", act="none", seed=3)
    note("half unaligned %s" % (hw,))
    assert_runs(layer, "half")
    ref = gpu_run(layer)
    parts = [gpu_run(layer, x=layer.x[i:i + 1]) for i in range(5)]
    assert np.array_equal(ref.view(np.uint16), np.concatenate(parts).view(np.uint16))
    plan = Plan.from_layer(layer)
    try:
        for off in (1, 2):
            flat = to_gpu(np.concatenate([np.zeros(off, np.float16), layer.x.ravel()]))
            ybuf = torch.full((off + ref.size + 8,), 7.0, dtype=torch.float16, device=device())
            y = ybuf[off:off + ref.size].view(ref.shape)
            plan.run(flat[off:].view(layer.x.shape), y)
            torch.cuda.synchronize()
            assert np.array_equal(y.cpu().numpy().view(np.uint16), ref.view(np.uint16))
            assert torch.all(ybuf[:off] == 7.0) and torch.all(ybuf[off + ref.size:] == 7.0)
    finally:
        plan.close()


def test_half_longest_runs_take_another_kernel():
    """2^28 + 5 images of one column: more workgroups than one launch takes."""
    import torch
    from paper_1911_09723_amd import Plan
    from synth import densify
    layer = make_layer(8, 8, 1, 1, 1, 0.5, storage="f16", act="none", seed=4, with_x=False)
    n = (1 << 28) + 5
    note("half longest run")
    plan = Plan.from_layer(layer)
    try:
        assert plan.run_kernel(n, 1, 1) == "strip"
        x = torch.randn((n, 8, 1, 1), device=device(), dtype=torch.float16)
        y = plan.run(x)
        w = to_gpu(densify(8, 8, 1, layer.row_ptr, layer.col_idx, layer.values).astype(np.float32))
        b = to_gpu(layer.bias)
        for i in range(0, n, 1 << 26):
            ref = x[i:i + (1 << 26)].view(-1, 8).float() @ w.T + b
            # one rounding to fp16 and fp32 sums of 8 terms
            assert torch.all((y[i:i + (1 << 26)].view(-1, 8).float() - ref).abs() <= 1e-3 * ref.abs() + 2e-5)
    finally:
        plan.close()
        torch.cuda.empty_cache()


def test_half_keeps_subnormals():
    """Subnormal fp16 values of X and of W reach the products: the result is
    exact (one weight of 1, or of 2^-20 times powers of two, a row)."""
    c = 96
    rng = np.random.default_rng(6)
    layer = make_layer(c, c, 7, 7, 3, 0.5, storage="f16", act="none", seed=6)
    layer.row_ptr, layer.col_idx = np.arange(c + 1, dtype=np.int32), np.arange(c, dtype=np.int32)
    layer.bias = np.zeros(c, np.float32)
    layer.values = np.ones(c, np.float32)
    layer.x = (rng.integers(-1023, 1024, layer.x.shape) * 2.0 ** -24).astype(np.float16)
    note("half subnormal x")
    assert_runs(layer, "half")
    assert np.array_equal(gpu_run(layer), layer.x)
    layer.values = np.full(c, 2.0 ** -20, np.float32)
    layer.x = (2.0 ** rng.integers(-4, 11, layer.x.shape)).astype(np.float16)
    note("half subnormal w")
    assert np.array_equal(gpu_run(layer).astype(np.float64), layer.x.astype(np.float64) * 2.0 ** -20)


@pytest.mark.parametrize("spec", [(70, 45, 8, 8, 5), (70, 45, 7, 7, 9), (70, 45, 1, 3, 30), (40, 96, 28, 28, 70),
                                  (96, 160, 13, 13, 400), (400, 80, 6, 6, 9), (128, 640, 4, 4, 3)],
                         ids=lambda s: "%d-%d-%dx%d-n%d" % s)
def test_half_non_finite_columns_leave_the_others_alone(spec):
    """The same bits in every column without an infinity or a NaN, of the same
    image and of the others in its tile."""
    cin, cout, h, w, n = spec
    layer = make_layer(cin, cout, h, w, n, 0.8, storage="f16", act="none", seed=cin + n)
    note("half columns %s" % (spec,))
    assert_runs(layer, "half")
    y = gpu_run(layer)
    x = layer.x.copy()
    x[0, 3, 0, 0] = np.inf
    x[n // 2, cin - 1, h - 1, w - 1] = np.nan
    x[n // 2, 5, h // 2, w // 2] = -np.inf
    finite = np.isfinite(x).all(axis=1)[:, None]
    assert int((~finite).sum()) == 3
    y2 = gpu_run(layer, x=x)
    same = y.view(np.uint16) == y2.view(np.uint16)
    assert (same | ~finite).all()
    assert not same.all()


# output channels one to three past a row tile, and second row tiles wholly past
# the last channel (two tiles a group, inputs of more than 320 channels)
@pytest.mark.parametrize("cin,cout", [(32, 33), (32, 18), (96, 3), (300, 17), (352, 40), (352, 33), (640, 16)])
def test_half_rows_past_the_last_channel_are_not_stored(cin, cout):
    """Whole units of the last image, 16-byte aligned: nothing behind y changes."""
    import torch
    from paper_1911_09723_amd import Plan
    layer = make_layer(cin, cout, 8, 8, 1, 0.2, storage="f16", act="none", seed=cin + cout)
    assert_runs(layer, "half")
    note("half rows past the last %d -> %d" % (cin, cout))
    plan = Plan.from_layer(layer)
    try:
        ybuf = torch.full((cout * 64 + 64 * 64,), 7.0, dtype=torch.float16, device=device())
        y = ybuf[:cout * 64].view(1, cout, 8, 8)
        plan.run(to_gpu(layer.x), y)
        torch.cuda.synchronize()
        assert_parity(layer, y.cpu().numpy(), what="%d -> %d" % (cin, cout))
        assert torch.all(ybuf[cout * 64:] == 7.0)
    finally:
        plan.close()


@pytest.mark.parametrize("hw", [(8, 8), (7, 7), (1, 1)])
@pytest.mark.parametrize("act", ["relu6", "none"])
def test_half_infinities_and_nans_stay_on_their_rows(hw, act):
    """Non-finite inputs reach the rows that store a weight at their channel
    and no other (the dense product alone would spread 0 * inf to all)."""
    layer = make_layer(70, 45, hw[0], hw[1], 4, 0.8, storage="f16", act=act, seed=17)
    x = layer.x.copy()
    x[0, 3, 0, 0] = np.inf
    x[1, 40, -1, -1] = -np.inf
    x[3, 69, -1, -1] = np.nan
    x[3, 12, 0, 0] = np.inf
    note("half non-finite %s %s" % (hw, act))
    assert_runs(layer, "half")
    y = gpu_run(layer, x=x).astype(np.float64)
    wd = densify(45, 70, 1, layer.row_ptr, layer.col_idx, layer.values)
    stored = densify(45, 70, 1, layer.row_ptr, layer.col_idx, np.ones_like(layer.values)) > 0
    finite = np.where(np.isfinite(x), x, 0).astype(np.float64)
    s = np.einsum("rc,nchw->nrhw", wd, finite) + layer.bias[None, :, None, None]
    for n, c, i, j in np.argwhere(~np.isfinite(x)):
        for r in np.flatnonzero(stored[:, c]):
            s[n, r, i, j] += wd[r, c] * float(x[n, c, i, j])
    if act == "relu6":
        s = np.where(np.isnan(s), 0.0, np.clip(s, 0, 6))  # a NaN clamps to the lower bound
    else:
        s = np.where(np.isnan(s), -np.inf, s)
    assert np.array_equal(np.isfinite(y), np.isfinite(s))
    ok = np.isfinite(s)
    assert np.array_equal(y[~ok], s[~ok])
    # 2^-11 of the value (one rounding to fp16) and fp32 sums of at most 70 terms
    assert np.all(np.abs(y[ok] - s[ok]) <= 2e-3 * np.abs(s[ok]) + 1e-4)
