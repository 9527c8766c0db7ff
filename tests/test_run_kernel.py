"""Which kernel a run takes (spconv_plan_run_kernel), on host-only plans: no GPU.

spconv_run launches what this call reports (one function decides for both), so
these cases pin the rules: forced kernels are honoured at every size, and the
automatic choice takes the kernels that the sizes and types ask for."""

import ctypes

import pytest

import paper_1911_09723_amd as sp
from paper_1911_09723_amd import Plan, spconv
from synth import make_layer


def run_kernel(layer, n, h, w, **options):
    plan = Plan.from_layer(layer, host_only=1, **options)
    try:
        return plan.run_kernel(n, h, w)
    finally:
        plan.close()


def layer_of(cin, cout, sparsity=0.9, **kw):
    return make_layer(cin, cout, 1, 1, 1, sparsity, seed=cin + cout, with_x=False, **kw)


@pytest.mark.parametrize("n,h,w", [(1, 14, 14), (256, 14, 14), (3, 7, 7), (5, 1, 3)])
@pytest.mark.parametrize("kernel,name", [(1, "strip"), (2, "direct"), (3, "indexed"), (4, "outer")])
def test_forced_kernels_run_at_every_size(kernel, name, n, h, w):
    assert run_kernel(layer_of(64, 96), n, h, w, kernel=kernel) == name
    assert run_kernel(layer_of(512, 512), n, h, w, kernel=kernel) == name


@pytest.mark.parametrize("cin,cout", [(600, 64), (1024, 96), (1030, 48), (1280, 320), (1300, 40)])
@pytest.mark.parametrize("n,h,w", [(1, 7, 7), (1, 8, 8), (3, 5, 5), (64, 7, 7)])
def test_forced_passes_run_at_every_size(cin, cout, n, h, w):
    assert run_kernel(layer_of(cin, cout), n, h, w, kernel=5) == "passes"


# (cin, cout, keywords of the layer, n, h, w, kernel)
AUTO = [
    (512, 512, {}, 1, 14, 14, "rows"),            # few columns
    (512, 512, {}, 256, 14, 14, "strip"),
    (128, 128, {}, 64, 56, 56, "lds rows"),       # up to 160 input channels, many columns
    (160, 960, {}, 128, 7, 7, "lds rows"),
    (161, 960, {}, 128, 7, 7, "strip"),
    (64, 128, {}, 64, 1, 3, "strip"),             # planes of fewer than 4 columns: no row kernel
    (512, 512, {"block_rows": 4}, 256, 14, 14, "outer"),
    (960, 160, {}, 128, 7, 7, "outer"),           # too wide for a strip
    (1280, 320, {}, 128, 7, 7, "passes"),
    (112, 672, {"block_rows": 4, "storage": "f16"}, 512, 14, 14, "half"),
    (1217, 64, {"storage": "f16"}, 64, 14, 14, "direct"),
    (8, 8, {}, 0, 14, 14, "none"),
    (8, 8, {}, 1, 0, 14, "none"),
]


# Runs where the other kernel is the faster one by half to three times (us on the LDS rows and on it)
LONG_ROWS = [
    (144, 1024, 0.8, {}, 24, 28, 28, "strip"),                   # 62, 40
    (136, 768, 0.5, {}, 189, 10, 10, "strip"),                   # 93, 58
    (80, 818, 0.7, {}, 44, 20, 20, "strip"),                     # 45, 33
    (96, 576, 0.5, {}, 6, 56, 56, "strip"),                      # 59, 41
    (152, 512, 0.5, {"block_rows": 2}, 87, 14, 14, "strip"),     # 77, 44
    (120, 576, 0.5, {"block_rows": 4}, 70, 20, 20, "outer"),     # 68, 40
    (160, 768, 0.5, {"block_rows": 4}, 12, 28, 28, "outer"),     # 77, 25
    (144, 960, 0.8, {"block_rows": 4}, 180, 12, 12, "outer"),    # 58, 34
]


# Runs whose X is past the L2, which the row kernel reads again for every output channel
WIDE_X = [
    (512, 64, 0.9, {}, 11, 28, 28, "strip"),                     # 17 us on the row kernel, 9 on this one
    (1024, 91, 0.9, {}, 8, 20, 20, "outer"),                     # 18, 9
    (512, 45, 0.9, {}, 3, 56, 56, "strip"),                      # 14, 8
    (1160, 128, 0.95, {}, 22, 14, 14, "outer"),                  # 20, 13
    (940, 128, 0.9, {}, 16, 10, 10, "outer"),                    # 14, 9 (a long chain of such reads)
    (1118, 184, 0.9, {}, 2, 28, 28, "outer"),                    # 16, 10
]


@pytest.mark.parametrize("cin,cout,s,kw,n,h,w,name", LONG_ROWS + WIDE_X)
def test_row_kernels_only_where_they_are_the_faster_ones(cin, cout, s, kw, n, h, w, name):
    assert run_kernel(layer_of(cin, cout, s, **kw), n, h, w) == name


@pytest.mark.parametrize("cin,cout,kw,n,h,w,name", AUTO)
def test_automatic_choice(cin, cout, kw, n, h, w, name):
    assert run_kernel(layer_of(cin, cout, **kw), n, h, w) == name


@pytest.mark.parametrize("option", ["group_lanes", "waves", "pipe_sets", "regions", "lane_cols", "reorder"])
def test_layout_options_keep_the_kernels_that_they_lay_out(option):
    """The half and the row kernels have no lane groups, bundles or strip
    parts: a caller who sets one of these gets a kernel that uses it."""
    value = {"group_lanes": 8, "waves": 5, "pipe_sets": 1, "regions": 2, "lane_cols": 4, "reorder": 0}[option]
    assert run_kernel(layer_of(256, 256), 4, 14, 14) == "rows"
    assert run_kernel(layer_of(256, 256), 4, 14, 14, **{option: value}) == "strip"
    assert run_kernel(layer_of(64, 96), 64, 28, 28) == "lds rows"
    assert run_kernel(layer_of(64, 96), 64, 28, 28, **{option: value}) in ("strip", "indexed")
    f16 = layer_of(64, 96, storage="f16")
    assert run_kernel(f16, 64, 28, 28) == "half"
    assert run_kernel(f16, 64, 28, 28, **{option: value}) == "strip"


@pytest.mark.parametrize("cin,cout,s,kw,h,w,name", [
    (1077, 10, 0.98, {}, 56, 56, "direct"),                   # us on the half kernel and on this one: 98, 9.7
    (890, 8, 0.95, {"block_rows": 2}, 28, 28, "direct"),      # 122, 14
    (420, 14, 0.98, {}, 28, 28, "strip"),                     # 21, 9
    (17, 8, 0.85, {"block_rows": 2}, 20, 20, "strip"),        # 11, 5
    (1002, 12, 0.95, {"block_rows": 4}, 7, 7, "direct"),      # 92, 49
    (477, 628, 0.98, {"block_rows": 4}, 2, 2, "outer"),       # 17, 9
    (112, 672, 0.9, {"block_rows": 4}, 14, 14, "half"),
    (1077, 64, 0.9, {}, 56, 56, "half"),
    (320, 628, 0.98, {"block_rows": 4}, 2, 2, "half"),
])
def test_half_kernel_where_its_products_are_worth_it(cin, cout, s, kw, h, w, name):
    """By the layer and the plane only: an image takes the same kernel, and
    gives the same bits, in every batch."""
    layer = layer_of(cin, cout, s, storage="f16", **kw)
    assert {run_kernel(layer, n, h, w) for n in (1, 26, 617, 4096)} == {name}


def test_half_kernel_only_where_its_workgroups_fit_one_launch():
    """A launch has fewer than 2^32 threads; the half kernel's workgroups take
    one tile each, so the longest runs take the kernel that loops over tiles."""
    layer = layer_of(8, 8, 0.5, storage="f16")
    assert run_kernel(layer, 1 << 27, 1, 1) == "half"
    assert run_kernel(layer, 1 << 30, 1, 1) == "strip"
    assert run_kernel(layer, 40 << 20, 7, 7) == "strip"
    assert run_kernel(layer_of(8, 8, 0.5, storage="f16", block_rows=4), 1 << 30, 1, 1) in ("strip", "outer")


def test_depthwise_stage_counts_output_columns():
    from synth import make_depthwise
    layer = layer_of(32, 64)
    kw, kb = make_depthwise(32, 5)
    plan = Plan.fused(64, 32, 1, layer.row_ptr, layer.col_idx, layer.values, layer.bias, "relu", kw, kb, "relu", 2,
                      host_only=1)
    try:
        assert plan.run_kernel(1, 15, 15) == "strip"
    finally:
        plan.close()


def test_arguments():
    lib = sp.load_library()
    k = ctypes.c_int32(7)
    plan = Plan.from_layer(layer_of(8, 8), host_only=1)
    try:
        assert lib.spconv_plan_run_kernel(None, 1, 1, 1, ctypes.byref(k)) == spconv.E_ARG
        assert lib.spconv_plan_run_kernel(plan.handle, 1, 1, 1, None) == spconv.E_ARG
        assert lib.spconv_plan_run_kernel(plan.handle, -1, 1, 1, ctypes.byref(k)) == spconv.E_ARG
        assert lib.spconv_plan_run_kernel(plan.handle, 1 << 16, 1 << 10, 1 << 10, ctypes.byref(k)) == spconv.E_SHAPE
    finally:
        plan.close()
