"""The first convolution on short and long runs (runs on an MI355X).

A short run shares the output channels of a pixel over several workgroups, a
long one gives all of them to one.  Each output is the same sum in the same
order either way, so an image alone and the same image among enough others
agree bit for bit; both agree with the oracle at |y - y_ref| <= 1e-5 * S + 1e-6
(S the sum of absolute terms of up to 72 fp32 products).
"""

import numpy as np
import pytest

import oracle
from gpu_util import note, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("cout,h,w,stride,act", [
    (1, 16, 16, 1, "none"),    # no channel to share
    (7, 1, 1, 1, "relu"),      # one pixel, fewer channels than two shares
    (9, 17, 16, 2, "relu6"),   # shares that do not divide the channels
    (33, 16, 17, 1, "none"),   # a plane that is not a multiple of the workgroup
])
def test_conv3x3_alone_and_among_others(cin, cout, h, w, stride, act):
    import torch
    from paper_1911_09723_amd import spconv_conv3x3_hwc
    rng = np.random.default_rng(cin * 100 + cout)
    n = 1024  # at least one workgroup an image
    x = rng.standard_normal((n, h, w, cin)).astype(np.float32)
    wt = rng.standard_normal((cout, 3, 3, cin)).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    ho, wo = (h - 1) // stride + 1, (w - 1) // stride + 1
    note("conv3x3 cin=%d cout=%d %dx%d stride %d %s" % (cin, cout, h, w, stride, act))
    gx, gw, gb = to_gpu(x), to_gpu(wt), to_gpu(b)
    y = torch.empty((n, cout, ho, wo), dtype=torch.float32, device="cuda")
    spconv_conv3x3_hwc(gx, gw, gb, act, stride, y, n, h, w, cin, cout)
    for i, m in ((0, 1), (n - 3, 3)):
        part = torch.full((m, cout, ho, wo), 9.5, dtype=torch.float32, device="cuda")
        spconv_conv3x3_hwc(gx[i:i + m].contiguous(), gw, gb, act, stride, part, m, h, w, cin, cout)
        torch.cuda.synchronize()
        assert torch.equal(part, y[i:i + m])
    y_ref, s = oracle.conv3x3_hwc_ref(x[:1], wt, b, act, stride)
    assert (np.abs(y[:1].cpu().numpy().astype(np.float64) - y_ref) <= 1e-5 * s + 1e-6).all()
