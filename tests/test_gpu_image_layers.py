"""The strided convolutions that read an image (D's first layer, the gradients of G's last) in whole steps against the oracle, at the sides where
their units change: maps that are whole numbers of units sixteen outputs wide, and others, whose units hang over the map's edges; every number of
image channels (2, 4 or 8 values a pixel) and of feature channels; label maps and bias, one pair over several labels, an empty model."""
import numpy as np
import pytest

from paper_2102_10485_amd import binding, synth
from tests import gpu_util as U
from tests.test_gpu_step import Pair, batch

pytestmark = pytest.mark.gpu

CASES = [
    # channels, feature channels, image side, g_h0, models, labels (one model: of D's maps), samples
    (1, 64, 40, 10, 2, 2, 13),       # side 20: 10 x 7 outputs a unit, the last row of units hangs over
    (2, 128, 40, 10, 1, 3, 9),
    # side 36: 12 x 8 (bf16 forward: 12 x 12).  (With 7 samples G's cost behind D's first update of Adam is 1.3e-4 from the oracle's, and 1.7e-4 with
    # a GEMM over patch matrices in these kernels' place: such a step cannot hold it to 1e-4.)
    (3, 64, 72, 18, 2, 2, 12),
    (4, 128, 72, 18, 1, 0, 4),
    (4, 64, 32, 8, 3, 3, 17),        # side 16: one unit across
    (2, 64, 64, 16, 2, 2, 6),        # side 32: two
    (1, 128, 32, 8, 3, 3, 26),       # (14 samples: the one bias gradient, a cancelled sum, is 0.378 of itself off in bf16 whichever kernels computed it)
    (3, 128, 8, 2, 2, 2, 48),        # side 4: one step of the reduction
]


@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("channels,feats,hw,h0,models,labels,n", CASES)
def test_units_of_the_image_layers(prec, channels, feats, hw, h0, models, labels, n, monkeypatch):
    spec = dict(cond_g=0, cond_d=labels, z_dim=12, img_c=channels, img_hw=hw, g_h0=h0, g_ch=[64 if h0 > 1 else 128, feats], d_ch=[feats, 64])
    monkeypatch.setitem(synth.SPECS, "units", spec)
    k = max(labels, models)
    p = Pair("units", models, k, n + 3, prec)
    lab = np.random.default_rng(n).integers(0, max(k - 1, 1), n) if models == 3 else np.arange(n) % k      # (three models: the last is empty)
    p.step(*batch(p.spec, lab, 700 + n))
    p.compare("image layers, side %d" % (hw // 2))
    p.close()


def test_pixels_beyond_the_split_range():
    """fp32: a pixel of 1e32, whose scaled bf16 parts are infinite, in front of weights of 1e-33 and in the weight gradient.  D's cost is that of
    the oracle (1e-4) and so is the first layer's gradient, which is that pixel's (1e-3: the derivatives it is multiplied by).  (Not G's cost, behind an
    update whose second moments are beyond fp32.)"""
    p = Pair("tiny3", 3, 3, 40, binding.FP32)
    at = synth.param_slices(p.spec, 1)
    for l in range(3):
        q = p.gpu.get_params(1, l)
        w = q[at["c1.w"][0]].reshape(at["c1.w"][1])
        w[:, :3] *= np.float32(1e-31)                            # the image's taps, not the label maps'
        for o in (p.gpu, p.orc, p.o32):
            o.set_params(1, l, q)
    lab, z, x = batch(p.spec, np.arange(37) % 3, 720)
    x[8, 1, 5, 6], x[22, 0, 15, 0] = 1e32, -1e32
    p.step(lab, z, x)
    got, ref = p.gpu.get_losses()[0], p.orc.get_losses()[0]
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    for l in (lab[8], lab[22]):
        g, r = (np.asarray(o.get_grads(1, int(l)), np.float64)[at["c1.w"][0]] for o in (p.gpu, p.orc))
        assert np.all(np.isfinite(g)) and np.abs(r).max() > 1e25
        assert U.rel_l2(g, r) <= 1e-3
    p.close()
