"""The strided convolutions that read an image (D's first layer, the gradients of G's last) in whole steps against the oracle, at the sides where
their units change: maps that are whole numbers of units sixteen outputs wide, and others, whose units hang over the map's edges; every number of
image channels (2, 4 or 8 values a pixel) and of feature channels; label maps and bias, one pair over several labels, an empty model.  The kernels' own results
(single operations) element by element: exactly, of whole numbers whose sums every order adds without rounding, and against 64-bit sums."""
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


@pytest.fixture(scope="module")
def ctxs():
    st = U.torch_mod().cuda.current_stream().cuda_stream
    c = {p: binding.Gan(binding.make_config(synth.SPECS["tiny3"], 3, 3, 48, p), st) for p in (binding.FP32, binding.BF16)}
    yield c
    for g in c.values():
        g.close()


class Layer:
    """One image-side layer's operands, NCHW and in the order of the samples, and what 64-bit sums make of them.  images [segments][n][cb][2 hs][2 hs],
    w [groups][cs][cb + maps][4][4], bias [groups][cs], dy [segments][n][cs][hs][hs]."""

    def __init__(self, g, bf, groups, images, w, bias, dy, nchw, maps, rng):
        torch = U.torch_mod()
        self.g, self.bf, self.groups, self.nchw, self.maps = g, bf, groups, nchw, maps
        self.S, self.n, self.cb, side, _ = images.shape
        self.cs, self.hs, self.G = w.shape[1], side // 2, len(groups)
        self.offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
        self.images, self.w, self.bias, self.dy = images, w, bias, dy
        perm = rng.permutation(self.n).astype(np.int32)
        caller = np.empty((self.n,) + images.shape[2:], np.float32)
        caller[perm] = images[0]
        nhwc = images.transpose(0, 1, 3, 4, 2).copy()
        if nchw:
            nhwc[0] = 7.0                                             # (not to be read)
        self.d_img, self.d_real, self.d_perm = U.dev(U.pack(nhwc, bf)), U.dev(caller), U.dev(perm)
        self.d_w = U.dev(np.ascontiguousarray(w.transpose(0, 3, 4, 2, 1), np.float32))
        self.d_bias, self.d_offs = U.dev(bias.astype(np.float32)), U.dev(self.offs)
        self.d_dy = U.dev(U.pack(dy.transpose(0, 1, 3, 4, 2), bf))
        self.out = torch.full((self.S * self.n * self.hs * self.hs * self.cs,), 77, dtype=torch.int16 if bf else torch.float32, device="cuda")
        self.grad = torch.full((self.G, 16 * (self.cb + maps) * self.cs + self.cs + 4), 77.0, device="cuda")

    def _parts(self):
        self.g.op_wgrad_parts(self.S, 1)
        return self.d_img.data_ptr(), self.d_real.data_ptr() if self.nchw else None, self.d_perm.data_ptr()

    def run(self, size_samples=None, size_models=None):
        """forward [segments][n][cs][hs][hs]; gradients of weights [groups][cs][cb + maps][16], biases [groups][cs], pixel sums [groups][cb]"""
        try:
            src = self._parts()
            self.g.op_image_conv(*src, self.d_w.data_ptr(), self.d_bias.data_ptr(), self.out.data_ptr(), self.d_offs.data_ptr(), self.G, self.n, self.cb, self.cs,
                                 self.hs, self.maps)
            self.g.op_image_wgrad(*src, self.d_dy.data_ptr(), self.grad.data_ptr(), self.d_offs.data_ptr(), self.G, self.n, self.cb, self.cs, self.hs, self.maps,
                                  size_samples, size_models)
        finally:
            self.g.op_wgrad_parts(1, 1)
        out = U.unpack(self.out, self.bf, (self.S, self.n, self.hs, self.hs, self.cs)).transpose(0, 1, 4, 2, 3)
        g, taps = self.grad.cpu().numpy(), 16 * (self.cb + self.maps) * self.cs
        return out, g[:, :taps].reshape(self.G, 16, self.cb + self.maps, self.cs).transpose(0, 3, 2, 1), g[:, taps:taps + self.cs], g[:, taps + self.cs:taps + self.cs + self.cb]

    def reference(self):
        hs = self.hs
        pad = np.zeros((self.S, self.n, self.cb + self.maps, 2 * hs + 2, 2 * hs + 2))
        pad[:, :, :self.cb, 1:-1, 1:-1] = self.images
        out = np.empty((self.S, self.n, self.cs, hs, hs))
        dw = np.zeros((self.G, self.cs, self.cb + self.maps, 16))
        db, px = np.zeros((self.G, self.cs)), np.zeros((self.G, self.cb))
        for l in range(self.G):
            a, b = self.offs[l], self.offs[l + 1]
            if self.maps:
                pad[:, a:b, self.cb + l, 1:-1, 1:-1] = 1.0
            p = np.stack([pad[:, a:b, :, ky:ky + 2 * hs:2, kx:kx + 2 * hs:2] for ky in range(4) for kx in range(4)], 3)      # [S][n][c][tap][hs][hs]
            p = p.transpose(0, 1, 4, 5, 2, 3).reshape(-1, (self.cb + self.maps) * 16).astype(np.float64)
            w = self.w[l].reshape(self.cs, -1).astype(np.float64)
            out[:, a:b] = (p @ w.T + self.bias[l]).reshape(self.S, b - a, hs, hs, self.cs).transpose(0, 1, 4, 2, 3)
            d = self.dy[:, a:b].transpose(0, 1, 3, 4, 2).reshape(-1, self.cs).astype(np.float64)
            dw[l] = (d.T @ p).reshape(self.cs, self.cb + self.maps, 16)
            db[l], px[l] = d.sum(0), self.images[:, a:b].sum(axis=(0, 1, 3, 4), dtype=np.float64)
        return out, dw, db, px

    def own_maps(self, dw):
        """what of the weights' gradient is written: the image's channels and every group's own label map"""
        return np.concatenate([dw[:, :, :self.cb]] + ([np.stack([dw[l, :, self.cb + l:self.cb + l + 1] for l in range(self.G)])] if self.maps else []), 2)


def layer(g, bf, groups, cb, cs, hs, segments, nchw, maps, rng, whole):
    n, G = int(sum(groups)), len(groups)
    draw = (lambda m, *s: rng.integers(-m, m + 1, s).astype(np.float32)) if whole else (lambda m, *s: U.round_to(rng.normal(size=s).astype(np.float32), bf))
    return Layer(g, bf, groups, draw(2, segments, n, cb, 2 * hs, 2 * hs), draw(1, G, cs, cb + maps, 4, 4), draw(3, G, cs), draw(3, segments, n, cs, hs, hs), nchw,
                 maps, rng)


EXACT = [
    # group sizes, sizing batch (of as many models that a model's samples are one tile if that may be so long), segments, segment 0 from the caller's batch, label maps
    ([3, 0, 2], 5, 2, True, True),         # a sample a tile
    ([5, 4], 2100, 2, True, False),        # tiles of three samples (bf16) and of five (fp32): full ones, ragged ones
    ([7], 4900, 1, False, False),          # one tile of all seven
]


@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("groups,size,segments,nchw,maps", EXACT)
@pytest.mark.parametrize("hs", [2, 4, 7, 14, 16, 18, 20, 32])
@pytest.mark.parametrize("cs", [64, 128])
@pytest.mark.parametrize("cb", [1, 2, 3, 4])
def test_sums_of_whole_numbers(ctxs, prec, groups, size, segments, nchw, maps, hs, cs, cb):
    """Pixels up to 2, weights up to 1, gradients and biases up to 3 in size: sums below 256 (forward: 80 of 2, and 3) and below 2^24, which bf16 and fp32 hold.  Every
    element is pinned that way: the last pixels of an image, whose 8-byte loads may reach behind it in bf16 with one or three channels, those of units that
    hang over the map, and what the rings of requests hold behind the last unit."""
    bf = prec == binding.BF16
    rng = np.random.default_rng([hs, cs, cb, size])
    x = layer(ctxs[prec], bf, groups, cb, cs, hs, segments, nchw, len(groups) if maps else 0, rng, True)
    got, want = x.run(size, 700), x.reference()
    assert np.abs(want[0]).max() < 256 and max(np.abs(a).max() for a in want[1:]) < 2 ** 24
    assert np.array_equal(got[0], want[0]), "forward"
    assert np.array_equal(x.own_maps(got[1]), x.own_maps(want[1])), "weights' gradient"
    assert np.array_equal(got[2], want[2]), "bias"
    some = np.array(groups) > 0                               # (no samples: no pixel sums are written)
    assert np.array_equal(got[3][some], want[3][some]), "pixel sums"


@pytest.mark.parametrize("prec,chain", [(binding.FP32, 48), (binding.BF16, 162)])
@pytest.mark.parametrize("hs,cs", [(16, 128), (18, 128), (16, 64)])
def test_long_tiles_are_added_in_chains(ctxs, prec, chain, hs, cs):
    """A tile of eighty samples, of two segments: a wave's accumulator takes at most `chain` sums of 16 pixels before they go to its partial sums.  Every addition rounds by
    2^-24 of the running sum at most, which grows as the root of the terms: a chain of c leaves an error of 2^-24 sqrt(c / 2) of the result at most (root mean square over the
    elements), of c sums of 16 pixels and of the partial sums behind them.  In one chain of more than a thousand the error is 1.5 (bf16) to 3 times this bound."""
    bf = prec == binding.BF16
    per = 80
    n, hb = per, 128 // cs
    x = layer(ctxs[prec], bf, [n], 3, cs, hs, 2, False, 0, np.random.default_rng([hs, cs]), False)
    (_, got, _, px), (_, want, _, px_want) = x.run(per * (700 if bf else 480), 700), x.reference()
    parts = -(-2 * n * -(-hs * hs // 16) // hb // chain) * hb
    assert U.rel_l2(got, want) <= 2.0 ** -24 * np.sqrt((chain + parts) / 2)
    # The sums of a channel's N pixels of variance 1: a lane adds twelve pixels of a unit at most in fp32 (an addition to k of them errs by 2^-24 sqrt(k / 3), root mean
    # square: twelve by 2^-24 sqrt(24), N of them by 2^-24 sqrt(2 N)), the units in double, and the result is rounded twice (2^-24 sqrt(N / 3) each).  Four times that.
    assert np.max(np.abs(px - px_want)) <= 4 * 2.0 ** -24 * np.sqrt((2 + 2 / 3) * x.images[:, :, 0].size)


@pytest.mark.parametrize("hs", [4, 8, 16])
@pytest.mark.parametrize("cs", [64, 128])
@pytest.mark.parametrize("cb", [1, 3, 4])
@pytest.mark.parametrize("nchw", [True, False])
def test_pixels_without_a_split(ctxs, hs, cs, cb, nchw):
    """fp32: two pixels of 1e32, whose scaled bf16 parts are infinite: the products around them are taken again in fp32, forward for 32 output pixels and the gradient for
    the whole tile.  Forward, every output is held to 2e-6 of the sum of its terms' sizes (a chain of 64 products rounds each at most 2^-24 of that); of the gradient, each
    (channel, tap) column to 4e-6 of its own largest term sums (chains of up to 512)."""
    rng = np.random.default_rng([hs, cs, cb])
    x = layer(ctxs[binding.FP32], False, [3], cb, cs, hs, 2, nchw, 0, rng, False)
    images = x.images.copy()
    images[0, 1, 0, hs, hs - 1], images[1, 2, cb - 1, 2 * hs - 1, 2 * hs - 1] = 1e32, -1e32
    x = Layer(x.g, False, [3], images, x.w, x.bias, x.dy, nchw, 0, rng)
    got, want = x.run(3), x.reference()
    size = Layer(x.g, False, [3], np.abs(images), np.abs(x.w), np.abs(x.bias), np.abs(x.dy), nchw, 0, rng).reference()
    for k, bound in ((0, 2e-6), (1, 4e-6), (2, 4e-6)):
        assert np.all(np.isfinite(got[k])) and np.all(np.abs(got[k] - want[k]) <= bound * size[k]), (k, np.max(np.abs(got[k] - want[k]) / size[k]))


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
