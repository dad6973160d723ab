"""Parity of the two rows next to the training step against the oracle (GPU): mixture sampling (Eq. 5: class draws
from the prior, then the per-label generators) and the one-way ANOVA F-statistic per channel (Section 4).

Class draws are integers decided in double on both sides: compared bit for bit.  Images: 1e-4 (fp32 storage) / 2e-2
(bf16 storage) relative L2 on the image scale.  F: all arithmetic is double on both sides and only the summation
order differs: 1e-9 relative."""
import numpy as np
import pytest

import oracle as O
from paper_2102_10485_amd import binding, synth
from tests import gpu_util as U
from tests.test_gpu_step import Pair, batch, TOL

pytestmark = pytest.mark.gpu


def _gpu_sample(p, prior, u, z, running=1):
    torch = U.torch_mod()
    n = len(u)
    shape = (n, p.spec["img_c"], p.spec["img_hw"], p.spec["img_hw"])
    out = torch.zeros(shape, dtype=torch.float32, device="cuda")
    labels = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    du, dz = torch.from_numpy(np.ascontiguousarray(u, np.float32)).cuda(), torch.from_numpy(np.ascontiguousarray(z, np.float32)).cuda()
    p.gpu.sample(prior, du.data_ptr(), dz.data_ptr(), n, out.data_ptr(), labels.data_ptr(), running)
    torch.cuda.synchronize()
    return out.cpu().numpy(), labels.cpu().numpy()


@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
def test_sample_small(prec):
    """Three tiny models with identical parameters on both sides (no training step in between: after one, single
    elements of the two parameter sets legitimately differ by 2 lr, which the near-cancelling running-statistics
    output would amplify; generation with trained statistics is covered in test_gpu_step.test_generate)."""
    p = Pair("tiny3", 3, 3, 64, prec)
    rng = np.random.default_rng(8)
    n = 50
    u = rng.random(n).astype(np.float32)
    u[:4] = [0.0, 0.25, 0.75, 0.99999994]                     # on the cumulative values of the prior below, and the ends
    zz = rng.normal(size=(n, p.spec["z_dim"])).astype(np.float32)
    prior = [0.25, 0.5, 0.25]
    for running in (1, 0):
        img, labels = _gpu_sample(p, prior, u, zz, running)
        rc, ref, ref_labels = p.orc.sample(prior, u, zz.astype(np.float64), use_running_stats=running)
        assert rc == 0
        np.testing.assert_array_equal(labels, ref_labels)
        assert U.rel_l2(img, ref, floor=0.1 * np.sqrt(ref.size)) <= TOL[prec]
    # a prior with empty classes, unnormalised
    img, labels = _gpu_sample(p, [0.0, 0.0, 5.0], u, zz)
    assert np.all(labels == 2)
    # bad priors are refused on the host
    with pytest.raises(binding.GanError):
        _gpu_sample(p, [0.0, 0.0, 0.0], u, zz)
    with pytest.raises(binding.GanError):
        _gpu_sample(p, [0.5, -0.5, 1.0], u, zz)
    p.close()


@pytest.mark.parametrize("channels,g_last", [(1, 64), (3, 128), (4, 64)])
@pytest.mark.parametrize("size", [1.0, 1e-34, 1e-35])
def test_small_features_in_front_of_the_image(channels, g_last, size, monkeypatch):
    """fp32: features so small that their bf16 parts would be lost unscaled, through the kernel onto the image.  Bound: three contractions
    of up to 5.7e-7 (a chain of 1024 multiply-adds, tests/test_fp32_products.py), their normalisations and tanh, doubled; without the
    scale the error is 1.6e-5 at 1e-34 and ten times that at 1e-35."""
    monkeypatch.setitem(synth.SPECS, "faint", dict(cond_g=0, cond_d=0, z_dim=20, img_c=channels, img_hw=16, g_h0=4, g_ch=[64, g_last], d_ch=[64, 64]))
    p = Pair("faint", 2, 2, 40, binding.FP32)
    at = synth.param_slices(p.spec, 0)
    for l in range(2):
        q = p.gpu.get_params(0, l)
        q[at["bn1.gamma"][0]] *= np.float32(size)
        q[at["ct2.w"][0]] *= np.float32(1e-4 / size)             # largest 1e30: within the range of the scaled parts
        p.gpu.set_params(0, l, q)
        p.orc.set_params(0, l, q)
    rng = np.random.default_rng(23)
    n = 37
    lab = (np.arange(n) % 2).astype(np.int32)
    z = rng.normal(size=(n, p.spec["z_dim"])).astype(np.float32)
    out = U.torch_mod().zeros((n, channels, 16, 16), device="cuda")
    dl, dz = U.dev(lab), U.dev(z)
    p.gpu.generate(dl.data_ptr(), dz.data_ptr(), n, out.data_ptr(), 1)
    rc, ref = p.orc.generate(lab, z.astype(np.float64), 1)
    assert rc == 0 and np.abs(ref).max() > 0
    assert U.rel_l2(out.cpu().numpy(), ref) <= 4e-6
    p.close()


@pytest.mark.parametrize("channels,g_last", [(1, 64), (3, 128), (4, 64)])
def test_values_beyond_the_split_range_through_the_generator(channels, g_last, monkeypatch):
    """fp32: one sample's noise holds a value whose parts are infinite, and every layer behind it sums far above 2^80.  Linear layer, transposed
    convolutions and the kernel onto the image compute what fp32 arithmetic gives (pixels of plus or minus one there), and the samples
    beside it are as accurate as ever."""
    monkeypatch.setitem(synth.SPECS, "bright", dict(cond_g=0, cond_d=0, z_dim=20, img_c=channels, img_hw=24, g_h0=6, g_ch=[64, g_last],
                                                    d_ch=[64, 64]))
    p = Pair("bright", 2, 2, 40, binding.FP32)
    rng = np.random.default_rng(29)
    n = 37
    lab = (np.arange(n) % 2).astype(np.int32)
    z = rng.normal(size=(n, p.spec["z_dim"])).astype(np.float32)
    z[8, 3], z[21, 0] = 1e38, -1e38
    out = U.torch_mod().zeros((n, channels, 24, 24), device="cuda")
    dl, dz = U.dev(lab), U.dev(z)
    p.gpu.generate(dl.data_ptr(), dz.data_ptr(), n, out.data_ptr(), 1)
    rc, ref = p.orc.generate(lab, z.astype(np.float64), 1)
    got = out.cpu().numpy()
    loud = np.isin(np.arange(n), [8, 21])
    assert rc == 0 and np.all(np.abs(ref[loud]) == 1.0)
    np.testing.assert_array_equal(got[loud], ref[loud])
    assert U.rel_l2(got[~loud], ref[~loud]) <= 4e-6                 # as for faint features above
    p.close()


def test_sample_config2_full_size_bf16():
    """6400 draws over 100 labels with a rank-Zipf prior: every label bit-exact; images of two labels against the
    oracle (with the running statistics every image depends on its own noise row only)."""
    w = synth.Workload(2)
    models = [0, 99]
    p = Pair("cifar", 100, 100, w.n, binding.BF16, seed=w.seed, oracle_models=models)
    rng = np.random.default_rng(9)
    prior = 1.0 / np.arange(1, 101) ** 1.1
    u = rng.random(w.n).astype(np.float32)
    z = rng.normal(size=(w.n, p.spec["z_dim"])).astype(np.float32)
    img, labels = _gpu_sample(p, prior, u, z)
    rc, want = O.draw_labels(prior, u)
    assert rc == 0
    np.testing.assert_array_equal(labels, want)
    assert np.bincount(labels, minlength=100)[0] > np.bincount(labels, minlength=100)[99]
    for k in models:
        rows = np.where(labels == k)[0]
        assert rows.size > 0
        rc, ref = p.orc.generate(np.full(rows.size, k, np.int32), z[rows].astype(np.float64), use_running_stats=1, only_model=k)
        assert U.rel_l2(img[rows], ref, floor=0.1 * np.sqrt(ref.size)) <= TOL[binding.BF16]
    p.close()


def _gpu_anova(gan, lab, img):
    torch = U.torch_mod()
    dl = torch.from_numpy(np.ascontiguousarray(lab, np.int32)).cuda()
    di = torch.from_numpy(np.ascontiguousarray(img, np.float32)).cuda()
    return gan.anova_f(dl.data_ptr(), di.data_ptr(), len(lab), img.shape[1])


@pytest.mark.parametrize("config", [1, 2, 4])
def test_anova_f_of_the_workloads(config):
    torch = U.torch_mod()
    w = synth.Workload(config)
    gan = binding.Gan(binding.make_config(w.spec, w.n_models, w.n_labels, w.n, binding.FP32), torch.cuda.current_stream().cuda_stream)
    lab = w.labels()
    img = w.images(lab)
    st, F = _gpu_anova(gan, lab, img)
    rc, ref = O.anova_f(lab, img, w.n_labels)
    assert st == 0 and rc == 0
    np.testing.assert_allclose(F, ref, rtol=1e-9)
    assert np.all(F > 10.0)
    gan.close()


def test_anova_f_edge_cases():
    torch = U.torch_mod()
    spec = synth.SPECS["tiny0"]                                 # unconditional networks: any number of labels
    C_, H_ = spec["img_c"], spec["img_hw"]
    gan = binding.Gan(binding.make_config(spec, 1, 5, 300, binding.FP32), torch.cuda.current_stream().cuda_stream)
    rng = np.random.default_rng(12)
    n = 257                                                     # ragged against the 256-thread reductions
    lab = rng.integers(0, 5, n).astype(np.int32)
    img = (rng.normal(size=(n, C_, H_, H_)) * 0.3 + 0.05 * lab[:, None, None, None]).astype(np.float32)
    st, F = _gpu_anova(gan, lab, img)
    rc, ref = O.anova_f(lab, img, 5)
    assert st == 0
    np.testing.assert_allclose(F, ref, rtol=1e-9)
    # labels outside the range are ignored; a class may be empty
    lab2 = lab.copy()
    lab2[lab2 == 3] = 9
    lab2[:3] = -1
    st, F2 = _gpu_anova(gan, lab2, img)
    rc, ref2 = O.anova_f(lab2, img, 5)
    assert st == 0 and rc == 0
    np.testing.assert_allclose(F2, ref2, rtol=1e-9)
    # one class only: no statistic
    st, F3 = _gpu_anova(gan, np.zeros(n, np.int32), img)
    assert st == binding.GAN_E_STATE and np.all(F3 == 0)
    # the worked example of the oracle's pins: F = 13
    vals = np.array([1, 2, 3, 2, 3, 4, 5, 6, 7], np.float32)
    ex = np.broadcast_to(vals[:, None, None, None], (9, C_, H_, H_)).copy()
    st, F4 = _gpu_anova(gan, np.array([0, 0, 0, 1, 1, 1, 2, 2, 2], np.int32), ex)
    assert st == 0
    np.testing.assert_allclose(F4, [13.0] * C_, rtol=1e-12)
    gan.close()


@pytest.mark.parametrize("hw,n", [(28, 37), (30, 10), (4, 70)])
def test_anova_f_odd_sizes_and_unaligned_images(hw, n):
    """Images whose pixel count is no multiple of the 256 floats one trip takes, and a buffer off 16-byte alignment."""
    torch = U.torch_mod()
    rng = np.random.default_rng(hw + n)
    lab = rng.integers(0, 5, n).astype(np.int32)
    img = np.tanh(rng.normal(size=(n, 3, hw, hw)) + 0.3 * lab[:, None, None, None]).astype(np.float32)
    rc, ref = O.anova_f(lab, img, 5)
    dl = torch.from_numpy(lab).cuda()
    for shift in (0, 1):
        buf = torch.zeros(img.size + shift, dtype=torch.float32, device="cuda")
        buf[shift:] = torch.from_numpy(img.reshape(-1)).cuda()
        st, F = binding.anova_f_static(dl.data_ptr(), buf.data_ptr() + 4 * shift, n, 5, 3, hw, torch.cuda.current_stream().cuda_stream)
        assert rc == 0 and st == binding.GAN_OK
        np.testing.assert_allclose(F, ref, rtol=1e-9)


@pytest.mark.parametrize("hw,n", [(5, 37), (7, 64), (2, 8192 + 37)])
def test_anova_f_odd_sides_and_more_images_than_one_trip(hw, n):
    """Pixel counts that are no multiple of 4 in an aligned buffer, and more than the 8192 images whose labels a block takes at once, with
    a label that occurs behind them only."""
    torch = U.torch_mod()
    rng = np.random.default_rng(hw + n)
    lab = rng.integers(0, 4, n).astype(np.int32)
    lab[-5:] = 4
    img = np.tanh(rng.normal(size=(n, 3, hw, hw)) + 0.3 * lab[:, None, None, None]).astype(np.float32)
    rc, ref = O.anova_f(lab, img, 5)
    dl, dx = U.dev(lab), U.dev(img)
    st, F = binding.anova_f_static(dl.data_ptr(), dx.data_ptr(), n, 5, 3, hw, torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and st == binding.GAN_OK
    np.testing.assert_allclose(F, ref, rtol=1e-9)


@pytest.mark.parametrize("n", [1023, 1025, 5003, 8192])
def test_anova_f_of_uneven_labels(n):
    """One label with most of the images (more than the four means a lane keeps between the passes), one with a single image, some with
    none, in lists that end inside and at the end of a wave."""
    rng = np.random.default_rng(n)
    lab = np.where(rng.random(n) < 0.9, 6, rng.integers(0, 4, n)).astype(np.int32)
    lab[n // 2] = 5
    img = np.tanh(rng.normal(size=(n, 2, 4, 4)) + 0.3 * lab[:, None, None, None]).astype(np.float32)
    rc, ref = O.anova_f(lab, img, 8)
    dl, dx = U.dev(lab), U.dev(img)
    st, F = binding.anova_f_static(dl.data_ptr(), dx.data_ptr(), n, 8, 2, 4, U.torch_mod().cuda.current_stream().cuda_stream)
    assert rc == 0 and st == binding.GAN_OK
    np.testing.assert_allclose(F, ref, rtol=1e-9)            # sums in double on both sides, as above


@pytest.mark.parametrize("n,K", [(8193, 3), (8193, 5), (24576, 12), (24577, 12), (40000, 2), (30000, 700)])
def test_anova_f_of_several_trips(n, K):
    """On both sides of the lines between lists of a label's images and sums without them: 8192 images, 2048 to a label, 24576 images."""
    rng = np.random.default_rng(n + K)
    lab = rng.integers(0, K, n).astype(np.int32)
    lab[rng.random(n) < 0.01] = K + 1                        # ignored
    img = np.tanh(rng.normal(size=(n, 2, 2, 2)) + 0.1 * (lab % 7)[:, None, None, None]).astype(np.float32)
    rc, ref = O.anova_f(lab, img, K)
    dl, dx = U.dev(lab), U.dev(img)
    st, F = binding.anova_f_static(dl.data_ptr(), dx.data_ptr(), n, K, 2, 2, U.torch_mod().cuda.current_stream().cuda_stream)
    assert rc == 0 and st == binding.GAN_OK
    np.testing.assert_allclose(F, ref, rtol=1e-9)            # sums in double on both sides, as above


def test_anova_f_after_a_failed_call_of_the_caller():
    """An error that some other HIP call of the thread left behind is not the analysis' own."""
    torch = U.torch_mod()
    rng = np.random.default_rng(4)
    n, K = 40, 3
    lab = (np.arange(n) % K).astype(np.int32)
    img = np.tanh(rng.normal(size=(n, 3, 16, 16)) + 0.3 * lab[:, None, None, None]).astype(np.float32)
    g = binding.Gan(binding.make_config(synth.SPECS["tiny3"], K, K, n, binding.FP32), torch.cuda.current_stream().cuda_stream)
    dl, dx = U.dev(lab), U.dev(img)
    torch.cuda.synchronize()
    assert g.lib.hipSetDevice(10000) != 0                    # refused by the runtime: no such device
    st, F = g.anova_f(dl.data_ptr(), dx.data_ptr(), n, 3)
    assert st == binding.GAN_OK
    np.testing.assert_allclose(F, O.anova_f(lab, img, K)[1], rtol=1e-9)
    g.close()
