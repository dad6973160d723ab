"""The parts of an update: the weight gradients' row splits added on the way, whole tiles of weights and quarters of them, the last layer's tiles in the
launch of the flat ranges, and the operand of the image-side layers written along with their weights.  Three contexts take the same steps:
plain, on a second stream (each layer's update in a launch of its own) and with every parameter read and set again between the steps (the operands
rebuilt from the parameters): the same sums in the same order, so parameters, moments and gradients are equal bit for bit.  That they are the
right ones is compared with the oracle where whole steps are."""
import numpy as np
import pytest

from paper_2102_10485_amd import binding, synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

CASES = [
    # image channels, G's channels, D's channels, g_h0, models, labels, D's label maps, samples
    (1, [128, 64], [64, 128], 4, 1, 10, 10, 64),          # 32 tiles a layer, row splits, several tables of one model
    (3, [128, 128], [128, 128], 4, 1, 1, 0, 40),          # no label maps
    (2, [128, 64], [64, 128], 4, 3, 3, 5, 48),            # several models, one without samples; maps of no table
    (4, [512, 256, 64], [64, 256, 512], 2, 1, 2, 2, 64),  # 512 tiles: quarters, the most that join
    (1, [512, 320, 64], [64, 320, 512], 2, 1, 2, 2, 64),  # 640: whole tiles, with row splits
]


@pytest.fixture(scope="module")
def ctxs():
    st = U.torch_mod().cuda.current_stream().cuda_stream
    c = {p: binding.Gan(binding.make_config(synth.SPECS["tiny3"], 3, 3, 48, p), st) for p in (binding.FP32, binding.BF16)}
    yield c
    for g in c.values():
        g.close()


@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("channels,g_ch,d_ch,h0,models,labels,maps,n", CASES)
def test_parts_of_the_update(prec, channels, g_ch, d_ch, h0, models, labels, maps, n):
    torch = U.torch_mod()
    spec = dict(cond_g=0, cond_d=maps, z_dim=12, img_c=channels, img_hw=h0 << len(g_ch), g_h0=h0, g_ch=g_ch, d_ch=d_ch)
    st = torch.cuda.current_stream().cuda_stream
    plain, side, again = ctxs = [binding.Gan(binding.make_config(spec, models, labels, n, prec, seed=5), st) for _ in range(3)]
    side.use_second_stream(True)
    for l in range(models):
        for which in (0, 1):
            p = synth.init_params(spec, which, np.random.default_rng([9, which, l]))
            for g in ctxs:
                g.set_params(which, l, p)
    rng = np.random.default_rng(n)
    for step in range(3):
        lab = np.arange(n) % labels
        empty = models - 1 if models > 1 and step == 1 else -1
        if empty >= 0:
            lab[lab == empty] = 0
        d_lab = torch.from_numpy(lab.astype(np.int32)).cuda()
        d_z = torch.from_numpy(rng.normal(size=(n, spec["z_dim"])).astype(np.float32)).cuda()
        d_x = torch.from_numpy(np.tanh(rng.normal(size=(n, channels, spec["img_hw"], spec["img_hw"]))).astype(np.float32)).cuda()
        for g in ctxs:
            g.train_step(d_lab.data_ptr(), d_z.data_ptr(), d_x.data_ptr(), n)
        torch.cuda.synchronize()
        for l in range(models):
            for which in (0, 1):
                want = (plain.get_params(which, l), *plain.get_opt_state(which, l)[:2], plain.get_grads(which, l))
                assert all(np.all(np.isfinite(w)) for w in want)
                for name, (at, _) in synth.param_slices(spec, which).items():        # of a model without samples: zero
                    if name.startswith("c") and name.endswith(".w"):
                        assert np.any(want[3][at]) == (l != empty), (step, l, which, name)
                for g in (side, again):
                    got = (g.get_params(which, l), *g.get_opt_state(which, l)[:2], g.get_grads(which, l))
                    for name, a, b in zip(("parameters", "m", "v", "gradients"), want, got):
                        assert np.array_equal(a, b), (step, l, which, name, np.abs(a - b).max())
                again.set_params(which, l, want[0])
    for g in ctxs:
        g.close()


def test_row_splits_are_added_in_the_stated_order(ctxs):
    """Bit for bit the sums that launch_sum_splits leaves: few values in many splits go through four sums, whose error is half to two thirds of one's."""
    torch = U.torch_mod()
    for prec, L, splits, cb, cs in [(binding.FP32, 1, 64, 64, 128), (binding.BF16, 1, 33, 64, 64), (binding.FP32, 3, 16, 64, 64), (binding.BF16, 1, 15, 64, 128),
                                    (binding.FP32, 1, 24, 128, 128), (binding.BF16, 1, 32, 128, 128), (binding.FP32, 10, 5, 256, 64)]:
        parts = np.random.default_rng(splits).normal(size=(splits, L, 16, cb, cs)).astype(np.float32)
        out = torch.full((L, 16, cb, cs), 7.0, device="cuda")
        ctxs[prec].op_split_sum(U.dev(parts).data_ptr(), out.data_ptr(), L, splits, cb, cs)
        chains = 4 if L * 4 * cb * cs < 65536 and splits >= 16 else 1
        sums = [np.zeros(parts.shape[1:], np.float32) for _ in range(chains)]
        for k in range(splits):
            sums[k % chains] = sums[k % chains] + parts[k]
        want = sums[0]
        for s in sums[1:]:
            want = want + s
        assert np.array_equal(out.cpu().numpy(), want), (prec, L, splits, cb, cs)
