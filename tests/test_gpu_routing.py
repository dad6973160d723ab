"""The routing kernel (GPU): large batches, many models, tables in LDS and beyond it.  The expected result is the definition itself, written out with numpy: a
stable partition of the flat batch by model (Eq. 5: pair k sees the samples of label k, in their order)."""
import numpy as np
import pytest

from paper_2102_10485_amd import binding, synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _step_and_routing(spec_name, n_models, n_labels, lab, seed):
    torch = U.torch_mod()
    spec = synth.SPECS[spec_name]
    n = len(lab)
    g = binding.Gan(binding.make_config(spec, n_models, n_labels, n, binding.BF16), torch.cuda.current_stream().cuda_stream)
    rng = np.random.default_rng(seed)
    z = rng.normal(size=(n, spec["z_dim"])).astype(np.float32)
    x = np.tanh(rng.normal(size=(n, spec["img_c"], spec["img_hw"], spec["img_hw"]))).astype(np.float32)
    dl, dz, dx = (torch.from_numpy(a).cuda() for a in (lab, z, x))
    g.train_step(dl.data_ptr(), dz.data_ptr(), dx.data_ptr(), n)
    jd, jg, cnt = g.get_losses()
    perm, offs = g.get_routing(n)
    g.close()
    return perm, offs, cnt, jd, jg


def _expected(lab, n_models):
    model = np.zeros_like(lab) if n_models == 1 else lab
    counts = np.bincount(model, minlength=n_models)
    return np.argsort(model, kind="stable").astype(np.int32), np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), counts


def test_one_pair_with_a_large_batch():
    rng = np.random.default_rng(1)
    lab = rng.integers(0, 4, 40000).astype(np.int32)                  # five trips of 512 samples for every wave
    perm, offs, cnt, jd, jg = _step_and_routing("tiny", 1, 4, lab, 2)
    eperm, eoffs, ecnt = _expected(lab, 1)
    assert np.array_equal(perm, eperm) and np.array_equal(offs, eoffs) and np.array_equal(cnt, ecnt)
    assert np.all(np.isfinite(jd)) and np.all(np.isfinite(jg))


def test_many_models_and_one_without_samples():
    L = 130                                                            # three trips of 64 models in the prefix scans
    rng = np.random.default_rng(3)
    lab = rng.integers(0, L, 1000).astype(np.int32)
    lab[lab == 7] = 8                                                  # one model without samples
    perm, offs, cnt, jd, jg = _step_and_routing("tiny0", L, L, lab, 4)
    eperm, eoffs, ecnt = _expected(lab, L)
    assert ecnt[7] == 0 and ecnt.min() == 0
    assert np.array_equal(perm, eperm) and np.array_equal(offs, eoffs) and np.array_equal(cnt, ecnt)
    assert np.all(np.isfinite(jd)) and np.all(np.isfinite(jg)) and jd[7] == 0 and jg[7] == 0


@pytest.mark.parametrize("L,n", [(1, 1), (3, 64), (64, 1025), (65, 8193), (2161, 3000), (2162, 3000), (2200, 5000)])
def test_shares_of_the_waves_and_tables_beyond_lds(L, n):
    """Sixteen waves share the batch 64 samples at a time, eight such groups in flight; labels outside the range are dropped wherever
    they stand; the tables of 2161 models are the largest that fit LDS (18 L + 1 integers in 152 KiB), those of more are in global memory."""
    rng = np.random.default_rng(L + n)
    lab = rng.integers(0, L, n).astype(np.int32)
    bad = rng.random(n) < 0.05
    if n > 1:
        bad[[0, n - 1]] = True
        lab[bad] = rng.choice([-2, -1, L, 1 << 30], int(bad.sum()))
    torch = U.torch_mod()
    spec = dict(synth.SPECS["tiny0"])
    g = binding.Gan(binding.make_config(spec, L, L, n, binding.BF16), torch.cuda.current_stream().cuda_stream)
    z = torch.randn((n, spec["z_dim"]), device="cuda")
    x = torch.randn((n, spec["img_c"], spec["img_hw"], spec["img_hw"]), device="cuda").tanh()
    dl = torch.from_numpy(lab).cuda()
    g.train_step(dl.data_ptr(), z.data_ptr(), x.data_ptr(), n)
    keep = np.flatnonzero(~bad) if n > 1 else np.arange(n)
    eperm, eoffs, ecnt = _expected(lab[keep], L)
    _, _, cnt, st = g.get_losses(check=False)
    perm, offs = g.get_routing(n)
    g.close()
    assert st == (binding.GAN_E_LABEL if n > 1 else binding.GAN_OK)
    assert np.array_equal(offs, eoffs) and np.array_equal(cnt, ecnt)
    assert np.array_equal(perm[:len(keep)], keep[eperm])
