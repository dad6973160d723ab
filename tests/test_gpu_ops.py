"""Per-kernel parity of the grouped implicit-GEMM engine against the oracle's direct loops (GPU).

Sizes span several 128-row tiles, a ragged tail, an empty group, and groups with different weights.
"""
import numpy as np
import pytest

import oracle as O
from paper_2102_10485_amd import binding, synth
from tests import fp32_products as F
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctxs():
    torch = U.torch_mod()
    torch.cuda.init()
    out = {}
    for prec in (binding.FP32, binding.BF16):
        cfg = binding.make_config(synth.SPECS["tiny"], 1, 4, 8, prec)
        out[prec] = binding.Gan(cfg, torch.cuda.current_stream().cuda_stream)
    yield out
    for g in out.values():
        g.close()


CASES = [
    # cb, cs, hs, group sizes
    (64, 128, 4, [5, 0, 19, 8]),
    (128, 64, 8, [3, 7]),
    (64, 64, 7, [9, 2, 4]),
    (256, 128, 2, [70, 1]),
    (128, 256, 4, [20, 5]),
    (64, 512, 2, [130]),
    (256, 512, 4, [33, 40]),       # 256-wide output tiles in both directions, several M-tiles per model
    (128, 128, 16, [3]),           # one sample is a whole 256-row tile
    (64, 128, 4, [1, 1, 2]),       # models with a single sample
    (64, 256, 8, [5, 0, 3]),       # down: 256-wide tiles of four samples each, ragged tails
    (256, 64, 8, [2, 7]),          # up: the same, per output phase
    (64, 256, 16, [2, 1]),         # down: one sample per 256-row tile
    (256, 64, 16, [1, 2]),         # up: one sample per tile
    (128, 64, 7, [3, 0, 6]),       # up: 256 x 128 tiles that do not share pixels
]


def tolerance(prec):
    return 2e-5 if prec == binding.FP32 else 1e-2


@pytest.mark.parametrize("tile_rows", [0, 64, 128, 256])
@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("cb,cs,hs,groups", CASES)
def test_conv_down_up_wgrad(ctxs, prec, cb, cs, hs, groups, tile_rows):
    """tile_rows: the forward-type kernel's tile height; with 256 the width follows the output channels (64, 128 or 256
    columns), and transposed convolutions in bf16 share the gathered pixels of two taps where the side allows it (not 2 and 7).  0: as a training step
    would choose for this size: 32 x 64 tiles with four groups of waves on a reduction, or 64 x 64 with two (256 -> 512 channels at side 4 down, 256 <- 64
    at sides 8 and 16 up).  Together the cases run every tile of the kernel without an epilogue, down and up."""
    torch = U.torch_mod()
    g = ctxs[prec]
    g.op_tile_rows(tile_rows)
    bf = prec == binding.BF16
    rng = np.random.default_rng(cb * 1000 + cs + hs)
    n = int(sum(groups))
    offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
    G = len(groups)
    W = U.round_to(rng.normal(0, 0.05, (G, cs, cb, 4, 4)), bf)          # [cs][cb][ky][kx] per group
    big = U.round_to(rng.normal(0, 1, (n, cb, 2 * hs, 2 * hs)), bf)     # NCHW for the oracle
    small = U.round_to(rng.normal(0, 1, (n, cs, hs, hs)), bf)
    w_up = np.ascontiguousarray(W.transpose(0, 3, 4, 2, 1)).reshape(G, 16, cb, cs)
    w_down = np.ascontiguousarray(W.transpose(0, 3, 4, 1, 2)).reshape(G, 16, cs, cb)
    d_offs = U.dev(offs)
    d_big = U.dev(U.pack(big.transpose(0, 2, 3, 1), bf))
    d_small = U.dev(U.pack(small.transpose(0, 2, 3, 1), bf))
    d_wup, d_wdown = U.dev(U.pack(w_up, bf)), U.dev(U.pack(w_down, bf))
    tol = tolerance(prec)

    # down: conv forward
    out = torch.zeros(n * hs * hs * cs, dtype=torch.int16 if bf else torch.float32, device="cuda")
    g.op_conv_down(d_big.data_ptr(), d_wdown.data_ptr(), out.data_ptr(), d_offs.data_ptr(), G, n, cb, cs, hs)
    got = U.unpack(out, bf, (n, hs, hs, cs)).transpose(0, 3, 1, 2)
    ref = np.concatenate([O.conv2d(big[offs[i]:offs[i + 1]], W[i], None) for i in range(G) if groups[i]])
    assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref)), "down"

    # up: transposed conv forward
    out = torch.zeros(n * 4 * hs * hs * cb, dtype=torch.int16 if bf else torch.float32, device="cuda")
    g.op_conv_up(d_small.data_ptr(), d_wup.data_ptr(), out.data_ptr(), d_offs.data_ptr(), G, n, cb, cs, hs)
    got = U.unpack(out, bf, (n, 2 * hs, 2 * hs, cb)).transpose(0, 3, 1, 2)
    ref = np.concatenate([O.conv_transpose2d(small[offs[i]:offs[i + 1]], W[i], None) for i in range(G) if groups[i]])
    assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref)), "up"

    # wgrad (fp32 output in both modes)
    dw = torch.full((G * 16 * cb * cs,), 7.0, dtype=torch.float32, device="cuda")
    g.op_conv_wgrad(d_big.data_ptr(), d_small.data_ptr(), dw.data_ptr(), d_offs.data_ptr(), G, n, cb, cs, hs)
    got = dw.cpu().numpy().reshape(G, 4, 4, cb, cs)
    for i in range(G):
        if groups[i] == 0:
            assert np.all(got[i] == 0)
            continue
        _, dW, _ = O.conv2d_bwd(big[offs[i]:offs[i + 1]], W[i], small[offs[i]:offs[i + 1]], need_dx=False)
        ref = dW.transpose(2, 3, 1, 0)                                   # [cs][cb][ky][kx] -> [ky][kx][cb][cs]
        assert np.max(np.abs(got[i] - ref)) <= 2e-5 * np.max(np.abs(ref)) * (50 if bf else 1), "wgrad group %d" % i


@pytest.mark.gpu
def test_probes_report_plausible_ceilings():
    """The register-only MFMA loop and the plain copy return rates of the right order for this chip."""
    U.torch_mod().cuda.set_device(0)
    bf = binding.probe_mfma(binding.BF16)
    fp = binding.probe_mfma(binding.FP32)
    cp = binding.probe_copy(1 << 28)
    assert 500.0 < bf < 2600.0          # published dense bf16 peak: 2.5 PFLOP/s
    assert 30.0 < fp < 170.0            # published fp32 matrix peak: 157.3 TFLOP/s
    assert 1000.0 < cp < 8200.0         # published HBM peak: 8 TB/s


@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("cin,cout,hs,groups", [(128, 128, 8, [3, 0, 2]), (128, 64, 16, [2, 1])])
def test_upsample_conv3_runs_on_the_transposed_convolution_engine(ctxs, prec, cin, cout, hs, groups):
    """The generator blocks the paper prints (Table 1: Upsample x2, then Conv k3 s1 p1) on the grouped k4 s2 p1
    transposed-convolution kernel with the summed taps W4 = A W3 A^T; reference: the oracle's literal upsampling
    followed by its 3 x 3 convolution."""
    from oracle import paper_nets as P
    torch = U.torch_mod()
    g = ctxs[prec]
    g.op_tile_rows(0)
    bf = prec == binding.BF16
    rng = np.random.default_rng(cin + cout + hs)
    n = int(sum(groups))
    offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
    G = len(groups)
    w3 = rng.normal(0, 0.05, (G, cout, cin, 3, 3))                       # [cout][cin][ky][kx] per group
    A = np.array([[0, 0, 1], [0, 1, 1], [1, 1, 0], [1, 0, 0]], float)
    w4 = U.round_to(np.einsum("ak,goikl,bl->gabio", A, w3, A), bf)       # [group][ky4][kx4][cin][cout], storage rounding
    small = U.round_to(rng.normal(0, 1, (n, cin, hs, hs)), bf)
    w_up = np.ascontiguousarray(w4.transpose(0, 1, 2, 4, 3)).reshape(G, 16, cout, cin)   # the kernel's [tap][cb][cs]
    d_offs = U.dev(offs)
    d_small = U.dev(U.pack(small.transpose(0, 2, 3, 1), bf))
    d_w = U.dev(U.pack(w_up, bf))
    out = torch.zeros(n * 4 * hs * hs * cout, dtype=torch.int16 if bf else torch.float32, device="cuda")
    g.op_conv_up(d_small.data_ptr(), d_w.data_ptr(), out.data_ptr(), d_offs.data_ptr(), G, n, cout, cin, hs)
    got = U.unpack(out, bf, (n, 2 * hs, 2 * hs, cout)).transpose(0, 3, 1, 2)
    # the summed taps are rounded to the storage type before the multiplication: the reference uses the same
    # rounded W4 through the pinned identity, and the literal form with the unrounded W3 bounds the difference
    ref4 = np.concatenate([O.conv_transpose2d(small[offs[i]:offs[i + 1]], w4[i].transpose(2, 3, 0, 1), None)
                           for i in range(G) if groups[i]])
    lit = np.concatenate([O.conv2d(P.upsample2(small[offs[i]:offs[i + 1]]), w3[i], None, 3, 1, 1)
                          for i in range(G) if groups[i]])
    tol = tolerance(prec)
    assert np.max(np.abs(got - ref4)) <= tol * np.max(np.abs(ref4))
    assert np.max(np.abs(got - lit)) <= (2e-5 if not bf else 2e-2) * np.max(np.abs(lit))


@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("cb,cs,hs,groups", [(64, 64, 32, [1, 1]), (64, 64, 64, [1]), (64, 128, 14, [3, 0, 2]), (128, 64, 5, [33, 1]),
                                             (8, 8, 7, [4]), (72, 136, 6, [5, 2]), (64, 256, 1, [70])])
def test_wgrad_row_decoding_and_narrow_tiles(ctxs, prec, cb, cs, hs, groups):
    """The weight gradient where its row decoding changes: sides of one K-chunk (32 rows in fp32, 64 in bf16) and above, sides
    that are no power of two (reciprocal products), a side of one, and outputs that fill no tile in either direction."""
    torch = U.torch_mod()
    g = ctxs[prec]
    bf = prec == binding.BF16
    rng = np.random.default_rng(cb + cs + hs)
    n, G = int(sum(groups)), len(groups)
    offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
    big = U.round_to(rng.normal(0, 1, (n, cb, 2 * hs, 2 * hs)), bf)
    small = U.round_to(rng.normal(0, 1, (n, cs, hs, hs)), bf)
    d_offs = U.dev(offs)
    d_big = U.dev(U.pack(big.transpose(0, 2, 3, 1), bf))
    d_small = U.dev(U.pack(small.transpose(0, 2, 3, 1), bf))
    dw = torch.full((G * 16 * cb * cs,), 7.0, dtype=torch.float32, device="cuda")
    g.op_conv_wgrad(d_big.data_ptr(), d_small.data_ptr(), dw.data_ptr(), d_offs.data_ptr(), G, n, cb, cs, hs)
    got = dw.cpu().numpy().reshape(G, 4, 4, cb, cs)
    for i in range(G):
        if groups[i] == 0:
            assert np.all(got[i] == 0)
            continue
        W = np.zeros((cs, cb, 4, 4))
        _, dW, _ = O.conv2d_bwd(big[offs[i]:offs[i + 1]], W, small[offs[i]:offs[i + 1]], need_dx=False)
        ref = dW.transpose(2, 3, 1, 0)
        # fp32 sums of up to 4096 products in another order; bf16 inputs are exact here, so only the sums differ too
        assert np.max(np.abs(got[i] - ref)) <= 2e-5 * np.max(np.abs(ref)), "wgrad group %d" % i


def test_fp32_values_without_a_bf16_split(ctxs):
    """fp32 contractions run on sums of bf16 parts.  Infinities, NaN and values that round to a bf16 infinity have no such parts:
    the results must be what fp32 arithmetic gives, and the other outputs must not notice.  Bounds as in the test above."""
    torch = U.torch_mod()
    g = ctxs[binding.FP32]
    cb, cs, hs, n = 64, 128, 4, 40
    rng = np.random.default_rng(11)
    big = rng.normal(0, 1, (n, 2 * hs, 2 * hs, cb)).astype(np.float32)
    small = rng.normal(0, 1, (n, hs, hs, cs)).astype(np.float32)
    big[3, 2, 5, 7], big[20, 0, 0, 1], big[31, 7, 7, 63], big[33, 4, 4, 0] = np.inf, -np.inf, np.nan, 3.4e38
    W = rng.normal(0, 0.05, (cs, cb, 4, 4)).astype(np.float32)
    offs = U.dev(np.array([0, n], np.int32))
    d_big, d_small = U.dev(big), U.dev(small)
    with np.errstate(all="ignore"):
        ref = O.conv2d(big.transpose(0, 3, 1, 2), W, None).transpose(0, 2, 3, 1)
        _, dW, _ = O.conv2d_bwd(big.transpose(0, 3, 1, 2), W, small.transpose(0, 3, 1, 2), need_dx=False)
        dW = dW.transpose(2, 3, 1, 0)
    for rows in (64, 128, 256):
        g.op_tile_rows(rows)
        out = torch.zeros((n, hs, hs, cs), device="cuda")
        d_w = U.dev(np.ascontiguousarray(W.transpose(2, 3, 0, 1)).reshape(16, cs, cb))
        g.op_conv_down(d_big.data_ptr(), d_w.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
        _same_classes(out.cpu().numpy(), ref)
    g.op_tile_rows(0)
    dw = torch.zeros((4, 4, cb, cs), device="cuda")
    g.op_conv_wgrad(d_big.data_ptr(), d_small.data_ptr(), dw.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
    _same_classes(dw.cpu().numpy(), dW)


def test_fp32_up_values_without_a_bf16_split(ctxs):
    """The same for the transposed convolution."""
    torch = U.torch_mod()
    g = ctxs[binding.FP32]
    cb, cs, hs, n = 64, 128, 4, 40
    rng = np.random.default_rng(12)
    small = rng.normal(0, 1, (n, hs, hs, cs)).astype(np.float32)
    small[3, 2, 3, 7], small[20, 0, 0, 1], small[31, 3, 3, 127], small[33, 1, 1, 0] = np.inf, -np.inf, np.nan, 3.4e38
    W = rng.normal(0, 0.05, (cs, cb, 4, 4)).astype(np.float32)
    offs = U.dev(np.array([0, n], np.int32))
    with np.errstate(all="ignore"):
        ref = O.conv_transpose2d(small.transpose(0, 3, 1, 2), W, None).transpose(0, 2, 3, 1)
    d_small, d_w = U.dev(small), U.dev(np.ascontiguousarray(W.transpose(2, 3, 1, 0)).reshape(16, cb, cs))
    for rows in (64, 128, 256):
        g.op_tile_rows(rows)
        out = torch.zeros((n, 2 * hs, 2 * hs, cb), device="cuda")
        g.op_conv_up(d_small.data_ptr(), d_w.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
        _same_classes(out.cpu().numpy(), ref)
    g.op_tile_rows(0)


@pytest.mark.parametrize("scales", [(1.0, 1.0), (1e-34, 1.0), (1.0, 1e-36), (1.2e-38, 1.0), (7e-40, 1e20), (1e-19, 1e-15), (1e15, 1e15)])
def test_fp32_products_are_no_less_accurate_than_a_chain_of_multiply_adds(ctxs, scales):
    """Operands of ordinary size, small, subnormal, and with sums beyond the range of the scaled parts.  What the bound tells apart is
    in tests/test_fp32_products.py."""
    torch = U.torch_mod()
    g = ctxs[binding.FP32]
    cb, cs, hs, n = 64, 64, 4, 3
    rng = np.random.default_rng(17)
    big = (rng.normal(size=(n, 2 * hs, 2 * hs, cb)) * scales[0]).astype(np.float32)
    small = (rng.normal(size=(n, hs, hs, cs)) * scales[0]).astype(np.float32)
    other = (rng.normal(size=(n, hs, hs, cs)) * scales[1]).astype(np.float32)
    w = (rng.normal(0, 0.05, (16, cb, cs)) * scales[1]).astype(np.float32)
    offs = U.dev(np.array([0, n], np.int32))
    d_big, d_small, d_other, d_wu, d_wd = U.dev(big), U.dev(small), U.dev(other), U.dev(w), U.dev(w.transpose(0, 2, 1))
    cols = F.columns_down(big)
    down, down_bound = F.reference(cols, w.reshape(16 * cb, cs))
    up, up_bound = F.reference(F.columns_up(small), w.transpose(0, 2, 1).reshape(16 * cs, cb))
    for rows in (64, 128, 256):
        g.op_tile_rows(rows)
        out = torch.zeros((n * hs * hs, cs), device="cuda")
        g.op_conv_down(d_big.data_ptr(), d_wd.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
        assert F.rel(out.cpu().numpy(), down) <= down_bound, rows
        out = torch.zeros((n * 4 * hs * hs, cb), device="cuda")
        g.op_conv_up(d_small.data_ptr(), d_wu.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
        assert F.rel(out.cpu().numpy(), up) <= up_bound, rows
    g.op_tile_rows(0)
    dw, dw_bound = F.reference(np.ascontiguousarray(cols.T), other.reshape(-1, cs))
    out = torch.zeros((16 * cb, cs), device="cuda")
    g.op_conv_wgrad(d_big.data_ptr(), d_other.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
    assert F.rel(out.cpu().numpy(), dw) <= dw_bound


def _same_classes(got, ref):
    with np.errstate(over="ignore"):
        ref = ref.astype(np.float32)                                     # what overflows in fp32 is an infinity there
    assert not np.isfinite(ref).all()
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    np.testing.assert_array_equal(got[inf], ref[inf])
    huge = np.isfinite(ref) & (np.abs(ref) > 1e30)
    assert np.all(np.abs(got[huge] / ref[huge] - 1) <= 2e-5)             # one product dwarfs the others there
    rest = np.isfinite(ref) & ~huge
    assert np.max(np.abs(got[rest] - ref[rest])) <= 2e-5 * np.max(np.abs(ref[rest]))


@pytest.mark.parametrize("cb,cs,hs,n", [(64, 128, 4, 40), (64, 256, 4, 200)])
def test_fp32_values_without_a_bf16_split_in_shared_reductions(ctxs, cb, cs, hs, n):
    """As above, on the tiles whose reduction several groups of waves share (the automatic choice at these sizes: 40 and 200 tiles)."""
    torch = U.torch_mod()
    g = ctxs[binding.FP32]
    g.op_tile_rows(0)
    rng = np.random.default_rng(13)
    big = rng.normal(0, 1, (n, 2 * hs, 2 * hs, cb)).astype(np.float32)
    big[3, 2, 5, 7], big[20, 0, 0, 1], big[31, 7, 7, 63], big[33, 4, 4, 0] = np.inf, -np.inf, np.nan, 3.4e38
    W = rng.normal(0, 0.05, (cs, cb, 4, 4)).astype(np.float32)
    with np.errstate(all="ignore"):
        ref = O.conv2d(big.transpose(0, 3, 1, 2), W, None).transpose(0, 2, 3, 1)
    out = torch.zeros((n, hs, hs, cs), device="cuda")
    offs, d_big, d_w = U.dev(np.array([0, n], np.int32)), U.dev(big), U.dev(np.ascontiguousarray(W.transpose(2, 3, 0, 1)).reshape(16, cs, cb))
    g.op_conv_down(d_big.data_ptr(), d_w.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
    _same_classes(out.cpu().numpy(), ref)


@pytest.mark.parametrize("rows", [0, 64, 128, 256])
def test_fp32_weights_without_a_bf16_split(ctxs, rows):
    """The weights' parts are made once and not where they are multiplied: weights beyond the parts' range must give what fp32 arithmetic
    gives (finite values and, with activations above one, infinities), in their columns and nowhere else, in both layouts."""
    torch = U.torch_mod()
    g = ctxs[binding.FP32]
    g.op_tile_rows(rows)
    cb, cs, hs, n = 64, 128, 4, 40
    rng = np.random.default_rng(14)
    big = rng.normal(0, 1, (n, 2 * hs, 2 * hs, cb)).astype(np.float32)
    small = rng.normal(0, 1, (n, hs, hs, cs)).astype(np.float32)
    W = rng.normal(0, 0.05, (cs, cb, 4, 4)).astype(np.float32)
    W[3, 5, 1, 2], W[70, 0, 0, 0], W[127, 63, 3, 3] = 3.3e38, 1e33, -3.3e38
    offs = U.dev(np.array([0, n], np.int32))
    with np.errstate(all="ignore"):
        down = O.conv2d(big.transpose(0, 3, 1, 2), W, None).transpose(0, 2, 3, 1)
        up = O.conv_transpose2d(small.transpose(0, 3, 1, 2), W, None).transpose(0, 2, 3, 1)
    d_big, d_small = U.dev(big), U.dev(small)
    d_wd, d_wu = U.dev(np.ascontiguousarray(W.transpose(2, 3, 0, 1))), U.dev(np.ascontiguousarray(W.transpose(2, 3, 1, 0)))
    out = torch.zeros((n, hs, hs, cs), device="cuda")
    g.op_conv_down(d_big.data_ptr(), d_wd.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
    _same_classes(out.cpu().numpy(), down)
    out = torch.zeros((n, 2 * hs, 2 * hs, cb), device="cuda")
    g.op_conv_up(d_small.data_ptr(), d_wu.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, cb, cs, hs)
    g.op_tile_rows(0)
    _same_classes(out.cpu().numpy(), up)


@pytest.mark.parametrize("tile_rows", [128, 256])
@pytest.mark.parametrize("cb,cs,hs,groups", [(128, 64, 12, [3, 0, 2]), (64, 64, 20, [2, 1]), (256, 64, 12, [4]), (64, 128, 28, [1, 1]), (256, 64, 5, [9])])
def test_conv_up_shared_pixels(ctxs, cb, cs, hs, groups, tile_rows):
    """Taps that share a stage of gathered pixels: sides that are no power of two, so that tiles start and end inside a row, and one side
    that the shared form does not take."""
    torch = U.torch_mod()
    g = ctxs[binding.BF16]
    g.op_tile_rows(tile_rows)
    rng = np.random.default_rng(cb + hs)
    n, G = int(sum(groups)), len(groups)
    offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
    W = U.round_to(rng.normal(0, 0.05, (G, cs, cb, 4, 4)), True)
    small = U.round_to(rng.normal(0, 1, (n, cs, hs, hs)), True)
    d_offs, d_small = U.dev(offs), U.dev(U.pack(small.transpose(0, 2, 3, 1), True))
    d_w = U.dev(U.pack(np.ascontiguousarray(W.transpose(0, 3, 4, 2, 1)).reshape(G, 16, cb, cs), True))
    out = torch.zeros(n * 4 * hs * hs * cb, dtype=torch.int16, device="cuda")
    g.op_conv_up(d_small.data_ptr(), d_w.data_ptr(), out.data_ptr(), d_offs.data_ptr(), G, n, cb, cs, hs)
    g.op_tile_rows(0)
    got = U.unpack(out, True, (n, 2 * hs, 2 * hs, cb)).transpose(0, 3, 1, 2)
    ref = np.concatenate([O.conv_transpose2d(small[offs[i]:offs[i + 1]], W[i], None) for i in range(G) if groups[i]])
    assert np.max(np.abs(got - ref)) <= tolerance(binding.BF16) * np.max(np.abs(ref))


@pytest.mark.parametrize("up,cin,cout,hs,groups", [
    (True, 64, 256, 4, [130]),             # tiles inside the first or last pixel row: two chunks, the fewest there are
    (True, 64, 512, 2, [1, 0, 70]),        # two and four chunks, a model of four rows
    (True, 192, 256, 5, [9, 2]),           # three channel lines, tiles that start inside a row
    (False, 64, 256, 4, [130, 1]),         # twelve chunks in tiles of the first and last pixel rows, sixteen in the others
    (False, 192, 512, 3, [30]),            # three channel lines
])
def test_tiles_multiplied_in_quarters(ctxs, up, cin, cout, hs, groups):
    """256 x 256 tiles in bf16: the smallest and odd numbers of chunks, rows past a model's end, exact products.  Inputs are small whole
    numbers, so sums are exact in fp32 and the result is the rounded exact one."""
    torch = U.torch_mod()
    g = ctxs[binding.BF16]
    g.op_tile_rows(256)
    rng = np.random.default_rng(cin + hs)
    n, G = int(sum(groups)), len(groups)
    offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
    cb, cs, side = (cout, cin, hs) if up else (cin, cout, 2 * hs)
    W = rng.integers(-3, 4, (G, cs, cb, 4, 4)).astype(np.float32)
    x = rng.integers(-3, 4, (n, cin, side, side)).astype(np.float32)
    d_offs, d_x = U.dev(offs), U.dev(U.pack(x.transpose(0, 2, 3, 1), True))
    d_w = U.dev(U.pack(np.ascontiguousarray(W.transpose(0, 3, 4, 2, 1) if up else W.transpose(0, 3, 4, 1, 2)).reshape(G, 16, cout, cin), True))
    out_side = 2 * hs if up else hs
    out = torch.zeros(n * out_side * out_side * cout, dtype=torch.int16, device="cuda")
    (g.op_conv_up if up else g.op_conv_down)(d_x.data_ptr(), d_w.data_ptr(), out.data_ptr(), d_offs.data_ptr(), G, n, cb, cs, hs)
    g.op_tile_rows(0)
    got = U.unpack(out, True, (n, out_side, out_side, cout)).transpose(0, 3, 1, 2)
    op = O.conv_transpose2d if up else O.conv2d
    ref = np.concatenate([op(x[offs[i]:offs[i + 1]], W[i], None) for i in range(G) if groups[i]])
    assert np.array_equal(got, U.round_to(ref, True))


@pytest.mark.parametrize("cb,cs,hs,groups", [
    (128, 256, 1, [3, 0, 130]),            # one chunk and three, the last one of two rows
    (128, 256, 2, [5, 16, 32, 33]),        # pixel rows in turn (16, 32 samples) and samples in turn
    (256, 512, 8, [1, 8, 9]),              # the same, one chunk a sample
    (384, 256, 4, [16, 7]),                # a tile over two taps
    (128, 512, 16, [1, 4]),                # chunks of four pixel rows; the top or bottom row's chunks left out
    (128, 256, 32, [2, 1]),                # the largest side
    (128, 256, 64, [1]), (192, 256, 4, [9]),       # not multiplied in quarters
])
def test_weight_gradient_in_quarters(ctxs, cb, cs, hs, groups):
    """256 x 256 tiles of the bf16 weight gradient: small whole numbers, so that every sum is exact in fp32."""
    torch = U.torch_mod()
    g = ctxs[binding.BF16]
    rng = np.random.default_rng(cb + hs)
    n, G = int(sum(groups)), len(groups)
    offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
    big = rng.integers(-3, 4, (n, 2 * hs, 2 * hs, cb)).astype(np.float32)
    small = rng.integers(-3, 4, (n, hs, hs, cs)).astype(np.float32)
    d_offs, d_big, d_small = U.dev(offs), U.dev(U.pack(big, True)), U.dev(U.pack(small, True))
    dw = torch.full((G, 4, 4, cb, cs), 7.0, dtype=torch.float32, device="cuda")
    g.op_conv_wgrad(d_big.data_ptr(), d_small.data_ptr(), dw.data_ptr(), d_offs.data_ptr(), G, n, cb, cs, hs)
    got = dw.cpu().numpy()
    pad = np.pad(big, ((0, 0), (1, 1), (1, 1), (0, 0)))
    for i in range(G):
        part = slice(offs[i], offs[i + 1])
        y = small[part].reshape(-1, cs)
        for ky in range(4):
            for kx in range(4):
                x = pad[part, ky:ky + 2 * hs:2, kx:kx + 2 * hs:2].reshape(-1, cb)
                assert np.array_equal(got[i, ky, kx], x.T @ y), (i, ky, kx)


@pytest.mark.parametrize("prec,cb,cs,hs,groups,segments,splits", [
    (binding.BF16, 128, 256, 8, [1, 3, 0], 2, 1),      # in quarters: one and three chunks to a segment
    (binding.BF16, 256, 256, 8, [8, 16], 2, 1),        # pixel rows in turn, seven and fourteen chunks, the first or last pixel row's left out
    (binding.BF16, 128, 256, 4, [16, 1], 2, 3),        # a share without rows; one of three of a chunk each
    (binding.BF16, 128, 256, 8, [16], 1, 2),           # the row that is left out at the start of a share and at the end of one
    (binding.BF16, 128, 512, 8, [16, 3], 2, 8),        # shares that are a pixel row, all of it left out
    (binding.BF16, 128, 256, 8, [16], 2, 16),          # shares that are half of one
    (binding.BF16, 128, 256, 8, [24], 2, 5),           # shares that start inside a pixel row
    (binding.BF16, 128, 256, 32, [2], 2, 7),
    (binding.BF16, 64, 256, 8, [8, 3], 2, 3), (binding.BF16, 128, 128, 4, [16, 5], 2, 2), (binding.BF16, 128, 64, 7, [5], 2, 3),       # other tiles
    (binding.FP32, 128, 256, 8, [8, 1], 2, 3), (binding.FP32, 128, 64, 7, [4, 0, 2], 2, 2), (binding.FP32, 64, 128, 4, [9], 2, 1),
])
def test_weight_gradient_of_segments_and_row_splits(ctxs, prec, cb, cs, hs, groups, segments, splits):
    """What a step's weight gradients run and the cases above do not: two segments, and rows shared among blocks.  Small whole numbers, so
    that every sum is exact in fp32, the parts' sum included."""
    torch = U.torch_mod()
    g, bf = ctxs[prec], prec == binding.BF16
    rng = np.random.default_rng(cb + cs + hs + splits)
    n, G = int(sum(groups)), len(groups)
    offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
    big = rng.integers(-3, 4, (segments, n, 2 * hs, 2 * hs, cb)).astype(np.float32)
    small = rng.integers(-3, 4, (segments, n, hs, hs, cs)).astype(np.float32)
    d_offs, d_big, d_small = U.dev(offs), U.dev(U.pack(big, bf)), U.dev(U.pack(small, bf))
    dw = torch.full((splits, G, 4, 4, cb, cs), 7.0, dtype=torch.float32, device="cuda")
    g.op_wgrad_parts(segments, splits)
    try:
        g.op_conv_wgrad(d_big.data_ptr(), d_small.data_ptr(), dw.data_ptr(), d_offs.data_ptr(), G, n, cb, cs, hs)
    finally:
        g.op_wgrad_parts(1, 1)
    got = dw.cpu().numpy().astype(np.float64)
    got = got.sum(axis=0)
    pad = np.pad(big, ((0, 0), (0, 0), (1, 1), (1, 1), (0, 0)))
    for i in range(G):
        part = slice(offs[i], offs[i + 1])
        y = small[:, part].reshape(-1, cs)
        for ky in range(4):
            for kx in range(4):
                x = pad[:, part, ky:ky + 2 * hs:2, kx:kx + 2 * hs:2].reshape(-1, cb)
                assert np.array_equal(got[i, ky, kx], x.T @ y), (i, ky, kx)


@pytest.mark.parametrize("mode", ["down", "up"])
def test_fp32_weights_up_to_two_gibibytes(ctxs, mode):
    """A weight block of 1.45 GB: its three bf16 planes together are beyond what a 32-bit byte offset reaches, each by itself is not."""
    torch = U.torch_mod()
    g = ctxs[binding.FP32]
    g.op_tile_rows(0)
    C, N, n = 4736, 4800, 3
    gen = torch.Generator(device="cuda").manual_seed(3)
    W = torch.randn((16, N, C), device="cuda", generator=gen) * 0.02
    offs = U.dev(np.array([0, n], np.int32))
    side = 2 if mode == "down" else 1
    x = torch.randn((n, side, side, C), device="cuda", generator=gen)
    out = torch.zeros((n, 3 - side, 3 - side, N), device="cuda")
    if mode == "down":
        g.op_conv_down(x.data_ptr(), W.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, C, N, 1)
    else:
        g.op_conv_up(x.data_ptr(), W.data_ptr(), out.data_ptr(), offs.data_ptr(), 1, n, N, C, 1)
    x, got = x.cpu().double(), out.cpu().double()
    ref = torch.zeros_like(got)
    for ky in (1, 2):                                                  # side 1: the inner taps, one pixel each
        for kx in (1, 2):
            w = W[ky * 4 + kx].cpu().double()
            if mode == "down":
                ref[:, 0, 0] += x[:, ky - 1, kx - 1] @ w.T
            else:
                ref[:, ky - 1, kx - 1] = x[:, 0, 0] @ w.T
    assert float((got - ref).abs().max()) <= tolerance(binding.FP32) * float(ref.abs().max())
