"""Building blocks of the networks as printed in the paper's Tables 1 and 2 against the oracle (GPU): the dropout
mask bit for bit (both sides implement Philox-4x32-10 from its definition), and the two linear maps that carry
"Upsample x2, then Conv k3 s1 p1" onto the k4 s2 p1 transposed-convolution kernel and its weight gradient back.
"""
import numpy as np
import pytest

from oracle import paper_nets as P
from paper_2102_10485_amd import binding, synth
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

A = np.array([[0, 0, 1], [0, 1, 1], [1, 1, 0], [1, 0, 0]], float)      # 4-tap filter = A . 3-tap filter, per axis


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


@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("ch,h,w,groups,p", [(16, 8, 8, [3, 0, 2], 0.25), (3, 5, 7, [1, 4], 0.25), (32, 4, 4, [6], 0.5),
                                             (8, 2, 2, [2, 2], 0.0)])
def test_dropout_mask_is_the_oracles_bit_for_bit(ctxs, prec, ch, h, w, groups, p):
    g = ctxs[prec]
    bf = prec == binding.BF16
    rng = np.random.default_rng(ch + h + len(groups))
    n = int(sum(groups))
    offs = np.concatenate([[0], np.cumsum(groups)]).astype(np.int32)
    x = U.round_to(rng.normal(0, 1, (n, ch, h, w)) + 3.0, bf)            # no zeros in the input: zeros mark dropped elements
    seed, step, layer, pass_id = 0x1234567811223344, 7, 3, 2
    d_x = U.dev(U.pack(x.transpose(0, 2, 3, 1), bf))
    g.op_dropout(d_x.data_ptr(), U.dev(offs).data_ptr(), len(groups), n, ch, h, w, p, seed, step, layer, pass_id)
    got = U.unpack(d_x, bf, (n, h, w, ch)).transpose(0, 3, 1, 2)
    for gi, cnt in enumerate(groups):
        if cnt == 0:
            continue
        keep = P.dropout_keep((cnt, ch, h, w), p, seed, gi, step, layer, pass_id)
        mine = got[offs[gi]:offs[gi + 1]]
        assert np.array_equal(mine != 0, keep), "group %d" % gi
        ref = x[offs[gi]:offs[gi + 1]] / (1.0 - p)
        assert np.allclose(mine[keep], ref[keep], rtol=1e-2 if bf else 1e-6, atol=0)
    if p == 0.0:
        assert np.array_equal(got, x)


@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("G,cb,cs", [(3, 8, 16), (2, 128, 64)])
def test_summed_taps_and_their_adjoint(ctxs, prec, G, cb, cs):
    torch = U.torch_mod()
    g = ctxs[prec]
    bf = prec == binding.BF16
    rng = np.random.default_rng(G * 100 + cb)
    w3 = rng.normal(0, 1, (G, 3, 3, cb, cs)).astype(np.float32)
    d_w3 = U.dev(w3.reshape(-1))
    dt = torch.int16 if bf else torch.float32
    d_w4 = torch.zeros(G * 16 * cb * cs, dtype=dt, device="cuda")
    d_w4t = torch.zeros(G * 16 * cb * cs, dtype=dt, device="cuda")
    g.op_w3_to_w4(d_w3.data_ptr(), d_w4.data_ptr(), d_w4t.data_ptr(), G, cb, cs)
    ref = np.einsum("ak,gklbs,cl->gacbs", A, w3.astype(np.float64), A)   # [G][4][4][cb][cs]
    got = U.unpack(d_w4, bf, (G, 4, 4, cb, cs))
    got_t = U.unpack(d_w4t, bf, (G, 4, 4, cs, cb))
    tol = 1e-2 if bf else 1e-6
    assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref))
    assert np.array_equal(got_t, got.transpose(0, 1, 2, 4, 3))
    # adjoint: <A w3 A^T, d4> == <w3, A^T d4 A>
    d4 = rng.normal(0, 1, (G, 4, 4, cb, cs)).astype(np.float32)
    d_d4 = U.dev(d4.reshape(-1))
    d_d3 = torch.full((G * 9 * cb * cs,), 5.0, dtype=torch.float32, device="cuda")
    g.op_dw4_to_dw3(d_d4.data_ptr(), d_d3.data_ptr(), G, cb, cs)
    got3 = d_d3.cpu().numpy().reshape(G, 3, 3, cb, cs)
    ref3 = np.einsum("ak,gacbs,cl->gklbs", A, d4.astype(np.float64), A)
    assert np.max(np.abs(got3 - ref3)) <= 1e-6 * np.max(np.abs(ref3))
    assert abs(np.sum(ref * d4) - np.sum(w3 * ref3)) <= 1e-9 * abs(np.sum(ref * d4))

@pytest.mark.parametrize("prec", [binding.FP32, binding.BF16])
@pytest.mark.parametrize("G,cb,cs,shift", [(2, 32, 64, 0),      # one tile of channels
                                           (2, 96, 192, 0),     # several both ways
                                           (2, 32, 96, 0),      # half a tile: the general kernels
                                           (2, 64, 64, 1),      # buffers that start off a 16-byte boundary
                                           (2, 7, 5, 0)])       # planes that are no whole number of 16-byte runs
def test_summed_taps_by_tiles(ctxs, prec, G, cb, cs, shift):
    """Small whole numbers: every sum is exact in both storage types, and what lies behind the results stays as it was."""
    torch = U.torch_mod()
    g = ctxs[prec]
    bf = prec == binding.BF16
    rng = np.random.default_rng(G * 1000 + cb + cs)
    plane, dt = cb * cs, torch.int16 if bf else torch.float32

    def put(values):
        t = torch.zeros(values.size + shift + 8, dtype=torch.float32, device="cuda")
        t[shift:shift + values.size] = U.dev(values.reshape(-1))
        return t

    w3 = rng.integers(-8, 9, (G, 3, 3, cb, cs)).astype(np.float32)
    d_w3 = put(w3)
    d_w4, d_w4t = (torch.full((G * 16 * plane + shift + 8,), 77, dtype=dt, device="cuda") for _ in range(2))
    g.op_w3_to_w4(d_w3[shift:].data_ptr(), d_w4[shift:].data_ptr(), d_w4t[shift:].data_ptr(), G, cb, cs)
    ref = np.einsum("ak,gklbs,cl->gacbs", A, w3.astype(np.float64), A)
    end = shift + G * 16 * plane
    assert np.array_equal(U.unpack(d_w4[shift:end].clone(), bf, (G, 4, 4, cb, cs)), ref)
    assert np.array_equal(U.unpack(d_w4t[shift:end].clone(), bf, (G, 4, 4, cs, cb)), ref.transpose(0, 1, 2, 4, 3))
    for t in (d_w4, d_w4t):
        assert torch.all(t[:shift] == 77) and torch.all(t[end:] == 77)
    d4 = rng.integers(-8, 9, (G, 4, 4, cb, cs)).astype(np.float32)
    d_d4, d_d3 = put(d4), torch.full((G * 9 * plane + shift + 8,), 77.0, device="cuda")
    g.op_dw4_to_dw3(d_d4[shift:].data_ptr(), d_d3[shift:].data_ptr(), G, cb, cs)
    end = shift + G * 9 * plane
    assert np.array_equal(d_d3[shift:end].cpu().numpy().reshape(G, 3, 3, cb, cs), np.einsum("ak,gacbs,cl->gklbs", A, d4.astype(np.float64), A))
    assert torch.all(d_d3[:shift] == 77) and torch.all(d_d3[end:] == 77)

