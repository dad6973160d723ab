"""The order in which a tile of the forward-type GEMM walks its reduction (csrc/k_order.h), on the host: every tap and channel line once,
at the right pixel and weight row, and nothing outside the operands -- also in the copies that go out behind the last chunk."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DOWN, UP = 0, 1
AHEAD = 3        # chunks behind the last one that a loop with two buffers still copies a part of


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("k_order") / "k_order.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "c", "k_order_host.cpp"), "-o", so], check=True)
    fn = ctypes.CDLL(so).k_order_walk

    def call(mode, cpl, lo, hi, first_gone, py, px, row, pxb, wtap, chunks):
        states = chunks + AHEAD
        out = [np.zeros(states, t) for t in (np.int32, np.int32, np.int32, np.uint32, np.uint32)]
        fn(mode, cpl, lo, hi, int(first_gone), py, px, ctypes.c_uint(row), ctypes.c_uint(pxb), ctypes.c_uint(wtap), chunks, states,
           *(a.ctypes.data_as(ctypes.c_void_p) for a in out))
        return [[int(v) for v in a] for a in out]
    return call


@pytest.mark.parametrize("mode,py,px", [(DOWN, 0, 0), (UP, 0, 0), (UP, 0, 1), (UP, 1, 0), (UP, 1, 1)])
@pytest.mark.parametrize("side", [1, 2, 4, 7])         # of the layer's smaller map
@pytest.mark.parametrize("C,N", [(64, 256), (192, 512)])
def test_every_copy_lies_inside_its_operand(walk, mode, py, px, side, C, N):
    samples, hin, step = 2, (2 * side if mode == DOWN else side), (2 if mode == DOWN else 1)
    pxb, row, wtap, cpl = 2 * C, 2 * C * hin, 2 * C * N, C // 64
    bias, slice_bytes = row + pxb, samples * hin * hin * pxb

    def gathered(y, x, tap):             # the input pixel under a tap, or None outside the map
        if mode == DOWN:
            iy, ix = 2 * y - 1 + (tap >> 2), 2 * x - 1 + (tap & 3)
        else:
            iy, ix = y + py - (tap >> 1), x + px - (tap & 1)
        return (iy, ix) if 0 <= iy < hin and 0 <= ix < hin else None

    for rows in {(0, 0), (side - 1, side - 1), (0, side - 1)}:      # pixel rows that a tile covers: the first, the last, all
        lo = hi = 4
        first_gone = False
        top, bottom = rows[1] == 0, rows[0] == side - 1
        if mode == DOWN:
            lo, hi, first_gone = (2 if top else 4), (2 if bottom else 4), top
        elif py == 0 and top:
            lo = 2
        elif py == 1 and bottom:
            lo, first_gone = 2, True
        chunks = (2 * (lo + hi) if mode == DOWN else lo) * cpl
        more, tap, line, aoff, woff = walk(mode, cpl, lo, hi, first_gone, py, px, row, pxb, wtap, chunks)
        assert more == [1] * chunks + [0] * AHEAD
        for i in range(chunks + AHEAD):
            assert woff[i] + (N - 1) * pxb + 128 <= 16 * wtap, (i, chunks)
            for n in range(samples):
                for y in range(rows[0], rows[1] + 1):
                    for x in range(side):
                        at = gathered(y, x, tap[i])
                        if at is None:
                            continue                   # masked
                        byte = ((n * hin + step * y) * hin + step * x) * pxb + aoff[i] - bias
                        assert 0 <= byte and byte + 128 <= slice_bytes, (i, chunks)
                        if more[i]:
                            assert byte == ((n * hin + at[0]) * hin + at[1]) * pxb + 128 * line[i]
        taps = {t for t in range(16 if mode == DOWN else 4)
                if any(gathered(y, x, t) for y in range(rows[0], rows[1] + 1) for x in range(-1, side + 1))}
        assert sorted(set(zip(tap[:chunks], line[:chunks]))) == sorted(zip(tap[:chunks], line[:chunks]))
        assert taps <= set(tap[:chunks])
        for t, w in {(tap[i], (woff[i] - 128 * line[i]) // wtap) for i in range(chunks)}:
            want = t if mode == DOWN else (2 * (t >> 1) + 1 - py) * 4 + 2 * (t & 1) + 1 - px
            assert w == want
