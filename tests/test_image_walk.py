"""What the image-side weight gradient requests of the feature gradient (csrc/image_walk.h), on the host: every value of a tile's samples once, at
its own address, and behind the last unit, where the buffer is empty, only offsets that cannot wrap its size round."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NO_PIXEL = 0xffffffff


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("image_walk") / "image_walk.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "c", "image_walk_host.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("esize", [2, 4])
@pytest.mark.parametrize("CS", [64, 128])
@pytest.mark.parametrize("side", [2, 4, 7, 14, 16, 18, 20, 32, 36, 48])      # 16, 32 and 48 in whole units of sixteen columns
def test_requests(lib, esize, CS, side):
    CB, j0, j1, nseg, ring = 3, 2, 4, 2, (6 if esize == 2 else 3)
    loads = 1 if esize == 2 else 2
    steps, units = lib.image_walk_steps(side, CB, CS), lib.image_walk_units(side, CB) * (j1 - j0) * nseg
    assert bool(lib.image_walk_even(side, CB, CS)) == (side % 16 == 0)
    want = units * steps
    asked = -(-want // ring) * ring + ring            # whole rounds of the ring, which runs one ahead
    per = side * side * CS * esize // 16              # 16-byte pieces of a sample
    seen = np.zeros((nseg, j1 - j0, per), int)
    for wave in range(4):
        for lane in range(64):
            out = [np.zeros(asked * k, t) for k, t in ((1, np.int32), (1, np.int32), (1, np.int32), (loads, np.uint32), (1, np.uint32))]
            lib.image_walk(esize, CB, side, CS, j0, j1, nseg, wave, lane, asked, *(a.ctypes.data_as(ctypes.c_void_p) for a in out))
            live, seg, j, off, uni = out
            off = off.reshape(asked, loads).astype(np.int64)
            assert np.all(live[:want] == 1) and np.all(live[want:] == 0)
            # an empty buffer refuses every offset; whether it does may hang on its size less the scalar part, so that stays zero
            assert np.all(uni[want:] == 0), (wave, lane, uni[want:].max())
            for i in range(loads):
                there = off[:want, i] != NO_PIXEL
                byte = (off[:want, i] + uni[:want])[there]
                assert np.all(uni[:want] < per * 16) and byte.min(initial=0) >= 0 and byte.max(initial=0) + 16 <= per * 16
                np.add.at(seen, (seg[:want][there], j[:want][there] - j0, byte // 16), 1)
    assert np.all(seen == 1)
