"""What the image-side weight gradient requests of the feature gradient (csrc/image_walk.h), on the host: every value of a tile's samples once, at
its own address, and behind the last unit, where the buffer is empty, only offsets that cannot wrap its size round.  And the tiles it takes them in."""
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


def tiles(lib, esize, size, counts):
    at, c = (ctypes.c_int * 2)(), (ctypes.c_int * len(counts))(*[int(v) for v in counts])
    return lib.image_walk_tiles(esize, size, len(counts), c, at), at[0], at[1]


@pytest.mark.parametrize("esize", [2, 4])
@pytest.mark.parametrize("L,size,n", [(1, 6400, 64), (1, 6400, 1), (10, 1280, 100), (100, 6400, 400), (100, 6400, 50), (8, 1024, 64), (20, 20000, 333)])
def test_small_calls_of_large_contexts(lib, esize, L, size, n):
    """A call of few samples has a block for nearly every sample, as long as that does not take more blocks than a full call: tiles as long as those of the
    sizing batch were a chain of their ten or more samples in a few blocks."""
    counts = np.full(L, n // L) + (np.arange(L) < n % L)
    got, _, _ = tiles(lib, esize, size, counts)
    assert got >= min(n, tiles(lib, esize, size, np.full(L, size // L))[0] // 2)


@pytest.mark.parametrize("esize", [2, 4])
@pytest.mark.parametrize("L", [1, 3, 10, 100, 479, 701, 2200])
def test_bound_of_the_tiles(lib, esize, L):
    """However the samples fall, no more tiles than the host launches blocks and holds partial sums for; none longer than at the sizing batch."""
    rng = np.random.default_rng(L)
    for _ in range(300):
        size = int(np.exp(rng.uniform(0, np.log(30000)))) + 1
        n = size if rng.random() < 0.3 else int(rng.integers(0, size + 1))
        p = rng.dirichlet(np.full(L, np.exp(rng.uniform(-5, 4))))
        counts = rng.multinomial(n, p / p.sum())
        got, bound, longest = tiles(lib, esize, size, counts)
        whole = tiles(lib, esize, size, [size] + [0] * (L - 1))[1]
        assert got <= bound <= max(whole, n) and bound <= n and longest <= -(-size // (480 if esize == 4 else 700))
    # evenly at the sizing batch: a round of blocks
    if L <= 100:
        assert tiles(lib, esize, 64 * L, np.full(L, 64))[0] <= (480 if esize == 4 else 700) + L
