"""The plan of the digit passes (csrc/radix_plan.h, compiled for the host), run
step by step on small arrays: whichever digits vary and however many low ones
the sample lets go, the first round has to write every element to the output in
the order of the digits it kept, and the second round has to sort it."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SKIP, SCATTER, COPY, REVERSE = range(4)
IN, A, B, OUT = range(4)
NOT_ASCENDING, NOT_DESCENDING, VALUES_NOT_ASCENDING = 1, 2, 4
PAIRS, KEYS64, KEYS = "pairs", "keys64", "keys"
RUNS, N = 32, 1 << 24

SHIM = """
#include "radix_plan.h"
extern "C" void plan(uint32_t flags, uint32_t var0, uint32_t var1, uint32_t near0, uint32_t near1,
                     const uint32_t *same, int runs, int64_t n, int passes, int two, int keys64,
                     int inplace, uint32_t *out)
{
    static_assert(sizeof(hvms::Ctl) == 83 * 4, "two rounds of eight steps of five words");
    hvms::plan_sort(hvms::Found{flags, var0, var1, near0, near1, same, runs, n}, passes, two,
                    keys64, inplace, (hvms::Ctl *)out);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__host__=", "-D__device__=",
                    "-I", os.path.join(ROOT, "paper_2409_03970_amd", "csrc"), str(src), "-o",
                    str(so)], check=True)
    f = ctypes.CDLL(str(so)).plan

    def call(kind, x, drop, inplace, n=N, third=0, alike=None):
        """The plan of sorting the uint64 words x with a sample that finds no two
        elements alike without their lowest `drop` digits, and all with fewer, and
        `third` elements that equal the one after next."""
        two = kind != KEYS
        hi, lo = x >> np.uint64(32), x & np.uint64(0xffffffff)
        flags = (bool((x[:-1] > x[1:]).any()) * NOT_ASCENDING
                 | bool((x[:-1] < x[1:]).any()) * NOT_DESCENDING
                 | (kind == PAIRS and bool((lo[:-1] > lo[1:]).any())) * VALUES_NOT_ASCENDING)
        same = (ctypes.c_uint32 * 8)(*[0 if d < drop else 8191 * RUNS for d in range(7)], third)
        for d, count in enumerate(alike or ()):
            same[d] = count
        near = [2**32 - 1] * 2
        for a, b in zip(x[:-1], x[1:]):
            d = int(a ^ b)
            if d:
                w = int(d >= 2**32)
                near[w] = min(near[w], (d >> 32 * w) - 1)
        var = [int(np.bitwise_or.reduce(w ^ w[0])) for w in (lo, hi)]
        out = (ctypes.c_uint32 * 83)()
        u = ctypes.c_uint32
        f(flags, var[0] if two else 0, u(var[1]), u(near[0]), u(near[1]), same,
          RUNS if two else 0, ctypes.c_int64(n), 8 if two else 4, int(two), int(kind == KEYS64), int(inplace), out)
        steps = np.array(out[:80]).reshape(2, 8, 5)
        return steps, out[80]
    return call


def _run(steps, x, kind, inplace):
    """The output buffer after one round's steps; None where nothing was
    written or a step read what another had overwritten."""
    buf = {IN: x.copy()}
    if inplace:
        buf[OUT] = buf[IN]
    done = [p for p in range(8) if steps[p][0] != SKIP]
    for j, p in enumerate(done):
        mode, src, dst, first, last = (int(v) for v in steps[p])
        assert src in buf and first == (j == 0) and last == (j == len(done) - 1)
        assert last == (dst == OUT) or kind != KEYS64
        same_array = src == dst or (inplace and {src, dst} == {IN, OUT})
        assert mode == COPY or not same_array, "a step scatters into the array it reads"
        word = buf[src]
        if mode == COPY:
            y = word.copy()
        elif mode == REVERSE:
            y = word[::-1].copy()
        else:
            digit = p if kind != KEYS else p + 4
            y = word[np.argsort((word >> np.uint64(8 * digit)) & np.uint64(255), kind="stable")]
        buf[dst] = y
        if inplace and dst in (IN, OUT):
            buf[IN] = buf[OUT] = y
    return buf.get(OUT)


def _words(need, rng):
    """24 words that vary in the digits of the mask `need`, and in no others."""
    x = rng.integers(0, 2**64, 24, dtype=np.uint64)
    for d in range(8):
        digit = np.uint64(255) << np.uint64(8 * d)
        if not need >> d & 1:
            x = (x & ~digit) | (x[0] & digit)
        else:
            x[0] &= ~digit
            x[1] |= digit
    return x


@pytest.mark.parametrize("inplace", (False, True))
@pytest.mark.parametrize("kind", (PAIRS, KEYS64, KEYS))
def test_every_plan_writes_the_output(plan, kind, inplace):
    rng = np.random.default_rng(1)
    dropped = 0
    for need, drop in itertools.product(range(1, 256), range(9)):
        if kind == KEYS:
            need &= 0xf0
        x = _words(need, rng)
        steps, low = plan(kind, x, drop, inplace)
        y = _run(steps[0], x, kind, inplace)
        assert y is not None, (need, drop, "no step writes the output")
        assert np.array_equal(np.sort(y), np.sort(x)), (need, drop)
        shift = np.uint64(8 * low)
        assert np.array_equal(y >> shift, np.sort(x) >> shift), (need, drop, low)
        assert low <= drop
        if low:
            dropped += 1
            z = _run(steps[1], y, kind, True)
            assert z is not None and np.array_equal(z, np.sort(x)), (need, drop, low)
    assert (dropped > 500) == (kind != KEYS)


@pytest.mark.parametrize("kind", (PAIRS, KEYS64))
@pytest.mark.parametrize("digit", range(8))
def test_heavy_value_and_its_like(plan, kind, digit):
    """Mostly one value, in all eight digits another now and then, and one element
    that differs from its neighbour from `digit` on: with many equal elements in the
    sample no digit above that one is left out, and with few the sample decides."""
    x = np.full(24, 0x0102030405060708, dtype=np.uint64)
    x[3], x[4] = 0xf1f2f3f4f5f6f7f8, 0                    # the top digit varies
    x[11] ^= np.uint64(3) << np.uint64(8 * digit)
    x[20] ^= np.uint64(0xff) << np.uint64(56)
    many = -(-RUNS * 8192 // 2048)
    assert plan(kind, x, 7, False, third=many)[1] == (digit if digit >= 2 else 0)
    assert plan(kind, x, 7, False, third=many - 1)[1] == 7
    y = x[x != x[11]]                                     # no like of the heavy value
    assert plan(kind, y, 7, False, third=many)[1] == 7
    assert plan(kind, x, 1, False, third=many)[1] == 0


@pytest.mark.parametrize("n,most", ((1 << 24, 0.5), (1 << 26, 0.5), (3 << 25, 0.75), (1 << 27, 1.0),
                                    (3 << 26, 1.5), (1 << 28, 2.0), (1 << 30, 2.0)))
def test_how_much_may_be_left_alike(plan, n, most):
    x = _words(255, np.random.default_rng(3))
    line = int(most * RUNS * 8192**2 / 2 / n)             # sampled neighbours alike
    for alike, low in ((line, 7), (line + 1, 2)):
        assert plan(KEYS64, x, 7, False, n=n, third=0, alike=(0, 0, alike))[1] == low


@pytest.mark.parametrize("inplace", (False, True))
@pytest.mark.parametrize("kind", (PAIRS, KEYS64, KEYS))
def test_presorted(plan, kind, inplace):
    x = np.sort(np.random.default_rng(2).integers(0, 2**64, 24, dtype=np.uint64))
    if kind == KEYS:
        x &= ~np.uint64(0xffffffff)
    for way in (x, x[::-1].copy()):
        steps, low = plan(kind, way, 7, inplace)
        assert low == 0 and np.array_equal(_run(steps[0], way, kind, inplace), x)
        assert all(s[0] in (SKIP, COPY, REVERSE) for s in steps[0])
