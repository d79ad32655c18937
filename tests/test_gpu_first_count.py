"""The first count of the digit passes and the counts that read the caller's
array: a single pair of elements out of order at the edges of a lane's load, a
wave, a tile and the array must not pass for presorted input, and passes whose
lower digits are constant count the caller's words, on and off the 16-byte
grid, with and without a ragged last tile."""
import numpy as np
import pytest
import torch

import paper_2409_03970_amd as hv

pytestmark = pytest.mark.gpu
DEV = "cuda"
KINDS = ("keys", "by_key", "pairs", "i64")
EDGES = (0, 1, 3, 63, 127, 255, 1023, 2047, 4095, 8191, 16383)


def _off(x, off):
    """x at `off` elements past an allocation's start."""
    buf = torch.empty(x.numel() + 8, dtype=x.dtype, device=DEV)
    view = buf[off:off + x.numel()]
    view.copy_(x)
    return view


def _check(kind, words, off, what):
    """Sorts `words` (int64) by the kind's entry point against torch."""
    n = words.numel()
    idx = torch.arange(n, device=DEV)
    if kind == "i64":
        x = _off(words, off)
        assert torch.equal(hv.sort_keys(x), torch.sort(words).values), what
        return
    k = _off(words.int(), off)
    want, order = torch.sort(words.int(), stable=True)
    if kind == "keys":
        assert torch.equal(hv.sort(k), want), what
    elif kind == "by_key":
        ko, vo = hv.sort_by_key(k, idx)
        assert torch.equal(ko, want) and torch.equal(vo, order), what
    else:
        v = _off(idx.int(), off)
        ko, vo = hv.sort_pairs(k, v)
        assert torch.equal(ko, want) and torch.equal(vo, order.int()), what


def _sizes(kind):
    return ((1 << 16, (1 << 16) + 5, 1 << 22) if kind in ("keys", "by_key")
            else (1 << 22, (1 << 22) + 5))


@pytest.mark.parametrize("off", (0, 1))
@pytest.mark.parametrize("kind", KINDS)
def test_one_pair_out_of_order(kind, off):
    for n in _sizes(kind):
        for rising in (True, False):
            for p in EDGES + (n - 2,):
                x = torch.arange(n, device=DEV) * 3
                if not rising:
                    x = x.flip(0).contiguous()
                a, b = x[p].clone(), x[p + 1].clone()
                x[p], x[p + 1] = b, a
                what = (kind, n, off, rising, p)
                print("first count", what, flush=True)
                _check(kind, x, off, what)


@pytest.mark.parametrize("off", (0, 1))
@pytest.mark.parametrize("kind", KINDS)
def test_lower_digits_constant(kind, off):
    for n in _sizes(kind):
        for shift in (8, 20, 32) if kind == "i64" else (8, 20):
            g = torch.Generator(device=DEV).manual_seed(n + shift)
            hi = 63 if kind == "i64" else 31
            x = torch.randint(-(1 << (hi - shift)), 1 << (hi - shift), (n,), device=DEV,
                              generator=g) << shift
            what = (kind, n, off, shift)
            print("constant digits", what, flush=True)
            _check(kind, x, off, what)


@pytest.mark.parametrize("kind,n", (("keys", 1 << 27), ("pairs", 5 << 23), ("i64", 5 << 23),
                                    ("by_key", 1 << 25)))
def test_largest_tiles(kind, n):
    for p in (16383, n - 2):
        x = torch.arange(n, device=DEV)
        x[p], x[p + 1] = p + 1, p
        print("first count", kind, n, p, flush=True)
        _check(kind, x, 0, (kind, n, p))
    # most keys out of order, a ragged last tile
    x = torch.arange(n + 5, device=DEV) * 40503 % 1000003 * 2039
    _check(kind, x, 0, (kind, n, "shuffled"))
    _check(kind, x, 1, (kind, n, "shuffled"))


@pytest.mark.parametrize("n", (1 << 16, 1 << 22, (1 << 22) + 5))
def test_first_pass_ranks(n):
    """Keys alone are ranked without order in the first pass: one digit for all
    but a few keys, two, and the largest digit beside a ragged tile's pads."""
    r = torch.arange(n, device=DEV)
    for what, x in (("few", torch.where(r % 4099 == 0, r % 251, 7) | ((r % 3) << 8)),
                    ("two", (r * 40503 >> 7) & 1 | ((r % 5) << 24)),
                    ("top", 255 - (r % 2) | ((r * 7919 % 1000) << 8)),
                    ("max", torch.where(r % 2 == 0, (1 << 31) - 1, r))):
        print("first ranks", n, what, flush=True)
        _check("keys", x, 0, (n, what))


@pytest.mark.parametrize("kind", ("i64", "pairs"))
def test_second_round_with_the_largest_tile(kind):
    """A group too long for the finish, planted where the sample of 2^19
    elements (element j at SplitMix64(j) * n / 2^64) does not look."""
    n = (5 << 23) + 4097
    print("second round", kind, n, flush=True)
    with np.errstate(over="ignore"):
        z = (np.arange(1 << 19, dtype=np.uint64) + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
        lo = ((z & np.uint64(0xffffffff)) * np.uint64(n)) >> np.uint64(32)
        seen = ((z >> np.uint64(32)) * np.uint64(n) + lo) >> np.uint64(32)
    rng = np.random.default_rng(9)
    at = np.setdiff1d(rng.integers(0, n, 40000), seen.astype(np.int64))
    x = rng.integers(-2**63, 2**63, n, dtype=np.int64)
    x[at] = (77 << 40) + rng.integers(0, 2**32, len(at))
    x = torch.from_numpy(x).to(DEV)
    want = torch.sort(x).values
    if kind == "i64":
        got = hv.sort_keys(x)
    else:
        ko, vo = hv.sort_pairs((x >> 32).int(), ((x & 0xffffffff) - 2**31).int())
        got = (ko.long() << 32) | (vo.long() + 2**31)
    assert torch.equal(got, want)
