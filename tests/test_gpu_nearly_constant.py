"""Nearly constant 64-bit keys and pairs at the sizes where a sample decides how
many low digits to leave out: hardly any two sampled elements differ, and what
does differ may lie below the digits left out.  Outputs hold a pattern before
the call, so an element that no launch writes shows."""
import pytest
import torch

import paper_2409_03970_amd as hv

pytestmark = pytest.mark.gpu
DEV = "cuda"
SIZES = (1 << 24, 20_000_001, (5 << 23) + 5)
POISON = 0x5A


def _words(what, n):
    """int64 keys: nearly all equal."""
    g = torch.Generator(device=DEV).manual_seed(n)

    def at(m):
        return torch.randint(0, n, (m,), device=DEV, generator=g)

    def draw(lo, hi, m):
        return torch.randint(lo, hi, (m,), device=DEV, generator=g)

    x = torch.zeros(n, dtype=torch.int64, device=DEV)
    if what == "one outlier":
        x[n // 3] = 1000
    elif what == "500 below 2^40":
        x[at(500)] = draw(1, 1 << 40, 500)
    elif what == "2000 in two bytes":
        x[at(2000)] = draw(1, 1 << 16, 2000)
    elif what == "two values":
        x = draw(0, 2, n) * 1000
    elif what == "both signs":                   # the top digit varies
        x[at(500)] = draw(-(1 << 62), 1 << 62, 500)
    elif what == "outliers beside the heavy value":
        x[at(30)] = draw(1, 1 << 20, 30)
        x[at(30)] = draw(-(1 << 62), 1 << 62, 30)
    elif what == "high constant word":
        x += 77 << 40
        x[at(500)] += draw(1, 1 << 30, 500)
    else:
        raise ValueError(what)
    return x


WORDS = ("one outlier", "500 below 2^40", "2000 in two bytes", "two values", "both signs",
         "outliers beside the heavy value", "high constant word")


def _poisoned(like):
    t = torch.empty_like(like)
    t.view(torch.uint8).fill_(POISON)
    return t


@pytest.mark.parametrize("what", WORDS)
@pytest.mark.parametrize("n", SIZES)
def test_keys64(n, what):
    print("nearly constant", n, what, flush=True)
    x = _words(what, n)
    want = torch.sort(x).values
    assert torch.equal(hv.sort_keys(x, out=_poisoned(x)), want)
    hv.sort_keys(x, out=x)
    assert torch.equal(x, want)


@pytest.mark.parametrize("count", (1, 500))
@pytest.mark.parametrize("n", SIZES)
def test_doubles(n, count):
    print("nearly constant doubles", n, count, flush=True)
    g = torch.Generator(device=DEV).manual_seed(count)
    x = torch.full((n,), 0.5, dtype=torch.float64, device=DEV)
    x[torch.randint(0, n, (count,), device=DEV, generator=g)] = \
        torch.rand(count, device=DEV, dtype=torch.float64, generator=g) * 0.99 + 0.01
    want = torch.sort(x).values
    assert torch.equal(hv.sort_keys(x, out=_poisoned(x)), want)


@pytest.mark.parametrize("where", ("apart", "both in place", "keys in place", "values in place"))
@pytest.mark.parametrize("what", WORDS)
def test_pairs(what, where):
    """The same words as pairs: the values hold what lies below the high word."""
    n = SIZES[0] + 3
    print("nearly constant pairs", what, where, flush=True)
    x = _words(what, n)
    want = torch.sort(x).values
    k, v = (x >> 32).int(), ((x & 0xffffffff) - 2**31).int()
    ko = k if where in ("both in place", "keys in place") else _poisoned(k)
    vo = v if where in ("both in place", "values in place") else _poisoned(v)
    hv.sort_pairs(k, v, ko, vo)
    assert torch.equal((ko.long() << 32) | (vo.long() + 2**31), want)


def test_one_key_and_few_values():
    n = SIZES[0]
    k = torch.full((n,), 7, dtype=torch.int32, device=DEV)
    v = torch.zeros(n, dtype=torch.int32, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(1)
    v[torch.randint(0, n, (500,), device=DEV, generator=g)] = \
        torch.randint(-1000, 1 << 30, (500,), device=DEV, generator=g, dtype=torch.int32)
    ko, vo = hv.sort_pairs(k, v, _poisoned(k), _poisoned(v))
    assert torch.equal(ko, k) and torch.equal(vo, torch.sort(v).values)
