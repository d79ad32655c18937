"""Digit passes (the library's own choice where no option is set) against the
CPU oracle: sizes around the tiles and chunks of each workgroup shape, every
kind of sort, in place, constant digits, presorted input, and the calls that
keep the merge passes (a workspace of the merge sort's size, a set option)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2409_03970_amd as hv
from paper_2409_03970_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"
KEYS = ("uniform", "sorted", "reverse", "distinct16", "zipf", "equal", "extremes", "organ_pipe",
        "negatives")


def _keys(n, dist, seed=0):
    if dist in inputs.DISTRIBUTIONS:
        return inputs.keys(n, dist, seed=seed, device=DEV)
    return inputs.adversarial_keys(n, dist, seed=seed, device=DEV)


@pytest.mark.parametrize("n", [(1 << 15) + 1, 2048 * 31 + 1, 1 << 16, (1 << 16) + 1, 100003,
                               1 << 17, (1 << 17) + 1, (1 << 19) + 2049, (1 << 22) - 1, 1 << 22,
                               8192 * 1025 + 1])
@pytest.mark.parametrize("dist", KEYS)
def test_keys_and_in_place(n, dist):
    print("digit passes", n, dist, flush=True)
    x = _keys(n, dist)
    want = oracle.sort(x.cpu().numpy())
    assert np.array_equal(hv.sort(x).cpu().numpy(), want)
    hv.sort(x, out=x)
    assert np.array_equal(x.cpu().numpy(), want)


def test_keys_largest_tile():
    n = (1 << 27) + 16384 + 5
    print("digit passes", n, flush=True)
    for dist in ("uniform", "zipf"):
        x = _keys(n, dist)
        assert torch.equal(hv.sort(x), torch.sort(x).values), dist


@pytest.mark.parametrize("dtype", [torch.float32, torch.uint32])
def test_mapped_keys(dtype):
    g = np.random.default_rng(3)
    bits = g.integers(0, 2**32, 70001, dtype=np.uint64).astype(np.uint32)
    bits[:6] = [0, 0x80000000, 0x7f800000, 0xff800000, 0x7fc00001, 0xffc00001]
    x = torch.from_numpy(bits.view(np.float32) if dtype == torch.float32 else bits).to(DEV)
    got = hv.sort_keys(x).cpu().numpy().view(np.uint32)
    ref = oracle.sort_f32(bits.view(np.float32)) if dtype == torch.float32 else \
        oracle.sort_u32(bits)
    assert np.array_equal(got, ref.view(np.uint32))


@pytest.mark.parametrize("n", [(1 << 15) + 1, 1 << 16, 2048 * 33 + 1, 1 << 17, 2048 * 65,
                               (1 << 22) + 8191])
@pytest.mark.parametrize("dist", ("uniform", "sorted", "reverse", "distinct16", "zipf", "equal"))
def test_by_key(n, dist):
    print("by key", n, dist, flush=True)
    k = _keys(n, dist)
    v = torch.arange(n, device=DEV, dtype=torch.int64) * 3 - 7
    ko, vo = hv.sort_by_key(k, v)
    ek, ev = oracle.sort_by_key_p64(k.cpu().numpy(), v.cpu().numpy().view(np.uint64))
    assert np.array_equal(ko.cpu().numpy(), ek)
    assert np.array_equal(vo.cpu().numpy().view(np.uint64), ev)
    hv.sort_by_key(k, v, keys_out=k, vals_out=vo)        # keys in place
    assert np.array_equal(k.cpu().numpy(), ek)
    assert np.array_equal(vo.cpu().numpy().view(np.uint64), ev)


@pytest.mark.parametrize("values", ("index", "reverse", "few", "random"))
@pytest.mark.parametrize("dist", ("uniform", "sorted", "reverse", "distinct16", "equal",
                                  "extremes"))
def test_pairs(dist, values):
    n = (1 << 22) + 8193
    print("pairs", n, dist, values, flush=True)
    k = _keys(n, dist)
    i = torch.arange(n, device=DEV, dtype=torch.int32)
    v = {"index": i, "reverse": i.flip(0).contiguous(), "few": (i * 7919) % 5 - 2,
         "random": _keys(n, "negatives", seed=5)}[values].to(torch.int32)
    ek, ev = oracle.sort_pairs(k.cpu().numpy(), v.cpu().numpy())
    ko, vo = hv.sort_pairs(k, v)
    assert np.array_equal(ko.cpu().numpy(), ek) and np.array_equal(vo.cpu().numpy(), ev)
    hv.sort_pairs(k, v, k, v)
    assert np.array_equal(k.cpu().numpy(), ek) and np.array_equal(v.cpu().numpy(), ev)


@pytest.mark.parametrize("what", ("wide", "small", "high", "sorted", "reverse", "normal",
                                  "special", "u64"))
def test_keys64(what):
    n = (1 << 22) + 8191
    print("64-bit keys", n, what, flush=True)
    g = np.random.default_rng(9)
    wide = g.integers(-2**63, 2**63, n, dtype=np.int64)
    x = {"wide": wide, "small": wide >> 50, "high": (wide >> 40) << 40, "sorted": np.sort(wide),
         "reverse": np.sort(wide)[::-1].copy(), "normal": g.standard_normal(n),
         "special": (wide & ~0xfffff).view(np.float64), "u64": wide.view(np.uint64)}[what]
    ref = {np.dtype("int64"): oracle.sort_i64, np.dtype("uint64"): oracle.sort_u64,
           np.dtype("float64"): oracle.sort_f64}[x.dtype](x).view(np.uint64)
    t = torch.from_numpy(x).to(DEV)
    assert np.array_equal(hv.sort_keys(t).cpu().numpy().view(np.uint64), ref)
    hv.sort_keys(t, out=t)
    assert np.array_equal(t.cpu().numpy().view(np.uint64), ref)


def test_merge_passes_where_the_workspace_or_an_option_asks_for_them():
    n = 300001
    x = _keys(n, "uniform")
    want = oracle.sort(x.cpu().numpy())
    L = hv.lib()
    merge = L.hvms_sort_workspace_bytes(n, 0, hv.Options(merge_ways=2))
    assert merge < L.hvms_sort_workspace_bytes(n, 0, None)
    for opts, nbytes in ((None, merge), ({"merge_ways": 4}, None), ({"wave_levels": 7}, None)):
        need = nbytes or L.hvms_sort_workspace_bytes(n, 0, hv._opts(opts))
        y = torch.empty_like(x)
        hv.hvms_sort_i32(x, y, torch.empty(need, dtype=torch.uint8, device=DEV), opts=opts)
        assert np.array_equal(y.cpu().numpy(), want), opts


def test_replayed_graph_on_a_side_stream():
    n = (1 << 22) + 3
    x = _keys(n, "uniform")
    y = torch.empty_like(x)
    ws = torch.empty(hv.lib().hvms_sort_workspace_bytes(n, 0, None), dtype=torch.uint8, device=DEV)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        hv.hvms_sort_i32(x, y, ws, stream=s)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        hv.hvms_sort_i32(x, y, ws, stream=s)
    for dist in ("uniform", "sorted", "zipf", "reverse"):   # other plans, same graph
        x.copy_(_keys(n, dist, seed=4))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, torch.sort(x).values), dist
        ws.fill_(0xA5)


def test_arrays_off_the_16_byte_grid():
    n = (1 << 22) + 77
    x = _keys(n + 1, "negatives")[1:]
    y = torch.empty(n + 3, dtype=torch.int32, device=DEV)[3:]
    assert torch.equal(hv.sort(x, out=y), torch.sort(x).values)
    v = _keys(n + 1, "uniform", seed=2)[1:]
    ko, vo = hv.sort_pairs(x, v, y, torch.empty(n + 1, dtype=torch.int32, device=DEV)[1:])
    ek, ev = oracle.sort_pairs(x.cpu().numpy(), v.cpu().numpy())
    assert np.array_equal(ko.cpu().numpy(), ek) and np.array_equal(vo.cpu().numpy(), ev)


def _unsampled(n, count, rng):
    """Positions that the sample of the digit choice does not read: element j
    of its 2^18 (at fewer than 2^25 elements) is at SplitMix64(j) * n / 2^64."""
    with np.errstate(over="ignore"):
        z = (np.arange(1 << 18, dtype=np.uint64) + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
        lo = ((z & np.uint64(0xffffffff)) * np.uint64(n)) >> np.uint64(32)
        seen = ((z >> np.uint64(32)) * np.uint64(n) + lo) >> np.uint64(32)
    free = np.ones(n, dtype=bool)
    free[seen.astype(np.int64)] = False
    return rng.choice(np.flatnonzero(free), count, replace=False)


@pytest.mark.parametrize("lengths", [tuple(range(2, 70)), (31, 32, 33, 34, 63, 64, 65, 66) * 20,
                                     (100, 1000, 8190, 8191, 8192), (8193,), (8256, 8447, 8449),
                                     (20000,), (2,) * 30000, (40,) * 65537])
@pytest.mark.parametrize("kind", ("i64", "pairs"))
def test_groups_left_alike_by_the_top_digits(lengths, kind):
    """Groups that share their upper words, planted where the sample does not
    look, so that the finish meets them: in a window, listed, too long, too
    many."""
    n = (1 << 24) + 12345
    print("groups", kind, lengths[:5], len(lengths), flush=True)
    rng = np.random.default_rng(len(lengths))
    x = rng.integers(-2**63, 2**63, n, dtype=np.int64)
    at = _unsampled(n, sum(lengths), rng)
    x[at] = np.repeat(rng.integers(-2**31, 2**31, len(lengths), dtype=np.int64) << 32, lengths)
    x[at] += rng.integers(0, 2**32, len(at), dtype=np.int64)
    x[at[:3]] = x[at[0]]                                  # and a few equal ones
    want = torch.sort(torch.from_numpy(x).to(DEV)).values
    if kind == "i64":
        got = hv.sort_keys(torch.from_numpy(x).to(DEV))
    else:
        k = torch.from_numpy((x >> 32).astype(np.int32)).to(DEV)
        v = torch.from_numpy((x & 0xffffffff).astype(np.uint32).view(np.int32) ^ -2**31).to(DEV)
        ko, vo = hv.sort_pairs(k, v)
        got = (ko.to(torch.int64) << 32) | ((vo.to(torch.int64) + 2**31) & 0xffffffff)
    assert torch.equal(got, want)


def test_a_long_group_in_order_and_one_out_of_order_at_its_end():
    n = (1 << 24) + 77
    rng = np.random.default_rng(4)
    x = rng.integers(-2**63, 2**63, n, dtype=np.int64)
    at = np.sort(_unsampled(n, 60000, rng))
    x[at[:30000]] = 5 << 40                               # equal: always in order
    x[at[30000:]] = (7 << 40) + np.arange(30000)          # ascending as they stand ...
    x[at[-1]] = 7 << 40                                   # ... but for the last
    want = torch.sort(torch.from_numpy(x).to(DEV)).values
    assert torch.equal(hv.sort_keys(torch.from_numpy(x).to(DEV)), want)
