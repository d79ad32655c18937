"""The work that users of this library have it do, as measurable cases.

Every case is one call (or one short training run) through the package's
public functions.  Sizes and distributions are those of the benchmark and the
tests: plain sorts from a thousand keys (where launches are the cost) to 2^30,
ragged sizes between them, every kind of key (int32, uint32, float32, int64,
float64), key-value pairs, a stable sort by key with 64-bit payloads, batches
of segments of uneven sizes with and without values, and the training of the
key-CDF model.
"""
import math

import torch

import paper_2409_03970_amd as hv
from paper_2409_03970_amd import inputs, tune

KEY_DISTS = ("uniform", "gaussian", "sorted", "reverse", "distinct16", "zipf", "mixture")


def listed():
    return [
        # a small lookup table or a batch of ids: the launches and the host path
        {"name": "sort_i32_1k", "kind": "sort", "dtype": "int32", "n": 1000, "dist": "uniform"},
        # scores of one request, ragged, a few block tiles
        {"name": "sort_f32_100k", "kind": "sort", "dtype": "float32", "n": 100_003,
         "dist": "normal"},
        # the benchmark's small plain sort
        {"name": "sort_i32_1m", "kind": "sort", "dtype": "int32", "n": 1 << 20,
         "dist": "uniform"},
        # the benchmark's headline size, random and presorted input
        {"name": "sort_i32_2p28", "kind": "sort", "dtype": "int32", "n": 1 << 28,
         "dist": "uniform"},
        {"name": "sort_i32_2p28_sorted", "kind": "sort", "dtype": "int32", "n": 1 << 28,
         "dist": "sorted"},
        # the benchmark's largest plain sort
        {"name": "sort_i32_2p30_mixture", "kind": "sort", "dtype": "int32", "n": 1 << 30,
         "dist": "mixture"},
        # 64-bit measurements (timestamps, distances), ragged
        {"name": "sort_f64_50m", "kind": "sort", "dtype": "float64", "n": 50_000_017,
         "dist": "normal"},
        # an index build over a skewed column: (key, row) pairs
        {"name": "sort_pairs_2p26_zipf", "kind": "pairs", "n": 1 << 26, "dist": "zipf",
         "values": "index"},
        # moving 8-byte records into key order, ragged
        {"name": "sort_by_key_30m", "kind": "by_key", "n": 30_000_001, "dist": "uniform"},
        # the benchmark's batch: 200,000 arrays of 1 to 65,536 keys
        {"name": "segmented_200k", "kind": "segmented", "nseg": 200_000, "lo": 1, "hi": 65_536},
        # the key-value batch of six distributions, one group of the benchmark's 50,000 segments
        {"name": "segmented_pairs_2k", "kind": "segmented_pairs", "nseg": 2000, "lo": 256,
         "hi": 4_194_304},
        # fitting the key-CDF model: forward, backward and Adam at the default batch
        {"name": "cdf_train_64k", "kind": "cdf_train", "batch": 65_536, "steps": 20,
         "sample": 1 << 20},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(("sort", "sort", "sort", "sort64", "pairs", "by_key", "segmented",
                       "segmented_pairs", "cdf_train"))
    if kind == "sort":
        dtype = rng.choice(("int32", "int32", "uint32", "float32"))
        dist = "normal" if dtype == "float32" else rng.choice(KEY_DISTS)
        return {"kind": kind, "dtype": dtype, "n": _log_int(rng, 1, 1 << 28), "dist": dist}
    if kind == "sort64":
        dtype = rng.choice(("int64", "float64"))
        return {"kind": "sort", "dtype": dtype, "n": _log_int(rng, 1, 1 << 27),
                "dist": "normal" if dtype == "float64" else rng.choice(("wide", "uniform"))}
    if kind == "pairs":
        return {"kind": kind, "n": _log_int(rng, 1, 1 << 27), "dist": rng.choice(KEY_DISTS),
                "values": rng.choice(("index", "random"))}
    if kind == "by_key":
        return {"kind": kind, "n": _log_int(rng, 1, 1 << 27), "dist": rng.choice(KEY_DISTS)}
    if kind == "segmented":
        return {"kind": kind, "nseg": _log_int(rng, 1, 150_000), "lo": 1,
                "hi": _log_int(rng, 64, 65_536)}
    if kind == "segmented_pairs":
        return {"kind": kind, "nseg": _log_int(rng, 1, 1500), "lo": 256,
                "hi": _log_int(rng, 1024, 4_194_304)}
    return {"kind": kind, "batch": _log_int(rng, 256, 65_536), "steps": rng.randint(2, 20),
            "sample": _log_int(rng, 1024, 1 << 20)}


def _i32_keys(n, dist, seed):
    # presorted input from a sort of uniform keys: the same for every run of a seed
    if dist in ("sorted", "reverse"):
        k = inputs.keys(n, "uniform", seed=seed, device="cuda").sort().values
        return k.flip(0) if dist == "reverse" else k
    return inputs.keys(n, dist, seed=seed, device="cuda")


def _keys(case, seed):
    n, dist, dtype = case["n"], case["dist"], case.get("dtype", "int32")
    dev = torch.device("cuda")
    if dist in ("normal", "wide"):
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        if dist == "normal":
            return torch.randn(n, generator=g, device=dev, dtype=getattr(torch, dtype))
        return torch.randint(-2**63, 2**63 - 1, (n,), generator=g, device=dev)
    k = _i32_keys(n, dist, seed)
    if dtype == "uint32":
        return k.view(torch.uint32)
    return k.to(torch.int64) if dtype == "int64" else k


def _random_i32(n, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    return torch.randint(-2**31, 2**31, (n,), generator=g, device="cuda").to(torch.int32)


def prepare(case, seed):
    """The inputs of one call and what a program keeps between calls: output
    arrays, and for the batches the tuned options and a workspace."""
    kind = case["kind"]
    if kind == "cdf_train":
        sample = inputs.keys(case["sample"], "mixture", seed=seed, device="cuda").sort().values
        return {"kind": kind, "sample": sample, "init": inputs.mlp_init(seed).cuda(),
                "batch": case["batch"], "steps": case["steps"], "seed": seed}
    if kind in ("segmented", "segmented_pairs"):
        pairs = kind == "segmented_pairs"
        # the sizes belong to the case, the keys to the seed
        sizes = inputs.log_uniform_sizes(case["nseg"], case["lo"], case["hi"], seed=0)
        offs = inputs.offsets_from_sizes(sizes)
        n = int(offs[-1])
        s = {"kind": kind, "n": n, "max_seg": int(sizes.max()), "off": offs.cuda()}
        if pairs:
            dists = inputs.segment_distributions(case["nseg"], seed=seed).tolist()
            s["keys"] = torch.cat([_i32_keys(m, inputs.DISTRIBUTIONS[d], seed + i)
                                   for i, (m, d) in enumerate(zip(sizes.tolist(), dists))])
            s["vals"] = torch.cat([torch.arange(m, dtype=torch.int32, device="cuda")
                                   for m in sizes.tolist()])
            s["vals_out"] = torch.empty_like(s["vals"])
        else:
            s["keys"] = inputs.keys(n, "uniform", seed=seed, device="cuda")
        s["out"] = torch.empty_like(s["keys"])
        s["opts"] = hv.Options(**(tune.tuned_options(kind, n) or {}))
        need = hv.lib().hvms_segmented_workspace_bytes(n, case["nseg"], s["max_seg"], int(pairs),
                                                       s["opts"])
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        return s
    keys = _keys(case, seed)
    s = {"kind": kind, "keys": keys, "out": torch.empty_like(keys)}
    if kind == "pairs":
        s["vals"] = (torch.arange(case["n"], dtype=torch.int32, device="cuda")
                     if case["values"] == "index" else _random_i32(case["n"], seed))
    elif kind == "by_key":
        s["vals"] = (_random_i32(case["n"], seed).to(torch.int64) << 20) + 12345
    if "vals" in s:
        s["vals_out"] = torch.empty_like(s["vals"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "sort":
        out = hv.sort_keys(s["keys"], out=s["out"])
        return out.view(torch.int32) if out.dtype == torch.uint32 else out
    if kind == "pairs":
        return hv.sort_pairs(s["keys"], s["vals"], s["out"], s["vals_out"])
    if kind == "by_key":
        return hv.sort_by_key(s["keys"], s["vals"], s["out"], s["vals_out"])
    if kind == "segmented":
        hv.hvms_segmented_sort_i32(s["keys"], s["out"], s["off"], s["n"], s["max_seg"], s["ws"],
                                   opts=s["opts"])
        return s["out"]
    if kind == "segmented_pairs":
        hv.hvms_segmented_sort_pairs_i32(s["keys"], s["vals"], s["out"], s["vals_out"], s["off"],
                                         s["n"], s["max_seg"], s["ws"], opts=s["opts"])
        return s["out"], s["vals_out"]
    return hv.cdf_train(s["init"].clone(), s["sample"], batch=s["batch"], steps=s["steps"],
                        seed=s["seed"])


def work(case):
    """Each key, value and payload read once and written once; for a training
    step its minibatch's keys, and the multiply-adds of forward and backward."""
    kind = case["kind"]
    if kind == "cdf_train":
        mults = 32 + 32 * 32 + 32
        return {"bytes": case["steps"] * case["batch"] * 4.0,
                "flops": case["steps"] * case["batch"] * 6.0 * mults}
    if kind in ("segmented", "segmented_pairs"):
        lo, hi = case["lo"], case["hi"]
        mean = (hi - lo) / math.log((hi + 1) / lo)
        return {"bytes": case["nseg"] * mean * (16.0 if kind == "segmented_pairs" else 8.0),
                "flops": 0.0}
    if kind == "sort":
        return {"bytes": case["n"] * (16.0 if case["dtype"].endswith("64") else 8.0), "flops": 0.0}
    return {"bytes": case["n"] * (24.0 if kind == "by_key" else 16.0), "flops": 0.0}


def _splitmix64(seed, k):
    """Output k of SplitMix64 as int64 bit patterns (wrapping arithmetic)."""
    def shr(x, b):
        return (x >> b) & ((1 << (64 - b)) - 1)

    def wrap(c):
        return c - (1 << 64) if c >= 1 << 63 else c

    z = seed + (k + 1) * wrap(0x9E3779B97F4A7C15)
    z = (z ^ shr(z, 30)) * wrap(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * wrap(0x94D049BB133111EB)
    return z ^ shr(z, 31)


def _exact_train(case, seed):
    s = prepare(case, seed)
    p = s["init"].double()
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    total, batch, h = s["sample"].numel(), case["batch"], 32
    k = torch.arange(batch, device="cuda", dtype=torch.int64)
    for step in range(1, case["steps"] + 1):
        r = _splitmix64(seed, ((step - 1) << 32) + k)
        i = (((r >> 32) & 0xFFFFFFFF) % total * ((1 << 32) % total) + (r & 0xFFFFFFFF)) % total
        x = (s["sample"][i].double() + 2.0**31) / 2.0**32
        t = i.double() / total
        w1, b1 = p[:h], p[h:2 * h]
        w2, b2 = p[2 * h:2 * h + h * h].view(h, h), p[2 * h + h * h:3 * h + h * h]
        w3, b3 = p[3 * h + h * h:4 * h + h * h], p[4 * h + h * h]
        z1 = x[:, None] * w1 + b1
        h1 = z1.clamp(min=0)
        z2 = h1 @ w2.t().contiguous() + b2
        h2 = z2.clamp(min=0)
        dy = 2 * (h2 @ w3 + b3 - t) / batch
        dz2 = dy[:, None] * w3 * (z2 > 0)
        dz1 = (dz2 @ w2) * (z1 > 0)
        g = torch.cat([(dz1 * x[:, None]).sum(0), dz1.sum(0),
                       (dz2.t().contiguous() @ h1).reshape(-1), dz2.sum(0),
                       (dy[:, None] * h2).sum(0), dy.sum().view(1)])
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - 1e-3 * (m / (1 - 0.9**step)) / ((v / (1 - 0.999**step)).sqrt() + 1e-8)
    return p, m, v


def exact(case, seed):
    kind = case["kind"]
    if kind == "cdf_train":
        return _exact_train(case, seed)
    s = prepare(case, seed)
    keys = s["keys"].view(torch.int32) if s["keys"].dtype == torch.uint32 else s["keys"]
    if kind == "sort":
        if s["keys"].dtype == torch.uint32:
            return (keys ^ -2**31).sort().values ^ -2**31
        return keys.sort().values
    if kind == "pairs":
        both = ((keys.to(torch.int64) << 32) + (s["vals"].to(torch.int64) + 2**31)).sort().values
        return ((both >> 32).to(torch.int32),
                ((both & 0xFFFFFFFF) - 2**31).to(torch.int32))
    if kind == "by_key":
        k, order = keys.sort(stable=True)
        return k, s["vals"][order]
    seg = torch.searchsorted(s["off"], torch.arange(s["n"], device="cuda"), right=True)
    both = (seg << 31) + keys          # keys lie in [0, 2^31)
    if kind == "segmented":
        return (both.sort().values & (2**31 - 1)).to(torch.int32)
    both, order = both.sort(stable=True)   # values ascend in each segment
    return (both & (2**31 - 1)).to(torch.int32), s["vals"][order]
