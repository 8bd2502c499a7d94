"""Workloads the library's speed is followed on: one sampling step over a batch of tuning tasks.

A pass is what a search loop does once per round with candidates that are already on the GPU:
k-means sweep over the list of k, knee, snap, Sample Synthesis + dedupe, through the entry points
of ``paper_2001_08743_amd.binding``, with the output buffers and workspaces the program keeps from
round to round.  Sizes are those of ``workloads.make_config`` / ``workloads.wide_space`` and of
the tests; ``draw`` spreads over the same ranges.

Inputs are made on the GPU (same recipe as ``workloads``): cardinalities uniform in a range, blob
centres uniform in the design space, blob weights uneven, point = round(centre + sigma * normal)
clipped to the knob, a share of rows replaced by uniform-random invalid rows; the visited set is
hashes of sampled rows, of random configurations and of configurations of other runs.
"""
import math
import random

import numpy as np
import torch

from paper_2001_08743_amd import binding

_BASE = dict(tasks=1, rows=256, ragged=False, d=8, card_lo=2, card_hi=32, wide=False, wide_frac=0.0, wide_lo=64, wide_hi=600,
             blobs_lo=4, blobs_hi=64, sigma=1.5, sigma_rel=0.0, invalid=0.05, ks="2:16", n_iter=30, visited=0, table=False,
             knee_chunk=0, warm=False, labels=False)


def _case(**kw):
    c = dict(_BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one task of a few hundred candidates, latency and launches count
        _case(name="single-tiny", rows=256, d=8, card_hi=16, blobs_lo=6, blobs_hi=6, sigma=1.0, invalid=0.0, ks="2:16", n_iter=30),
        # one conv2d layer tuned by itself
        _case(name="single-conv", rows=4096, d=12, card_lo=3, card_hi=24, blobs_lo=16, blobs_hi=16, ks="2:64", n_iter=50, visited=4096),
        # the layers of a model tuned together, ordinary sizes
        _case(name="batch-conv", tasks=64, rows=1024, d=12, card_lo=3, card_hi=24, blobs_lo=8, blobs_hi=24, ks="2:32", n_iter=30,
              visited=65536),
        # the full-model sweep: the benchmark's default workload
        _case(name="full-model", tasks=256, rows=4096, d=24, ks="1:64", n_iter=50, visited=1048576),
        # a later search round of the same layers: candidates of uneven number, centroids of the last
        # round as the start, labels kept
        _case(name="warm-ragged", tasks=24, rows=3001, ragged=True, d=21, ks="4:48:4", n_iter=20, visited=20001, warm=True, labels=True),
        # Algorithm 1 as printed: the sweep stops at the knee; the visited set lives in a device table
        _case(name="knee-table", tasks=256, rows=4096, d=24, ks="8:64", n_iter=50, visited=262144, table=True, knee_chunk=8),
        # one very large clustering, powers of two for k
        _case(name="large-single", rows=1048576, d=16, blobs_lo=128, blobs_hi=128, sigma=2.0, invalid=0.0, ks="16,32,64,128,256", n_iter=20),
        # candidate pools of some ten thousand rows each, odd sizes and an odd number of knobs
        _case(name="pools-ragged", tasks=6, rows=60013, ragged=True, d=23, blobs_lo=16, blobs_hi=48, ks="8,16,24,32,48,64,96", n_iter=20,
              visited=8192),
        # many small clusters of ordinary tasks (k beyond 64)
        _case(name="many-clusters", tasks=16, rows=2500, ragged=True, d=24, blobs_lo=32, blobs_hi=64, ks="72,96,128", n_iter=20, visited=4096),
        # byte knobs at the interface's largest number of knobs
        _case(name="knobs-32", tasks=32, rows=2048, d=32, blobs_lo=8, blobs_hi=24, ks="2:32:2", n_iter=30, visited=16384),
        # design spaces with split knobs of some hundred choices
        _case(name="wide-batch", tasks=64, rows=2048, d=40, wide=True, wide_frac=0.3, blobs_lo=8, blobs_hi=24, sigma_rel=0.02, ks="2:32",
              n_iter=30, visited=4096),
        # ... and of thousands of choices
        _case(name="wide-thousands", tasks=16, rows=1900, ragged=True, d=27, wide=True, wide_frac=0.4, wide_hi=5000, blobs_lo=8, blobs_hi=24,
              sigma_rel=0.02, ks="2:40:2", n_iter=20, visited=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges of the listed ones."""
    kind = rng.choice(["single", "batch", "full", "warm", "knee", "large", "pools", "many", "knobs32", "wide", "thousands"])
    sigma = round(rng.uniform(0.8, 2.5), 2)
    blobs = dict(blobs_lo=rng.randint(4, 12), blobs_hi=rng.randint(16, 64))
    if kind == "single":
        rows, top = _log_int(rng, 200, 4096), rng.randint(8, 64)
        return _case(rows=rows, d=rng.randint(4, 31), sigma=sigma, ks="2:%d" % top, n_iter=rng.randint(20, 50), visited=_log_int(rng, 16, 8192), **blobs)
    if kind == "batch":
        return _case(tasks=_log_int(rng, 4, 128), rows=_log_int(rng, 300, 4096), ragged=rng.random() < 0.5, d=rng.randint(6, 31), sigma=sigma,
                     ks="2:%d" % rng.randint(12, 48), n_iter=rng.randint(20, 50), visited=_log_int(rng, 64, 131072), **blobs)
    if kind == "full":
        return _case(tasks=rng.randint(96, 224), rows=rng.randint(2000, 4096), ragged=rng.random() < 0.3, d=rng.randint(16, 30), sigma=sigma,
                     ks="1:%d" % rng.randint(40, 64), n_iter=rng.randint(30, 50), visited=_log_int(rng, 4096, 1048576), **blobs)
    if kind == "warm":
        return _case(tasks=_log_int(rng, 2, 64), rows=_log_int(rng, 500, 4096), ragged=True, d=rng.randint(9, 31), sigma=sigma,
                     ks="4:%d:4" % rng.randint(16, 64), n_iter=rng.randint(10, 30), visited=_log_int(rng, 64, 65536), warm=True, labels=True, **blobs)
    if kind == "knee":
        return _case(tasks=_log_int(rng, 4, 256), rows=_log_int(rng, 500, 4096), d=rng.randint(8, 31), sigma=sigma, ks="8:%d" % rng.randint(24, 64),
                     n_iter=rng.randint(20, 50), visited=_log_int(rng, 256, 262144), table=True, knee_chunk=rng.choice([4, 8, 16]), **blobs)
    if kind == "large":
        return _case(rows=_log_int(rng, 100000, 1000000), d=rng.randint(10, 20), blobs_lo=64, blobs_hi=128, sigma=sigma, invalid=0.0,
                     ks=rng.choice(["16,32,64,128,256", "16,32,64", "50,100,200", "64,128"]), n_iter=rng.randint(10, 20))
    if kind == "pools":
        return _case(tasks=rng.randint(1, 8), rows=_log_int(rng, 6000, 100000), ragged=True, d=rng.randint(10, 31), sigma=sigma,
                     ks=rng.choice(["8,16,24,32,48,64,96", "8,16,32,64", "20,40,80"]), n_iter=rng.randint(10, 20), visited=_log_int(rng, 64, 16384), **blobs)
    if kind == "many":
        return _case(tasks=_log_int(rng, 2, 32), rows=rng.randint(1500, 4096), ragged=rng.random() < 0.5, d=rng.randint(12, 31), sigma=sigma,
                     ks=rng.choice(["72,96,128", "65,80", "100,200"]), n_iter=rng.randint(10, 20), visited=_log_int(rng, 64, 8192), **blobs)
    if kind == "knobs32":
        return _case(tasks=_log_int(rng, 4, 64), rows=rng.randint(500, 3000), ragged=rng.random() < 0.5, d=32, sigma=sigma, ks="2:%d:2" % rng.randint(16, 40),
                     n_iter=rng.randint(15, 30), visited=_log_int(rng, 64, 32768), **blobs)
    if kind == "wide":
        return _case(tasks=_log_int(rng, 4, 64), rows=rng.randint(500, 2048), ragged=rng.random() < 0.5, d=rng.randint(20, 63), wide=True, wide_frac=0.3,
                     wide_hi=rng.randint(200, 2000), sigma_rel=0.02, ks="2:%d" % rng.randint(12, 32), n_iter=rng.randint(15, 30),
                     visited=_log_int(rng, 64, 8192), **blobs)
    return _case(tasks=_log_int(rng, 2, 24), rows=rng.randint(500, 2500), ragged=True, d=rng.randint(16, 48), wide=True, wide_frac=0.4,
                 wide_hi=rng.randint(2500, 8000), sigma_rel=0.02, ks="2:%d:2" % rng.randint(16, 40), n_iter=rng.randint(10, 20),
                 visited=_log_int(rng, 64, 8192), **blobs)


def _ks(case):
    text = case["ks"]
    if ":" in text:
        p = [int(x) for x in text.split(":")]
        return list(range(p[0], p[1] + 1, p[2] if len(p) > 2 else 1))
    return [int(x) for x in text.split(",")]


def _sizes(case):
    if not case["ragged"]:
        return [case["rows"]] * case["tasks"]
    rng = random.Random(case["rows"] * 1000 + case["tasks"])        # sizes belong to the case, values to the seed
    return [max(1, int(case["rows"] * rng.uniform(0.35, 1.0))) for _ in range(case["tasks"])]


def prepare(case, seed):
    dev = torch.device("cuda:0")
    rng = random.Random(seed)
    g = torch.Generator(device=dev).manual_seed(seed)
    T, d, ks = case["tasks"], case["d"], _ks(case)
    sizes = _sizes(case)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    ld = (n + 63) // 64 * 64

    def cards_of():
        if rng.random() < case["wide_frac"]:
            return rng.randint(case["wide_lo"], case["wide_hi"])
        return rng.randint(case["card_lo"], case["card_hi"])

    cards = np.array([[cards_of() for _ in range(d)] for _ in range(T)], dtype=np.uint16)
    # rows: blobs of uneven weight per task
    cd = torch.from_numpy(cards.astype(np.float32)).to(dev)
    sizes_t = torch.tensor(sizes, device=dev)
    task = torch.repeat_interleave(torch.arange(T, device=dev), sizes_t, output_size=n)
    nb = [rng.randint(case["blobs_lo"], max(case["blobs_lo"], case["blobs_hi"])) for _ in range(T)]
    bmax = max(nb)
    live = torch.arange(bmax, device=dev)[None, :] < torch.tensor(nb, device=dev)[:, None]
    weight = -torch.log(torch.rand((T, bmax), generator=g, device=dev).clamp_min(1e-12)) * live
    cum = torch.cumsum(weight / weight.sum(1, keepdim=True), 1)
    centre = torch.rand((T, bmax, d), generator=g, device=dev) * (cd[:, None, :] - 1)
    pick = torch.rand(n, generator=g, device=dev)
    which = (cum[task] < pick[:, None]).sum(1)
    which = torch.minimum(which, torch.tensor(nb, device=dev)[task] - 1)
    spread = torch.clamp(cd * case["sigma_rel"], min=case["sigma"])
    rows = centre[task, which] + spread[task] * torch.randn((n, d), generator=g, device=dev)
    top = cd[task] - 1
    rows = torch.minimum(torch.round(rows).clamp_min(0), top)
    spoiled = torch.rand(n, generator=g, device=dev) < case["invalid"]
    uniform = torch.floor(torch.rand((n, d), generator=g, device=dev) * (top + 1)).minimum(top)
    rows = torch.where(spoiled[:, None], uniform, rows)
    knob = torch.int16 if case["wide"] else torch.uint8
    rows = rows.to(knob)
    X = torch.zeros((d, ld), dtype=knob, device=dev)
    X[:, :n] = rows.T
    valid = torch.zeros(ld, dtype=torch.uint8, device=dev)
    valid[:n] = (~spoiled).to(torch.uint8)

    sfx = "_u16" if case["wide"] else ""
    # two-byte knobs whose cardinalities are at most 2048 carry the caller's promise
    flags = binding.F_VALUES_BELOW_2048 if case["wide"] and int(cards.max()) <= 2048 else 0
    s = dict(case=case, X=X, ld=ld, d=d, off=off, ks=ks, cards=cards, valid=valid, sfx=sfx, flags=flags,
             salts=np.arange(T, dtype=np.uint64), init=None, visited=None, table=None)

    nv = case["visited"]
    if nv:
        # half rows of this batch, a quarter random configurations of it, the rest hashes of other runs
        own = torch.randint(0, n, (nv // 2,), generator=g, device=dev)
        rt = torch.randint(0, T, (nv // 4,), generator=g, device=dev)
        rc = torch.floor(torch.rand((nv // 4, d), generator=g, device=dev) * cd[rt]).minimum(cd[rt] - 1).to(knob)
        cfg = torch.cat([rows[own], rc]).contiguous()
        salt = torch.cat([task[own], rt]).to(torch.int64).contiguous()
        h = binding.cham_hash_rows(cfg, salt, _sfx=sfx)
        other = torch.randint(-2 ** 63, 2 ** 63 - 1, (nv - h.numel(),), generator=g, device=dev, dtype=torch.int64)
        h = torch.cat([h, other])
        if case["table"]:
            slots = 1 << max(4, (4 * nv - 1).bit_length())
            s["table"] = torch.empty(slots, dtype=torch.int64, device=dev)
            binding.cham_visited_table_clear(s["table"])
            binding.cham_visited_table_insert_hashes(s["table"], h)
        else:
            sign = torch.tensor(-2 ** 63, dtype=torch.int64, device=dev)
            s["visited"] = torch.sort(h ^ sign).values ^ sign          # ascending as unsigned words

    if case["warm"]:
        # centroids of the round before: means of a few candidates each
        parts = []
        for k in ks:
            at = torch.from_numpy(off[:-1]).to(dev)[:, None, None] + \
                (torch.rand((T, k, 3), generator=g, device=dev) * sizes_t[:, None, None]).long().minimum(sizes_t[:, None, None] - 1)
            parts.append(rows[at].double().mean(2))
        s["init"] = torch.cat(parts, 1).contiguous()

    # output buffers and workspaces the program keeps
    n_k, kmax, ksum = len(ks), ks[-1], sum(ks)
    f64 = dict(dtype=torch.float64, device=dev)
    i32 = dict(dtype=torch.int32, device=dev)
    u8 = dict(dtype=torch.uint8, device=dev)
    s["sweep"] = dict(centroids=torch.zeros((T, ksum, d), **f64), counts=torch.zeros((T, ksum), **i32), inertia=torch.zeros((T, n_k), **f64),
                      status=torch.zeros((T, n_k), **i32), chosen=torch.zeros(T, **i32),
                      labels=torch.zeros((n_k, ld), **u8) if case["labels"] else None, trace=None)
    s["snap"] = dict(labels_sel=torch.zeros(ld, **u8), pick_row=torch.zeros((T, kmax), **i32), pick_cfg=torch.zeros((T, kmax, d), dtype=knob, device=dev))
    s["synth"] = dict(out_cfg=torch.zeros((T, kmax, d), dtype=knob, device=dev), out_flag=torch.zeros((T, kmax), **u8), out_count=torch.zeros(T, **i32))
    size = binding.cham_sweep_knee_workspace_bytes if case["knee_chunk"] else binding.cham_sweep_workspace_bytes
    s["sweep_ws"] = torch.empty(max(256, size(ld, d, off, ks, case["n_iter"], flags, _sfx=sfx)), **u8)
    lib = binding.load()
    to, k32 = np.ascontiguousarray(off), np.asarray(ks, dtype=np.int32)
    for name in ("snap", "synth"):
        need = getattr(lib, "cham_%s_workspace_bytes%s" % (name, sfx))(ld, d, to.ctypes.data, T, k32.ctypes.data, n_k)
        if need < 0:
            raise RuntimeError("cham_%s_workspace_bytes: %d" % (name, need))
        s[name + "_ws"] = torch.empty(max(256, need), **u8)
    return s


def run(s):
    case, sfx = s["case"], s["sfx"]
    X, ld, d, off, ks = s["X"], s["ld"], s["d"], s["off"], s["ks"]
    start = dict(init_centroids=s["init"], flags=s["flags"], out=s["sweep"], workspace=s["sweep_ws"], _sfx=sfx)
    if case["knee_chunk"]:
        sw = binding.cham_kmeans_sweep_knee(X, ld, d, off, ks, case["n_iter"], threshold=2.5, chunk=case["knee_chunk"], **start)
        chosen = sw["chosen"]
    else:
        sw = binding.cham_kmeans_sweep(X, ld, d, off, ks, case["n_iter"], **start)
        chosen = binding.cham_select_k(sw["inertia"], sw["status"], 2.5, chosen=s["sweep"]["chosen"])
    sn = binding.cham_snap_centroids(X, ld, d, off, ks, chosen, sw["centroids"], out=s["snap"], workspace=s["snap_ws"], _sfx=sfx)
    last = dict(task_salt=s["salts"], out=s["synth"], workspace=s["synth_ws"], _sfx=sfx)
    picks = (sn["labels_sel"], sn["pick_row"], sn["pick_cfg"])
    if s["table"] is not None:
        sy = binding.cham_synthesize_table(X, ld, d, off, s["cards"], s["valid"], ks, chosen, *picks, s["table"], **last)
    else:
        sy = binding.cham_synthesize(X, ld, d, off, s["cards"], s["valid"], ks, chosen, *picks, s["visited"], **last)
    return [sw["centroids"], sw["counts"], sw["inertia"], sw["status"], sw["labels"], chosen, *picks,
            sy["out_cfg"], sy["out_flag"], sy["out_count"]]


def work(case):
    """Bytes: every knob read once, every output written once.  Operations: a multiply and an add per
    knob, row and centroid in every labelling pass; an iteration reaches its fixed point after
    about half of its steps (23.8 of 51 passes measured on the full-model workload).  A sweep that
    stops at the knee needs its first two values of k."""
    ks = _ks(case)
    n = sum(_sizes(case))
    size = 2 if case["wide"] else 1
    ksum = sum(ks)
    out = case["tasks"] * (ksum * (8 * case["d"] + 4) + len(ks) * 12 + ks[-1] * (2 * size * case["d"] + 5) + 8) + n * (1 + (len(ks) if case["labels"] else 0))
    evals = n * (sum(ks[:2]) if case["knee_chunk"] else ksum) * (1 + case["n_iter"]) * 0.5
    return {"bytes": n * (size * case["d"] + 1) + out, "flops": evals * 2 * case["d"]}


def tolerance(case):
    """Labels, counts, picks and configurations are whole numbers and have to be the same; centroids are
    quotients of whole numbers.  The loss is a sum of up to 2^20 doubles whose order is free: between the
    library's own kernel families it differs by up to 6e-16, and a plain running sum over 2^20 terms is
    up to 5e-14 away from the exactly rounded one."""
    return {"rel": 5e-14, "max": 5e-14, "differ": 0.0}
