"""What this framework is timed on: passes of its public entry points as a
user's program makes them, over the range of sizes, models and options in use.

A case is a dict of plain values; `kind` says which entry points its pass goes
through:

  job      reset, sweeps, then the observables and the tiling (or its hash): a
           plain sampling run, the form of the benchmark's workloads
  step     a few more sweeps of a chain that is kept, and its tiling: the
           smallest calls (animations, convergence checks, interactive use)
  resume   a stored tiling is imported, swept on and exported (checkpoints)
  exact    one exact sample by coupling from the past, and its tiling
  batch    many independent domino chains in one call, and every tiling
  served   a burst of requests to the server, and every result

Outputs are whole numbers and bytes (heights, faces, counts, digests) except
the densities, which are quotients of whole numbers.
"""
import hashlib
import math

import numpy as np

import paper_1804_07250_amd as tl
from paper_1804_07250_amd import serving, workloads

MODELS = {"domino": tl.TL_DOMINO, "lozenge": tl.TL_LOZENGE, "sixvertex": tl.TL_SIXVERTEX}
COLOURS = {"domino": 2, "lozenge": 3, "sixvertex": 4}


def listed():
    return [
        # the smallest call: ten more sweeps of a kept chain, and its tiling
        dict(name="step_aztec32", kind="step", model="domino", n=32, weights="uniform", sweeps=10),
        # the per-face density job of the benchmark: a sample after every sweep
        dict(name="density_aztec64", kind="job", model="domino", n=64, weights="uniform", sweeps=1000, obs_every=1,
             obs_bin=1, out="tiling"),
        # the benchmark's headline job
        dict(name="aztec2048", kind="job", model="domino", n=2048, weights="uniform", sweeps=10000, obs_every=100,
             obs_bin=64, out="hash"),
        # a figure of the two-periodic Aztec diamond: weighted decisions, an odd order
        dict(name="two_periodic1001", kind="job", model="domino", n=1001, weights="two_periodic", wa=1.0, wb=0.5,
             sweeps=2000, obs_every=0, obs_bin=1, out="tiling"),
        # the benchmark's lozenge job (volume weight, 64 x 64 volume bins)
        dict(name="hexagon1024", kind="job", model="lozenge", a=1024, b=1024, c=1024, weights="volume", wa=1999.0,
             wb=2000.0, sweeps=20000, obs_every=200, obs_bin=64, out="tiling"),
        # the benchmark's weighted six-vertex job
        dict(name="sixv1024", kind="job", model="sixvertex", n=1024, weights="sixvertex", wa=1.0, wb=1.0, wc=2.0,
             sweeps=2000, obs_every=100, obs_bin=64, out="tiling"),
        # one-bit decisions of a height model, a ragged size, the paper's random colour order
        dict(name="sixv777_random", kind="job", model="sixvertex", n=777, weights="uniform", sweeps=1000,
             obs_every=250, obs_bin=1, order=1, out="tiling"),
        # a checkpoint of an uneven hexagon picked up again (lazy Metropolis)
        dict(name="resume_hexagon", kind="resume", model="lozenge", a=301, b=200, c=157, weights="volume", wa=9.0,
             wb=10.0, metropolis=True, sweeps=300),
        # the L-shaped six-vertex domain of the paper, bins every 50 sweeps
        dict(name="lshape_sixv400", kind="job", model="sixvertex", shape="l", n=400, cut_w=160, cut_h=200,
             weights="uniform", sweeps=1000, obs_every=50, obs_bin=16, out="tiling"),
        # the batched form: chains of uneven orders as in the benchmark, one GPU's worth of tilings taken home
        dict(name="batch512", kind="batch", chains=512, lo=16, hi=512, weights="two_periodic", wa=1.0, wb=0.5,
             sweeps=5000),
        # the served form: a burst of the benchmark's request mix
        dict(name="served24", kind="served", requests=24, sweeps=2000, slots=64, budget_mib=1024),
        # exact sampling, the benchmark's six-vertex case
        dict(name="exact_sixv128", kind="exact", model="sixvertex", n=128, weights="uniform"),
    ]


# ------------------------------------------------------------------- drawing

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _weighted(rng, model):
    """A weight choice of the model: uniform, or the weights it is used with."""
    if rng.random() < 0.4:
        c = dict(weights="uniform")
    elif model == "domino":
        c = rng.choice([dict(weights="two_periodic", wa=1.0, wb=rng.choice([0.5, 0.25, 0.75])),
                        dict(weights="volume_bw", wa=5.0, wb=4.0, wc=rng.choice([2.0, 4.0]), wd=3.0)])
    elif model == "lozenge":
        c = rng.choice([dict(weights="volume", wa=9.0, wb=10.0), dict(weights="volume", wa=1999.0, wb=2000.0)])
    else:
        c = rng.choice([dict(weights="sixvertex", wa=1.0, wb=1.0, wc=2.0),
                        dict(weights="sixvertex", wa=4.0, wb=1.0, wc=4.0)])
    if rng.random() < 0.3:
        c["metropolis"] = True
    return c


def _shape(rng, model, lo, hi):
    if model == "lozenge":
        a, b, c = (_log_int(rng, lo, hi) for _ in range(3))
        return dict(a=a, b=b, c=c)
    return dict(n=_log_int(rng, lo, hi))


# Site updates a drawn plain case may ask for, by whether its decisions are
# one-bit: about the time of the largest listed one at the rates of the models.
_MOST_UPDATES = {("domino", True): 6e10, ("domino", False): 1e10, ("lozenge", True): 1.5e10,
                 ("lozenge", False): 6e9, ("sixvertex", True): 1e10, ("sixvertex", False): 3e9}


def _sweeps(rng, case, lo, hi):
    most = _MOST_UPDATES[(case["model"], case["weights"] == "uniform")]
    if case.get("order"):
        most /= 3
    return max(1, min(_log_int(rng, lo, hi), int(most / (_sites(case) * COLOURS[case["model"]]))))


def draw(rng):
    kind = rng.choice(["job", "job", "job", "job", "job", "mask", "mask", "step", "step", "resume", "resume",
                       "exact", "batch", "served"])
    model = rng.choice(["domino", "domino", "lozenge", "sixvertex"])
    if kind == "batch":
        lo = _log_int(rng, 8, 64)
        hi = _log_int(rng, 2 * lo, 512)
        c = dict(kind="batch", chains=_log_int(rng, 16, 512), lo=lo, hi=hi, sweeps=_log_int(rng, 100, 5000))
        c.update(dict(weights="uniform") if rng.random() < 0.4 else
                 dict(weights="two_periodic", wa=1.0, wb=rng.choice([0.5, 0.25])))
        if rng.random() < 0.25:
            c.update(order=1)
        return c
    if kind == "served":
        return dict(kind="served", requests=rng.randint(2, 32), sweeps=_log_int(rng, 100, 2000),
                    slots=rng.choice([8, 64]), budget_mib=rng.choice([16, 1024]))
    if kind == "exact":
        if model == "lozenge":
            c = dict(kind="exact", model=model, **_shape(rng, model, 3, 20))
        else:
            c = dict(kind="exact", model=model, n=_log_int(rng, 6, 64 if model == "domino" else 100))
        if model == "sixvertex" and rng.random() < 0.4:
            c.update(weights="sixvertex", wa=1.0, wb=1.0, wc=2.0, n=min(c["n"], 64))
        elif model == "lozenge" and rng.random() < 0.4:
            c.update(weights="volume", wa=9.0, wb=10.0)
        else:
            c.update(weights="uniform")
        return c
    if kind == "step":
        c = dict(kind="step", model=model, **_shape(rng, model, 8, 400), **_weighted(rng, model))
        c["sweeps"] = _sweeps(rng, c, 1, 100)
        return c
    if kind == "resume":
        c = dict(kind="resume", model=model, **_shape(rng, model, 16, 500), **_weighted(rng, model))
        c["sweeps"] = _sweeps(rng, c, 10, 1000)
        return c
    c = dict(kind="job", model=model)
    if kind == "mask":
        if model == "domino":
            w, h = _log_int(rng, 16, 900), 2 * _log_int(rng, 8, 450)
            c.update(shape="rectangle", w=w, h=h)
        elif model == "sixvertex":
            n = _log_int(rng, 24, 700)
            c.update(shape="l", n=n, cut_w=max(1, (2 * n) // 5), cut_h=n // 2)
        else:
            c.update(shape="triangles", **_shape(rng, model, 8, 300))
    else:
        c.update(_shape(rng, model, 16, 2048 if model == "domino" else 1024))
    c.update(_weighted(rng, model))
    if rng.random() < 0.25:
        c["order"] = 1
    c["sweeps"] = _sweeps(rng, c, 100, 20000)
    # a sample every so many sweeps, as many as a density map takes
    c["obs_every"] = rng.choice([0, max(1, c["sweeps"] // rng.choice([10, 40, 100]))])
    c["obs_bin"] = rng.choice([1, 16, 64])
    c["out"] = rng.choice(["tiling", "hash"])
    return c


# ----------------------------------------------------------- domains, weights

def _l_shape(n, cut_w, cut_h):
    """The n x n square without its north-east cut_w x cut_h corner."""
    m = np.ones((n, n), dtype=np.uint8)
    m[n - cut_h:, n - cut_w:] = 0
    return m


def _hexagon_triangles(a, b, c):
    """The hexagon's unit triangles as a mask: those whose corners all satisfy
    -b <= x - y <= a in the sheared box (shifted by c)."""
    h, w = b + c, a + c
    y, x = np.mgrid[0:h, 0:w]

    def inside(X, Y):
        return (X - Y >= -b) & (X - Y <= a)

    low = inside(x, y) & inside(x + 1, y) & inside(x + 1, y + 1)
    up = inside(x, y) & inside(x, y + 1) & inside(x + 1, y + 1)
    return np.stack([low, up], axis=2).astype(np.uint8)


def _domain(case):
    model = MODELS[case["model"]]
    shape = case.get("shape")
    if shape == "l":
        return tl.domain(model, mask=_l_shape(case["n"], case["cut_w"], case["cut_h"]))
    if shape == "rectangle":
        return tl.domain(model, mask=np.ones((case["h"], case["w"]), dtype=np.uint8))
    if shape == "triangles":
        return tl.domain(model, mask=_hexagon_triangles(case["a"], case["b"], case["c"]))
    if case["model"] == "lozenge":
        return tl.domain(model, a=case["a"], b=case["b"], c=case["c"])
    return tl.domain(model, n=case["n"])


def _weights(case):
    kind = {"uniform": tl.TL_W_UNIFORM, "two_periodic": tl.TL_W_TWO_PERIODIC, "volume": tl.TL_W_VOLUME,
            "sixvertex": tl.TL_W_SIXVERTEX, "volume_bw": tl.TL_W_VOLUME_BW}[case["weights"]]
    w = [case[k] for k in ("wa", "wb", "wc", "wd") if k in case]
    return tl.weights(kind, *w, rule=tl.TL_METROPOLIS if case.get("metropolis") else tl.TL_HEATBATH)


def _options(case):
    return tl.options(obs_every=case.get("obs_every", 0), obs_bin=case.get("obs_bin", 1),
                      colour_order=case.get("order", 0))


def _cells(case):
    """Faces, vertices or points of the case's export."""
    if case["model"] == "domino":
        return case["w"] * case["h"] if case.get("shape") == "rectangle" else 4 * case["n"] ** 2
    if case["model"] == "lozenge":
        return (case["a"] + case["c"] + 1) * (case["b"] + case["c"] + 1)
    return (case["n"] + 1) ** 2


def _sites(case):
    if case["model"] == "domino":
        return _cells(case) if case.get("shape") == "rectangle" else 2 * case["n"] ** 2
    if case["model"] == "lozenge":
        a, b, c = case["a"], case["b"], case["c"]
        return a * b + b * c + a * c
    return case["n"] ** 2 - case.get("cut_w", 0) * case.get("cut_h", 0)


# --------------------------------------------------------------------- passes

def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        # the benchmark's orders over the case's range; the seed keys the chains
        orders = workloads.batch_orders(case["chains"], case["lo"], case["hi"])
        batch = serving.Batch([tl.domain(tl.TL_DOMINO, n=n) for n in orders], _weights(case),
                              [seed + i for i in range(len(orders))], _options(case))
        batch.autotune(4)
        return dict(case=case, batch=batch)
    if kind == "served":
        # sizes, weights and rule of the request mix; a burst has no arrival times
        jobs = []
        for r in workloads.serve_requests(case["requests"], seed=seed):
            w = tl.weights(tl.TL_W_SIXVERTEX, *r["w2"], rule=tl.TL_METROPOLIS)
            jobs.append((tl.domain(tl.TL_SIXVERTEX, n=r["N"]), w, seed + r["seed"]))
        return dict(case=case, jobs=jobs, server=serving.Server(case["budget_mib"] << 20, case["slots"]))
    sampler = tl.Sampler(_domain(case), _weights(case), seed, _options(case))
    state = dict(case=case, seed=seed, sampler=sampler)
    if kind == "resume":
        # the checkpoint: the chain's own state some way into the run
        sampler.sweep(2 * case["sweeps"])
        state["checkpoint"], state["at"] = sampler.export(), 2 * case["sweeps"]
    sampler.sync()
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        batch = state["batch"]
        batch.reset()
        batch.sweep(case["sweeps"])
        return np.concatenate([batch.export(i).reshape(-1) for i in range(batch.n)])
    if kind == "served":
        server = state["server"]
        tickets = [server.submit(dom, w, seed, case["sweeps"]) for dom, w, seed in state["jobs"]]
        results = [server.wait(t) for t in tickets]
        return dict(status=np.array([r["status"] for r in results]), sweeps=np.array([r["sweeps"] for r in results]),
                    scalar=np.array([r["scalar_now"] for r in results]), hash=np.stack([_digest(r["hash"]) for r in results]))
    sampler = state["sampler"]
    if kind == "step":
        sampler.sweep(case["sweeps"])
        return sampler.export()
    if kind == "resume":
        sampler.import_(state["checkpoint"], state["at"])
        sampler.sweep(case["sweeps"])
        return sampler.export()
    sampler.reset(state["seed"])
    if kind == "exact":
        info = sampler.cftp(28)
        return dict(info=info, tiling=sampler.export())
    sampler.sweep(case["sweeps"])
    out = {}
    if case["obs_every"]:
        out["observables"] = sampler.observables()
    if case["out"] == "hash":
        out["hash"] = _digest(sampler.hash())
    else:
        out["tiling"] = sampler.export()
    return out


def _digest(text):
    return np.frombuffer(bytes.fromhex(text), dtype=np.uint8)


# ----------------------------------------------------------------------- work

# 32-bit operations of one Philox4x32-10 call (ten rounds of two products and
# two three-way exclusive ors), which draws a bit for each of 128 sites, and of
# testing and flipping a word of 32 sites in one colour step.
_PHILOX_OPS, _STEP_OPS = 40, 16


def _plane_count(case):
    """Bits a decision needs: one where every threshold is a half, two on
    average where bits are compared until they differ."""
    return 1.0 if case["weights"] == "uniform" else 2.0


def _updates_ops(updates, planes):
    return updates * (planes * _PHILOX_OPS / 128.0 + _STEP_OPS / 32.0)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        lo, hi = case["lo"], case["hi"]
        n2 = (lo * lo + lo * hi + hi * hi) / 3.0 * case["chains"]   # mean square order, all chains
        return {"bytes": n2 * (1.0 + 4.0), "flops": _updates_ops(2 * n2 * case["sweeps"], _plane_count(case))}
    if kind == "served":
        n2 = sum(n * n for n in workloads.SERVE_SIZES) / len(workloads.SERVE_SIZES) * case["requests"]
        return {"bytes": n2 / 4.0, "flops": _updates_ops(n2 * case["sweeps"], 1.5)}
    sites = _sites(case)
    # the packed state read and written, and the export where it comes home
    state = sites / 2.0 if case["model"] == "domino" else sites / 4.0
    export = _cells(case) * (1 if case["model"] == "domino" else 4)
    sweeps = case.get("sweeps", 0)
    if kind == "exact":
        # two chains over the doubling rounds: about n^2 sweeps for a domain of side n
        sweeps = 4 * sites
    moved = state + (32 if case.get("out") == "hash" else export) + (export if kind == "resume" else 0)
    if case.get("obs_every"):
        bins = _cells(case) / case["obs_bin"] ** 2
        moved += 8 * bins + (sweeps // case["obs_every"]) * state / 2
    return {"bytes": float(moved), "flops": _updates_ops(float(sites) * sweeps, _plane_count(case))}


# ---------------------------------------------------------------------- exact

_MASK = np.uint64(0xFFFFFFFF)


def _philox(c0, c1, c2, c3, key):
    """Philox4x32-10 (Salmon et al. 2011) of arrays of counters, as 64-bit integers."""
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    c0, c1, c2, c3 = (np.asarray(v, dtype=np.uint64) for v in (c0, c1, c2, c3))
    for _ in range(10):
        p0, p1 = c0 * np.uint64(0xD2511F53), c2 * np.uint64(0xCD9E8D57)
        c0, c1, c2, c3 = ((p1 >> np.uint64(32)) ^ c1 ^ np.uint64(k0), p1 & _MASK,
                          (p0 >> np.uint64(32)) ^ c3 ^ np.uint64(k1), p0 & _MASK)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1, c2, c3


def _aztec_job(n, seed, sweeps, every, B):
    """The uniform Aztec chain in plain numpy: faces as partner directions
    (0 north, 1 south, 2 east, 3 west, 255 outside), one Philox bit per vertex
    and colour step, and the horizontal-face counts of the samples."""
    Y, X = np.mgrid[-n:n, -n:n]
    inside = np.abs(2 * X + 1) + np.abs(2 * Y + 1) <= 2 * n
    half = np.where(Y >= 0, n - Y, n + Y + 1)      # faces of a row: x in [-half, half)
    F = np.where(inside, np.where((X + half) % 2 == 0, 2, 3), 255).astype(np.uint8)
    total = 2 * n
    bins = -(-total // B)
    counts = np.zeros((bins, bins), dtype=np.uint64)

    def count():
        horiz = np.zeros((bins * B, bins * B), dtype=np.uint64)
        horiz[:total, :total] = (F == 2) | (F == 3)
        return horiz.reshape(bins, B, bins, B).sum(axis=(1, 3))

    steps = []
    for c in (0, 1):
        y, x = np.mgrid[1 - n:n, 1 - n:n]
        at = (np.abs(x) + np.abs(y) <= n - 1) & ((x + y) % 2 == c)
        y, x = y[at], x[at]
        r, k = (x + y + n - 1) // 2, (y - x + n - 1) // 2
        key = np.unique(np.stack([k >> 7, r]), axis=1, return_inverse=True)
        steps.append((y + n, x + n, key[0], key[1].reshape(-1), (k >> 5) & 3, np.uint64(1) << (k & 31).astype(np.uint64)))
    samples = 0
    for t in range(sweeps):
        for c, (y, x, groups, which, word, bit) in enumerate(steps):
            draws = np.stack(_philox(groups[0], groups[1], np.full(groups.shape[1], t), np.full(groups.shape[1], c), seed))
            up = (draws[word, which] & bit) == 0       # the top bit of the uniform: u < 2^31
            sw, se, nw, ne = F[y - 1, x - 1], F[y - 1, x], F[y, x - 1], F[y, x]
            flat = (sw == 2) & (se == 3) & (nw == 2) & (ne == 3)
            tall = (sw == 0) & (nw == 1) & (se == 0) & (ne == 1)
            for move, (a, b, d, e) in ((flat & up, (0, 0, 1, 1)), (tall & ~up, (2, 3, 2, 3))):
                yy, xx = y[move], x[move]
                F[yy - 1, xx - 1], F[yy - 1, xx], F[yy, xx - 1], F[yy, xx] = a, b, d, e
        if every and (t + 1) % every == 0:
            counts += count()
            samples += 1
    cells = np.zeros((bins * B, bins * B))
    cells[:total, :total] = inside
    cells = cells.reshape(bins, B, bins, B).sum(axis=(1, 3))
    density = np.where((cells > 0) & (samples > 0), counts / (max(samples, 1) * np.maximum(cells, 1.0)), 0.0)
    return F, counts, count(), density, samples


def exact(case, seed):
    """Densities are the only outputs that are not whole numbers or bytes: the
    small uniform Aztec jobs are run in plain numpy for them (whole)."""
    if (case["kind"] != "job" or case["model"] != "domino" or case.get("shape") or case["weights"] != "uniform"
            or case.get("order") or not case["obs_every"] or case["n"] ** 2 * case["sweeps"] > 5e6):
        return None
    F, counts, now, density, samples = _aztec_job(case["n"], seed, case["sweeps"], case["obs_every"], case["obs_bin"])
    out = dict(observables=dict(sweeps=case["sweeps"], samples=samples, scalar_now=int(now.sum()),
                                scalar_sum=int(counts.sum()), bin_sum=counts, bin_now=now, bin_density=density))
    if case["out"] == "hash":
        rows = b"".join(hashlib.sha256(row.tobytes()).digest() for row in F)
        out["hash"] = _digest(hashlib.sha256(rows).hexdigest())
    else:
        out["tiling"] = F
    return out
