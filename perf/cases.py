"""The work that programs have this library do, as cases that can be timed.

Every case is a whole call sequence of a user's program: one or many annealing
runs from their descriptors to their records (and, where the program asks for
them, configurations, weighted averages and overlap distributions), or a batch
of requests through the continuous-batching server.  A descriptor determines
its run, so a case's inputs are its descriptors, with every seed drawn from
the case's seed.

  listed()             the cases, from one small run to the full-size ones
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  what the program holds before the call
  run(state)           one pass through the public entry points
  work(case)           bytes and operations the pass cannot do without
  exact(case, seed)    what run returns, in plain 64-bit torch / numpy, for
                       the cases small enough
"""
import math
import os

import numpy as np
import torch

import paper_2207_05535_amd as pa
import workloads as W

TUNED = {"": None, "fm": "tuning_cache.json", "two_pop": "tuning_cache_two_pop.json",
         "serving": "tuning_cache_serving.json"}
# lattice sizes whose launch shapes the caches hold
TUNED_L = {"fm": (8, 16, 24, 32, 64), "two_pop": (32,)}
OVERLAP = {"none": W.Q_NONE, "shift": W.Q_INDEX_SHIFT, "two_pop": W.Q_TWO_POP, "wang": W.Q_WANG,
           "wang_rdm": W.Q_WANG_RDM}
W_FLOATS = 14   # the FP64 fields of a weighted-average record, then n_included


def _case(kind, **kw):
    """A case of plain values: `runs` runs of one descriptor shape (for the
    batch and the server, of every size in `sizes`)."""
    c = dict(kind=kind, repr="msc", model="fm", sizes="", L=0, runs=1, R=1000, theta=10, K=101, beta_f=1.0,
             resampling="multinomial", overlap="none", qhist=False, tuned="", M=0)
    c.update(kw)
    return c


def listed():
    return [
        # one small run, read back whole: latency, launches and the host's
        # share of creating a context count (L = 8 ferromagnet, R = 1000)
        _case("run", name="one_small_run", L=8, state=True),
        # the same path driven step by step, each record read as it is made
        # (a program that adapts or stops on what it sees)
        _case("steps", name="step_by_step", L=16, model="ea", R=2000, theta=3, K=31, beta_f=3.0,
              resampling="nearest", overlap="shift"),
        # a spin glass on a lattice size without a kernel of its own, ragged
        # population, nearest-integer resampling, overlap histograms
        _case("run", name="odd_lattice", L=20, model="ea", R=5003, theta=5, K=101, beta_f=3.0,
              resampling="nearest", overlap="shift", qhist=True),
        # the benchmark's headline run: L = 64 ferromagnet, R = 1e5, whole
        # schedule, with the cached launch shapes and its weighted average
        _case("run", name="fm_L64_R100k", L=64, R=100_000, K=200, beta_f=0.6, tuned="fm", M=1),
        # two populations on one spin-glass sample for unbiased overlaps
        _case("run", name="ea_two_populations", L=32, model="ea", R=200_000, K=301, beta_f=3.0, overlap="two_pop",
              tuned="two_pop"),
        # many runs of uneven size in one context, combined by their
        # free-energy weights
        _case("batch", name="batch_uneven", sizes="8,16,24,32", runs=256, R=2000, K=150, beta_f=0.6, tuned="fm",
              M=256),
        # the bias-versus-M pool: thousands of tiny runs weighted in groups
        _case("pool", name="bias_pool", L=10, runs=3840, R=100, theta=1, K=61, beta_f=0.6),
        # overlap estimators from permutation pairings on one sample
        _case("overlaps", name="permutation_pairs", L=32, model="ea", runs=16, R=20_000, K=61, beta_f=2.4,
              overlap="wang", qhist=True, M=16),
        # the theta = infinity limit: only reweighting and resampling remain
        _case("run", name="theta_infinite", L=16, runs=256, R=20_000, theta=-1, K=89, beta_f=0.44, M=256),
        # one byte per spin: the representation for lattices of any size
        _case("run", name="bytes_L64", repr="int8", L=64, R=20_000, K=51, beta_f=0.6),
        # a lattice beyond the bit-packed representation's sizes
        _case("run", name="bytes_L128", repr="int8", L=128, model="ea", R=2000, K=21, beta_f=1.0, overlap="shift"),
        # a stream of spin-glass requests of mixed sizes through the server
        _case("serve", name="serve_mixed", model="ea", sizes="16,24,32,48,64", runs=2, R=50_000, K=61, beta_f=3.0,
              overlap="shift", tuned="serving"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _even(rng, lo, hi):
    return 2 * _log(rng, lo // 2, hi // 2)


def _fit(c, flips):
    """The population of c reduced until it attempts at most `flips` flips."""
    N = sum(int(x) ** 2 for x in c["sizes"].split(",")) if c["sizes"] else c["L"] ** 2
    npop = 2 if c["overlap"] == "two_pop" else 1
    per = N * c["runs"] * npop * max(c["theta"], 1) * c["K"]
    c["R"] = max(50, min(c["R"], int(flips / per)))
    return c


def draw(rng):
    kind = rng.choice(("run", "run", "run", "steps", "tuned", "two_pop", "batch", "pool", "overlaps", "theta",
                       "bytes", "bytes", "serve"))
    ea = rng.random() < 0.5
    common = dict(model="ea" if ea else "fm", beta_f=rng.choice((1.0, 2.0, 3.0) if ea else (0.5, 0.6, 1.0)),
                  resampling=rng.choice(("multinomial", "nearest")), overlap=rng.choice(("none", "shift")))
    if kind == "run":   # any even size that the bit-packed path holds on chip
        return _fit(_case("run", L=_even(rng, 4, 90), R=_log(rng, 300, 100_000), theta=rng.choice((1, 3, 5, 10, 20)),
                          K=_log(rng, 21, 201), qhist=rng.random() < 0.3 and common["overlap"] == "shift",
                          **common), 1e11)
    if kind == "steps":
        return _fit(_case("steps", L=_even(rng, 4, 64), R=_log(rng, 300, 20_000), theta=rng.choice((1, 3, 10)),
                          K=_log(rng, 21, 101), **common), 2e10)
    if kind == "tuned":
        return _fit(_case("run", L=rng.choice(TUNED_L["fm"]), R=_log(rng, 5000, 150_000), K=_log(rng, 51, 201),
                          beta_f=0.6, tuned="fm", M=1), 4e11)
    if kind == "two_pop":
        return _fit(_case("run", L=32, model="ea", R=_log(rng, 5000, 200_000), K=_log(rng, 61, 301), beta_f=3.0,
                          overlap="two_pop", resampling=common["resampling"], tuned="two_pop"), 1e12)
    if kind == "batch":
        n = _log(rng, 16, 256)
        return _fit(_case("batch", sizes=rng.choice(("8,16,24,32", "8,16", "10,12,20", "16,32,48")), runs=n,
                          R=_log(rng, 500, 4000), K=_log(rng, 31, 150), beta_f=0.6, M=n), 3e11)
    if kind == "pool":
        return _fit(_case("pool", L=rng.choice((8, 10, 12)), runs=30 * _log(rng, 8, 128), R=_log(rng, 60, 200),
                          theta=rng.choice((1, 5)), K=61, beta_f=0.6), 2e10)
    if kind == "overlaps":
        n = _log(rng, 2, 16)
        return _fit(_case("overlaps", L=_even(rng, 8, 32), model="ea", runs=n, R=_log(rng, 1000, 20_000),
                          K=_log(rng, 21, 61), beta_f=2.4, overlap=rng.choice(("wang", "wang_rdm")), qhist=True,
                          M=n), 2e11)
    if kind == "theta":
        n = _log(rng, 16, 256)
        return _case("run", L=rng.choice((8, 10, 16)), runs=n, R=_log(rng, 2000, 20_000), theta=-1,
                     K=_log(rng, 31, 89), beta_f=0.44, M=n, resampling=common["resampling"])
    if kind == "bytes":
        return _fit(_case("run", repr="int8", L=_even(rng, 8, 200), R=_log(rng, 300, 30_000),
                          theta=rng.choice((1, 5, 10)), K=_log(rng, 11, 51), **common), 4e10)
    return _fit(_case("serve", model="ea", sizes=rng.choice(("16,24,32,48,64", "16,32,64", "24,48")),
                      runs=rng.choice((1, 2)), R=_log(rng, 5000, 50_000), K=_log(rng, 31, 61), beta_f=3.0,
                      overlap="shift", tuned="serving"), 1.3e11)


# ------------------------------------------------------------------ inputs

def _runs(case, seed):
    beta = np.array(W.linear_schedule(case["beta_f"], case["K"]))
    sizes = [int(x) for x in case["sizes"].split(",")] if case["sizes"] else [case["L"]]
    res = W.NEAREST_INT if case["resampling"] == "nearest" else W.MULTINOMIAL
    out = []
    for L in sizes:
        for _ in range(case["runs"]):
            m = len(out)
            d = W.run_desc(L, W.EA_PMJ if case["model"] == "ea" else W.FM,
                           seed=W.RUN_SEED_BASE + (int(seed) << 20) + m,
                           # the overlap runs share one sample, requests have their own
                           disorder_seed=W.DISORDER_SEED_BASE + (int(seed) << 20) + (m if case["kind"] == "serve" else 0),
                           R=case["R"], theta=case["theta"], K=case["K"], beta_f=case["beta_f"], resampling=res,
                           overlap=OVERLAP[case["overlap"]], qhist=int(case["qhist"]))
            d["beta"] = beta   # one array for every run, as a program would keep it
            out.append(d)
    return out


def prepare(case, seed):
    st = {"case": case, "runs": _runs(case, seed), "cache": None}
    if TUNED[case["tuned"]]:
        st["cache"] = os.path.join(os.path.dirname(os.path.abspath(pa.__file__)), TUNED[case["tuned"]])
    if case["kind"] == "serve":
        from paper_2207_05535_amd.serve import Server
        room = sum(pa.pa_server_footprint(d, case["repr"]) for d in st["runs"])
        st["server"] = Server(room + room // 8 + (64 << 20), max_slots=16, repr_=case["repr"],
                              tuning_cache=st["cache"])
    return st


# -------------------------------------------------------------------- pass

def _fields(obs):
    return {f: obs[f] for f in obs.dtype.names}


def _wavg(w):
    """A weighted-average record array as its FP64 fields and its run counts."""
    return {"W": w.view(np.float64).reshape(w.shape + (W_FLOATS + 1,))[..., :W_FLOATS],
            "n_included": w["n_included"]}


POOL_M = (1, 4, 16, 30)


def run(state):
    case, runs = state["case"], state["runs"]
    if case["kind"] == "serve":
        return _serve(state)
    ctx = pa.Context(runs, case["repr"])
    if state["cache"]:
        ctx.autotune(steps=3, cache_path=state["cache"])   # applies the cached launch shapes
    out = {}
    if case["kind"] == "steps":
        out["seen"] = _fields(np.stack([ctx.step(i, read=True)[0, 0] for i in range(1, case["K"])]))
    else:
        ctx.run(1, case["K"])
    if case["kind"] == "pool":
        for M in POOL_M:
            out["M%d" % M] = _wavg(ctx.weighted_average(M))
    else:
        out["obs"] = _fields(ctx.obs())
    if case["M"]:
        kind = pa.PA_W_FULL | (pa.PA_W_EXCLUDE_LARGE_FAMILY if case["kind"] == "overlaps" else 0)
        out["avg"] = _wavg(ctx.weighted_average(case["M"], kind))
        if case["qhist"]:
            out["P_q"] = ctx.weighted_qhist(case["M"], kind)
    if case["qhist"]:
        out["qhist"] = ctx.qhist(0)
    if case["kind"] == "overlaps":
        out["pair_status"], out["pairs"] = ctx.pairing(0)
    if case.get("state"):
        out["spins"], out["E"], out["families"], out["counts"] = ctx.state(0)
    ctx.close()
    return out


def _serve(state):
    srv, runs = state["server"], state["runs"]
    waiting, active, done = list(range(len(runs))), {}, {}
    while waiting or active:
        while waiting:
            slot = srv.admit(runs[waiting[0]])
            if slot is None:
                break
            active[slot] = waiting.pop(0)
        for slot in srv.step():
            q = active.pop(slot)
            done[q] = srv.read_obs(slot, runs[q], sync=False)
            srv.release(slot)
    srv.stream.synchronize()
    return _fields(np.stack([done[q][1][:, 0] for q in range(len(runs))]))


# -------------------------------------------------------------------- work

def work(case):
    """Per temperature step every lattice is read and written once (children
    gathered, swept and measured in one visit) with its energy and label; an
    attempted flip takes at least 3.5 integer operations (a site's share of
    the random bits that decide it), a theta = infinity draw one generator
    call.  Records are written once."""
    sizes = [int(x) for x in case["sizes"].split(",")] if case["sizes"] else [case["L"]]
    npop = 2 if case["overlap"] == "two_pop" else 1
    site = 1.0 if case["repr"] == "int8" else 0.125
    nbytes = ops = 0.0
    for L in sizes:
        reps = case["runs"] * npop * case["R"]
        lattice = 0.0 if case["theta"] < 0 else L * L * site
        nbytes += (case["K"] - 1) * (reps * (2 * lattice + 16) + 144.0 * case["runs"] * npop)
        ops += (case["K"] - 1) * reps * (40.0 if case["theta"] < 0 else 3.5 * L * L * case["theta"])
    return {"bytes": nbytes, "flops": ops}


# ------------------------------------------------------------------- exact
#
# The method in plain torch (Sec. II B of the paper under the documented
# random-number contract): int64 tensors for the generator and every integer,
# FP64 for the sums, all runs of the case (equal shapes) at once.

M32 = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, k0, k1):
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57   # modulo 2^64
        c0, c1, c2, c3 = ((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _mulhi(hi, lo, s):
    """floor((hi 2^32 + lo) s / 2^64) for 32-bit words hi, lo and s < 2^63."""
    sh, sl = s >> 32, s & M32

    def parts(a, b):
        p = a * b
        return (p >> 32) & M32, p & M32
    h1, l1 = parts(hi, sl)
    h2, l2 = parts(lo, sh)
    h0, _ = parts(lo, sl)
    h3, l3 = parts(hi, sh)
    mid = h0 + l1 + l2
    return ((h3 + ((h1 + h2 + l3 + (mid >> 32)) >> 32)) << 32) + ((h1 + h2 + l3 + (mid >> 32)) & M32)


def _simulate(runs):
    """Records of runs of one shape (one population each): per temperature the
    tensors E [run][replica] and M, and ln Q and A [run]; None if a population
    leaves its capacity."""
    d = runs[0]
    L, N, R, beta, n = d["L"], d["L"] ** 2, d["R"], d["beta"], len(runs)
    dev = "cuda" if torch.cuda.is_available() else "cpu"

    def ints(v, *shape):
        return torch.tensor(v, dtype=torch.int64, device=dev).reshape(shape)
    k0 = ints([r["seed"] & M32 for r in runs], n, 1, 1)
    k1 = ints([(r["seed"] >> 32) & M32 for r in runs], n, 1, 1)
    b32 = torch.arange(32, device=dev)
    site = torch.arange(N, device=dev)
    y, x = site // L, site % L
    nb = [y * L + (x + 1) % L, y * L + (x - 1) % L, ((y + 1) % L) * L + x, ((y - 1) % L) * L + x]
    JR = torch.ones(n, N, dtype=torch.int64, device=dev)
    JD = JR.clone()
    if d["model"] == W.EA_PMJ:
        o = _philox(site[None], 0, 0, 5 << 28, ints([r["disorder_seed"] & M32 for r in runs], n, 1),
                    ints([(r["disorder_seed"] >> 32) & M32 for r in runs], n, 1))
        JR, JD = 1 - 2 * (o[0] & 1), 1 - 2 * (o[1] & 1)
    J = [JR, JR[:, nb[1]], JD, JD[:, nb[3]]]

    def spread(lo, hi, count):   # bits of (lo | hi << 32) over replicas 64 g + b
        w = torch.stack([lo, hi], -1)[..., None] >> b32 & 1
        return w.reshape(*lo.shape[:-1], -1)[..., :count]

    G = (R + 63) // 64
    o = _philox(site[None, :, None], torch.arange(G, device=dev)[None, None], 0, 4 << 28, k0, k1)
    s = 1 - 2 * spread(o[0], o[1], R)
    call = torch.arange(16, device=dev).reshape(16, 1, 1, 1)

    def energy(s):
        return -(s * (JR[..., None] * s[:, nb[0]] + JD[..., None] * s[:, nb[2]])).sum(1)

    A = np.full(n, N * math.log(2.0))
    E = energy(s)
    out = [(E, s.sum(1), np.zeros(n), A)]
    for i in range(1, len(beta)):
        Rp = s.shape[2]
        db = beta[i] - beta[i - 1]
        xs = np.exp(-(db * (4.0 * np.arange(N + 1))))
        Emin = E.amin(1)
        k = (E - Emin[:, None]) >> 2
        lnQ = np.log(torch.tensor(xs, device=dev)[k].sum(1).cpu().numpy()) - math.log(Rp) - db * Emin.cpu().numpy()
        A = A + lnQ
        X = torch.tensor(np.floor(xs * 2.0 ** 40).astype(np.int64), device=dev)[k]
        cum = X.cumsum(1)
        SX = cum[:, -1:]
        if d["resampling"] == W.MULTINOMIAL:
            o = _philox(torch.arange(R, device=dev)[None], 0, i, 3 << 28, k0[:, 0], k1[:, 0])
            parent = torch.searchsorted(cum, _mulhi(o[1], o[0], SX), right=True).sort(1).values
        else:
            count, rem = R * X // SX, R * X % SX
            t = torch.zeros_like(rem)
            for _ in range(32):
                rem = rem << 1
                t = (t << 1) | (rem >= SX)
                rem = torch.where(rem >= SX, rem - SX, rem)
            u = _philox(torch.arange(Rp, device=dev)[None], 0, i, 2 << 28, k0[:, 0], k1[:, 0])[0]
            parent = torch.repeat_interleave(torch.arange(Rp, device=dev), (count + (u < t))[0])[None]
            if not 0 < parent.shape[1] <= d["R_cap"]:
                return None
        Rc = parent.shape[1]
        G = (Rc + 63) // 64
        s = torch.gather(s, 2, parent[:, None].expand(n, N, Rc)).contiguous()
        T = [int(math.floor(math.exp(-(beta[i] * 4.0 * q)) * 2.0 ** 32)) for q in (1, 2)]
        for sweep in range(d["theta"]):
            for colour in range(2):
                at = ((x + y) % 2 == colour).nonzero().flatten()
                o = _philox(at[None, None, :, None] | call << 20, torch.arange(G, device=dev), i, 1 << 28 | sweep,
                            k0, k1)
                u = (spread(o[0], o[1], Rc) << (31 - 2 * call)).sum(0) + (spread(o[2], o[3], Rc) << (30 - 2 * call)).sum(0)
                dE = 2 * s[:, at] * sum(j[:, at, None] * s[:, m[at]] for j, m in zip(J, nb))
                flip = (dE <= 0) | ((dE == 4) & (u < T[0])) | ((dE == 8) & (u < T[1]))
                s[:, at] = torch.where(flip, -s[:, at], s[:, at])
        E = energy(s)
        out.append((E, s.sum(1), lnQ, A))
    return out


def _average(sim, runs, M):
    """Weighted averages (Sec. IV, full weights) over consecutive groups of M."""
    N, R, beta = runs[0]["L"] ** 2, runs[0]["R"], runs[0]["beta"]
    g = len(runs) // M
    out = np.zeros((g, len(beta), W_FLOATS))
    cum = 0.0
    for i, (E, mag, lnQ, A) in enumerate(sim):
        E, mag = E.double(), mag.double().abs()
        e, e2, m, m2 = ((v.mean(1).cpu().numpy() / q).reshape(g, M) for v, q in (
            (E, N), (E * E, N * N), (mag, N), (mag * mag, N * N)))
        c = beta[i] ** 2 * N * (E.var(1, unbiased=False).cpu().numpy().reshape(g, M) / N ** 2)
        chi = beta[i] * N * (mag.var(1, unbiased=False).cpu().numpy().reshape(g, M) / N ** 2)
        a = (math.log(R) + A).reshape(g, M)
        w = np.exp(a - a.max(1, keepdims=True))
        w /= w.sum(1, keepdims=True)
        mean = lambda v: (w * v).sum(1)  # noqa: E731
        spread = lambda v: (w * (v - mean(v)[:, None]) ** 2).sum(1)  # noqa: E731
        if i == 0:
            F = A.reshape(g, M)[:, 0]
        else:
            ap, lq = last, lnQ.reshape(g, M)
            cum = cum + np.log((np.exp(ap - ap.max(1, keepdims=True)) * np.exp(lq)).sum(1) /
                               np.exp(ap - ap.max(1, keepdims=True)).sum(1))
            F = F0 + cum
        if i == 0:
            F0 = F
        last = a
        out[:, i] = np.stack([mean(e), mean(e2), mean(c) + beta[i] ** 2 * N * spread(e), mean(c), mean(m), mean(m2),
                              mean(chi) + beta[i] * N * spread(m), mean(chi), 0 * F, 0 * F, 0 * F, F,
                              ((w - 1.0 / M) ** 2).mean(1),
                              np.expm1(A.reshape(g, M).var(1)) / M ** 2], -1)
    return out


def exact(case, seed):
    runs = _runs(case, seed)
    flips = len(runs) * case["R"] * case["L"] ** 2 * max(case["theta"], 0) * case["K"]
    small = 0 < flips <= 4e9 and case["theta"] * case["K"] <= 4000 and case["L"] ** 2 * case["R"] <= 1 << 21
    if case["kind"] not in ("run", "steps", "pool") or not small or case["overlap"] == "two_pop":
        return None
    if case["runs"] > 1 and case["resampling"] == "nearest":
        return None
    sim = _simulate(runs)
    if sim is None:
        return None
    if case["kind"] == "pool":
        return {"M%d" % M: {"W": _average(sim, runs, M), "n_included": None} for M in POOL_M}
    lnQ, A = (np.stack([r[q] for r in sim], 1)[:, None] for q in (2, 3))
    out = {"obs": {f: None for f in pa.PA_OBS_DTYPE.names}}
    out["obs"].update(lnQ=lnQ, A=A)
    if case["kind"] == "steps":
        out["seen"] = {f: None for f in pa.PA_OBS_DTYPE.names}
        out["seen"].update(lnQ=lnQ[0, 0, 1:], A=A[0, 0, 1:])
    if case["M"] and case["overlap"] == "none":
        out["avg"] = {"W": _average(sim, runs, case["M"]), "n_included": None}
    return out
