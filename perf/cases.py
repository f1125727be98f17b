"""The workloads that the library's speed is measured on.

A case is a dict of plain values.  ``prepare`` makes what a program that uses
the library has in hand (data, graph, chain, result buffers), ``run`` is one
pass through the public entry points and returns its results, ``work`` counts
the bytes and operations that the pass cannot do without, and ``exact`` gives
the same results by a plain 64-bit sampler written here with torch and numpy
(on the GPU where there is one), which shares no code with the library.

Kinds of cases:

* ``sweeps``: a resident chain runs one more call of ``sweeps`` sweeps and
  leaves its posterior mean and variance in device memory, with the trace of
  (tau, lam, beta0) -- the ordinary use of the sampler;
* ``step``: one sweep and the state read back to the host, as a program does
  that puts its own update between the sweeps;
* ``solve``: from host observations to host results on a graph that the
  program keeps: a new chain, its sweeps, the posterior mean and variance;
* ``batch``: many chains of uneven sizes advanced by shared launches.
"""
import functools
import math

import numpy as np
import torch

from paper_1702_05518_amd import gmrf, inputs

# the fields of a case and their defaults; "name" is left out of drawn cases
DEFAULTS = dict(kind="sweeps", graph="lattice", rows=0, cols=0, stencil=8, n=0, rho=1.0,
                precision="f32", sweeps=100, burn_in=0, intercept=False, hyper=True,
                capture=False, binomial=False, trials=0.0, rng=1, chains=0, noise=0.1)


def full(case):
    return {**DEFAULTS, **case}


def listed():
    return [
        # The smallest call: a small image, one sweep, the state on the host
        # (a sampler whose caller updates something else between sweeps).
        dict(name="step_48x40_f64", kind="step", rows=48, cols=40, precision="f64", sweeps=1),
        # The paper's simulated image: 50 x 50, intercept, burn-in, trace.
        dict(name="image_50x50_f64", rows=50, cols=50, precision="f64", intercept=True,
             sweeps=500, burn_in=100, noise=1.0),
        # The small 4-neighbour lattice of the test suite and the benchmark.
        dict(name="lattice_64x64_s4_f64", rows=64, cols=64, stencil=4, precision="f64",
             sweeps=200),
        # An ordinary photograph-sized image of odd sides, with the intercept.
        dict(name="lattice_509x517_f32", rows=509, cols=517, precision="f32", intercept=True,
             sweeps=100),
        # The benchmark's lattice in both precisions.
        dict(name="lattice_2048_f32", rows=2048, cols=2048, precision="f32", sweeps=40),
        dict(name="lattice_2048_f64", rows=2048, cols=2048, precision="f64", sweeps=40),
        # A lattice far beyond the last-level cache.
        dict(name="lattice_4096_f32", rows=4096, cols=4096, precision="f32", sweeps=20),
        # The irregular map of the paper's size, swept as a captured graph.
        dict(name="graph_15k_f64", graph="delaunay", n=15000, rho=0.95, precision="f64",
             sweeps=200, capture=True, noise=0.2),
        # A large irregular map.
        dict(name="graph_300k_f32", graph="delaunay", n=300000, rho=0.95, precision="f32",
             sweeps=100, noise=0.2),
        # The paper's election example: binomial counts, Polya-Gamma draws.
        dict(name="binomial_14926_f64", graph="delaunay", n=14926, rho=0.995, precision="f64",
             binomial=True, trials=250.0, intercept=True, sweeps=10),
        # Many chains at once, the benchmark's mix of sizes at a smaller count.
        dict(name="batch_32_f32", kind="batch", chains=32, stencil=4, rho=0.95, precision="f32",
             sweeps=50),
        # Host observations to host results for one image.
        dict(name="solve_512_f64", kind="solve", rows=512, cols=512, precision="f64",
             sweeps=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: the kind, then its sizes spread
    over the logarithm, and its options."""
    kind = rng.choice(["lattice", "lattice", "lattice", "graph", "graph", "binomial", "step",
                       "solve", "batch"])
    prec = rng.choice(["f32", "f64"])
    if kind == "graph":
        return dict(graph="delaunay", n=_log_int(rng, 500, 300000), precision=prec,
                    rho=rng.choice([0.95, 1.0]), intercept=rng.random() < 0.3,
                    sweeps=rng.randint(20, 100), noise=0.2, capture=rng.random() < 0.3)
    if kind == "binomial":
        return dict(graph="delaunay", n=_log_int(rng, 300, 14926), precision=prec,
                    rho=rng.choice([0.95, 0.995]), binomial=True, intercept=True,
                    trials=float(rng.choice([20.0, 80.0, 250.0])), sweeps=rng.randint(3, 10))
    if kind == "batch":
        return dict(kind="batch", chains=2 * rng.randint(2, 16), precision=prec, rho=0.95,
                    stencil=rng.choice([4, 8]), sweeps=rng.randint(10, 50))
    big = {"step": 300, "solve": 800}.get(kind, 2500)
    rows, cols = _log_int(rng, 16, big), _log_int(rng, 16, big)
    paired = kind == "lattice" and rng.random() < 0.25
    if paired:
        cols = -(-cols // 4) * 4
    most = max(10, min(60, 160000000 // (rows * cols)))
    case = dict(kind="sweeps" if kind == "lattice" else kind, rows=rows, cols=cols,
                stencil=rng.choice([4, 8]), precision=prec, intercept=rng.random() < 0.3,
                sweeps=1 if kind == "step" else rng.randint(10, most),
                burn_in=0 if kind == "step" else rng.choice([0, 0, 5]))
    if kind == "lattice":
        case.update(hyper=rng.random() < 0.9, capture=rng.random() < 0.3,
                    rng=2 if paired else 1)
    return case


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
@functools.lru_cache(maxsize=64)
def _map(n, map_seed):
    """An irregular map: its sites, adjacency and coloring.  One map serves
    many data sets, so it depends on its size alone."""
    pts, row_ptr, col = inputs.delaunay_graph(n, data_seed=map_seed)
    return pts, row_ptr, col, _first_fit(row_ptr, col)


def _first_fit(row_ptr, col):
    """The smallest color that no lower-numbered neighbour has, in id order."""
    color = []
    rp, cl = row_ptr.tolist(), col.tolist()
    for i in range(len(rp) - 1):
        used = {color[j] for j in cl[rp[i]:rp[i + 1]] if j < i}
        c = 0
        while c in used:
            c += 1
        color.append(c)
    return np.array(color, dtype=np.int32)


def _jobs(c, seed):
    """The chains of a case: dicts of shape (lattice or map), y, trials, seed."""
    rng = np.random.Generator(np.random.PCG64(seed))
    if c["kind"] == "batch":
        sizes = np.random.Generator(np.random.PCG64(4 + c["chains"]))   # of the mix, not the data
        jobs = []
        for i in range(c["chains"]):
            if i < c["chains"] // 2:
                side = int(sizes.integers(32, 513))
                y = inputs.image_observations(side, side, 0.1, int(rng.integers(1 << 30)))[1]
                jobs.append(dict(lattice=(side, side, c["stencil"]), map=None, y=y, rho=1.0))
            else:
                m = _map(int(sizes.integers(1000, 50001)), 100 + i)
                y = inputs.smooth_field(m[0]) + 0.2 * rng.standard_normal(m[0].shape[0])
                jobs.append(dict(lattice=None, map=m, y=y, rho=c["rho"]))
    elif c["graph"] == "lattice":
        y = inputs.image_observations(c["rows"], c["cols"], c["noise"], seed)[1]
        jobs = [dict(lattice=(c["rows"], c["cols"], c["stencil"]), map=None, y=y, rho=c["rho"])]
    else:
        m = _map(c["n"], 3)
        field = inputs.smooth_field(m[0])
        if c["binomial"]:
            eta = 0.3 + 0.5 * field + 0.3 * rng.standard_normal(c["n"])
            trials = np.ceil(c["trials"] * np.exp(0.8 * rng.standard_normal(c["n"])))
            trials = trials.astype(np.int32)
            trials[rng.random(c["n"]) < 0.022] = 0       # areas without data
            y = rng.binomial(trials, 1.0 / (1.0 + np.exp(-eta))).astype(np.float64)
            jobs = [dict(lattice=None, map=m, y=y, trials=trials, rho=c["rho"])]
        else:
            y = field + c["noise"] * rng.standard_normal(c["n"])
            jobs = [dict(lattice=None, map=m, y=y, rho=c["rho"])]
    for i, j in enumerate(jobs):
        j.update(seed=1000 + seed, instance=i)
    return jobs


def _graph(job):
    if job["lattice"]:
        return gmrf.Graph(lattice=job["lattice"], rho=job["rho"])
    _, row_ptr, col, color = job["map"]
    return gmrf.Graph(row_ptr=row_ptr, col_idx=col, color=color,
                      num_colors=int(color.max()) + 1, rho=job["rho"])


def _chain(c, job, graph):
    return gmrf.Chain(graph, job["y"], seed=job["seed"], instance=job["instance"],
                      precision=gmrf.FP64 if c["precision"] == "f64" else gmrf.FP32_ACC64,
                      burn_in=c["burn_in"], intercept=c["intercept"],
                      trials=job.get("trials"), beta0_var=1000.0 if c["binomial"] else 0.0,
                      rng_version=c["rng"])


def prepare(case, seed):
    c = full(case)
    jobs = _jobs(c, seed)
    graphs = [_graph(j) for j in jobs]
    s = dict(case=c, jobs=jobs, graphs=graphs)
    if c["kind"] == "solve":
        return s
    s["chains"] = [_chain(c, j, g) for j, g in zip(jobs, graphs)]
    if c["kind"] == "step":
        return s
    n = sum(g.n for g in graphs)
    s["mean"] = torch.empty(n, dtype=torch.float64, device="cuda")
    s["var"] = torch.empty(n, dtype=torch.float64, device="cuda")
    if c["kind"] == "batch":
        s["batch"] = gmrf.Batch(s["chains"])
    else:
        s["chains"][0].enable_trace(c["sweeps"])     # the first call's sweeps
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "solve":
        chain = _chain(c, s["jobs"][0], s["graphs"][0])
        chain.sweep(c["sweeps"], hyper=c["hyper"])
        mean, var, _ = chain.posterior_stats()
        return {"mean": mean, "var": var}
    if c["kind"] == "step":
        x, tau, lam, _ = s["chains"][0].sweep(1, hyper=c["hyper"]).get_state()
        return {"x": x, "tau": tau, "lam": lam}
    if c["kind"] == "batch":
        s["batch"].sweep(c["sweeps"], hyper=c["hyper"], capture=c["capture"])
    else:
        s["chains"][0].sweep(c["sweeps"], hyper=c["hyper"], capture=c["capture"])
    at = 0
    for chain in s["chains"]:
        chain.posterior_stats_device(s["mean"][at:at + chain.n], s["var"][at:at + chain.n])
        at += chain.n
    out = {"mean": s["mean"], "var": s["var"]}
    if c["kind"] == "sweeps":
        out["trace"] = s["chains"][0].trace_buf
    return out


def work(case):
    """Per sweep the field is read and written and y read once (the next
    sweep's precisions need a sum over the whole field); the accumulators are
    read and written once in a call, and the mean and variance written once.
    A site update is counted as its neighbour sum and edge terms, about 40
    operations for the normal and 15 for the rest; a Polya-Gamma term as 80."""
    c = full(case)
    real = 8 if c["precision"] == "f64" else 4
    if c["kind"] == "batch":
        sizes = np.random.Generator(np.random.PCG64(4 + c["chains"]))
        half = c["chains"] // 2
        n = sum(int(sizes.integers(32, 513)) ** 2 for _ in range(half))
        n += sum(int(sizes.integers(1000, 50001)) for _ in range(c["chains"] - half))
        deg = 5.0
    elif c["graph"] == "lattice":
        n, deg = c["rows"] * c["cols"], float(c["stencil"])
    else:
        n, deg = c["n"], 6.0
    adjacency = 0.0 if c["graph"] == "lattice" and c["kind"] != "batch" else 4.0 * deg
    per_sweep = n * (3.0 * real + adjacency)
    flops = n * (2.5 * deg + 55.0)
    if c["binomial"]:
        terms = n * c["trials"] * math.exp(0.32)      # the mean of the lognormal counts
        flops += 80.0 * terms
    once = n * (32.0 + 16.0)
    if c["kind"] == "solve":
        once = n * (8.0 + 16.0)                       # y up, mean and variance down
    if c["kind"] == "step":
        once = n * (32.0 + 8.0)
    return {"bytes": per_sweep * c["sweeps"] + once, "flops": flops * c["sweeps"]}


# --------------------------------------------------------------------------
# the same results in 64 bits
# --------------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 words; counters are ints or int64 tensors below 2^32."""
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        pa, pb = 0xD2511F53 * c0, 0xCD9E8D57 * c2     # tensors wrap at 64 bits
        c0, c1, c2, c3 = (((pb >> 32) & _M32) ^ c1 ^ k0, pb & _M32,
                          ((pa >> 32) & _M32) ^ c3 ^ k1, pa & _M32)
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1, c2, c3


def _unit(hi, lo):
    m = (hi << 20) | (lo >> 12)
    return ((m.to(torch.float64) if torch.is_tensor(m) else float(m)) + 0.5) * 2.0 ** -52


def _normals(ids, t, instance, seed, branch=None):
    w = _philox(ids, t, instance, 0, seed)
    r = torch.sqrt(-2.0 * torch.log(_unit(w[0], w[1])))
    a = 2.0 * math.pi * _unit(w[2], w[3])
    z = r * torch.cos(a)
    return z if branch is None else torch.where(branch, r * torch.sin(a), z)


def _scalar_normal(seed, c0, t, instance, tag):
    w = _philox(c0, t, instance, tag, seed)
    return math.sqrt(-2.0 * math.log(_unit(w[0], w[1]))) * math.cos(2 * math.pi * _unit(w[2], w[3]))


def _gamma(shape, rate, seed, t, instance, tag):
    """Marsaglia and Tsang's Gamma variate."""
    d = shape - 1.0 / 3.0
    for k in range(64):
        z = _scalar_normal(seed, 2 * k, t, instance, tag)
        cz = z / math.sqrt(9.0 * d)
        if cz <= -1.0:
            continue
        log_v = 3.0 * math.log1p(cz)
        w = _philox(2 * k + 1, t, instance, tag, seed)
        if math.log(_unit(w[0], w[1])) < 0.5 * z * z + d * (log_v - math.expm1(log_v)):
            return d * math.exp(log_v) / rate
    raise FloatingPointError("no Gamma variate in 64 attempts")


def _pg_terms(z, site, j, t, instance, seed):
    """PG(1, 2 z) of each term (Devroye's method as given by Polson, Scott and
    Windle, 2013): terms still without a variate are drawn together."""
    T, pi = 0.64, math.pi
    out = torch.zeros_like(z)
    used = torch.zeros_like(site)

    def uniform(k):
        u = used[k]
        used[k] = u + 1
        w = _philox(site[k], t, instance, 0x80000000 | (j[k] << 10) | (u >> 1), seed)
        odd = (u & 1) == 1
        return _unit(torch.where(odd, w[2], w[0]), torch.where(odd, w[3], w[1]))

    K = pi * pi / 8.0 + 0.5 * z * z
    p = pi / (2.0 * K) * torch.exp(-K * T)
    cdf = lambda v: 0.5 * torch.special.erfc(-v / math.sqrt(2.0))  # noqa: E731
    q = 2.0 * (torch.exp(-z) * cdf((T * z - 1.0) / math.sqrt(T))
               + torch.exp(z) * cdf(-(T * z + 1.0) / math.sqrt(T)))
    right = p / (p + q)
    todo = torch.arange(z.numel(), device=z.device)
    while todo.numel():
        x = torch.zeros(todo.numel(), dtype=torch.float64, device=z.device)
        is_right = uniform(todo) < right[todo]
        k = todo[is_right]
        x[is_right] = T - torch.log(uniform(k)) / K[k]
        left = torch.nonzero(~is_right)[:, 0]
        tail = left[z[todo[left]] < 1.0 / T]
        while tail.numel():            # the normal tail, kept with exp(-z^2 x / 2)
            search, e1 = tail, torch.zeros(todo.numel(), dtype=torch.float64, device=z.device)
            while search.numel():
                k = todo[search]
                a = -torch.log(uniform(k))
                b = -torch.log(uniform(k))
                e1[search] = a
                search = search[a * a > 2.0 * b / T]
            v = T / (1.0 + T * e1[tail]) ** 2
            x[tail] = v
            k = todo[tail]
            tail = tail[uniform(k) > torch.exp(-0.5 * z[k] * z[k] * v)]
        steep = left[z[todo[left]] >= 1.0 / T]
        while steep.numel():           # Michael, Schucany and Haas
            k = todo[steep]
            mu = 1.0 / z[k]
            nrm = torch.sqrt(-2.0 * torch.log(uniform(k))) * torch.cos(2 * pi * uniform(k))
            my = mu * nrm * nrm
            v = mu + 0.5 * mu * my - 0.5 * mu * torch.sqrt(4.0 * my + my * my)
            v = torch.where(uniform(k) > mu / (mu + v), mu * mu / v, v)
            x[steep] = v
            steep = steep[v >= T]

        def term(n, v):
            h = n + 0.5
            r = 2.0 / (pi * v)
            return torch.where(v > T, pi * h * torch.exp(-0.5 * h * h * pi * pi * v),
                               pi * h * r * torch.sqrt(r) * torch.exp(-2.0 * h * h / v))

        s = term(0, x)
        y = uniform(todo) * s
        open_ = torch.ones_like(x, dtype=torch.bool)
        ok = torch.zeros_like(open_)
        for n in range(1, 201):
            s = s - term(n, x) if n & 1 else s + term(n, x)
            hit = open_ & ((y <= s) if n & 1 else (y > s))
            if n & 1:
                ok |= hit
            open_ &= ~hit
            if not bool(open_.any()):
                break
        out[todo[ok]] = 0.25 * x[ok]
        todo = todo[~ok]
    return out


class _Sampler:
    """The chromatic Gibbs sampler in 64 bits on padded neighbour tables."""

    def __init__(self, c, job, dev):
        self.c, self.seed, self.instance = c, job["seed"], job["instance"]
        self.rho = job["rho"]
        if job["lattice"]:
            rows, cols, st = job["lattice"]
            r = torch.arange(rows, device=dev)[:, None].expand(rows, cols)
            q = torch.arange(cols, device=dev)[None, :].expand(rows, cols)
            offs = [(a, b) for a in (-1, 0, 1) for b in (-1, 0, 1)
                    if (a or b) and (st == 8 or a * b == 0)]
            n = rows * cols
            nb = torch.stack([torch.where((r + a >= 0) & (r + a < rows) & (q + b >= 0) & (q + b < cols),
                                          (r + a) * cols + q + b, n).reshape(-1)
                              for a, b in offs], 1)
            color = ((r + q) % 2 if st == 4 else 2 * (r % 2) + q % 2).reshape(-1)
        else:
            _, row_ptr, col, clr = job["map"]
            n = row_ptr.size - 1
            deg = np.diff(row_ptr)
            table = np.full((n, int(deg.max())), n, dtype=np.int64)
            at = np.arange(col.size) - np.repeat(row_ptr[:-1], deg)
            table[np.repeat(np.arange(n), deg), at] = col
            nb, color = torch.from_numpy(table).to(dev), torch.from_numpy(clr.astype(np.int64)).to(dev)
        self.n, self.nb, self.dev = n, nb, dev
        self.deg = (nb < n).sum(1).to(torch.float64)
        self.sites = [torch.nonzero(color == k)[:, 0] for k in range(int(color.max()) + 1)]
        self.keys = [(ids, None) for ids in self.sites]
        if c["rng"] == 2:              # a color's sites paired by rank
            self.keys = []
            for ids in self.sites:
                rank = torch.arange(ids.numel(), device=dev)
                self.keys.append((ids[rank - (rank & 1)], (rank & 1) == 1))
        self.y = torch.from_numpy(job["y"]).to(dev)
        self.trials = job.get("trials")
        if self.trials is not None:
            m = torch.from_numpy(self.trials.astype(np.int64)).to(dev)
            self.term_site = torch.repeat_interleave(torch.arange(n, device=dev), m)
            start = torch.cumsum(m, 0) - m
            self.term_j = torch.arange(int(m.sum()), device=dev) - start[self.term_site]
            self.y = self.y - 0.5 * m.to(torch.float64)
        self.x = torch.zeros(n + 1, dtype=torch.float64, device=dev)   # the last entry stays 0
        self.s1 = torch.zeros(n, dtype=torch.float64, device=dev)
        self.s2 = torch.zeros(n, dtype=torch.float64, device=dev)
        self.tau = self.lam = 1.0
        self.b0, self.n_acc, self.trace = 0.0, 0, []

    def sweep(self, t):
        c, n, x = self.c, self.n, self.x
        psi = None
        if self.trials is not None:
            tilt = 0.5 * torch.abs(self.b0 + x[:n])
            terms = _pg_terms(tilt[self.term_site], self.term_site, self.term_j, t,
                              self.instance, self.seed)
            psi = torch.zeros(n, dtype=torch.float64, device=self.dev)
            psi.index_add_(0, self.term_site, terms)
        for ids, (key, branch) in zip(self.sites, self.keys):
            s = x[self.nb[ids]].sum(1)
            z = _normals(key, t, self.instance, self.seed, branch)
            if psi is None:
                Q = self.tau * self.deg[ids] + self.lam
                b = self.lam * (self.y[ids] - self.b0)
            else:
                Q = self.tau * self.deg[ids] + psi[ids]
                b = self.y[ids] - psi[ids] * self.b0
            x[ids] = (b + self.tau * self.rho * s) / Q + z / torch.sqrt(Q)
        f = x[:n]
        if t >= c["burn_in"]:
            self.s1 += self.b0 + f
            self.s2 += (self.b0 + f) ** 2
            self.n_acc += 1
        if c["hyper"]:
            edges = torch.zeros((), dtype=torch.float64, device=self.dev)
            for k in range(self.nb.shape[1]):
                other = self.nb[:, k]
                edges += torch.where(other < n, (f - x[other]) ** 2, 0.0).sum()
            q = float((1.0 - self.rho) * (self.deg * f * f).sum() + 0.5 * self.rho * edges)
            rank = n - 1 if self.rho == 1.0 else n
            if psi is not None:
                if c["intercept"]:
                    P = float(psi.sum()) + 1.0 / 1000.0
                    self.b0 = (float((self.y - psi * f).sum()) / P
                               + _scalar_normal(self.seed, 0, t, self.instance, 3) / math.sqrt(P))
            else:
                if c["intercept"]:
                    self.b0 = (float((self.y - f).mean()) + math.sqrt(1.0 / (n * self.lam))
                               * _scalar_normal(self.seed, 0, t, self.instance, 3))
                sse = float(((self.y - self.b0 - f) ** 2).sum())
                self.lam = _gamma(1.0 + 0.5 * n, 1.0 + 0.5 * sse, self.seed, t, self.instance, 2)
            self.tau = _gamma(1.0 + 0.5 * rank, 1.0 + 0.5 * q, self.seed, t, self.instance, 1)
        self.trace.append((self.tau, self.lam, self.b0))

    def stats(self):
        N = self.n_acc
        return self.s1 / N, (self.s2 - self.s1 * self.s1 / N) / (N - 1.0)


def exact(case, seed):
    c = full(case)
    jobs = _jobs(c, seed)
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    samplers = []
    for job in jobs:
        s = _Sampler(c, job, dev)
        for t in range(c["sweeps"]):
            s.sweep(t)
        samplers.append(s)
    if c["kind"] == "step":
        s = samplers[0]
        return {"x": s.x[:s.n], "tau": s.tau, "lam": s.lam}
    stats = [s.stats() for s in samplers]
    out = {"mean": torch.cat([m for m, _ in stats]), "var": torch.cat([v for _, v in stats])}
    if c["kind"] == "sweeps":
        out["trace"] = torch.tensor(samplers[0].trace, dtype=torch.float64)
    return out
