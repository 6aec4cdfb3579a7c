"""Performance cases of the framework: what its users have it do, through its
public entry points, over the sizes that the benchmark, the tests and the
serving trace use.

Two ways of working are covered:

* ``direct``: a program that holds its data in device memory and runs one
  request on its own stream (``gvm_plain_run_noalloc``);
* ``batch``: eight SPMD ranks that share the GPU through the manager, each
  with its request in its shared-memory space (``gvm_submit`` / ``gvm_wait``
  on the zero-copy region), every copy to and from the device included.

A case is ``{"way", "kernel", "n"}``: the kernel (vecadd, vecmul, bs, sgemm,
ep) and the request size, per rank for a batch.  The inputs have the
distributions of the framework's own workloads: vectors U[-1, 1]; options
S U[5, 30], K U[1, 100], T U[0.25, 10]; matrices N(0, 1); random EP keys.
"""

import math
import os

import numpy as np
import torch

from paper_1511_07658_amd import gvm as G

KERNELS = {"vecadd": G.GVM_K_VECADD, "vecmul": G.GVM_K_VECMUL, "bs": G.GVM_K_BLACKSCHOLES,
           "sgemm": G.GVM_K_SGEMM, "ep": G.GVM_K_EP}
RATE = float(np.float32(0.02))
VOLATILITY = float(np.float32(0.30))
RANKS = 8


def case(way, kernel, n, name=None):
    c = {"way": way, "kernel": kernel, "n": n}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # two of the uneven workload's lengths, odd as most of them are: a short
        # one, where a call is mostly latency, and a long one
        case("direct", "vecadd", 491127, "vecadd_491127"),
        case("direct", "vecadd", 14520833, "vecadd_uneven"),
        # the vector multiply of the model validation, 16M elements
        case("direct", "vecmul", 1 << 24, "vecmul_16m"),
        # a ragged book of options, and the batch workload's four million
        case("direct", "bs", 300001, "bs_300001"),
        case("direct", "bs", 4 << 20, "bs_4m"),
        # matrix products: the serving range's smallest, a ragged one, the
        # 8-rank workload's size and the serving range's largest
        case("direct", "sgemm", 256, "sgemm_256"),
        case("direct", "sgemm", 517, "sgemm_517"),
        case("direct", "sgemm", 1024, "sgemm_1024"),
        case("direct", "sgemm", 2048, "sgemm_2048"),
        # the EP-like tally at one work unit, the smallest of its validation
        case("direct", "ep", 1 << 15, "ep_32k"),
        # whole steps of eight ranks through the manager: the matrix product
        # with its copies over the link, and the EP-like tally, which has none
        # to speak of
        case("batch", "sgemm", 1024, "batch8_sgemm_1024"),
        case("batch", "ep", 1 << 24, "batch8_ep_16m"),
    ]


def draw(rng):
    def log2(lo, hi):
        return int(2.0 ** rng.uniform(lo, hi))

    if rng.random() < 0.2:
        kernel = rng.choice(["sgemm", "vecadd", "bs", "ep"])
        n = {"sgemm": lambda: 64 * rng.randint(4, 16) - rng.choice([0, 0, rng.randint(1, 63)]),
             "vecadd": lambda: log2(18, 20), "bs": lambda: log2(17, 20), "ep": lambda: log2(15, 24)}[kernel]()
        return case("batch", kernel, n)
    kernel = rng.choice(["vecadd", "vecmul", "bs", "sgemm", "sgemm", "ep"])
    if kernel == "sgemm":  # multiples of 64 as the workloads draw them, and any size
        n = 64 * rng.randint(4, 32) if rng.random() < 0.4 else log2(6, 11)
    else:
        n = log2(*{"vecadd": (19, 24), "vecmul": (19, 24), "bs": (17, 22), "ep": (15, 24)}[kernel])
    return case("direct", kernel, n)


def work(c):
    n, ranks = c["n"], RANKS if c["way"] == "batch" else 1
    nbytes = 4 * (G.in_elems(KERNELS[c["kernel"]], n) + G.out_elems(KERNELS[c["kernel"]], n))
    flops = {"vecadd": n, "vecmul": n,
             # per option: the logarithm, the two exponentials of the discount
             # and of each density, root and divisions as one operation each,
             # two fifth-degree polynomials, the two prices
             "bs": 50 * n,
             "sgemm": 2 * n ** 3,
             # binary64 operations per pair of the method: both uniforms and
             # the radius, and for an accepted pair (pi / 4) the transform
             # and the tally
             "ep": (9 + math.pi / 4 * 9) * n}[c["kernel"]]
    return {"bytes": ranks * nbytes, "flops": ranks * flops}


# ------------------------------------------------------------------ inputs

def device_input(c, seed):
    """The packed input of one request in device memory."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, kernel = c["n"], c["kernel"]
    if kernel == "ep":
        return torch.randint(-2 ** 63, 2 ** 63 - 1, (2,), generator=g, device="cuda")
    if kernel == "sgemm":
        return torch.randn(2 * n * n, generator=g, device="cuda")
    x = torch.rand((3 if kernel == "bs" else 2) * n, generator=g, device="cuda")
    if kernel == "bs":
        for part, lo, hi in ((x[:n], 5.0, 30.0), (x[n:2 * n], 1.0, 100.0), (x[2 * n:], 0.25, 10.0)):
            part.mul_(hi - lo).add_(lo)
        return x
    return x.mul_(2.0).sub_(1.0)


def host_input(c, seed, rank, into):
    """The packed input of one rank's request, written to its shared memory."""
    g = np.random.Generator(np.random.PCG64(np.random.SeedSequence([seed, rank])))
    n, kernel = c["n"], c["kernel"]
    if kernel == "ep":
        into.view(np.uint64)[:] = g.integers(0, 2 ** 64, size=2, dtype=np.uint64)
    elif kernel == "sgemm":
        g.standard_normal(out=into, dtype=np.float32)
    else:
        g.random(out=into, dtype=np.float32)
        if kernel == "bs":
            for part, lo, hi in ((into[:n], 5.0, 30.0), (into[n:2 * n], 1.0, 100.0), (into[2 * n:], 0.25, 10.0)):
                part *= hi - lo
                part += lo
        else:
            into *= 2.0
            into -= 1.0


# ------------------------------------------------------------------ ways

class Direct:
    """Device buffers of one request, as a program that reuses them holds them."""

    def __init__(self, c, seed):
        self.kernel, self.n = KERNELS[c["kernel"]], c["n"]
        self.x = device_input(c, seed)
        if c["kernel"] == "ep":
            self.out = torch.empty(12, dtype=torch.int64, device="cuda")
            self.result = (self.out[:2].view(torch.float64), self.out[2:])
        else:
            self.out = torch.empty(G.out_elems(self.kernel, self.n), device="cuda")
            self.result = self.out
        self.stream = torch.cuda.current_stream().cuda_stream
        G.lib()

    def run(self):
        G.check(G.gvm_plain_run_noalloc(self.kernel, self.x.data_ptr(), self.out.data_ptr(), self.n, RATE, VOLATILITY,
                                        self.stream), "gvm_plain_run_noalloc")
        return self.result


class Manager:
    """The manager and its eight attached ranks, up while a batch is."""

    SPACE = 96 << 20   # shared memory per rank, cut into regions of one request each
    REGIONS = 6
    up = None
    users = 0

    @classmethod
    def acquire(cls):
        if cls.up is None:
            cls.up = cls()
        cls.users += 1
        return cls.up

    @classmethod
    def release(cls):
        cls.users -= 1
        if cls.users == 0:
            cls.up.spaces = None
            cls.up = None
            G.check(G.gvm_shutdown(), "gvm_shutdown")

    def __init__(self):
        name = "gvm.perf.%d" % os.getpid()
        cfg = G.gvm_config_default(nranks=RANKS, shm_bytes_per_rank=self.SPACE, staging_bytes=16 << 20,
                                   hbm_budget_bytes=1 << 30, batch_window_us=1_000_000, name=name)
        G.check(G.gvm_init(cfg), "gvm_init")
        self.spaces = []
        for r in range(RANKS):
            G.check(G.gvm_attach_ns(name, r), "gvm_attach")
            self.spaces.append(G.gvm_rank_buffer(r, self.SPACE))
        self.free = list(range(self.REGIONS))


class Results(list):
    """The ranks' results where they lie, in shared memory that their owner keeps mapped."""

    def __init__(self, results, owner):
        super().__init__(results)
        self.owner = owner


class Batch:
    """Eight ranks' requests, each in its rank's shared-memory space."""

    def __init__(self, c, seed):
        self.kernel, self.n = KERNELS[c["kernel"]], c["n"]
        self.region = None
        self.manager = Manager.acquire()
        self.region = self.manager.free.pop()
        ni, no = G.in_elems(self.kernel, self.n), G.out_elems(self.kernel, self.n)
        elems = Manager.SPACE // 4 // Manager.REGIONS // 1024 * 1024
        out_at = (ni + 1023) // 1024 * 1024
        if out_at + no > elems:
            raise ValueError("a request of this size does not fit its region")
        self.ins, self.outs, self.result = [], [], []
        for r in range(RANKS):
            space = self.manager.spaces[r][self.region * elems:(self.region + 1) * elems]
            host_input(c, seed, r, space[:ni])
            self.ins.append(space[:ni])
            self.outs.append(space[out_at:out_at + no])
            if c["kernel"] == "ep":
                self.result.append((self.outs[r].view(np.float64)[:2], self.outs[r].view(np.int64)[2:]))
            else:
                self.result.append(self.outs[r])

    def run(self):
        tickets = [G.check(G.gvm_submit(r, self.kernel, self.ins[r], self.outs[r], self.n), "gvm_submit")
                   for r in range(RANKS)]
        for r in range(RANKS):
            G.check(G.gvm_wait(r, tickets[r]), "gvm_wait")
        return Results(self.result, self)

    def __del__(self):
        if self.region is not None:
            self.ins = self.outs = self.result = None
            self.manager.free.append(self.region)
            self.manager = None
            Manager.release()


def prepare(c, seed):
    return (Batch if c["way"] == "batch" else Direct)(c, seed)


def run(state):
    return state.run()


# ------------------------------------------------------------------ 64 bits

def exact_request(c, x):
    """What one request returns for its packed input `x` (on the GPU), in 64 bits."""
    n, kernel = c["n"], c["kernel"]
    if kernel == "ep":
        return exact_ep(x.cpu().numpy().view(np.uint64), n)
    x = x.double()
    if kernel == "vecadd":
        return x[:n] + x[n:]
    if kernel == "vecmul":
        return x[:n] * x[n:]
    if kernel == "sgemm":
        return (x[:n * n].view(n, n) @ x[n * n:].view(n, n)).reshape(-1)
    s, k, t = x[:n], x[n:2 * n], x[2 * n:]
    vol = VOLATILITY * torch.sqrt(t)
    d1 = (torch.log(s / k) + (RATE + 0.5 * VOLATILITY ** 2) * t) / vol
    d2 = d1 - vol
    kd = k * torch.exp(-RATE * t)

    def cdf(z):
        return 0.5 * torch.erfc(-z / math.sqrt(2.0))

    return torch.cat([s * cdf(d1) - kd * cdf(d2), kd * cdf(-d2) - s * cdf(-d1)])


def exact_ep(key, n):
    """The tally of n pairs: numpy's Philox generator gives the words (it
    steps its counter before the first block, so it starts one below zero)."""
    words = np.random.Philox(counter=(1 << 256) - 1, key=int(key[0]) | int(key[1]) << 64)
    sums, counts = [0.0, 0.0], np.zeros(10, np.int64)
    done = 0
    while done < n:
        m = min(n - done, 1 << 22)
        w = words.random_raw(2 * m)
        u = torch.from_numpy((w >> np.uint64(11)).astype(np.float64)).cuda() * 2.0 ** -53
        x, y = 2.0 * u[0::2] - 1.0, 2.0 * u[1::2] - 1.0
        t = x * x + y * y
        ok = (t > 0.0) & (t <= 1.0)
        x, y, t = x[ok], y[ok], t[ok]
        f = torch.sqrt(-2.0 * torch.log(t) / t)
        x, y = x * f, y * f
        sums[0] += float(x.sum())
        sums[1] += float(y.sum())
        ring = torch.maximum(x.abs(), y.abs()).to(torch.int64)
        counts += torch.bincount(ring, minlength=10)[:10].cpu().numpy()
        done += m
    return np.array(sums), counts


def exact(c, seed):
    if c["way"] == "direct":
        return exact_request(c, device_input(c, seed))
    got = []
    for r in range(RANKS):
        x = np.empty(G.in_elems(KERNELS[c["kernel"]], c["n"]), np.float32)
        host_input(c, seed, r, x)
        if c["kernel"] == "ep":
            got.append(exact_ep(x.view(np.uint64), c["n"]))
        else:
            got.append(exact_request(c, torch.from_numpy(x).cuda()).cpu().numpy())
    return got
