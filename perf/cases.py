"""The calls this library spends its time on, as cases that can be timed and compared one by one.

Each case is one step of a program that owns an embedding table (or the two dense tables of the
quotient-remainder decomposition): `prepare` makes the table, brings it to the state that such a program
has after running for a while, and lays out a short cycle of batches; `run` takes the next batch of the
cycle through the public entry points, with the caller's own output buffers, as a training or serving loop
does; every pass has a step number of its own.

Four kinds:
  serve  lookup_or_insert + gather_pool                                   (the forward)
  train  lookup_or_insert + gather_pool + apply_grad_adagrad, and, on tables whose keys expire,
         expire_sweep                                                     (forward and backward)
  sync   a training step + export_touched                                 (incremental synchronisation)
  qr     qr_gather_pool                                                   (two dense tables, no lookup)

What a pass returns.  Pooled rows, the number of expired keys, and (sync) the message with the exported keys,
rows and accumulators.  Row numbers are left out: which row a new key gets is not specified and differs from run to
run.  The rows that an update wrote come back where the next pass pools them, and whole in the sync cases.
The cycle lets every state run for any number of passes in a steady mix: keys that one batch of it brings
are found again a cycle later (no expiry), or have expired by then and are counted and admitted anew
(expiry shorter than the cycle), or stay below a high admission threshold and miss every time.
"""
import math

import numpy as np
import torch

from paper_2209_07663_amd.binding import Table, mono_qr_gather_pool

DEVICE = "cuda:0"
LR, EPS, GRAD_SIGMA = 0.05, 1e-8, 0.1
HEAD = 1 << 16                                   # ranks whose probabilities are summed exactly
M1, M2 = 0xD6E8FEB86659FD93, 0xA5A5A5A5A5A5A5A5  # odd multipliers that spread the ranks over the ID space


def _case(name, kind, capacity_log2, dim, samples, slots, lam, alpha, universe_bits, bf16=False, threshold=1,
          expire=0, hashes=1, min_len=1, fill=0.0, batches=8, noalloc=False):
    """lam, min_len: a bag holds Poisson(lam) + min_len IDs; alpha: Zipf exponent of the IDs, 0 = uniform;
    fill: share of the table that the hottest IDs take before the first pass; batches: length of the cycle."""
    return dict(name=name, kind=kind, capacity_log2=capacity_log2, dim=dim, samples=samples, slots=slots,
                lam=float(lam), min_len=min_len, alpha=float(alpha), universe_bits=universe_bits, bf16=bf16,
                threshold=threshold, expire=expire, hashes=hashes, fill=float(fill), batches=batches, noalloc=noalloc)


def listed():
    return [
        # One serving request: sixteen candidates with the 26 multi-hot slots of the repository's workloads, all
        # of whose IDs the table knows.  Latency and launches are all there is.
        _case("serve_request", "serve", 22, 32, 16, 26, 3, 1.05, 32),
        # configs[0] of the benchmark: one batch of 4096 uniform IDs, dim 16, 2^16 rows, lookup and gather.
        _case("serve_uniform_4k", "serve", 16, 16, 4096, 1, 0, 0, 20, batches=6),
        # A mini-batch of online training: 256 samples, keys expire, new ones keep coming in.
        _case("train_minibatch", "train", 20, 32, 256, 26, 3, 1.1, 40, threshold=2, expire=10, batches=14),
        # The same in the largest batch that the allocation-free update takes, on a table without expiry.
        _case("train_noalloc_200k", "train", 22, 16, 1960, 26, 3, 1.05, 32, batches=8, noalloc=True),
        # User-history slots: long, ragged and often empty bags, a dimension that is no power of two, and the
        # two-hash occurrence filter.
        _case("train_history_ragged", "train", 22, 36, 10007, 3, 23, 1.1, 40, threshold=3, expire=6, hashes=2,
              min_len=0, batches=8),
        # Wide rows (dim 512, bf16), a few slots per sample.
        _case("train_wide_bf16", "train", 20, 512, 4099, 8, 2, 1.1, 40, bf16=True, batches=6),
        # configs[1] as a full training step: half of the table holds the hottest IDs, the tail stays below the
        # admission threshold and misses at every step.
        _case("train_cfg2", "train", 24, 32, 65536, 26, 3, 1.05, 32, threshold=255, fill=0.5, batches=12),
        # configs[2], the largest: 26 M IDs a step, dim 64, every key known after the first cycle.
        _case("train_cfg3", "train", 26, 64, 131072, 40, 4, 1.1, 40, batches=4),
        # configs[3]: a stream whose tail never stops changing.  About a million keys come in and about as many
        # expire at every step, at the load that follows from it.
        _case("train_cfg4_stream", "train", 25, 32, 65536, 26, 3, 1.1, 40, expire=20, batches=24),
        # configs[4]: 2^28 rows in bf16, sparsely filled, a million one-hot IDs a step, a sweep every step.
        _case("train_cfg5_bf16", "train", 28, 64, 262144, 4, 0, 1.2, 63, bf16=True, threshold=2, expire=50, batches=56),
        # The hashing baseline: configs[1]'s batch over two dense tables of 2^24 rows, forward only.
        _case("qr_pool", "qr", 24, 32, 65536, 26, 3, 1.05, 48, batches=3),
        # Incremental synchronisation: the keys that a training step touched leave for the serving side.
        _case("sync_touched", "sync", 22, 64, 1024, 26, 3, 1.1, 40, batches=8),
    ]


def draw(rng):
    """One more case of the ranges above: 400 to 8 M IDs, dims 4 to 512, fp32 and bf16, short and long bags."""
    kind = rng.choice(("serve", "train", "train", "train", "sync", "qr"))
    dim = rng.choice((4, 8, 16, 20, 32, 36, 48, 64, 100, 128, 256, 512))
    long_bags = rng.random() < 0.25
    lam = round(rng.uniform(6, 40), 1) if long_bags else rng.choice((0.0, 1.0, 2.0, 3.0, 4.0))
    min_len = 0 if lam > 0 and rng.random() < 0.3 else 1
    slots = rng.choice((1, 2, 3, 4, 8, 13, 26, 40))
    top = min(8e6, 2.5e8 / dim) if kind != "sync" else 3e5
    n = math.exp(rng.uniform(math.log(400), math.log(top)))
    samples = max(1, int(n / (slots * (lam + min_len))))
    alpha = rng.choice((0.0, 1.05, 1.1, 1.2))
    if kind == "qr":
        m = rng.randint(16, 24 if dim <= 32 else 20)
        return _without_name(_case("", "qr", m, dim, samples, slots, lam, alpha, 2 * m, bf16=rng.random() < 0.5,
                                   min_len=min_len, batches=3))
    expire = rng.choice((0, 0, 4, 8)) if kind == "train" else 0
    batches = expire + 4 if expire else 4
    c = _case("", kind, 16, dim, samples, slots, lam, alpha, rng.randint(32, 63) if alpha else rng.randint(20, 30),
              bf16=rng.random() < 0.5, threshold=rng.randint(1, 3), expire=expire, hashes=rng.choice((1, 1, 1, 2)),
              min_len=min_len, batches=batches)
    stored = distinct(c, _ids(c) * batches)      # no more than this many keys are ever stored
    c["capacity_log2"] = min(25, max(12, math.ceil(math.log2(stored / 0.75)) + rng.choice((0, 0, 1, 2))))
    c["noalloc"] = kind == "train" and _ids(c) < 2.4e5 and rng.random() < 0.3
    return _without_name(c)


def _without_name(c):
    return {k: v for k, v in c.items() if k != "name"}


# ---- inputs ----------------------------------------------------------------------------------------------


def _weights(alpha, universe):
    """Zipf weights of the ranks 1..HEAD, and of all ranks beyond together (their sum as an integral)."""
    head = np.arange(1, min(HEAD, universe) + 1, dtype=np.float64) ** -alpha
    if universe <= HEAD:
        return head, 0.0
    e = 1.0 - alpha
    return head, ((HEAD + 0.5) ** e - (universe + 0.5) ** e) / -e


def _ranks(case, n, gen):
    """n ranks (from 0) of the case's distribution, on the device."""
    universe = 1 << case["universe_bits"]
    if case["alpha"] == 0:
        return torch.randint(0, min(universe, (1 << 63) - 1), (n,), device=DEVICE, generator=gen)
    head, tail = _weights(case["alpha"], universe)
    cdf = torch.from_numpy(np.cumsum(head) / (head.sum() + tail)).to(DEVICE)
    u = torch.rand(n, device=DEVICE, generator=gen, dtype=torch.float64)
    r = torch.searchsorted(cdf, u, right=True)
    if tail > 0:                                 # beyond the head the sum is an integral and is inverted as one
        e, share = 1.0 - case["alpha"], float(cdf[-1])
        v = ((u - share) / (1.0 - share)).clamp(0.0, 1.0)
        lo, hi = (HEAD + 0.5) ** e, (universe + 0.5) ** e
        far = (lo + v * (hi - lo)).pow(1.0 / e).clamp(HEAD + 1.0, min(float(universe), 2.0 ** 63 - 2.0 ** 12))
        r = torch.where(u < share, r, far.to(torch.int64) - 1)
    return r.clamp_(max=universe - 1)


def _spread(ranks, bits):
    """A bijection of [0, 2^bits): hot ranks are no neighbouring integers."""
    mask = (1 << bits) - 1
    for m in (M1, M2):
        ranks = (ranks * (m - (1 << 64))) & mask
        ranks = ranks ^ (ranks >> (bits // 2 + 1))
    return ranks


def _batch(case, gen):
    bags = case["samples"] * case["slots"]
    if case["lam"] > 0:
        lengths = torch.poisson(torch.full((bags,), case["lam"], device=DEVICE), generator=gen).to(torch.int64)
        lengths += case["min_len"]
    else:
        lengths = torch.ones(bags, dtype=torch.int64, device=DEVICE)
    offsets = torch.zeros(bags + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(lengths, 0, out=offsets[1:])
    keys = _spread(_ranks(case, int(offsets[-1]), gen), case["universe_bits"])
    return keys, offsets


def _fill(table, case, gen):
    """The hottest IDs come back from a snapshot."""
    count = int(case["fill"] * table.capacity)
    for lo in range(0, count, 1 << 21):
        k = _spread(torch.arange(lo, min(count, lo + (1 << 21)), device=DEVICE), case["universe_bits"])
        values = torch.randn((k.shape[0], case["dim"]), device=DEVICE, generator=gen).mul_(0.05)
        acc = torch.rand(k.shape[0], device=DEVICE, generator=gen)
        table.mono_table_import(k, values, acc, torch.zeros(k.shape[0], dtype=torch.int32, device=DEVICE))


class State:
    """What the program keeps: the table, its output buffers, and the batches that its loader has put on the GPU."""

    def __init__(self, case, seed):
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(seed)
        self.kind, self.noalloc, self.expire = case["kind"], case["noalloc"], case["expire"]
        self.batches = [_batch(case, gen) for _ in range(case["batches"])]
        bags, dim = case["samples"] * case["slots"], case["dim"]
        self.pooled = torch.empty((bags, dim), device=DEVICE)
        self.passes = self.step = 0
        if self.kind == "qr":
            dtype = torch.bfloat16 if case["bf16"] else torch.float32
            self.tables = [torch.randn((1 << case["capacity_log2"], dim), device=DEVICE, generator=gen).mul_(0.05).to(dtype)
                           for _ in range(2)]
            return
        most = max(1, bags - 1, *(k.shape[0] for k, _ in self.batches))
        self.table = Table(1 << case["capacity_log2"], dim, seed, case["threshold"], case["expire"], case["bf16"],
                           max_ids=most, max_bags=bags, device=DEVICE, filter_hashes=case["hashes"])
        self.rows = torch.empty(most, dtype=torch.int32, device=DEVICE)
        self.expired = torch.zeros(1, dtype=torch.int64, device=DEVICE)
        if self.kind != "serve":
            self.grad = torch.randn((bags, dim), device=DEVICE, generator=gen).mul_(GRAD_SIGMA)
        if self.kind == "sync":                  # the message to the serving side, as large as a step can make it
            most = int(1.25 * _ids(case)) + 4096
            self.message = {"keys": np.zeros(most, np.int64), "rows": np.zeros((most, dim), np.float32),
                            "acc": np.zeros(most, np.float32)}
        if case["fill"] > 0:
            _fill(self.table, case, gen)
        else:                                    # the cycle has gone round before
            for _ in range(1 if case["expire"] else case["threshold"]):
                for keys, _ in self.batches:
                    self.table.mono_lookup_or_insert(keys, self.step, self.rows[: keys.shape[0]])
                    if self.expire:
                        self.table.mono_expire_sweep(self.step)
                    self.step += 1


def prepare(case, seed):
    return State(case, seed)


def run(s):
    keys, offsets = s.batches[s.passes % len(s.batches)]
    s.passes += 1
    if s.kind == "qr":
        return mono_qr_gather_pool(s.tables[0], s.tables[1], keys, offsets, s.pooled)
    t, rows, step = s.table, s.rows[: keys.shape[0]], s.step
    s.step += 1
    t.mono_lookup_or_insert(keys, step, rows)
    t.mono_gather_pool(rows, offsets, s.pooled)
    if s.kind == "serve":
        return s.pooled
    if s.noalloc:
        t.mono_apply_grad_adagrad_noalloc(rows, offsets, s.grad, LR, EPS)
    else:
        t.mono_apply_grad_adagrad(rows, offsets, s.grad, LR, EPS)
    if s.kind == "sync":
        delta = t.mono_export_touched()
        for part, to in s.message.items():
            to[: delta["n"]] = delta[part]
        return {"pooled": s.pooled, "n": delta["n"], "message": s.message}
    if s.expire:
        t.mono_expire_sweep(step, s.expired)
        return {"pooled": s.pooled, "expired": s.expired}
    return s.pooled


# ---- what a pass cannot do without -----------------------------------------------------------------------


def _ids(case):
    return case["samples"] * case["slots"] * (case["lam"] + case["min_len"])


def distinct(case, n):
    """Expected number of distinct IDs among n."""
    universe = 1 << case["universe_bits"]
    if case["alpha"] == 0:
        return -universe * math.expm1(-n / universe)
    head, tail = _weights(case["alpha"], universe)
    total = head.sum() + tail
    u = float(-np.expm1(-n * head / total).sum())
    if tail > 0:                                 # the ranks beyond, in geometric steps
        edge = np.exp(np.linspace(math.log(HEAD), math.log(universe), 400))
        mid = np.sqrt(edge[1:] * edge[:-1])
        u += float((np.diff(edge) * -np.expm1(-n * mid ** -case["alpha"] / total)).sum())
    return u


def work(case):
    """Compulsory bytes: each ID, offset, row number, distinct row, gradient and pooled row once; of a table, the
    eight keys of one bucket per distinct ID, its last-seen step and its optimizer state."""
    n, bags, dim = _ids(case), case["samples"] * case["slots"], case["dim"]
    row, pooled = dim * (2 if case["bf16"] else 4), 4 * dim * bags
    if case["kind"] == "qr":
        half = 1 << case["capacity_log2"]
        parts = distinct(case, n)
        rows = half * -math.expm1(-parts / half)          # remainders of scrambled IDs are uniform, quotients too
        return {"bytes": 8 * n + 8 * bags + 2 * row * rows + pooled, "flops": 2 * n * dim}
    u = distinct(case, n)
    if case["fill"] > 0:                                  # only the hottest IDs have rows
        stored = case["fill"] * (1 << case["capacity_log2"])
        head, tail = _weights(case["alpha"], 1 << case["universe_bits"])
        e = 1.0 - case["alpha"]
        present = float(-np.expm1(-n * head / (head.sum() + tail)).sum())
        edge = np.exp(np.linspace(math.log(HEAD), math.log(stored), 400))
        mid = np.sqrt(edge[1:] * edge[:-1])
        present += float((np.diff(edge) * -np.expm1(-n * mid ** -case["alpha"] / (head.sum() + tail))).sum())
    else:
        present = u if case["threshold"] == 1 or not case["expire"] else 0.5 * u
    b = 8 * n + 4 * n + 8 * bags + 68 * u + row * present + pooled
    f = n * dim
    if case["kind"] != "serve":
        b += pooled + (row + 16) * present
        f += n * dim + 6 * present * dim
    if case["kind"] == "sync":
        b += (8 + 4 * dim + 4) * present
    if case["expire"]:
        b += 4 * min(distinct(case, n * case["expire"]), 31 / 32 * (1 << case["capacity_log2"]))
    return {"bytes": b, "flops": f}


def tolerance(case):
    """fp32 sums in another order; rows that an update rounds to bf16 may fall to the other side of a tie."""
    return {"rel": 1e-2 if case["bf16"] and case["kind"] in ("train", "sync") else 1e-5}
