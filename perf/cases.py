"""The work that a user of this framework has it do, as cases that can be timed.

Three kinds of case ("op"):

  slice   one time slice of one sketch (Alg. 4): the packets of the slice, the
          end of the slice, and the cardinalities of the monitored hosts by
          one of the estimate calls ("api");
  query   the estimate call alone, on a slice that is closed already;
  batch   one time slice of several independent sketches: their packets are
          copied into the batch's buffers and the captured slice is replayed;
  train   one minibatch step of the learned estimator.

Traffic has the shape of streams.py's workloads: Zipf(1.1) activity over the
population, Pareto(1.1) numbers of opposite hosts clipped at 1e5.  The window
is full before the first pass (the slices of a stream are cycled), so that
every pass is one of the steady state.
"""
from __future__ import annotations

import math

import torch

from paper_1812_00282_amd import learned, streams, train
from paper_1812_00282_amd.batch import Batch
from paper_1812_00282_amd.sketch import Config, Sketch

_M32 = 0xFFFFFFFF
_SEED_A, _SEED_B = 0xA5A5, 0x5A5A
_WINDOWS = (0.02, 0.1, 0.25, 0.5, 1.0)      # window lengths asked for together, as shares of k


def _slice(name, log2_pool, width, k, g, packets, hosts, population, api, counter=0, block_log2=0, partition=0,
           op="slice", kprime=0):
    c = {"op": op, "log2_pool": log2_pool, "width": width, "k": k, "g": g, "packets": packets, "hosts": hosts,
         "population": population, "api": api, "counter": counter, "block_log2": block_log2, "partition": partition,
         "kprime": kprime}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # An edge router's sketch: the smallest calls, launches and latency.
        _slice("slice_small", 16, 8, 4, 128, 25_000, 1000, 1000, "direct"),
        # The narrowest counters (nibbles), the shortest window.
        _slice("slice_nibble_k2", 26, 4, 2, 128, 25_000, 1000, 1000, "direct"),
        # A few suspicious hosts looked up on a large sketch between slices.
        _slice("query_16_hosts", 28, 8, 60, 1024, 5_000_000, 16, 1_000_000, "direct", op="query"),
        # Training states of the learned estimator: background traffic and the
        # distance histograms and features of some hundred probe hosts.
        _slice("states_331_probes", 28, 8, 60, 1024, 2_500_000, 331, 1_000_000, "states"),
        # A 40 Gb/s link, all 1M hosts, closed form and learned estimates.
        _slice("slice_40g_learned", 28, 8, 60, 1024, 5_000_000, 1_000_000, 1_000_000, "learned"),
        # A fixed list of monitored hosts (planned once), Fig. 5's partition.
        _slice("slice_planned", 27, 8, 16, 1024, 1_250_007, 250_007, 500_000, "planned", partition=1),
        # Several windows at once, long window in 16-bit counters.
        _slice("windows_k256", 28, 16, 256, 1024, 1_000_000, 100_003, 1_000_000, "windows"),
        # The paper's setting of Sec. 5: 10-bit counters packed exactly, k = 300.
        _slice("slice_exact_k300", 27, 10, 300, 1024, 1_000_000, 20_011, 1_000_000, "partitioned"),
        # The baseline of Sec. 5: distance recorders, the whole pool each slide.
        _slice("vdre_k300", 28, 9, 300, 1024, 1_000_000, 1000, 1_000_000, "direct", counter=1),
        # Locality-blocked VATs, all 1M hosts of a 40 Gb/s link.
        _slice("slice_40g_blocked", 28, 8, 60, 1024, 5_000_000, 1_000_000, 1_000_000, "direct", block_log2=6),
        # Sixteen sketches of mixed geometry advanced together by a graph.
        {"name": "batch_16", "op": "batch", "members": 16, "pool_lo": 20, "pool_hi": 26, "mix": 4, "lo": 5.0, "hi": 7.0},
        # One step of the learned estimator's training.
        {"name": "train_4096", "op": "train", "rows": 4096},
    ]


def _log_int(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n))


def draw(rng):
    op = rng.choice(["slice"] * 5 + ["query", "batch", "train"])
    if op == "train":
        return {"op": "train", "rows": _log_int(rng, 64, 65536)}
    if op == "batch":
        lo = rng.randint(16, 22)
        hi = min(26, lo + rng.randint(1, 5))
        return {"op": "batch", "members": rng.randint(2, min(16, 2 ** (28 - hi))), "pool_lo": lo, "pool_hi": hi, "mix": rng.randrange(1 << 16), "lo": round(rng.uniform(3.0, 5.0), 3), "hi": round(rng.uniform(5.2, 6.6), 3)}
    c = rng.randint(16, 28)
    k = _log_int(rng, 2, 300)
    counter = 1 if rng.random() < 0.15 else 0
    need = (k + 1 if counter else 2 * k + 1)
    need = (need - 1).bit_length()
    width = rng.choice([need] + [w for w in (4, 8, 16) if w >= need])
    g = rng.choice([64, 100, 128, 256, 384, 512, 1000, 1024, 1024, 2048])
    block = rng.choice([3, 5, 6]) if rng.random() < 0.12 else 0
    apis = ["direct", "direct"]
    if op == "slice":
        apis += ["partitioned", "windows"] if not block else []
        apis += ["planned"] if not block else []
        apis += ["hist"] if k <= 256 else []
        apis += ["states", "learned"] if k <= 61 else []
    api = rng.choice(apis)
    few = api in ("hist", "states") or op == "query"
    hosts = _log_int(rng, 1, 4096 if few else (1 << 26) // g)
    packets = _log_int(rng, 1000, 4_000_000) if c >= 22 else _log_int(rng, 1000, 400_000)
    return _slice("", c, width, k, g, packets, hosts, max(hosts, _log_int(rng, 1000, 500_000)), api, counter, block,
                  rng.randint(0, 1), op, rng.randint(1, k) if api in ("direct", "partitioned", "planned") and rng.random() < 0.4 else 0)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _i32(x):
    """int64 tensor of 32-bit values -> int32 tensor with the same bits."""
    return (x - (x >= 2**31).to(torch.int64) * 2**32).to(torch.int32)


def _u32(x):
    return x.to(torch.int64) & _M32


def _window(case):
    """The window estimated (0 in a case stands for the longest, k)."""
    return case["kprime"] or case["k"]


def _windows(case):
    return sorted({max(1, int(round(s * case["k"]))) for s in _WINDOWS})


def _traffic(case, seed):
    """(hosts to estimate, the stream's slices) on the GPU."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    H, n = case["population"], case["packets"]
    aips = torch.randint(0, 2**32, (H,), generator=gen, device=dev, dtype=torch.int64)
    u = torch.rand(H, generator=gen, device=dev, dtype=torch.float64).clamp_min(1e-12)
    card = u.pow(-1.0 / 1.1).floor().clamp(1, 100_000)
    rank = torch.randperm(H, generator=gen, device=dev).to(torch.float64) + 1.0
    cdf = torch.cumsum(rank.pow(-1.1), 0)
    cdf = cdf / cdf[-1].clone()
    # as many different slices as fill the window, at most 64 and 2.5 GB
    S = max(2, min(2 * case["k"], 64, 320_000_000 // n))
    pairs = torch.empty((S, n, 2), dtype=torch.int32, device=dev)
    for s in range(S):
        h = torch.searchsorted(cdf, torch.rand(n, generator=gen, device=dev, dtype=torch.float64)).clamp_max(H - 1)
        j = (torch.rand(n, generator=gen, device=dev, dtype=torch.float64) * card[h]).to(torch.int64)
        a = aips[h]
        pairs[s, :, 0] = _i32(a)
        pairs[s, :, 1] = _i32((a * 0x9E37 + j * 0x85EBCA6B + 0x1234567) & _M32)
    hosts = _i32(aips[torch.randperm(H, generator=gen, device=dev)[: case["hosts"]]])
    return hosts.contiguous(), pairs


def _config(case):
    return Config(case["log2_pool"], case["width"], case["k"], case["g"], case["partition"], _SEED_A, _SEED_B,
                  case["counter"], case["block_log2"])


def _before(case):
    """Slices run before the first pass: the window is full."""
    return 2 * case["k"] if case["k"] <= 64 else case["k"] + 8


def _prepare_slice(case, seed):
    hosts, pairs = _traffic(case, seed)
    sk = Sketch(_config(case))
    for s in range(_before(case)):
        sk.ingest(pairs[s % pairs.shape[0]])
        sk.close_slice()
    st = {"case": case, "sk": sk, "hosts": hosts, "pairs": pairs, "next": _before(case)}
    if case["api"] == "planned":
        sk.plan(hosts)
    if case["api"] == "learned":
        theta = train.load()
        st["weights"] = learned.pack(theta, learned.new_weights())
        env = train.load_envelope()
        if (env["k"], env["g"], env["log2_pool"], env["width"]) == (case["k"], case["g"], case["log2_pool"], case["width"]):
            learned.set_envelope(st["weights"], env)
    if case["op"] == "query":
        sk.ingest(pairs[st["next"] % pairs.shape[0]])
        sk.close_slice()
        st["pairs"] = None
    return st


def _members(case):
    return streams.batch_members(case["mix"], case["members"], (case["pool_lo"], case["pool_hi"]))


_BATCH_SLICES, _BATCH_BEFORE = 4, 6


def _batch_traffic(case, seed):
    dev = torch.device("cuda")
    members = _members(case)
    hosts, slices = [], []
    for i, m in enumerate(members):
        gen = torch.Generator(device=dev)
        gen.manual_seed(int(seed) * 64 + i)
        hosts.append(torch.randint(-2**31, 2**31, (m.n_hosts,), generator=gen, device=dev, dtype=torch.int64).to(torch.int32))
    for s in range(_BATCH_SLICES):
        counts = streams.batch_packet_counts(int(seed) & 0xFFFF, len(members), s, case["lo"], case["hi"])
        slices.append([streams.member_slice_torch(m, hosts[i], s, int(counts[i]), dev) for i, m in enumerate(members)])
    return members, hosts, slices


def _prepare_batch(case, seed):
    members, hosts, slices = _batch_traffic(case, seed)
    caps = [max(sl[i].shape[0] for sl in slices) for i in range(len(members))]
    b = Batch([Sketch(Config(m.log2_pool, m.width, m.k, m.g, 0, m.seed, m.seed + 1)) for m in members], caps, hosts)
    for s in range(_BATCH_BEFORE):
        b.load(slices[s % _BATCH_SLICES])
        b.slice()
    b.autotune()
    b.capture()
    return {"case": case, "batch": b, "slices": slices, "next": _BATCH_BEFORE}


def _prepare_train(case, seed):
    """A minibatch of states like the training set's: sparse histograms of
    hosts over the whole range of cardinalities, and a network in training."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    n, k, g = case["rows"], 60, 1024

    def rand(*s):
        return torch.rand(*s, generator=gen, device=dev, dtype=torch.float64)

    truth = torch.exp(rand(n) * math.log(1e6))
    live = g * (1.0 - (1.0 - 0.011) * torch.exp(-truth / g))
    share = torch.rand((n, k), generator=gen, device=dev, dtype=torch.float64) * (rand(n, k) < 0.5)
    share = share / share.sum(1, keepdim=True).clamp_min(1e-9)
    hist = torch.floor(share * live[:, None]).to(torch.int32)
    total = hist.sum(1)
    full = torch.cat([hist, (g - total)[:, None].to(torch.int32)], 1).contiguous()
    est = (g * math.log(1.0 - 0.011) - g * torch.log(((g - total).clamp_min(1)) / g)).to(torch.float32)
    x, r = learned.features(full, est, k, g, 0.011)
    y = torch.log(truth).to(torch.float32)
    theta = train.load() + 0.01 * torch.randn(learned.MLP_PARAMS, generator=gen, device=dev)
    return {"case": case, "x": x, "r": r, "y": y, "theta": theta, "m": torch.zeros_like(theta), "v": torch.zeros_like(theta),
            "grad": torch.zeros_like(theta), "loss": torch.zeros(1, device=dev),
            "weights": learned.pack(theta, learned.new_weights()), "step": 0}


def prepare(case, seed):
    if case["op"] == "train":
        return _prepare_train(case, seed)
    if case["op"] == "batch":
        return _prepare_batch(case, seed)
    return _prepare_slice(case, seed)


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _estimate(st):
    case, sk, hosts = st["case"], st["sk"], st["hosts"]
    api, kp = case["api"], _window(case)
    if api == "direct":
        return sk.estimate(hosts, kp)[:2]
    if api == "partitioned":
        return sk.estimate(hosts, kp, partitioned=True)[:2]
    if api == "planned":
        return sk.estimate_run(kp)[:2]
    if api == "hist":
        return sk.estimate(hosts, kp, want_hist=True)
    if api == "windows":
        return (sk.estimate_windows(hosts, _windows(case)),)
    if api == "learned":
        return learned.estimate_learned(sk, hosts, st["weights"], partitioned=True)
    est, _, hist = sk.estimate(hosts, want_live=False, want_hist=True)
    occupancy = train.cfg_active_fraction(sk.census(), case["k"], case["log2_pool"])
    x, r = learned.features(hist, est, case["k"], case["g"], occupancy)
    return est, hist, x, r


def run(state):
    op = state["case"]["op"]
    if op == "query":
        return list(_estimate(state))
    if op == "slice":
        s = state["next"]
        state["next"] = s + 1
        sk = state["sk"]
        sk.ingest(state["pairs"][s % state["pairs"].shape[0]])
        sk.close_slice()
        return [*_estimate(state), sk.pool]
    if op == "batch":
        b, s = state["batch"], state["next"]
        state["next"] = s + 1
        b.load(state["slices"][s % _BATCH_SLICES])
        b.replay()
        torch.cuda.current_stream().wait_stream(b.stream)
        return [[b.est[i], b.live[i], sk.pool] for i, sk in enumerate(b.sketches)]
    t = state
    t["step"] += 1
    learned.fill(t["grad"], 0.0)
    learned.fill(t["loss"], 0.0)
    learned.train_step(t["weights"], t["x"], t["r"], t["y"], t["grad"], t["loss"])
    learned.adam(t["theta"], t["grad"], t["m"], t["v"], t["step"], lr=3e-3)
    learned.pack(t["theta"], t["weights"])
    return [t["grad"], t["loss"], t["m"], t["v"]]


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
_NET = 2 * (64 * 64 + 64 * 64 + 64)     # flops of the network for one host
_HASH = 8                                # operations of one mix (H of one VAT)


def _work_slice(case):
    pool = 2 ** case["log2_pool"] * case["width"] / 8
    hosts, g, k, n = case["hosts"], case["g"], case["k"], case["packets"]
    out = {"direct": 8, "partitioned": 8, "planned": 8, "hist": 8 + 4 * (k + 1), "windows": 4 * len(_windows(case)),
           "learned": 8, "states": 4 + 4 * (k + 1) + 128 + 4}[case["api"]]
    lookups = min(hosts * g * case["width"] / 8, pool)
    b, f = hosts * (4 + out), hosts * g * _HASH
    if case["api"] == "learned":
        f += hosts * _NET
    if case["op"] == "query":
        return {"bytes": b + lookups, "flops": f}
    # the packets, the counters that they set, the pool once (Z_p of Eq. 11
    # and the lookups), and the counters that the slide looks over
    slide = 2 * pool if case["counter"] else 2 * pool / max(1, 2 * k - 1)
    return {"bytes": b + 8 * n + min(n, 2 ** case["log2_pool"]) * case["width"] / 8 + pool + min(slide, pool),
            "flops": f + n * 3 * _HASH}


def work(case):
    if case["op"] == "train":
        n = case["rows"]
        return {"bytes": n * (128 + 8) + learned.MLP_PARAMS * 4 * 7 + learned.MLP_WEIGHT_BYTES, "flops": 3 * n * _NET}
    if case["op"] == "batch":
        b = f = 0.0
        n = 0.5 * (10 ** case["lo"] + 10 ** case["hi"])          # packets of a member, about
        for m in _members(case):
            w = _work_slice(_slice("", m.log2_pool, m.width, m.k, m.g, int(n), m.n_hosts, m.n_hosts, "direct"))
            b, f = b + w["bytes"], f + w["flops"]
        return {"bytes": b, "flops": f}
    return _work_slice(case)


# ---------------------------------------------------------------------------
# The same values in 64 bits, from the slice in which each counter was last
# set (a counter is active for k' iff that slice is among the last k')
# ---------------------------------------------------------------------------
def _mix(h):
    h = h ^ (h >> 16)
    h = (h * 0x85EBCA6B) & _M32
    h = h ^ (h >> 13)
    h = (h * 0xC2B2AE35) & _M32
    return h ^ (h >> 16)


def _pid(cfg, aip, i):
    key = _mix(aip ^ cfg.seed_a)
    if cfg.block_log2 == 0:
        return _mix(key ^ ((i * 0x9E3779B9) & _M32)) >> (32 - cfg.log2_pool)
    bm = (1 << cfg.block_log2) - 1
    x = _mix(key ^ (((i >> cfg.block_log2) * 0x9E3779B9) & _M32)) >> (32 - cfg.log2_pool)
    return (x & ~bm) | (i & bm)


def _set(last, cfg, pairs, t):
    for part in pairs.split(1 << 23):
        vid = (_mix(_u32(part[:, 1]) ^ cfg.seed_b) * cfg.g) >> 32
        last[_pid(cfg, _u32(part[:, 0]), vid)] = t


def _true_hist(last, cfg, hosts, t):
    """Distances below k of every host's VATs: (hosts, k + 1), the rest last."""
    k, g = cfg.k, cfg.g
    i = torch.arange(g, device=hosts.device)
    out = []
    for part in hosts.split(max(1, (1 << 23) // g)):
        d = (t - last[_pid(cfg, _u32(part)[:, None], i[None, :])]).clamp_max(k).to(torch.int64)
        row = torch.arange(part.numel(), device=hosts.device)[:, None] * (k + 1)
        out.append(torch.bincount((d + row).reshape(-1), minlength=part.numel() * (k + 1)).reshape(-1, k + 1))
    return torch.cat(out)


def _closed_form(cfg, hist, pool_hist, kp):
    N = float(2 ** cfg.log2_pool)
    zv = (cfg.g - hist[:, :kp].sum(1)).clamp_min(1).to(torch.float64) / cfg.g
    zp = max(1.0, N - float(pool_hist[:kp].sum())) / N
    return cfg.g * (math.log(zp) - torch.log(zv))


def _network(theta, x, r):
    p = theta.to(torch.float64)
    w1, b1, w2, b2, w3, b3 = (p[o:o + max(1, math.prod(s))].reshape(s) for o, s in learned.OFFSETS.values())
    a = torch.nn.functional.gelu(x @ w1.T + b1)
    return torch.nn.functional.gelu(a @ w2.T + b2) @ w3 + b3 + r


def _pool_hist(last, k, t):
    h = torch.zeros(k + 1, dtype=torch.int64, device=last.device)
    for part in last.split(1 << 26):
        h += torch.bincount((t - part).clamp_max(k).to(torch.int64), minlength=k + 1)
    return h


def _exact_slice(case, seed):
    hosts, pairs = _traffic(case, seed)
    cfg = _config(case)
    k, t = cfg.k, _before(case)
    last = torch.full((2 ** cfg.log2_pool,), -(1 << 20), dtype=torch.int32, device=hosts.device)
    for s in range(max(0, t - k + 1), t + 1):
        _set(last, cfg, pairs[s % pairs.shape[0]], s)
    pool_hist = _pool_hist(last, k, t)
    hist = _true_hist(last, cfg, hosts, t)
    api = case["api"]
    end = [] if case["op"] == "query" else [None]
    if api == "windows":
        return [torch.stack([_closed_form(cfg, hist, pool_hist, kp) for kp in _windows(case)], 1), *end]
    est = _closed_form(cfg, hist, pool_hist, _window(case))
    if api in ("direct", "partitioned", "planned"):
        return [est, None, *end]
    if api == "hist":
        return [est, None, None, *end]
    occ = float(pool_hist[:k].sum()) / 2 ** cfg.log2_pool
    r = torch.log(est.clamp_min(1.0))
    if api == "states":
        return [est, None, None, r, *end]
    x = torch.zeros((hosts.numel(), 64), dtype=torch.float64, device=hosts.device)
    x[:, :k] = hist[:, :k].to(torch.float64) / cfg.g
    x[:, k] = hist[:, :k].sum(1).to(torch.float64) / cfg.g
    x[:, k + 1] = occ
    x[:, k + 2] = r / 16
    est_l = torch.exp(_network(train.load(), x, r))
    off = ~torch.isfinite(est_l.to(torch.float32))
    env = train.load_envelope()
    if (env["k"], env["g"], env["log2_pool"], env["width"]) == (cfg.k, cfg.g, cfg.log2_pool, cfg.width):
        seen = x.to(torch.bfloat16).to(torch.float32)      # the range is one of rounded features
        lo, hi = (torch.from_numpy(env[e]).to(seen.device) for e in ("lo", "hi"))
        off |= ((seen < lo) | (seen > hi)).any(1)
    return [torch.where(off, est, est_l), est, *end]


def _exact_batch(case, seed):
    members, hosts, slices = _batch_traffic(case, seed)
    out, t = [], _BATCH_BEFORE
    for i, m in enumerate(members):
        cfg = Config(m.log2_pool, m.width, m.k, m.g, 0, m.seed, m.seed + 1)
        last = torch.full((2 ** cfg.log2_pool,), -(1 << 20), dtype=torch.int32, device=hosts[i].device)
        for s in range(max(0, t - cfg.k + 1), t + 1):
            _set(last, cfg, slices[s % _BATCH_SLICES][i], s)
        out.append([_closed_form(cfg, _true_hist(last, cfg, hosts[i], t), _pool_hist(last, cfg.k, t), cfg.k), None, None])
    return out


def _bf16(x):
    return x.to(torch.bfloat16).to(torch.float64)


def _exact_train(case, seed):
    """The step as it is defined: sums, biases, GELU and the output layer are
    exact; features, W1, W2, the activations and the gradients that enter a
    product are values of 16 bits."""
    s = _prepare_train(case, seed)
    x = _i32((s["x"].to(torch.int64) & 0xFFFF) << 16).view(torch.float32).to(torch.float64)
    p = s["theta"].to(torch.float64)
    w1, b1, w2, b2, w3, b3 = (p[o:o + max(1, math.prod(q))].reshape(q) for o, q in learned.OFFSETS.values())
    w1, w2 = _bf16(w1), _bf16(w2)

    def slope(z):
        return 0.5 * (1 + torch.erf(z / math.sqrt(2))) + z * torch.exp(-z * z / 2) / math.sqrt(2 * math.pi)

    z1 = x @ w1.T + b1
    a1 = _bf16(torch.nn.functional.gelu(z1))
    z2 = a1 @ w2.T + b2
    a2 = _bf16(torch.nn.functional.gelu(z2))
    e = torch.exp(a2 @ w3 + b3 + s["r"].to(torch.float64) - s["y"].to(torch.float64))
    do = torch.sign(e - 1) * e / case["rows"]
    dz2 = do[:, None] * w3 * slope(z2)
    dz1 = (_bf16(dz2) @ w2) * slope(z1)
    g = torch.cat([(_bf16(dz1).T @ x).reshape(-1), dz1.sum(0), (_bf16(dz2).T @ a1).reshape(-1), dz2.sum(0), do @ a2,
                   do.sum().reshape(1)])
    return [g, torch.abs(e - 1).mean().reshape(1), 0.1 * g, 0.001 * g * g]


def exact(case, seed):
    if case["op"] == "train":
        return _exact_train(case, seed)
    if case["op"] == "batch":
        return _exact_batch(case, seed)
    return _exact_slice(case, seed)
