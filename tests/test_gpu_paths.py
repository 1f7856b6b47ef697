"""Kernel variants chosen by size, each at the sizes where it can go wrong,
against the CPU oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1812_00282_amd.sketch import Config, Sketch  # noqa: E402
from test_gpu_learned import test_gradient_parity as gradient_parity  # noqa: E402
from test_gpu_parity import _check_estimates, _check_state, _pair, _u32  # noqa: E402

pytestmark = pytest.mark.gpu


def _stream(rng, n, hosts, peers, hot=0.0):
    """n packets of `hosts` hosts; a share `hot` of them is one single pair."""
    p = np.empty((n, 2), dtype=np.uint32)
    p[:, 0] = hosts[rng.integers(0, hosts.size, n)]
    p[:, 1] = rng.integers(0, peers, n)
    p[rng.random(n) < hot] = (hosts[0], 7)
    return p


# Counters set by compare-and-swap: one packet, one workgroup's share and its
# remainder, several tiles per workgroup; counters that share words with hot
# ones, words that straddle, the filter's slots taken by several counters.
@pytest.mark.parametrize("w,k,c,n", [(4, 7, 9, 1), (4, 7, 20, 1_200_003), (3, 3, 10, 1025), (7, 60, 18, 300_001),
                                     (10, 300, 16, 1_100_000), (15, 300, 12, 4097)])
def test_ingest_hot_counters(w, k, c, n):
    rng = np.random.default_rng(c * 100 + w)
    hosts = rng.integers(0, 2**32, 500, dtype=np.uint64).astype(np.uint32)
    gpu, ref = _pair(Config(c, w, k, 64, seed_a=3, seed_b=4))
    for t in range(3):
        p = _stream(rng, n, hosts, 5000, hot=0.4)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
        _check_state(gpu, ref, f"slice {t}")


# The direct gather: lanes per host and hosts per workgroup change with the
# number of hosts, gathers in flight with g; odd and even k, one host, the
# remainder of a workgroup's hosts; with and without histograms.
@pytest.mark.parametrize("c,w,k,g,n_hosts,b", [
    (14, 8, 60, 1024, 1, 0), (14, 8, 61, 1000, 17, 0), (12, 4, 7, 64, 2049, 0), (16, 10, 300, 257, 33, 0),
    (14, 16, 256, 100, 4100, 0), (13, 5, 9, 1, 9000, 0), (16, 8, 13, 300, 40_000, 3), (15, 7, 60, 3, 33_000, 0)])
def test_direct_gather_shapes(c, w, k, g, n_hosts, b):
    rng = np.random.default_rng(c * 1000 + g)
    gpu, ref = _pair(Config(c, w, k, g, seed_a=1, seed_b=2, block_log2=b))
    hosts = rng.integers(0, 2**32, n_hosts, dtype=np.uint64).astype(np.uint32)
    for t in range(5):
        p = _stream(rng, 4000, hosts, 3000)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    for kp in sorted({1, 2, k}):
        _check_estimates(gpu, ref, hosts, kprime=kp, hist=(kp == k and k <= 256), what=f"k'={kp}")
    if k <= 256:
        kps = sorted({1, 2, 3, (k + 1) // 2, k - 1, k})
        est = gpu.estimate_windows(hosts, kps).cpu().numpy().astype(np.float64)
        for j, kp in enumerate(kps):
            one, _, _ = gpu.estimate(hosts, kprime=kp)
            np.testing.assert_array_equal(est[:, j], one.cpu().numpy().astype(np.float64))


# Which path answers depends on lookups and pool size: bitmaps copied to LDS
# (up to 2^20 ATs, from 2M lookups), partitioned lookups (from 2^23 ATs), both
# sides of the rules; subgroups of even size, windows of few subgroups.
@pytest.mark.parametrize("c,w,k,g,n_hosts", [
    (5, 7, 9, 1024, 2100), (20, 8, 60, 1024, 2048), (16, 10, 300, 2048, 1500), (18, 4, 7, 100, 30_001),
    (20, 16, 256, 33, 70_000), (19, 8, 61, 1000, 2500), (23, 8, 60, 1024, 48_000), (23, 8, 60, 2048, 24_577),
    (26, 8, 61, 1024, 6_200), (27, 4, 7, 64, 49_153), (28, 8, 60, 1024, 1_537), (28, 10, 300, 100, 20_000)])
def test_estimate_routes(c, w, k, g, n_hosts):
    from paper_1812_00282_amd import _lib, learned as L

    rng = np.random.default_rng(c * 1000 + g)
    cfg = Config(c, w, k, g, seed_a=5, seed_b=6)
    gpu, ref = _pair(cfg)
    hosts = rng.integers(0, 2**32, n_hosts, dtype=np.uint64).astype(np.uint32)
    some = hosts[rng.permutation(n_hosts)[:200]]
    for t in range(4):
        p = _stream(rng, 60_000 if c > 10 else 50, some if c > 20 else hosts, 2**32)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    gpu.plan(hosts)
    for kp in sorted({1, 3, k}):
        want = kp == k
        _, r_live, r_hist = ref.estimate(hosts, kprime=kp, want_hist=want)
        one, live, hist = gpu.estimate(hosts, kprime=kp, want_hist=want, partitioned=True)
        est, plive, phist = gpu.estimate_run(kp, want_hist=want)
        np.testing.assert_array_equal(_u32(live), r_live)
        np.testing.assert_array_equal(_u32(plive), r_live)
        assert torch.equal(one, est)
        if want:
            np.testing.assert_array_equal(_u32(hist), r_hist)
            assert torch.equal(hist, phist)
        dlive = gpu.estimate(hosts, kprime=kp)[1]
        assert torch.equal(live, dlive)
    if k + 3 <= _lib.MLP_FEATURES:
        gen = torch.Generator().manual_seed(k)
        wts = L.pack((torch.randn(_lib.MLP_PARAMS, generator=gen) * 0.05).cuda(), L.new_weights())
        d, dcf = L.estimate_learned(gpu, hosts, wts)
        for e, cf in (L.estimate_learned(gpu, hosts, wts, partitioned=True), L.estimate_learned_run(gpu, wts)):
            assert torch.equal(d, e) and torch.equal(dcf, cf)


# Streaming kernels with the exact width at compile time: every width, a pool
# of one group and one with a ragged last round, blocks shorter than a group
# and blocks that cut groups, both counters, census and bitmap (live counts).
@pytest.mark.parametrize("w", [1, 2, 3, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15])
@pytest.mark.parametrize("counter,c", [(0, 5), (0, 14), (1, 5), (1, 14)])
def test_exact_width_streams(w, counter, c):
    k = (1 << w) - 1 if counter else ((1 << w) - 1) // 2
    if k < 1:
        pytest.skip("a 1-bit AT has no window")
    k = min(k, 16 if c == 5 else 5000)
    rng = np.random.default_rng(w * 10 + counter)
    gpu, ref = _pair(Config(c, w, k, 64, seed_a=1, seed_b=2, counter=counter, partition=w & 1))
    hosts = rng.integers(0, 2**32, 300, dtype=np.uint64).astype(np.uint32)
    for t in range(min(2 * k + 3, 40)):
        p = _stream(rng, 40 if c == 5 else 2000, hosts, 5000)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
        if t % 4 == 3 or t < 3:
            _check_state(gpu, ref, f"slice {t}")
            np.testing.assert_array_equal(gpu.census(), ref.census())
            np.testing.assert_array_equal(_u32(gpu.estimate(hosts)[1]), ref.estimate(hosts)[1])


# Batch members on both sides of the rule that sends lookups through LDS, with
# windows of all kinds, against the single-sketch calls; eager and replayed, and
# with hosts set again after the capture.
def test_batch_sliced_members():
    from paper_1812_00282_amd.batch import Batch
    from paper_1812_00282_amd.sketch import Sketch

    geo = [(16, 8, 60, 1024, 3000), (20, 7, 60, 1000, 4001), (21, 16, 200, 2048, 1500), (23, 8, 9, 300, 30_011),
           (12, 4, 7, 33, 70_000), (24, 8, 60, 1024, 2500), (18, 8, 60, 100, 50)]
    cfgs = [Config(c, w, k, g, seed_a=c, seed_b=w) for c, w, k, g, _ in geo]
    rng = np.random.default_rng(8)
    hosts = [rng.integers(0, 2**32, x[4], dtype=np.uint64).astype(np.uint32) for x in geo]
    kp = [60, 13, 200, 4, 3, 60, 60]
    b = Batch([Sketch(c) for c in cfgs], [20_000] * len(geo), hosts, kprime=kp)
    solo = [Sketch(c) for c in cfgs]
    for t in range(5):
        sl = [_stream(rng, int(rng.integers(1, 20_000)), h, 4000) for h in hosts]
        b.load(sl)
        if t < 2:
            b.slice()
        else:
            if t == 2:
                b.capture()
            b.replay()
        b.synchronize()
        for i, sk in enumerate(solo):
            sk.ingest(sl[i])
            sk.close_slice()
            est, live, _ = sk.estimate(hosts[i], kprime=kp[i])
            assert torch.equal(b.live[i], live) and torch.equal(b.est[i], est), (t, i)


# Training takes 32 or 64 samples per workgroup, and beyond 256 workgroups
# several times over: gradients and loss against the FP64 network.
@pytest.mark.parametrize("n", [1, 33, 2048, 2049, 16_385])
def test_training_sample_tiles(n):
    gradient_parity(n)


# The closed form by parts of the bitmap (2^26 ATs and more, window k): two,
# four and eight parts, one lane per host and several, locality blocks of one
# word, of two and more, the last block cut short; with and without live counts.
@pytest.mark.parametrize("c,w,k,g,n_hosts,b", [
    (26, 8, 60, 1024, 3100, 0), (27, 4, 7, 100, 40_003, 0), (28, 8, 60, 1000, 30_000, 0), (28, 4, 3, 7, 500_009, 0),
    (26, 8, 60, 1000, 110_001, 5), (28, 8, 20, 2048, 100_001, 6), (27, 8, 60, 1500, 300_000, 7)])
def test_estimate_by_parts(c, w, k, g, n_hosts, b):
    rng = np.random.default_rng(c * 1000 + g)
    gpu, ref = _pair(Config(c, w, k, g, seed_a=5, seed_b=6, block_log2=b))
    hosts = rng.integers(0, 2**32, n_hosts, dtype=np.uint64).astype(np.uint32)
    some = hosts[:300]
    for t in range(3):
        p = _stream(rng, 200_000, some, 2**32)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    est, live, _ = gpu.estimate(hosts)
    _, r_live, _ = ref.estimate(some)
    np.testing.assert_array_equal(_u32(live)[:300], r_live)
    pieces = [gpu.estimate(hosts[i:i + 300]) for i in range(0, n_hosts, max(300, n_hosts // 20))]   # few hosts: gathered
    for j, (e, lv, _) in enumerate(pieces):
        i = j * max(300, n_hosts // 20)
        assert torch.equal(live[i:i + 300], lv) and torch.equal(est[i:i + 300], e)
    alone, _, _ = gpu.estimate(hosts, want_live=False)
    assert torch.equal(est, alone)


# The host list's own buffer as the live counts' or the estimates' output, at a
# size that is otherwise answered by parts and at one that is not.
@pytest.mark.parametrize("n_hosts", [300, 3100])
def test_estimate_over_its_hosts(n_hosts):
    rng = np.random.default_rng(n_hosts)
    gpu = Sketch(Config(26, 8, 60, 1024, seed_a=5, seed_b=6))
    hosts = torch.from_numpy(rng.integers(0, 2**32, n_hosts, dtype=np.uint64).astype(np.uint32).view(np.int32)).cuda()
    gpu.ingest(_stream(rng, 200_000, hosts.cpu().numpy().view(np.uint32)[:300], 2**32))
    gpu.close_slice()
    est, live, _ = gpu.estimate(hosts)
    over = hosts.clone()
    e, _, _ = gpu.estimate(over, out=(torch.empty_like(est), over, None))
    assert torch.equal(over, live) and torch.equal(e, est)
    over = hosts.clone()
    gpu.estimate(over, out=(over.view(torch.float32), None, None))
    assert torch.equal(over.view(torch.float32), est)
