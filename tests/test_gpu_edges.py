"""Edges of the estimate calls: launches past a grid's limit, workspaces between
two layouts, outputs over the host list."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1812_00282_amd import _lib  # noqa: E402
from paper_1812_00282_amd.sketch import Config, Sketch  # noqa: E402
from test_gpu_parity import _pair, _tol  # noqa: E402

pytestmark = pytest.mark.gpu


def _hosts(rng, n):
    return rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)


def _packets(rng, n, hosts):
    return np.stack([hosts[rng.integers(0, hosts.size, n)], _hosts(rng, n)], 1)


def test_windows_of_2_24_hosts():
    """One host per workgroup (rows of 8191 distances) and 2^24 hosts: more
    workgroups of 256 threads than one grid takes."""
    k, n = 8191, 2**24
    rng = np.random.default_rng(24)
    gpu, ref = _pair(Config(14, 14, k, 1, seed_a=1, seed_b=2))
    hosts = torch.randint(-2**31, 2**31, (n,), device="cuda", dtype=torch.int64,
                          generator=torch.Generator("cuda").manual_seed(1)).to(torch.int32)
    for t in range(3):
        p = _packets(rng, 3000, hosts[:2000].cpu().numpy().view(np.uint32))
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    est = gpu.estimate_windows(hosts, [1, k])
    for j, kp in enumerate((1, k)):
        one, _, _ = gpu.estimate(hosts, kprime=kp)
        assert torch.equal(est[:, j], one), kp
        few = torch.cat([hosts[:500], hosts[-500:]]).cpu().numpy().view(np.uint32)
        r_est, _, _ = ref.estimate(few, kprime=kp)
        got = torch.cat([est[:500, j], est[-500:, j]]).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - r_est) <= _tol(r_est, ref.g)), kp


def test_run_needs_the_plans_workspace():
    """A plan may be laid out with fewer hosts per subgroup, and more run padding,
    than the least workspace a plan may be given holds: a run that states less
    than its plan's layout is refused, one that states all of it is answered."""
    rng = np.random.default_rng(5)
    n = 20_011                                   # 742 subgroups of 27, not 527 of 38
    gpu = Sketch(Config(28, 8, 60, 1024, seed_a=3, seed_b=4))
    hosts = _hosts(rng, n)
    gpu.ingest(_packets(rng, 50_000, hosts[:300]))
    gpu.close_slice()
    full = gpu.workspace_bytes(n)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    h = torch.from_numpy(hosts.view(np.int32)).cuda()
    lib, est = _lib.lib(), torch.empty(n, dtype=torch.float32, device="cuda")
    _lib.check(lib.vate_estimate_plan(gpu.handle, h.data_ptr(), n, ws.data_ptr(), full, None), gpu.handle)

    def run(stated):
        return lib.vate_estimate_run(gpu.handle, n, 60, est.data_ptr(), None, None, ws.data_ptr(), stated, None)

    assert run(full - 256) == _lib.VATE_E_INVAL
    _lib.check(run(full), gpu.handle)
    torch.cuda.synchronize()
    assert torch.equal(est, gpu.estimate(hosts)[0])
    # planned with less: the larger subgroups' layout, which then is enough
    refused, least = 0, full
    while least - refused > 256:
        mid = (refused + least) // 512 * 256
        if lib.vate_estimate_plan(gpu.handle, h.data_ptr(), n, ws.data_ptr(), mid, None) == _lib.VATE_OK:
            least = mid
        else:
            refused = mid
    _lib.check(lib.vate_estimate_plan(gpu.handle, h.data_ptr(), n, ws.data_ptr(), least, None), gpu.handle)
    assert least < full
    _lib.check(run(least), gpu.handle)
    torch.cuda.synchronize()
    assert torch.equal(est, gpu.estimate(hosts)[0])


@pytest.mark.parametrize("at", [0, 1000, 290_000])
def test_outputs_over_the_host_list(at):
    """The calls with a workspace read the whole host list before they write: an
    output buffer may hold it, here from word `at` on."""
    from paper_1812_00282_amd import learned as L

    rng = np.random.default_rng(at)
    n, k = 300_000, 60
    gpu = Sketch(Config(16, 8, k, 64, seed_a=3, seed_b=4))
    hosts = torch.from_numpy(_hosts(rng, n).view(np.int32)).cuda()
    gpu.ingest(_packets(rng, 50_000, hosts.cpu().numpy().view(np.uint32)))
    gpu.close_slice()
    wts = L.pack((torch.randn(_lib.MLP_PARAMS, generator=torch.Generator().manual_seed(1)) * 0.05).cuda(),
                 L.new_weights())
    ws = torch.empty(gpu.workspace_bytes(n), dtype=torch.uint8, device="cuda")
    lib = _lib.lib()

    def over(words):                             # a buffer of that many words with the host list in it
        b = torch.zeros(max(words, at + n), dtype=torch.int32, device="cuda")
        b[at:at + n] = hosts
        return b, b.data_ptr() + 4 * at

    est, live, hist = gpu.estimate(hosts, kprime=7, want_hist=True)
    free = torch.empty(n, dtype=torch.float32, device="cuda")
    for shape, which in ((n, "est"), (n, "live"), (n * (k + 1), "hist")):
        b, h = over(shape)
        e, lv, hi = (b.data_ptr() if which == x else None for x in ("est", "live", "hist"))
        _lib.check(lib.vate_estimate_ws(gpu.handle, h, n, 7, e or free.data_ptr(), lv, hi, ws.data_ptr(), ws.numel(),
                                        None), gpu.handle)
        want = {"est": est.view(torch.int32), "live": live, "hist": hist}[which].reshape(-1)
        assert torch.equal(b[:shape], want), which
    kps = np.array([1, 7, 59, 60], dtype=np.uint32)
    want = gpu.estimate_windows(hosts, kps)
    b, h = over(4 * n)
    _lib.check(lib.vate_estimate_multi_ws(gpu.handle, h, n, kps.ctypes.data, 4, b.data_ptr(), ws.data_ptr(),
                                          ws.numel(), None), gpu.handle)
    assert torch.equal(b[:4 * n].view(torch.float32).reshape(n, 4), want)
    learned, cf = L.estimate_learned(gpu, hosts, wts)
    b, h = over(n)
    _lib.check(lib.vate_estimate_learned_ws(gpu.handle, h, n, wts.data_ptr(), b.data_ptr(), free.data_ptr(),
                                            ws.data_ptr(), ws.numel(), None), gpu.handle)
    assert torch.equal(b[:n].view(torch.float32), learned) and torch.equal(free, cf)


# Census workgroups add into the census itself or into partial censuses: 256
# workgroups and more, 16384 additions and more, windows at the LDS histogram's
# limit and beyond, for every container, exact widths and both counters.
@pytest.mark.parametrize("c,w,k,counter", [
    (22, 8, 60, 0), (23, 8, 60, 0), (22, 7, 32, 0), (22, 7, 33, 0), (21, 16, 300, 0), (22, 16, 300, 0), (22, 4, 7, 0),
    (23, 4, 7, 1), (16, 13, 4000, 0), (16, 14, 4096, 0), (16, 14, 4097, 0), (21, 9, 300, 1), (22, 9, 300, 1)])
def test_census_additions(c, w, k, counter):
    rng = np.random.default_rng(c * 1000 + k)
    gpu, ref = _pair(Config(c, w, k, 64, seed_a=1, seed_b=2, counter=counter))
    hosts = _hosts(rng, 3000)
    for t in range(4):
        p = _packets(rng, 60_000, hosts)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
        np.testing.assert_array_equal(gpu.census(), ref.census())
    _, r_live, _ = ref.estimate(hosts[:300], kprime=max(1, k // 2))
    live = gpu.estimate(hosts[:300], kprime=max(1, k // 2))[1]
    np.testing.assert_array_equal(live.cpu().numpy().view(np.uint32), r_live)


# Lookups that fill their slots and lookups that don't, on pools from those whose
# bits a cache line holds to the largest that goes through LDS: gathered, or by
# slices with 16 or 32 VATs a thread, one round of hosts per workgroup or several.
@pytest.mark.parametrize("c,w,k,g,n_hosts", [
    (10, 8, 60, 1024, 20_000), (13, 8, 60, 1024, 40_000), (16, 4, 7, 128, 130_000), (16, 8, 60, 100, 130_000),
    (18, 7, 60, 16, 400_000), (18, 8, 60, 24, 300_000), (20, 8, 60, 5, 500_000), (20, 16, 300, 64, 60_000),
    (21, 8, 60, 8, 700_000), (21, 8, 60, 17, 500_000), (22, 8, 60, 12, 600_000), (22, 10, 300, 400, 50_000),
    (23, 8, 60, 16, 900_000), (23, 8, 60, 128, 130_000), (23, 4, 7, 200, 130_000)])
def test_lookups_by_slots(c, w, k, g, n_hosts):
    rng = np.random.default_rng(c * 1000 + g)
    gpu, ref = _pair(Config(c, w, k, g, seed_a=5, seed_b=6))
    hosts = _hosts(rng, n_hosts)
    for t in range(3):
        p = _packets(rng, min(200_000, 2**c // 8), hosts)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    few = np.r_[hosts[:700], hosts[-700:]]
    pick = lambda x: torch.cat([x[:700], x[-700:]]).cpu().numpy()
    kps = sorted({1, 2, k})
    windows = gpu.estimate_windows(hosts, kps)
    for j, kp in enumerate(kps):
        r_est, r_live, r_hist = ref.estimate(few, kprime=kp, want_hist=k <= 256)
        est, live, hist = gpu.estimate(hosts, kprime=kp, want_hist=k <= 256)
        np.testing.assert_array_equal(pick(live).view(np.uint32), r_live)
        assert np.all(np.abs(pick(est).astype(np.float64) - r_est) <= _tol(r_est, g))
        if k <= 256:
            np.testing.assert_array_equal(pick(hist).view(np.uint32), r_hist)
        one, lone, _ = gpu.estimate(hosts, kprime=kp)
        assert torch.equal(one, est) and torch.equal(lone, live) and torch.equal(windows[:, j], est)


# One lane per host: many hosts with fewer VATs than four lanes hold; both sides
# of the rule, k and below, every kind of counter.
@pytest.mark.parametrize("c,w,g,k,n_hosts,b", [
    (12, 8, 1, 60, 131_073, 0), (24, 8, 63, 60, 140_001, 0), (24, 8, 64, 60, 140_001, 0), (25, 4, 16, 7, 200_003, 0),
    (24, 7, 17, 60, 131_072, 0), (24, 16, 33, 300, 104_000, 0), (22, 8, 40, 60, 150_001, 3)])
def test_one_lane_per_host(c, w, g, k, n_hosts, b):
    rng = np.random.default_rng(c * 1000 + g)
    gpu, ref = _pair(Config(c, w, k, g, seed_a=7, seed_b=8, block_log2=b))
    hosts = _hosts(rng, n_hosts)
    for t in range(3):
        p = _packets(rng, 100_000, hosts)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    for kp in sorted({1, 2, k}):
        r_est, r_live, _ = ref.estimate(hosts, kprime=kp)
        est, live, _ = gpu.estimate(hosts, kprime=kp)
        np.testing.assert_array_equal(live.cpu().numpy().view(np.uint32), r_live)
        assert np.all(np.abs(est.cpu().numpy().astype(np.float64) - r_est) <= _tol(r_est, g))


# Gathers per host from which the bitmap is taken by parts, and one fewer: two,
# four and eight parts, VATs and blocks of one, two and eight words.
@pytest.mark.parametrize("c,g,n_hosts,b", [
    (26, 2, 900_000, 0), (26, 3, 600_001, 0), (27, 3, 600_001, 0), (28, 4, 500_003, 0), (28, 5, 400_001, 0),
    (28, 33, 60_000, 0), (27, 70, 600_001, 5), (27, 100, 500_001, 5), (28, 300, 400_001, 6), (28, 330, 300_000, 6),
    (27, 300, 800_001, 8), (28, 600, 530_000, 8), (26, 16, 200_001, 3), (26, 24, 200_001, 3), (28, 20, 200_000, 1),
    (28, 100, 50_000, 3)])
def test_few_gathers_by_parts(c, g, n_hosts, b):
    rng = np.random.default_rng(c * 1000 + g)
    gpu, ref = _pair(Config(c, 4, 7, g, seed_a=9, seed_b=10, block_log2=b))
    hosts = _hosts(rng, n_hosts)
    for t in range(3):
        p = _packets(rng, 300_000, hosts[:4000])
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    est, live, _ = gpu.estimate(hosts)
    few = np.r_[hosts[:4000], hosts[-300:]]
    r_est, r_live, _ = ref.estimate(few)
    pick = lambda x: torch.cat([x[:4000], x[-300:]]).cpu().numpy()
    np.testing.assert_array_equal(pick(live).view(np.uint32), r_live)
    assert np.all(np.abs(pick(est).astype(np.float64) - r_est) <= _tol(r_est, g))
    for i in range(0, n_hosts, 40_000):                    # few hosts: gathered
        e, lv, _ = gpu.estimate(hosts[i:i + 2000])
        assert torch.equal(live[i:i + 2000], lv) and torch.equal(est[i:i + 2000], e)


# Histograms and windows of many hosts with few VATs: 16 to 256 hosts per
# workgroup, rows that fit fewer, the remainder of a workgroup's hosts.
@pytest.mark.parametrize("c,w,k,g,n_hosts,counter", [
    (18, 8, 60, 1, 400_003, 0), (24, 8, 60, 20, 300_001, 0), (24, 4, 7, 60, 200_001, 0), (25, 8, 61, 128, 120_001, 0),
    (24, 16, 256, 9, 180_001, 0), (22, 7, 60, 16, 500_000, 0), (24, 8, 59, 300, 70_001, 1), (24, 16, 100, 40, 20_000, 0)])
def test_many_hosts_per_workgroup(c, w, k, g, n_hosts, counter):
    rng = np.random.default_rng(c * 1000 + g)
    gpu, ref = _pair(Config(c, w, k, g, seed_a=7, seed_b=8, counter=counter))
    hosts = _hosts(rng, n_hosts)
    for t in range(3):
        p = _packets(rng, 200_000, hosts)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    few = np.r_[hosts[:1500], hosts[-1500:]]
    pick = lambda x: torch.cat([x[:1500], x[-1500:]]).cpu().numpy()
    kps = sorted({1, 2, 3, k - 1, k})
    windows = gpu.estimate_windows(hosts, kps)
    for j, kp in enumerate(kps):
        r_est, r_live, r_hist = ref.estimate(few, kprime=kp, want_hist=True)
        est, live, hist = gpu.estimate(hosts, kprime=kp, want_hist=True)
        np.testing.assert_array_equal(pick(live).view(np.uint32), r_live)
        np.testing.assert_array_equal(pick(hist).view(np.uint32), r_hist)
        assert np.all(np.abs(pick(est).astype(np.float64) - r_est) <= _tol(r_est, g))
        assert torch.equal(hist.sum(1), torch.full((n_hosts,), g, device="cuda"))
        one, lone, _ = gpu.estimate(hosts, kprime=kp)
        assert torch.equal(one, est) and torch.equal(lone, live) and torch.equal(windows[:, j], est)


# Counters set by swaps or put without a look, by how many packets meet on a word:
# both sides of the words' and the packets' limits, one packet a thread and four,
# hot counters, widths whose counters straddle words, both kinds of counter.
@pytest.mark.parametrize("c,w,k,counter,n", [
    (16, 4, 2, 0, 8191), (16, 4, 2, 0, 8192), (16, 4, 7, 0, 2_097_152), (18, 4, 7, 0, 40_000), (19, 4, 7, 1, 300_001),
    (14, 3, 3, 0, 1536), (18, 3, 3, 0, 262_145), (16, 7, 60, 0, 262_143), (16, 7, 60, 0, 262_144), (15, 10, 300, 1, 30_001),
    (17, 15, 300, 0, 262_144), (22, 10, 300, 0, 262_145), (10, 4, 7, 0, 5)])
def test_ingest_words(c, w, k, counter, n):
    rng = np.random.default_rng(c * 1000 + w)
    gpu, ref = _pair(Config(c, w, k, 64, seed_a=3, seed_b=4, counter=counter))
    hosts = _hosts(rng, 20_000)
    for t in range(3):
        p = _packets(rng, n, hosts)
        p[rng.random(n) < 0.2] = (hosts[0], 7)
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
        pool = gpu.read_state()[0]
        assert np.array_equal(pool, ref.packed_pool()), t


def test_batch_ingest_words():
    from paper_1812_00282_amd.batch import Batch

    geo = [(16, 4, 7, 200_000), (18, 3, 3, 131_072), (18, 10, 300, 131_073), (14, 7, 60, 20_000), (20, 4, 7, 150_000)]
    rng = np.random.default_rng(4)
    pairs = [_pair(Config(c, w, k, 64, seed_a=c, seed_b=w)) for c, w, k, _ in geo]
    hosts = [_hosts(rng, 5000) for _ in geo]
    b = Batch([g for g, _ in pairs], [n for *_, n in geo], hosts)
    for t in range(3):
        sl = [_packets(rng, n, h) for (*_, n), h in zip(geo, hosts)]
        b.load(sl)
        b.slice()
        b.synchronize()
        for (gpu, ref), p in zip(pairs, sl):
            ref.ingest(p)
            ref.close_slice()
            assert np.array_equal(gpu.read_state()[0], ref.packed_pool()), t


# Hosts set again after the capture: a list that would go through LDS in a graph
# that has no such launch is gathered, and a graph that has one gathers a short list.
@pytest.mark.parametrize("first,then", [(100, 4000), (4000, 100)])
def test_batch_hosts_set_after_capture(first, then):
    from paper_1812_00282_amd.batch import Batch

    rng = np.random.default_rng(first)
    pairs = [_pair(Config(c, 8, 60, 1024, seed_a=c, seed_b=2)) for c in (20, 24)]
    lists = [_hosts(rng, first), _hosts(rng, 300)]
    b = Batch([g for g, _ in pairs], [20_000] * 2, lists)

    def slices(step):
        sl = [_packets(rng, 20_000, h[:50]) for h in lists]
        b.load(sl)
        step()
        b.synchronize()
        for (_, ref), p in zip(pairs, sl):
            ref.ingest(p)
            ref.close_slice()

    slices(b.slice)
    b.capture()
    slices(b.replay)
    lists[0] = _hosts(rng, then)
    h = torch.from_numpy(lists[0].view(np.int32)).cuda()
    est = torch.full((then,), float("nan"), device="cuda")
    live = torch.full((then,), -1, dtype=torch.int32, device="cuda")
    assert _lib.lib().vate_batch_set_io(b._h, 0, b.pairs[0].data_ptr(), b.pairs[0].shape[0], h.data_ptr(), then, 60,
                                        est.data_ptr(), live.data_ptr()) == _lib.VATE_OK
    for _ in range(3):
        slices(b.replay)
        for (_, ref), hosts, lv, e in ((pairs[0], lists[0], live, est), (pairs[1], lists[1], b.live[1], b.est[1])):
            r_est, r_live, _ = ref.estimate(hosts)
            np.testing.assert_array_equal(lv.cpu().numpy().view(np.uint32), r_live)
            assert np.all(np.abs(e.cpu().numpy().astype(np.float64) - r_est) <= _tol(r_est, 1024))
