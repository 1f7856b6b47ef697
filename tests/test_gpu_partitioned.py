"""The partitioned lookups at sizes whose calls take them: 3 * 2^47 lookups times
ATs (doubling beyond 2^28 ATs), pools of 2^23 ATs and more.  Every geometry
against the CPU oracle and bit for bit against the gathers."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1812_00282_amd import _lib, learned as L  # noqa: E402
from paper_1812_00282_amd.sketch import Config, Sketch  # noqa: E402
from test_gpu_parity import _pair, _tol, _u32  # noqa: E402

pytestmark = pytest.mark.gpu


def _hosts(rng, n):
    return rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)


def _packets(rng, n, hosts):
    return np.stack([hosts[rng.integers(0, hosts.size, n)], _hosts(rng, n)], 1)


def _least(c):
    """Lookups from which a pool of 2^c ATs is partitioned."""
    return 3 << 47 >> c if c <= 28 else 3 << 19 << (c - 28)


def _learned_weights():
    gen = torch.Generator().manual_seed(3)
    return L.pack((torch.randn(_lib.MLP_PARAMS, generator=gen) * 0.05).cuda(), L.new_weights())


@pytest.mark.parametrize("c,w,k,g,partition,counter,n_hosts", [
    (28, 16, 300, 1024, 0, 0, 1_700),     # 16-bit ATs, 16-bit distances, 7 hosts per subgroup
    (26, 16, 129, 64, 1, 0, 100_001),     # 16-bit ATs, Fig. 5's blocks, hundreds of hosts per subgroup
    (27, 8, 60, 33, 1, 0, 100_003),       # g does not divide the workgroup size, below a wavefront
    (27, 4, 7, 32, 0, 0, 100_000),        # nibbles; g divides it, below a wavefront
    (28, 8, 60, 1, 0, 0, 1_700_003),      # one VAT per host, as many hosts per subgroup as histograms fit
    (28, 8, 60, 3, 1, 1, 530_001),        # byte recorders, three VATs
    (27, 9, 300, 100, 0, 1, 32_001),      # exact 9-bit recorders, 16-bit distances
    (25, 8, 100, 2048, 0, 0, 6_200),      # blocks shorter than a slice: a block lookup per AT
    (28, 8, 60, 256, 0, 0, 300_000),      # 147 hosts per subgroup, two subgroups per finalize workgroup
    (26, 7, 60, 1024, 1, 0, 6_301),       # exact 7-bit ATs, a ragged last subgroup
    (24, 8, 61, 1024, 0, 0, 24_700),      # 16 slices, odd k
    (29, 4, 7, 1024, 0, 0, 3_100),        # beyond 2^28 ATs: histograms partitioned, the closed form by parts
])
def test_partitioned_geometries_across_the_rule(c, w, k, g, partition, counter, n_hosts):
    assert n_hosts * g >= _least(c) and c >= 23
    rng = np.random.default_rng(c * 1000 + k + g)
    gpu, ref = _pair(Config(c, w, k, g, partition=partition, counter=counter, seed_a=c + g, seed_b=k))
    hosts = _hosts(rng, n_hosts)
    for t in range(3):
        p = _packets(rng, 200_000, hosts[: 1 + n_hosts // 20])
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    few = np.r_[hosts[:400], hosts[n_hosts // 2: n_hosts // 2 + 400], hosts[-400:]]
    pick = lambda x: torch.cat([x[:400], x[n_hosts // 2: n_hosts // 2 + 400], x[-400:]])
    gpu.plan(hosts)
    kps = sorted({1, 2, k})
    windows = gpu.estimate_windows(hosts, kps)
    for j, kp in enumerate(kps):
        hist = kp == k
        r_est, r_live, r_hist = ref.estimate(few, kprime=kp, want_hist=hist)
        est, live, h = gpu.estimate(hosts, kprime=kp, want_hist=hist, partitioned=True)
        np.testing.assert_array_equal(_u32(pick(live)), r_live)
        assert np.all(np.abs(pick(est).cpu().numpy().astype(np.float64) - r_est) <= _tol(r_est, g)), kp
        if hist:
            np.testing.assert_array_equal(_u32(pick(h)), r_hist)
            assert torch.equal(h.sum(1), torch.full((n_hosts,), g, device="cuda"))
            assert torch.equal(h[:, :k].sum(1).to(torch.int32), live)
        one, dlive, _ = gpu.estimate(hosts, kprime=kp)
        assert torch.equal(live, dlive) and torch.equal(est, one)
        assert torch.equal(windows[:, j], est)
        pest, plive, _ = gpu.estimate_run(kp)
        assert torch.equal(plive, live) and torch.equal(pest, est)
    if k + 3 <= _lib.MLP_FEATURES:
        wts = _learned_weights()
        d, dcf = L.estimate_learned(gpu, hosts, wts)
        for e, cf in (L.estimate_learned(gpu, hosts, wts, partitioned=True), L.estimate_learned_run(gpu, wts)):
            assert torch.equal(d, e) and torch.equal(dcf, cf)


# A plan on such a pool outlives slices and other hosts' estimates in other workspaces.
def test_plan_across_the_rule():
    rng = np.random.default_rng(11)
    n, g, c = 7001, 1024, 27
    assert n * g >= _least(c)
    gpu, ref = _pair(Config(c, 8, 20, g, partition=1, seed_a=5, seed_b=6))
    hosts, others = _hosts(rng, n), _hosts(rng, n)
    gpu.plan(hosts)
    for t in range(4):
        p = _packets(rng, 100_000, hosts[:500])
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
        gpu.estimate(others, kprime=3, partitioned=True)
        for kp in (3, 20):
            _, live, _ = gpu.estimate_run(kp)
            np.testing.assert_array_equal(_u32(live[:600]), ref.estimate(hosts[:600], kprime=kp)[1])
            assert torch.equal(live, gpu.estimate(hosts, kprime=kp)[1])


# Both sides of the rule beyond 2^28 ATs: the same answers by parts of the bitmap,
# partitioned and gathered.
@pytest.mark.parametrize("n_hosts", [1_000, 3_000, 6_200])
def test_2_30_counters(n_hosts):
    rng = np.random.default_rng(n_hosts)
    gpu = Sketch(Config(30, 4, 7, 1024, seed_a=5, seed_b=6))
    hosts = _hosts(rng, n_hosts)
    for t in range(3):
        gpu.ingest(_packets(rng, 500_000, hosts[:300]))
        gpu.close_slice()
    for kp in (3, 7):
        est, live, hist = gpu.estimate(hosts, kprime=kp, want_hist=True, partitioned=True)
        for e, lv, _ in (gpu.estimate(hosts, kprime=kp), gpu.estimate(hosts, kprime=kp, partitioned=True)):
            assert torch.equal(live, lv) and torch.equal(est, e)
        assert torch.equal(hist[:, :kp].sum(1).to(torch.int32), live)
        for i in range(0, n_hosts, 500):                 # few hosts: gathered
            e, lv, h = gpu.estimate(hosts[i:i + 500], kprime=kp, want_hist=True)
            assert torch.equal(live[i:i + 500], lv) and torch.equal(est[i:i + 500], e)
            assert torch.equal(hist[i:i + 500], h)
    assert int(live.max()) > 0


# The fixed scratch near its limit: 7,800 hosts, whose even subgroups (31) fit it
# by 0.3 MB, 7,850, whose do not; then fewer hosts, another window, in the same array.
def test_noalloc_partitioned():
    rng = np.random.default_rng(9)
    gpu, ref = _pair(Config(28, 8, 60, 1024, seed_a=7, seed_b=8))
    hosts = _hosts(rng, 7_850)
    for t in range(3):
        p = _packets(rng, 300_000, hosts[:400])
        gpu.ingest(p)
        ref.ingest(p)
        gpu.close_slice()
        ref.close_slice()
    lib = _lib.lib()
    for n, kp, hist in ((7_800, 60, True), (1_600, 30, True), (7_850, 2, False), (6_200, 60, False), (7_800, 60, True)):
        assert n * 1024 >= _least(28)
        h = torch.from_numpy(hosts[:n].view(np.int32)).cuda()
        need = ctypes.c_size_t()
        _lib.check(lib.vate_estimate_workspace_bytes(gpu.handle, n, ctypes.byref(need)), gpu.handle)
        est = torch.full((n,), float("nan"), device="cuda")
        live = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        hi = torch.full((n, 61), -1, dtype=torch.int32, device="cuda")
        _lib.check(lib.vate_estimate_noalloc(gpu.handle, h.data_ptr(), n, kp, est.data_ptr(), live.data_ptr(),
                                             hi.data_ptr() if hist else None, None), gpu.handle)
        torch.cuda.synchronize()
        e, lv, dh = gpu.estimate(h, kprime=kp, want_hist=hist)
        assert torch.equal(live, lv) and torch.equal(est, e)
        if hist:
            assert torch.equal(hi, dh)
        np.testing.assert_array_equal(_u32(live[:500]), ref.estimate(hosts[:500], kprime=kp)[1])
