"""Kernel variants chosen by size, each at the sizes where it can go wrong,
against the CPU oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1812_00282_amd.sketch import Config  # noqa: E402
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
