"""GPU parity on both sides of the sizes at which a wavefront of the list kernels takes a tile of 8192 elements, half of one or
a quarter, with many and with few selected entries, flat, per tensor and as a second level, in all forms of the call.  Against
the CPU oracle, bit for bit."""
import numpy as np
import pytest

from paper_2305_12201_amd import binding, workloads
from tests import test_gpu_multilevel as levels
from tests import test_gpu_routes as routes
from tests import test_gpu_threshold as threshold
from tests.gpu_util import assert_same, check, gpu_compress, oracle_compress

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

TILE = 8192
FB, NC = binding.FLAG_FORCE_FALLBACK, binding.FLAG_NO_COMMIT


def gradient(n, seed):
    """Normal, a tenth of it a hundred times larger and in one place: sub-tiles without a candidate list among the others."""
    g = workloads.normal_gradient(n, 1e-4, seed=seed)
    g[n // 3:n // 3 + n // 10] *= 100.0
    return g


@pytest.mark.parametrize("cf", [10.0, 20.0, 100.0])
@pytest.mark.parametrize("tiles", [511, 512, 1023, 1024, 1535, 1536, 3071, 3072])
def test_limits(tiles, cf):
    """Quarter tiles with up to 511 tiles (up to 1535 at CF 10 and 20), half tiles with up to 1023 (3071), tiles above: the limits are
    on a bound that is a tile higher than a flat call's own number."""
    n = tiles * TILE - 3
    g, r = gradient(n, tiles), workloads.normal_gradient(n, 1e-5, seed=1)
    ref = oracle_compress(g, r, [cf])
    without = ref[3].copy()
    without[ref[0]] = ref[1]
    for flags, res in ((0, ref[3]), (FB, ref[3]), (NC, without)):
        got = gpu_compress(g, r, [cf], flags=flags)
        assert got[4]["internal_error"] == 0
        assert_same(got, (ref[0], ref[1], ref[2], res), f"{tiles} tiles, CF {cf}, flags {flags}")


@pytest.mark.parametrize("n", [2_000_003, 6_000_001])
def test_forms(n):
    g, r = gradient(n, 7), workloads.normal_gradient(n, 1e-5, seed=8)
    check(g, r, [10.0, 100.0, 1000.0], 1, what="three CFs")
    check(g, r, [3.0, 300.0], 0, workloads.offsets_of([n // 2, 64, 20_001, 300_000, n - n // 2 - 320_065]), what="tensors")
    for cf in (10.0, 200.0):
        routes.check_randomk(g, r, [cf], seed=5, what=f"Random-k, CF {cf}")
    count = threshold.check(g, r, 2e-3, what="threshold that fits")
    threshold.check(g, r, 2e-3, capacity=count - 1, what="threshold, one too few")


@pytest.mark.parametrize("rel", [4.0, 100.0])
def test_second_level(rel):
    n = 5_000_001
    val = gradient(n, 9)
    idx = (2 * np.arange(n, dtype=np.int64)).astype(np.int32)
    res = np.full(2 * n, 0.5, np.float32)
    res[idx] = 0.0
    levels.check_recompress(idx, val, rel, res, None, what=f"rel {rel}")


def test_streamed_messages():
    """1.5 million pairs and more in a call without a scan step, whose message goes through LDS: sub-tiles with and without
    lists, a message that starts off a multiple of four pairs, Random-k, a second level with and without a residual; and a message
    of every second entry, which does not."""
    n = 26_000_003
    g, r = gradient(n, 11), workloads.normal_gradient(n, 1e-5, seed=12)
    off = workloads.offsets_of([1_000_001, 25_000_000, 2])
    for cfs, commit, seg in (([12.0], 0, None), ([3.0], 0, None), ([15.0, 200.0], 0, off), ([2.0], 0, None), ([2.0, 100.0], 0, off)):
        check(g, r, cfs, commit, seg, what=f"CFs {cfs}")
    routes.check_randomk(g, r, [10.0], seed=3, what="Random-k")
    idx = (2 * np.arange(n, dtype=np.int64)).astype(np.int32)
    res = np.full(2 * n, 0.5, np.float32)
    res[idx] = 0.0
    levels.check_recompress(idx, g, 9.0, res, None, what="second level")
