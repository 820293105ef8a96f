"""GPU parity of direct calls, the flat Top-k calls of at most 524,288 elements whose sampling kernel counts all of them, and
of the calls just above that: bins with few entries, with more than a gather list holds, of one key, at either end of the
keys.  Against the CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2305_12201_amd import binding, workloads
from tests import test_gpu_multilevel as levels
from tests.gpu_util import assert_same, check, gpu_compress, oracle_compress

pytestmark = pytest.mark.gpu

LIMIT = 524_288
VALUES = {
    "normal": lambda n, rng: rng.standard_normal(n) * 1e-3,
    "one value": lambda n, rng: rng.choice([-0.25, 0.25], n),
    "few values": lambda n, rng: rng.choice([-0.5, 0.25, 0.125, 1.0], n, p=[0.1, 0.6, 0.2, 0.1]),
    "close together": lambda n, rng: 1.0 + rng.integers(0, 3000, n) * 2.0 ** -23,
    "tiny": lambda n, rng: rng.standard_normal(n) * 1e-41,
    "tiny and ordinary": lambda n, rng: np.where(rng.random(n) < 0.02, rng.standard_normal(n), rng.standard_normal(n) * 1e-20),
    "huge": lambda n, rng: rng.standard_normal(n) * 1e30,
    "infinite": lambda n, rng: np.where(rng.random(n) < 0.3, rng.choice([np.inf, -np.inf], n), rng.standard_normal(n)),
    "NaN": lambda n, rng: np.where(rng.random(n) < 0.01, np.nan, rng.standard_normal(n)),
}


@pytest.mark.parametrize("values", list(VALUES))
@pytest.mark.parametrize("n", [1, 1024, 8193, 65_537, LIMIT, LIMIT + 1])
def test_values(n, values):
    with np.errstate(over="ignore"):
        g = VALUES[values](n, np.random.default_rng(n)).astype(np.float32)
    z = np.zeros(n, np.float32)
    for cfs, commit in (([10.0], 0), ([2.0, 30.0, 1000.0], 1)):
        check(g, z, cfs, commit, what=f"{values}, n {n}, CFs {cfs}")


@pytest.mark.parametrize("cfs,commit", [([1.0], 0), ([1.5, 4.0], 1), ([100.0, 3.0], 0), ([2.0, 3.0, 5.0, 8.0, 300.0], 4)])
def test_iterations_unaligned_without_commit(cfs, commit):
    n = 300_001
    res = workloads.normal_gradient(n, 1e-4, seed=5)
    comp = binding.Compressor(n, cfs, commit)
    buf = torch.zeros(n + 4, dtype=torch.float32, device="cuda")
    r = buf[3:3 + n]
    r.copy_(torch.from_numpy(res))
    for it in range(3):
        g = workloads.resnet_like_gradient(n, seed=it)
        ref = oracle_compress(g, res, cfs, commit)
        without = ref[3].copy()
        without[ref[0]] = ref[1]
        got = gpu_compress(g, res, cfs, commit, flags=binding.FLAG_NO_COMMIT)
        assert_same(got, (ref[0], ref[1], ref[2], without), f"without commit, iteration {it}")
        idx, val, stats = comp(torch.from_numpy(g).cuda(), r)
        assert_same((idx.cpu().numpy(), val.cpu().numpy(), stats.cpu().numpy(), r.cpu().numpy()), ref, f"iteration {it}")
        assert comp.status()["internal_error"] == 0
        res = ref[3]


@pytest.mark.parametrize("k1", [1000, 40_001, LIMIT])
def test_second_level(k1):
    rng = np.random.default_rng(k1)
    idx = (2 * np.arange(k1, dtype=np.int64)).astype(np.int32)
    res = np.full(2 * k1, 0.5, np.float32)
    res[idx] = 0.0
    for val in (rng.standard_normal(k1), rng.choice([-0.25, 0.25, 1.0], k1)):
        for rel in (2.0, 16.0):
            levels.check_recompress(idx, val.astype(np.float32), rel, res, None, what=f"k1 {k1}, rel {rel}")
