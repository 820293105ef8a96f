"""GPU parity where the k-th largest magnitude is zero or next to it: gradients that are mostly zeros of both signs, flat and
per tensor, whose zeros the streaming pass counts instead of listing.  Against the CPU oracle, bit for bit."""
import numpy as np
import pytest

from oracle import oracle
from paper_2305_12201_amd import binding, workloads
from tests import test_gpu_multilevel as levels
from tests.gpu_util import check

pytestmark = pytest.mark.gpu


def mostly_zeros(n, share, seed):
    """`share` of the entries Normal(0, 1e-3), in runs of 650 or alone; the others +0 or -0."""
    rng = np.random.default_rng(seed)
    v = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    live = np.repeat(rng.random(n // 650 + 1) < share, 650)[:n] if seed % 2 else rng.random(n) < share
    return np.where(live, v, np.where(rng.random(n) < 0.5, np.float32(0.0), np.float32(-0.0))).astype(np.float32)


@pytest.mark.parametrize("n", [20_000, 200_000, 1_000_003])
@pytest.mark.parametrize("cfs,commit", [([10.0], 0), ([20.0], 0), ([21.0], 0), ([4.0, 100.0], 0), ([4.0, 100.0], 1), ([2.0, 19.0, 300.0], 1)])
def test_flat(n, cfs, commit):
    for seed in (1, 2):
        g = mostly_zeros(n, 0.05, seed)
        check(g, np.where(g == 0, g, np.float32(0)), cfs, commit, what=f"n {n}, CFs {cfs}, seed {seed}")
    check(g, np.zeros(n, np.float32), cfs, commit, flags=binding.FLAG_FORCE_FALLBACK, what="forced")


def test_threshold_on_either_side_of_zero():
    """Exactly, one fewer and one more entries than there are non-zero ones; nothing but zeros."""
    n, live = 300_000, 3000
    for count in (live - 1, live, live + 1, 0):
        g = np.zeros(n, np.float32)
        g[np.random.default_rng(count).permutation(n)[:count]] = workloads.normal_gradient(max(count, 1), 1e-3, seed=3)[:count]
        check(g, np.zeros(n, np.float32), [100.0], what=f"{count} non-zero")


@pytest.mark.parametrize("cfs,commit", [([10.0], 0), ([5.0, 40.0], 1)])
def test_tensors(cfs, commit):
    sizes = [9000, 8192, 131_072, 64, 40_004, 650_000, 16_384, 300_000]
    g = mostly_zeros(sum(sizes), 0.05, 3)
    check(g, np.zeros_like(g), cfs, commit, workloads.offsets_of(sizes), what=f"tensors, CFs {cfs}")


def test_second_level():
    n = 400_000
    val = mostly_zeros(n, 0.05, 2)
    idx = (3 * np.arange(n, dtype=np.int64)).astype(np.int32)
    res = np.full(3 * n, 0.5, np.float32)
    res[idx] = 0.0
    for rel in (10.0, 30.0):
        levels.check_recompress(idx, val, rel, res, None, what=f"rel {rel}")
