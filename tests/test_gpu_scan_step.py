"""GPU parity of the calls that have a scan step of their own, those of more than 6144 tiles of 8192 elements (smaller ones
resolve the threshold and the offsets in the emit step), in all their forms, against the CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2305_12201_amd import binding, workloads
from tests import test_gpu_multilevel as levels
from tests import test_gpu_randomk as randomk
from tests import test_gpu_threshold as threshold
from tests.gpu_util import assert_same, gpu_compress, oracle_compress

pytestmark = [pytest.mark.gpu, pytest.mark.fullsize, pytest.mark.timeout(300)]

LIMIT = 6144 * 8192
FB, NC = binding.FLAG_FORCE_FALLBACK, binding.FLAG_NO_COMMIT


@pytest.fixture(scope="module")
def inputs():
    n = LIMIT + 20_003
    return workloads.normal_gradient(n, 1e-3, seed=1), workloads.normal_gradient(n, 1e-4, seed=2)


def check_all_flags(g, r, cfs, commit, seg, run, ref, what):
    """The ordinary call, the exact route and the call without commit share one oracle result."""
    without = ref[3].copy()
    without[ref[0]] = ref[1]
    for flags, res in ((0, ref[3]), (FB, ref[3]), (NC, without)):
        got = run(g, r, cfs, commit, seg, flags)
        assert got[4]["internal_error"] == 0, what
        assert_same(got, (ref[0], ref[1], ref[2], res), f"{what}, flags {flags}")


@pytest.mark.parametrize("n", [LIMIT, LIMIT + 1])
def test_topk_on_both_sides_of_the_limit(inputs, n):
    g, r = inputs[0][:n], inputs[1][:n]
    check_all_flags(g, r, [20.0], 0, None, gpu_compress, oracle_compress(g, r, [20.0]), f"n {n}")


def test_tensors(inputs):
    """One tensor of several slices of the scan (4096 tiles each), small ones, and some of one tile and a few."""
    g, r = inputs
    off = workloads.offsets_of([34_000_007, 64, 1_200_001, 8_193, 5, g.size - 35_208_270])
    check_all_flags(g, r, [20.0, 300.0], 1, off, gpu_compress, oracle_compress(g, r, [20.0, 300.0], 1, off), "tensors")


def test_randomk(inputs):
    g, r = inputs
    off = workloads.offsets_of([36_000_001, 700, g.size - 36_000_701])
    for cfs, commit, seg in (([10.0], 0, None), ([10.0, 50.0], 0, off)):
        res = r.copy()
        ref = (*oracle.randomk_compress(g, res, cfs, 11, commit, seg), res)
        check_all_flags(g, r, cfs, commit, seg, lambda a, b, c, d, e, f: randomk.gpu_randomk(a, b, c, 11, d, e, f), ref, "Random-k")


def test_threshold_that_fits_and_one_too_few(inputs):
    g, r = inputs
    count = threshold.check(g, r, 2.5e-3, what="fits")
    threshold.check(g, r, 2.5e-3, capacity=count, what="exactly")
    threshold.check(g, r, 2.5e-3, capacity=count - 1, what="one too few")


def test_second_level(inputs):
    val = inputs[0]
    idx = (2 * np.arange(val.size, dtype=np.int64) + 1).astype(np.int32)
    res = np.full(2 * val.size + 5, 0.25, np.float32)
    res[idx] = 0.0
    ref_res = res.copy()
    ref = oracle.recompress(idx, val, 10.0, ref_res)
    for flags in (0, FB):
        levels.assert_recompress_same(levels.gpu_recompress(idx, val, 10.0, res, flags=flags), ref, ref_res, val.size, f"flat, flags {flags}")
    counts = [36_000_001, 700, val.size - 36_000_701]
    levels.check_recompress(idx, val, 10.0, None, counts, what="tensors")
