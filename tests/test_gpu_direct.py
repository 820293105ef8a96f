"""GPU parity of direct calls, the flat Top-k calls of at most 524,288 elements whose sampling kernel counts all of them, and
of the calls just above that: bins with few entries, with more than a gather list holds, of one key, at either end of the
keys.  Against the CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2305_12201_amd import binding, workloads
from tests import test_gpu_multilevel as levels
from tests.gpu_util import assert_same, check, cut_again, gpu_compress, oracle_compress

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


# bins of 0.27 % in magnitude, or coarser ones, with more than 4096 of 524,288 entries
FULL = {
    "within a tenth": lambda n, rng: rng.choice([-1.0, 1.0], n) * rng.uniform(1e-3, 1.1e-3, n),
    "255 values": lambda n, rng: np.clip(np.round(rng.standard_normal(n) * 20), -127, 127) * 1e-4,
    "one value above others": lambda n, rng: np.where(rng.random(n) < 0.5, 1e-3, rng.standard_normal(n) * 1e-5),
    "denormal": lambda n, rng: rng.integers(-5000, 5000, n) * 2.0 ** -149,
}


@pytest.mark.parametrize("values", list(FULL))
@pytest.mark.parametrize("n", [16_385, 131_072, 262_145, LIMIT])
def test_full_bins(n, values):
    """Several CFs' bins at once, full ones among ordinary ones; units of the last chunk that are not there; a residual."""
    rng = np.random.default_rng(n)
    g = FULL[values](n, rng).astype(np.float32)
    r = np.where(rng.random(n) < 0.1, g, 0.0).astype(np.float32)
    full = 0
    for cfs, commit in (([100.0], 0), ([10.0], 0), ([2.0, 30.0, 1000.0], 0), ([1.5, 2.0, 3.0, 4.0, 5.0, 8.0, 10.0, 1.0], 5)):
        comp = binding.Compressor(n, cfs, commit)
        for res in (np.zeros(n, np.float32), r):
            got = gpu_compress(g, res, cfs, commit, comp=comp)
            full += cut_again(comp.workspace)
            assert_same(got, oracle_compress(g, res, cfs, commit), f"{values}, n {n}, CFs {cfs}")
    assert full or n < LIMIT   # (of the largest size, some are)


def test_full_bins_replayed_and_side_by_side():
    """The queue and the counts of such a call start anew with each replay of a graph, and belong to its workspace."""
    n, cfs = LIMIT - 5, [4.0, 50.0]
    rng = np.random.default_rng(1)
    g = [FULL[v](n, rng).astype(np.float32) for v in ("within a tenth", "255 values")]
    dg = [torch.from_numpy(x).cuda() for x in g]
    comp = [binding.Compressor(n, cfs, 0) for _ in g]
    r = [torch.zeros(n, device="cuda") for _ in g]
    streams, graphs = [torch.cuda.Stream() for _ in g], []
    for i in range(2):
        comp[i](dg[i], r[i])
        torch.cuda.synchronize()
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[i]):
            comp[i](dg[i], r[i])
    res = [np.zeros(n, np.float32) for _ in g]
    for x in r:
        x.zero_()
    torch.cuda.synchronize()
    for it in range(4):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                graphs[i].replay()
        torch.cuda.synchronize()
        for i in range(2):
            ref = oracle_compress(g[i], res[i], cfs)
            assert cut_again(comp[i].workspace)
            assert_same((comp[i].out_idx.cpu().numpy(), comp[i].out_val.cpu().numpy(), comp[i].out_stats.cpu().numpy(), r[i].cpu().numpy()), ref, f"replay {it}")
            res[i] = ref[3]


def test_full_bins_cost():
    """A full bin costs a few waits of the workgroups for each other, 10 to 50 us, and not a walk over all lists by each of them,
    ten times the call."""
    n, times = LIMIT, []
    comp = binding.Compressor(n, [100.0], 0)
    for values in (VALUES["normal"], FULL["within a tenth"]):
        g = torch.from_numpy(values(n, np.random.default_rng(2)).astype(np.float32)).cuda()
        r, ts = torch.zeros(n, device="cuda"), []
        for _ in range(30):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            r.zero_()
            a.record()
            for _ in range(4):
                comp(g, r, flags=binding.FLAG_NO_COMMIT)
                r.zero_()
            b.record()
            b.synchronize()
            ts.append(a.elapsed_time(b))
        times.append(float(np.median(ts)))
    assert times[1] < 4.0 * times[0], times
