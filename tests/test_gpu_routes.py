"""GPU parity at the edges of the dispatch: sizes, CF counts and value distributions at which a call changes from one
kernel form or route to another, against the CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2305_12201_amd import binding, workloads
from tests.gpu_util import assert_same, check, cut_again, gpu_compress, oracle_compress
from tests.test_gpu_randomk import check as check_randomk

pytestmark = pytest.mark.gpu

FB = binding.FLAG_FORCE_FALLBACK


@pytest.mark.parametrize("n_cf", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("n", [9_001, 300_007])
def test_randomk_forms(n_cf, n):
    """The Random-k pass is compiled for 1, 2, 3, 4 and 8 CFs; a call with five takes the form for eight."""
    cfs = [2.0, 7.5, 10.0, 33.0, 100.0, 160.0, 300.0, 1000.0][:n_cf]
    g = workloads.resnet_like_gradient(n, seed=n)
    r = workloads.normal_gradient(n, 1e-5, seed=n_cf)
    check_randomk(g, r, cfs, seed=n + n_cf, commit=n_cf - 1, what=f"{n_cf} CFs, highest sent")
    check_randomk(g, r, cfs, seed=n - n_cf, commit=0, what=f"{n_cf} CFs, lowest sent")


def _mass(n, seed, share, value, rest):
    """n entries, about `share` of them exactly +-value, the others Normal(0, rest)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    g = (rng.standard_normal(n) * rest).astype(np.float32)
    hit = rng.random(n) < share
    g[hit] = np.where(rng.random(int(hit.sum())) < 0.5, -value, value).astype(np.float32)
    return g


@pytest.mark.parametrize("flags", [0, FB])
@pytest.mark.parametrize("n,share,cf", [(131_073, 0.5, 3.0), (300_007, 0.2, 10.0), (600_011, 0.5, 3.0), (900_007, 0.2, 10.0), (1_200_001, 0.9, 1.5),
                                        (700_001, 0.05, 25.0)])
def test_mass_of_equal_values(n, share, cf, flags):
    """The k-th largest is one of many equal values: its bin holds more entries than a gather list, on the exact route
    after the lists have been collected again too (at the two smallest sizes only there: without the flag the calls are direct)."""
    for value, rest in ((1e-3, 1e-3), (0.0, 1e-3), (np.float32(1.25), 1e-6)):
        g = _mass(n, n, share, value, rest)
        check(g, np.zeros(n, np.float32), [cf], flags=flags, what=f"mass of {value}")
        check(g, np.zeros(n, np.float32), [cf, 4 * cf, 40 * cf], 1, flags=flags, what=f"mass of {value}, three CFs")


@pytest.mark.parametrize("n,direct", [(400_003, True), (700_003, False)])
def test_wide_bracket_is_cut_twice(n, direct):
    """Magnitudes over hundreds of octaves and a mass of equal ones below: bins far wider than 2^11 keys, and still too
    full when they are cut the first time, by the plan step or, in a direct call, by the emit step."""
    rng = np.random.Generator(np.random.PCG64(5))
    g = np.exp(rng.uniform(-80.0, 0.0, n)).astype(np.float32)
    g[rng.random(n) < 0.5] = np.float32(1e-30)
    for cf in (2.0, 2.5, 3.0):
        for cfs in ([cf], [cf, 10.0 * cf]):
            comp = binding.Compressor(n, cfs, 0)
            got = gpu_compress(g, np.zeros(n, np.float32), cfs, 0, comp=comp)
            assert_same(got, oracle_compress(g, np.zeros(n, np.float32), cfs), f"cfs {cfs}")
            if cf != 2.0:
                continue
            # The k-th largest is one of the equal values.  They lie below 2^-48, where one bin of the sample takes in all
            # keys, so the bracket's bins are 2^18 keys wide, the first cut leaves 2^7, and those are as full as before.
            assert got[4]["fallback_segments"] == 1 and got[4]["narrow_fallback_segments"] == 1, got[4]
            assert cut_again(comp.workspace) == direct


@pytest.mark.parametrize("n_cf", [1, 2, 3, 5, 8])
def test_plan_of_every_cf_count(n_cf):
    """The search of the histograms is split over the workgroup in as many ways as there are CFs."""
    n = 900_001
    cfs = [2.0, 5.0, 10.0, 33.0, 100.0, 160.0, 300.0, 1000.0][:n_cf]
    g = workloads.resnet_like_gradient(n, seed=n_cf)
    r = workloads.normal_gradient(n, 1e-5, seed=2)
    for flags in (0, FB):
        check(g, r, cfs, n_cf // 2, flags=flags, what=f"{n_cf} CFs")


def test_some_tensors_take_the_exact_route():
    """Layerwise: tensors of several workgroups, of one, and small ones; some full of equal values, some ordinary."""
    sizes = [700_001, 64, 20_000, 1_100_003, 8_193, 600_000, 5, 70_001]
    off = workloads.offsets_of(sizes)
    n = int(off[-1])
    g = workloads.normal_gradient(n, 1e-3, seed=3)
    for t in (0, 2, 5):
        g[off[t]:off[t + 1]] = _mass(sizes[t], t, 0.6, 1e-3, 1e-4)
    rng = np.random.Generator(np.random.PCG64(9))
    g[off[3]:off[4]] = np.exp(rng.uniform(-80.0, 0.0, sizes[3])).astype(np.float32)
    g[off[3]:off[4]][rng.random(sizes[3]) < 0.5] = np.float32(1e-30)
    r = np.zeros(n, np.float32)
    for flags in (0, FB):
        check(g, r, [2.5], 0, off, flags=flags, what="layerwise, one CF")
        check(g, r, [2.5, 10.0], 1, off, flags=flags, what="layerwise, two CFs")


def test_exact_route_gives_up_a_wait_that_cannot_end():
    """The workgroups of the exact route wait for each other.  With an arrival that never comes every kernel still ends and
    the call reports an internal error; the next call on the same workspace is right again."""
    stall = FB | binding.FLAG_STALL_FALLBACK
    n = 600_001
    g, z = workloads.normal_gradient(n, 1e-3, seed=1), np.zeros(n, np.float32)
    off = workloads.offsets_of([200_000, 5, 8_193, n - 208_198])
    for cfs, commit, seg in (([10.0], 0, None), ([10.0, 100.0, 1000.0], 2, None), ([10.0, 100.0], 0, off)):
        comp = binding.Compressor(n, cfs, commit, seg)
        for run in (lambda r, f: comp(torch.from_numpy(g).cuda(), r, flags=f), lambda r, f: comp.randomk(torch.from_numpy(g).cuda(), r, seed=7, flags=f)):
            run(torch.zeros(n, device="cuda"), stall)
            assert comp.status()["internal_error"] == 1
        got = gpu_compress(g, z, cfs, commit, seg, flags=FB, comp=comp)
        assert got[4]["internal_error"] == 0
        assert_same(got, oracle_compress(g, z, cfs, commit, seg), "the call after")
    with pytest.raises(binding.GravacError):
        comp(torch.from_numpy(g).cuda(), torch.zeros(n, device="cuda"), flags=binding.FLAG_STALL_FALLBACK)


def _coarse(x, bits):
    """float32 values with only the top `bits` bits of the mantissa: many equal magnitudes, 2^(23 - bits) keys apart."""
    return (np.ascontiguousarray(x).view(np.uint32) & np.uint32(0xFFFFFFFF << (23 - bits) & 0xFFFFFFFF)).view(np.float32)


@pytest.mark.parametrize("n,bits", [(250_007, 5), (1_000_003, 7), (2_500_001, 8)])
def test_long_gather_lists(n, bits):
    """Located bins with hundreds to thousands of entries, few distinct keys among them: the gather lists are longer than
    their heads, and ties are spread over many tiles."""
    g = _coarse(workloads.normal_gradient(n, 1e-3, seed=n), bits)
    z = np.zeros(n, np.float32)
    for cf in (3.0, 10.0, 50.0):
        check(g, z, [cf], what=f"cf {cf}")
    check(g, z, [3.0, 10.0, 50.0], 1, what="three CFs")
    sizes = [8_193, n // 3, 100, n - n // 3 - 8_193 - 100]
    check(g, z, [10.0], 0, workloads.offsets_of(sizes), what="layerwise")


@pytest.mark.parametrize("n", [3 * 8_192 + 5, 200_003])
@pytest.mark.parametrize("cf", [1.2, 2.0, 2.8, 4.0, 6.0])
def test_lists_of_many_rounds(n, cf):
    """Sub-tiles with up to 383 listed candidates (the last one, which is ragged, with as many as it has), in buffers on and off a
    16-byte boundary."""
    g = workloads.normal_gradient(n, 1e-3, seed=n)
    r = workloads.normal_gradient(n, 1e-4, seed=n + 1)
    check(g, r, [cf], what="one CF")
    check(_coarse(g, 7), np.zeros(n, np.float32), [cf, 10.0 * cf], 0, what="ties, two CFs")
    check_randomk(g, r, [cf], seed=n, commit=0, what="Random-k")
    dg = torch.empty(n + 1, device="cuda")[1:]
    dr = torch.empty(n + 1, device="cuda")[1:]
    dg.copy_(torch.from_numpy(g))
    dr.copy_(torch.from_numpy(r))
    idx, val, stats = binding.Compressor(n, [cf], 0)(dg, dr)
    got = (idx.cpu().numpy(), val.cpu().numpy(), stats.cpu().numpy(), dr.cpu().numpy())
    assert_same(got, oracle_compress(g, r, [cf]), "off a 16-byte boundary")


@pytest.mark.parametrize("cfs", [[1.2], [1.9], [2.6, 20.0]])
def test_long_lists_of_ragged_sub_tiles(cfs):
    """Tensors whose last, ragged sub-tile keeps a list whatever it holds: up to 1023 candidates, among sub-tiles without a list and
    behind them, in tensors of one tile and of several."""
    tails = [1023, 1022, 900, 640, 513, 512, 511, 449, 385, 384, 383, 129]
    sizes = [tiles * 8_192 + rest * 1_024 + t for i, t in enumerate(tails) for tiles, rest in ((1, i % 8), (3 + i, (5 * i) % 8))]
    off = workloads.offsets_of(sizes)
    n = int(off[-1])
    g = workloads.normal_gradient(n, 1e-3, seed=n)
    r = workloads.normal_gradient(n, 1e-4, seed=1)
    check(g, r, cfs, 0, off, what="tensors")
    check(_coarse(g, 7), np.zeros(n, np.float32), cfs, len(cfs) - 1, off, what="tensors, ties")
    check(g, r, cfs, 0, off, flags=FB, what="tensors, exact route")
    for t in range(0, len(sizes), 5):
        check(g[off[t]:off[t + 1]], r[off[t]:off[t + 1]], cfs, what=f"{sizes[t]} elements alone")


@pytest.mark.parametrize("n", [1, 8_192, 8_193, 8 * 8_192, 8 * 8_192 + 1, 64 * 8_192, 64 * 8_192 + 1, 72 * 8_192 + 5])
def test_workgroup_and_group_boundaries(n):
    """Tile counts around a workgroup of the emit step (8 tiles) and around a partial sum of the tiles' counts (64)."""
    g = workloads.normal_gradient(n, 1e-3, seed=n)
    r = workloads.normal_gradient(n, 1e-4, seed=n + 1)
    for cf in (1.0, 10.0, 1000.0):
        check(g, r, [cf], what=f"n {n} cf {cf}")


def test_tensors_that_start_inside_a_group():
    """Layerwise: tensors of more than 64 tiles that start anywhere between two partial sums."""
    sizes = [9 * 8_192 + 3, 130 * 8_192 + 1, 5, 64 * 8_192, 8_193, 200 * 8_192 - 7]
    off = workloads.offsets_of(sizes)
    n = int(off[-1])
    g = workloads.resnet_like_gradient(n, seed=1)
    r = workloads.normal_gradient(n, 1e-5, seed=2)
    check(g, r, [10.0, 100.0], 0, off, what="lowest sent")
    check(_coarse(g, 6), np.zeros(n, np.float32), [20.0], 0, off, what="ties")


def _gapped(n, count, seed, spread):
    """Ascending distinct indices in runs: gaps from one entry to many tiles of 8192."""
    rng = np.random.Generator(np.random.PCG64(seed))
    step = np.maximum(1, np.exp(rng.uniform(0.0, spread, count))).astype(np.int64)
    idx = np.cumsum(step) - 1
    return idx[idx < n].astype(np.int32)


@pytest.mark.parametrize("W", [1, 2, 8, 9, 33, 65])
@pytest.mark.parametrize("n,spread", [(40 * 8_192 + 11, 4.0), (700 * 8_192 - 5, 9.0), (2_000 * 8_192, 12.5)])
def test_decompression_of_gapped_messages(W, n, spread):
    """Tile boundaries across gaps of every length; tiles named by no worker, by one (applied together, up to 512 pairs)
    and by several; entries outside the buffer are ignored; with and without a workspace."""
    msgs = [_gapped(n + 20_000, 3_000 + 97 * w, 100 * W + w, spread) for w in range(W)]
    if W > 1:
        msgs[1] = msgs[1][:0]                                            # a worker without pairs
        msgs[0] = np.unique(np.concatenate([msgs[0], np.arange(3 * 8_192, 3 * 8_192 + 512),    # exactly 512 pairs of one worker ...
                                            np.arange(5 * 8_192, 5 * 8_192 + 513)])).astype(np.int32)   # ... and one more
    rng = np.random.Generator(np.random.PCG64(W))
    vals = [rng.standard_normal(m.size).astype(np.float32) for m in msgs]
    base = rng.standard_normal(n).astype(np.float32)
    idx, val, counts = np.concatenate(msgs), np.concatenate(vals), [m.size for m in msgs]
    ref = base.copy()
    keep = [m < n for m in msgs]
    oracle.decompress_update(np.concatenate([m[k] for m, k in zip(msgs, keep)]), np.concatenate([v[k] for v, k in zip(vals, keep)]),
                             [int(k.sum()) for k in keep], -0.0125, ref)
    i, v = torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda()
    for ws in (None, torch.empty(binding.gravac_decompress_workspace_bytes(W, n), dtype=torch.uint8, device="cuda")):
        d = torch.from_numpy(base.copy()).cuda()
        binding.gravac_decompress_update(i, v, counts, -0.0125, d, workspace=ws)
        assert np.array_equal(d.cpu().numpy().view(np.uint32), ref.view(np.uint32)), f"workspace {ws is not None}"


@pytest.mark.parametrize("count", [65_535, 65_536])
def test_tile_boundaries_on_both_sides_of_their_two_forms(count):
    """Eight messages with gaps from one entry to a tile, 2^19 pairs together and eight fewer: boundaries found four rows of
    pairs and one row at a time."""
    n, W = 70_000_000, 8
    msgs = [_gapped(n, count, w, 9.0) for w in range(W)]
    assert all(m.size == count for m in msgs)
    rng = np.random.Generator(np.random.PCG64(count))
    val = rng.standard_normal(W * count).astype(np.float32)
    ref = np.zeros(n, np.float32)
    oracle.decompress_update(np.concatenate(msgs), val, [count] * W, 0.5, ref)
    d = torch.zeros(n, device="cuda")
    ws = torch.empty(binding.gravac_decompress_workspace_bytes(W, n), dtype=torch.uint8, device="cuda")
    binding.gravac_decompress_update(torch.from_numpy(np.concatenate(msgs)).cuda(), torch.from_numpy(val).cuda(), [count] * W, 0.5, d, workspace=ws)
    assert np.array_equal(d.cpu().numpy().view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("n", [4_000_001, 8 * 1024 * 1024, 8 * 1024 * 1024 + 1, 24 * 1024 * 1024, 24 * 1024 * 1024 + 1])
@pytest.mark.parametrize("W", [2, 9])
def test_decompression_of_whole_tiles(n, W):
    """Tiles moved whole, in buffers on both sides of the sizes between which their rows are stored through the caches; the
    last tile ragged, a buffer that starts off a 16-byte boundary moved element by element."""
    step = 6 * W
    msgs = [np.arange(w, n, step, dtype=np.int32) for w in range(W - 1)] + [np.arange(0, n, step, dtype=np.int32)]
    rng = np.random.Generator(np.random.PCG64(n + W))
    vals = [rng.random(m.size, dtype=np.float32) - np.float32(0.5) for m in msgs]
    base = rng.random(n + 1, dtype=np.float32)
    idx, val, counts = np.concatenate(msgs), np.concatenate(vals), [m.size for m in msgs]
    ref = base[1:].copy()
    oracle.decompress_update(idx, val, counts, -0.0125, ref)
    i, v = torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda()
    ws = torch.empty(binding.gravac_decompress_workspace_bytes(W, n), dtype=torch.uint8, device="cuda")
    for w in (None, ws):
        for off in ((0, 1) if n < 5_000_000 else (0,)):
            d = torch.empty(n + off, device="cuda")[off:]
            d.copy_(torch.from_numpy(base[1:]))
            binding.gravac_decompress_update(i, v, counts, -0.0125, d, workspace=w)
            assert np.array_equal(d.cpu().numpy().view(np.uint32), ref.view(np.uint32)), f"workspace {w is not None}, offset {off}"


@pytest.mark.parametrize("n", [200_003, (1 << 19) - 1, 1 << 19, 1_500_001])
@pytest.mark.parametrize("scale", [1e-30, 1e-12, 1e-5, 1.0, 3e4, 1e8])
def test_sample_window(n, scale):
    """Magnitudes inside, below and above the finely binned octaves of the sample, of tensors read whole and of sampled ones;
    thresholds far below the largest entries, and infinities among the entries the octaves are found from."""
    rng = np.random.Generator(np.random.PCG64(n))
    g = (rng.standard_normal(n) * scale).astype(np.float32)
    z = np.zeros(n, np.float32)
    check(g, z, [10.0, 300.0], 0, what="normal")
    wide = (np.exp(rng.uniform(-30.0, 0.0, n)) * scale).astype(np.float32)
    check(wide, z, [1.5, 10.0], 0, what="thirty octaves and a low CF")
    g[rng.random(n) < 0.02] = np.inf
    check(g, z, [10.0], 0, what="infinities")
