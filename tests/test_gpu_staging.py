"""GPU parity of the streaming pass where its wavefronts' staging of entries can go wrong: sub-tiles of 1024 with none, a
few, exactly 512 and more entries that some bracket concerns, with and without a candidate list (384 candidates), ragged
and unaligned ones.  Against the CPU oracle, bit for bit, over two iterations."""
import numpy as np
import pytest
import torch

from paper_2305_12201_amd import binding, workloads
from tests.gpu_util import assert_same, oracle_compress

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1023, 1024, 8192 * 17 + 1, 300_032])
@pytest.mark.parametrize("cfs,commit", [([2.0], 0), ([1.0], 0), ([2.5, 2.7], 1), ([1.5, 100.0], 1), ([100.0, 1.5], 0),
                                        ([10.0, 100.0, 1000.0], 2), ([3.0, 2.0, 20.0, 200.0], 1),
                                        ([2.0, 3.0, 5.0, 8.0, 20.0], 3)])
def test_staged_rows(n, cfs, commit):
    # half of the sub-tiles' entries large in turn, so that full, half-full and empty ones follow each other
    scale = np.repeat(np.resize([1.0, 1e-3, 0.05, 1.0, 1.0], n // 512 + 1), 512)[:n].astype(np.float32)
    comp = binding.Compressor(n, cfs, commit)
    for shift in (0, 1):   # a buffer aligned to 16 bytes, and one that is not
        res = workloads.normal_gradient(n, 1e-4, seed=5)
        buf = torch.zeros(n + 4, dtype=torch.float32, device="cuda")
        r = buf[shift:shift + n]
        r.copy_(torch.from_numpy(res))
        for it in range(2):
            g = workloads.normal_gradient(n, 1e-3, seed=n + it) * scale
            idx, val, stats = comp(torch.from_numpy(g).cuda(), r)
            ref = oracle_compress(g, res, cfs, commit)
            assert comp.status()["internal_error"] == 0
            assert_same((idx.cpu().numpy(), val.cpu().numpy(), stats.cpu().numpy(), r.cpu().numpy()), ref,
                        f"n {n}, CFs {cfs}, shift {shift}, iteration {it}")
            res = ref[3]
