"""GPU parity at the edges of the dispatch: sizes, CF counts and value distributions at which a call changes from one
kernel form or route to another, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

from paper_2305_12201_amd import workloads
from tests.test_gpu_randomk import check as check_randomk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_cf", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("n", [9_001, 300_007])
def test_randomk_forms(n_cf, n):
    """The Random-k pass is compiled for 1, 2, 3, 4 and 8 CFs; a call with five takes the form for eight."""
    cfs = [2.0, 7.5, 10.0, 33.0, 100.0, 160.0, 300.0, 1000.0][:n_cf]
    g = workloads.resnet_like_gradient(n, seed=n)
    r = workloads.normal_gradient(n, 1e-5, seed=n_cf)
    check_randomk(g, r, cfs, seed=n + n_cf, commit=n_cf - 1, what=f"{n_cf} CFs, highest sent")
    check_randomk(g, r, cfs, seed=n - n_cf, commit=0, what=f"{n_cf} CFs, lowest sent")
