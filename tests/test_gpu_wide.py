"""Launched rounds with a wave per gap (k_grant_wide): few and many list blocks (sixteen and eight waves each, and
more than it takes), list blocks of one lane and of 64, records that many lanes pass, bounded rounds, against the
oracle (small batches in the mode that leaves them to these kernels too, see full_tick_check)."""
import numpy as np
import pytest

from gen import make_workload
from test_gpu_parity import full_tick_check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2509_19086_amd as P
    return P.Engine(0)


@pytest.mark.parametrize("caps,windows,gaps_each", [(1, 1, 64), (2, 2, 65), (64, 8, 1), (57, 9, 1), (64, 16, 1), (64, 17, 1)])
def test_list_blocks(engine, oracle, caps, windows, gaps_each):
    # a window twice as long begins a list block: 1, 6, 512, 513, 1024 and 1088 of them
    wl = make_workload("stress", 2, n_gaps=caps * windows * gaps_each, n_jobs=400)
    wl.W = np.tile(np.repeat(200 * 2 ** np.arange(windows), gaps_each), caps).astype(np.int32)
    wl.C = np.repeat(np.arange(30000, 30000 + 1500 * caps, 1500)[:caps], windows * gaps_each).astype(np.int32)
    wl.max_rounds = 12
    full_tick_check(engine, oracle, wl, policies=[0, 3], resolve_modes=(0,))


@pytest.mark.parametrize("name,gaps,jobs", [("large", 700, 3000), ("stress", 1100, 2000), ("medium", 333, 5000)])
@pytest.mark.parametrize("max_rounds", [1, 2, 3, 8])
def test_bounded_rounds(engine, oracle, name, gaps, jobs, max_rounds):
    wl = make_workload(name, gaps, n_gaps=gaps, n_jobs=jobs)
    wl.max_rounds = max_rounds
    full_tick_check(engine, oracle, wl, policies=[1], resolve_modes=(0,))
