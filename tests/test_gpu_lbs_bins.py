"""Load-balancing simulation: guide tables with cells that have to be searched, and strata sorted in bins of 64 lanes,
trial by trial against the oracle."""
import numpy as np
import pytest

import workloads as W
from paper_2402_02447_amd import lbs
from test_gpu_lbs import check, check_all

pytestmark = pytest.mark.gpu

CUM, ENDS = W.length_histogram_piecewise_uniform(), W.LENGTH_STRATUM_END
LOCAL = (lbs.LBS_LOCAL_RASTER, lbs.LBS_LOCAL_SNAKE)


def _cum(hist):
    return np.concatenate([[0], np.cumsum(hist)]).astype(np.uint32)


SPIKE = _cum(np.where(np.arange(512) == 99, 4_000_000, 1))     # one length holds nearly everything


# (gpus per node, local batch, quota): what of 64 / gpus_per_node rows the strata fill
@pytest.mark.parametrize("gpn,batch,quota", [
    (8, 16, [6, 3, 2, 5]), (4, 32, [12, 6, 4, 10]), (2, 44, [20, 12, 12, 0]),       # two bins, full
    (8, 12, [6, 3, 2, 1]), (16, 7, [3, 2, 1, 1]), (8, 9, [0, 8, 0, 1]),                       # two bins, padded
    (4, 16, [5, 2, 3, 6]), (8, 8, [3, 2, 1, 2]), (16, 4, [1, 1, 1, 1]), (1, 64, [16, 16, 16, 16]),  # one bin, full
    (8, 5, [2, 1, 1, 1]), (1, 3, [1, 0, 1, 1]), (16, 1, [0, 0, 1, 0]),                        # one bin, padded
    (8, 16, [9, 3, 2, 2]), (16, 16, [6, 3, 2, 5]), (8, 21, [7, 7, 7, 0]),                     # do not fit
])
def test_quotas_that_fit_in_bins_and_quotas_that_do_not(gpn, batch, quota):
    batch = sum(quota)
    for n_nodes in (1, 9, 67):     # fewer nodes than a wavefront takes at a time, and numbers it does not divide
        for method in LOCAL:
            check(CUM, ENDS, method, batch, gpn, gpn * n_nodes, quota, seed=31 * gpn + n_nodes, n=7, first=3)
        check_all(CUM, ENDS, batch, gpn, gpn * n_nodes, quota, seed=17 * gpn + n_nodes, n=7, first=11)


# Full bins of nodes of 4 and 8: numbers of nodes that leave wavefronts and groups of lanes without a node, and odd numbers where
# two nodes share a register.  Slots whose rows change parity inside a bin ([5, 2, 3, 6]) and ones that do not.
@pytest.mark.parametrize("gpn,batch,quota,nodes", [
    (8, 16, [6, 3, 2, 5], (19, 22, 33, 50, 128, 131)), (8, 16, [5, 2, 3, 6], (32, 64, 97)),
    (8, 8, [3, 2, 1, 2], (31, 45, 65, 130, 255)), (4, 16, [5, 2, 3, 6], (9, 61, 67, 129, 256)), (4, 32, [12, 6, 4, 10], (17, 33, 65, 130)),
])
def test_full_bins_by_number_of_nodes(gpn, batch, quota, nodes):
    import torch
    for n_nodes in nodes:
        check_all(CUM, ENDS, batch, gpn, gpn * n_nodes, quota, seed=n_nodes, n=5, first=2)
    # one method alone: more trials than are resident at once
    n = 6 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    for n_nodes, method in zip((nodes[0], nodes[1], nodes[-1]), LOCAL + LOCAL[:1]):
        check(CUM, ENDS, method, batch, gpn, gpn * n_nodes, quota, seed=5 * n_nodes, n=n)


# Each number of registers a node of full bins can lie in, by all five methods at once and by one alone, and the columns in registers where cells
# have to be searched.  Which form a size takes is a fitted cost: test_fake_device.py looks that these tests leave none out.
@pytest.mark.parametrize("gpn,batch,quota,n_nodes,n,searched", [
    (8, 16, [6, 3, 2, 5], 23, 7, False), (8, 16, [6, 3, 2, 5], 47, 7, False), (8, 16, [6, 3, 2, 5], 113, 301, False),   # two bins: 8, 16, 32 registers
    (8, 8, [3, 2, 1, 2], 39, 7, False), (8, 8, [3, 2, 1, 2], 79, 7, False), (8, 8, [3, 2, 1, 2], 255, 301, False),      # one bin
    (4, 32, [12, 6, 4, 10], 51, 7, False), (4, 32, [12, 6, 4, 10], 113, 301, False),                                    # two bins: 16, 32
    (4, 16, [5, 2, 3, 6], 99, 7, False), (4, 16, [5, 2, 3, 6], 255, 301, False),                                        # one bin
    (8, 16, [6, 3, 2, 5], 27, 7, True), (8, 4, [1, 1, 1, 1], 51, 7, True),
])
def test_forms_of_full_bins(gpn, batch, quota, n_nodes, n, searched):
    cum = SPIKE if searched else CUM
    check_all(cum, ENDS, batch, gpn, gpn * n_nodes, quota, seed=n_nodes, n=n, first=5)
    for method in LOCAL:
        check(cum, ENDS, method, batch, gpn, gpn * n_nodes, quota, seed=7 * n_nodes, n=n, first=1 << 40)


@pytest.mark.parametrize("kind", ["gaps", "spike", "rare_tail", "wide_strata", "one_length"])
def test_histograms_whose_cells_have_to_be_searched(kind):
    rng = np.random.default_rng(5)
    ends, quota = (100, 300, 700, 1000), [3, 2, 1, 2]
    if kind == "gaps":          # most lengths do not occur
        hist = np.where(rng.random(1000) < 0.1, rng.integers(1, 9, 1000), 0)
        hist[[50, 200, 500, 999]] = 3
    elif kind == "spike":       # one length holds nearly everything
        hist = np.ones(1000, np.int64)
        hist[411] = 4_000_000
    elif kind == "rare_tail":
        hist = (1e6 / (1 + np.arange(1000.0)) ** 2 + 1).astype(np.int64)
    elif kind == "wide_strata":  # more than 256 lengths in a stratum
        hist, ends, quota = np.full(1000, 977), (1000,), [8]
    else:
        hist, ends, quota = np.zeros(1000, np.int64), (1000,), [8]
        hist[999] = 5
    for method in range(5):
        check(_cum(hist), ends, method, 8, 8, 8 * 5, quota, seed=3, n=20)
    check_all(_cum(hist), ends, 8, 8, 8 * 5, quota, seed=4, n=20)


def test_largest_token_counts_in_sixteen_bits_and_beyond_and_a_single_gpu():
    for max_len in (1023, 1024):    # 64 x 1023 fits in half a register, 64 x 1024 does not
        hist = np.zeros(max_len, np.int64)
        hist[-1] = 7
        check_all(_cum(hist), (max_len,), 64, 1, 5, [64], seed=1, n=4)
        check(_cum(hist), (max_len,), lbs.LBS_GLOBAL, 64, 1, 1, [64], seed=1, n=4)


@pytest.mark.parametrize("gpn,n_nodes,batch,quota", [(1, 1, 3, [1, 0, 1, 1]), (2, 4, 2, [1, 0, 0, 1]), (4, 3, 3, [1, 1, 1, 0])])
def test_many_short_trials_on_both_sides_of_the_line(gpn, n_nodes, batch, quota):
    """Few nodes and small pools: beyond sixty trials a workgroup the sorted pools take over from the bins."""
    import torch
    line = 60 * 32 * torch.cuda.get_device_properties(0).multi_processor_count
    for n in (line, line + 1):
        check(CUM, ENDS, lbs.LBS_LOCAL_SNAKE, batch, gpn, gpn * n_nodes, quota, seed=n, n=n)
