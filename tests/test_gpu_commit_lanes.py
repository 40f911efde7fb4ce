"""The commit's decisions where its straight block hands over to the general path:
equal rank keys, lanes that run out, columns that outgrow the LDS pool, slots
around the two chunks of a peak.  On the GPU against the oracle, compared exactly
(needs an MI355X)."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest

from paper_2405_06856_amd import workloads as wl
from tests.test_gpu_short_tiles import ROOMY, aladdin, check, period, uneven  # noqa: F401  (aladdin: a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [1, 63, 64, 65, 150])
@pytest.mark.parametrize("R", [0, 1])
def test_equal_keys_rank_by_index(aladdin, W, R):  # noqa: F811
    """Every request is the same, so workers with as many requests have equal keys."""
    t = wl.make_trace("equal%d" % W, 780 + W, W=W, R=R, Q=400, kv_capacity=5000, model=wl.BASE_MODEL)
    t = dataclasses.replace(t, res_l_in=np.full_like(t.res_l_in, 200), res_l_pred=np.full_like(t.res_l_pred, 300),
                            res_generated=np.zeros_like(t.res_generated), q_l_in=np.full_like(t.q_l_in, 200),
                            q_l_pred=np.full_like(t.q_l_pred, 300))
    for diag in (True, False):
        check(aladdin, t, [(400, period(400, 130), diag)])


@pytest.mark.parametrize("size", [63, 64, 126, 127, 128, 129])
@pytest.mark.parametrize("diag", [True, False])
def test_peaks_around_the_chunk_edges(aladdin, size, diag):  # noqa: F811
    t = uneven([size, size + 1, 3, 0, size], 260, 790 + size, kv_capacity=120000, model=ROOMY)
    check(aladdin, t, [(200, period(200, 200), diag), (60, period(60, 20), diag)], slots=600)


@pytest.mark.parametrize("diag", [True, False])
def test_columns_beyond_the_pool(aladdin, diag):  # noqa: F811
    """More columns than the pool holds, so copies are dropped and made again, one
    worker growing past the room its copy was given; capacities that bind."""
    sizes = [2600, 2400, 2300, 2200, 2100, 900, 40, 0]
    t = uneven(sizes, 420, 801, kv_capacity=900000, model=ROOMY)
    load = np.array([int((t.res_l_in[a:b] + t.res_generated[a:b]).sum())
                     for a, b in zip(t.res_offsets[:-1], t.res_offsets[1:])])
    t = dataclasses.replace(t, kv_capacity=(load + 30000).astype(t.kv_capacity.dtype))
    check(aladdin, t, [(420, period(420, 140), diag)], slots=3000)
