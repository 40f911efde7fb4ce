"""Tile lengths, slot counts and worker counts at the edges where the evaluator
changes its path, on the GPU against the oracle, compared exactly (needs an
MI355X)."""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import pytest

from oracle import ref
from paper_2405_06856_amd import workloads as wl

pytestmark = pytest.mark.gpu

# a decode worker whose batch limit is about 4000 requests
ROOMY = dataclasses.replace(wl.BASE_MODEL, ttft_slo=math.inf, c3=0.0, c2=wl.BASE_MODEL.decode_slo / 4000, k2=1e-12)

INT_FIELDS = ("n_feasible", "near_tie", "kv_peak_chosen", "kv_excess_min")


@pytest.fixture(scope="module")
def aladdin():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2405_06856_amd import aladdin as mod
    return mod


def uneven(sizes, Q, seed, kv_capacity, model=wl.BASE_MODEL, in_dist=wl.SHORT_IN, out_dist=wl.SHORT_OUT):
    """A trace whose worker w holds sizes[w] requests."""
    sizes = np.asarray(sizes)
    R = int(sizes.max(initial=0))
    t = wl.make_trace("uneven%d" % seed, seed, W=sizes.size, R=R, Q=Q, kv_capacity=kv_capacity, model=model,
                      in_dist=in_dist, out_dist=out_dist)
    keep = (np.arange(R)[None, :] < sizes[:, None]).reshape(-1)
    return dataclasses.replace(
        t, res_offsets=np.concatenate([[0], np.cumsum(sizes)]).astype(t.res_offsets.dtype),
        res_l_in=t.res_l_in[keep], res_l_pred=t.res_l_pred[keep], res_generated=t.res_generated[keep],
        res_t_dec=None if t.res_t_dec is None else t.res_t_dec[keep])


def oracle(t, hb):
    return ref.place_hb(t.n_workers, t.kv_capacity, t.res_offsets, t.res_l_in, t.res_l_pred, t.res_generated, t.model,
                        t.q_l_in, t.q_l_pred, hb, res_t_dec=t.res_t_dec)


def period(Q, H):
    hb = np.zeros(Q, np.int32)
    hb[H::H] = 1
    return hb


def check(aladdin, t, calls, tile=1024, slots=0):
    """Places the trace in the given calls [(queries, heartbeats before each, diagnostics)]."""
    ev = aladdin.Evaluator(0, tile=tile)
    ev.load_trace(t, slots_per_worker=slots)
    a, workers = 0, []
    hb = np.concatenate([np.asarray(h, np.int32) for _, h, _ in calls])
    want = oracle(dataclasses.replace(t, q_l_in=t.q_l_in[:hb.size], q_l_pred=t.q_l_pred[:hb.size], arrivals=None), hb)
    for n, h, diag in calls:
        print("call", a, n, "tile", tile, "diag", diag, flush=True)
        got = ev.place(t.q_l_in[a:a + n], t.q_l_pred[a:a + n], diag=diag, hb_before=np.asarray(h, np.int32))
        workers.append(got.worker)
        if diag:
            for f in INT_FIELDS:
                g, w = got.diag[f].astype(np.int64), getattr(want, f)[a:a + n].astype(np.int64)
                assert np.array_equal(g, w), (f, a, np.flatnonzero(g != w)[:10])
        a += n
    summ = ev.summary()
    ev.close()
    workers = np.concatenate(workers)
    assert np.array_equal(workers, want.worker), np.flatnonzero(workers != want.worker)[:10]
    for f in ("B", "sum_c", "sum_r", "peak"):
        assert np.array_equal(summ[f].astype(np.int64), getattr(want, f)), f
    return want


@pytest.mark.parametrize("diag", [True, False])
@pytest.mark.parametrize("H", [1, 63, 64, 65, 255, 256, 257, 300])
def test_window_lengths(aladdin, H, diag):
    """Heartbeat windows at the edges of query groups and of short tiles, with
    more feasible workers than a wave holds; every constraint set in turn."""
    Q = 130 if H == 1 else 3 * H + 7
    for model in (wl.BASE_MODEL, dataclasses.replace(wl.BASE_MODEL, ttft_slo=math.inf),
                  dataclasses.replace(wl.BASE_MODEL, k1=-1e-7, k1q=1e-9)):
        t = wl.make_trace("window", 700 + H, W=150, R=20, Q=Q, kv_capacity=16000, model=model)
        want = check(aladdin, t, [(Q, period(Q, H), diag)])
        assert (want.worker >= 0).any()


@pytest.mark.parametrize("history", [False, True])
def test_slot_counts(aladdin, history):
    """Workers with slot counts at the edges of a wave, of the two-load scan, of
    the staged ends and of the small build, next to empty ones."""
    sizes = [0, 1, 63, 64, 65, 127, 128, 129, 0, 254, 255, 256, 257, 510, 511, 512, 513, 700, 0, 3]
    for cap in (40000, 400000):
        t = uneven(sizes, 400, 710, cap)
        if history:
            t = wl.with_decode_history(t, 711)
        for diag in (True, False):
            check(aladdin, t, [(400, period(400, 50), diag)])
            check(aladdin, t, [(400, np.zeros(400), diag)])


def test_calls_that_need_different_tables(aladdin):
    """Short and long calls with and without diagnostics on one state: each finds
    what its tiles read, whatever the call before it built."""
    t = wl.make_trace("levels", 720, W=40, R=30, Q=3000, kv_capacity=25000, model=wl.BASE_MODEL)
    rng = np.random.default_rng(721)
    calls, left = [], 3000
    for n in (10, 300, 20, 500, 1, 256, 257, 64, 300, 7, 400):
        for diag in (False, True):
            n = min(n, left)
            hb = np.zeros(n, np.int32)
            if n and rng.random() < 0.6:
                hb[0] = int(rng.integers(0, 4))
            calls.append((n, hb, diag))
            left -= n
    check(aladdin, t, [c for c in calls if c[0]])


@pytest.mark.parametrize("diag", [True, False])
def test_many_requests_to_one_worker(aladdin, diag):
    """One worker takes more requests in one window than a wave, or a scan's
    stage, holds."""
    t = wl.make_trace("pile", 730, W=1, R=3, Q=1500, kv_capacity=4000000,
                      model=ROOMY)
    hb = np.zeros(1500, np.int32)
    hb[[200, 1490]] = [3, 200]
    want = check(aladdin, t, [(1500, hb, diag)], tile=4096)
    assert (want.worker >= 0).all()


@pytest.mark.parametrize("diag", [True, False])
def test_full_slot_ranges(aladdin, diag):
    """Slot ranges that fill to the last slot and wrap while requests finish."""
    t = wl.make_trace("wrap", 740, W=9, R=6, Q=1200, kv_capacity=60000, model=wl.BASE_MODEL)
    rng = np.random.default_rng(741)
    hb = ((rng.random(1200) < 0.05) * rng.integers(1, 120, 1200)).astype(np.int32)
    most = 0  # requests on the fullest worker before any heartbeat or at the end
    for k in [*np.flatnonzero(hb), 1200]:
        if k:
            p = dataclasses.replace(t, q_l_in=t.q_l_in[:k], q_l_pred=t.q_l_pred[:k], arrivals=None)
            most = max(most, int(oracle(p, hb[:k]).B.max()))
    for slots in (most, most + 1, most + 17):
        check(aladdin, t, [(700, hb[:700], diag), (500, hb[700:], not diag)], slots=slots)


@pytest.mark.parametrize("diag", [True, False])
def test_columns_beyond_the_pool(aladdin, diag):
    """Capacity binds on workers whose slots do not all fit the wave's LDS."""
    # the residents' peaks lie between 385854 and 507692: about 20 of the roomy
    # workers, 900 slots each, take a query (the wave's LDS holds 14336 entries)
    t = uneven([1000 - 3 * i for i in range(60)], 1000, 750, 450000, model=ROOMY)
    want = check(aladdin, t, [(1000, np.zeros(1000), diag)])
    assert np.unique(want.worker).size > 16


@pytest.mark.parametrize("R", [0, 2])
def test_more_workers_than_ranks_in_lds(aladdin, R):
    t = wl.make_trace("wide", 760, W=4500, R=R, Q=330, kv_capacity=12000, model=wl.BASE_MODEL)
    for diag in (True, False):
        check(aladdin, t, [(330, period(330, 110), diag)])


@pytest.mark.parametrize("H", [0, 40, 300])
def test_sweep_with_empty_and_full_clusters(aladdin, H):
    """A sweep whose scenarios run from one worker to more than a wave, empty at
    the start, capacity from nearly none to ample."""
    rng = np.random.default_rng(770)
    scen = [wl.Scenario(n_workers=W, gpus_per_worker=1, kv_capacity=cap, model=wl.BASE_MODEL.scaled(f))
            for W in (1, 63, 64, 65, 200) for cap, f in ((600, 1.0), (9000, 0.7), (90000, 1.0))]
    q_in = wl._lengths(rng, *wl.SHORT_IN, 900).astype(np.int32)
    q_pred = wl._lengths(rng, *wl.SHORT_OUT, 900).astype(np.int32)
    Hs = np.full(len(scen), H, np.int32)
    print("sweep", len(scen), "H", H, flush=True)
    ev = aladdin.Evaluator(0)
    rej, first, workers, _ = ev.sweep(scen, q_in, q_pred, want_workers=True, heartbeat_every=Hs, want_answer=True)
    ev.close()
    orej, ofirst, oworkers = ref.sweep(scen, q_in, q_pred, want_workers=True, heartbeat_every=Hs)
    assert np.array_equal(workers, oworkers), np.argwhere(workers != oworkers)[:5]
    assert np.array_equal(rej, orej) and np.array_equal(first, ofirst)
