"""Retrieval's selection where it can go wrong: banks around the batch and wave edges, open gates
(more admissible entries than are ranked at once), and banks whose best entries all fall to one lane,
which keeps four and has the rest looked for again. Exact against the fp64 oracle."""

from __future__ import annotations

import math

import numpy as np
import pytest

import paper_2607_21848_amd as rv
from oracle import retrieval as ORT
from tests.gpu_helpers import dev, host, same_bits_f32

pytestmark = pytest.mark.gpu


def _check(bank, query, chunk, k, *, tau_c=1e6, tau_v=math.pi, delta=0, first=0, E=2.0, w_v=0.5):
    args = (E, w_v, tau_c, tau_v, delta, first, k)
    want_i, want_s, want_c = ORT.retrieve(bank, query, chunk, *args)
    print(f"N={len(bank)} Q={len(query)} k={k} counts {want_c.tolist()[:4]}", flush=True)
    idx, score, count, sel = rv.retrieve_chunks(dev(bank), dev(query), dev(chunk), E=E, w_v=w_v, tau_c=tau_c, tau_v=tau_v,
                                                delta=delta, first_candidate=first, k=k, frames_per_chunk=3)
    assert np.array_equal(host(count), want_c) and np.array_equal(host(idx), want_i)
    assert same_bits_f32(host(score), want_s.astype(np.float32)).all()
    assert np.array_equal(host(sel), ORT.frame_selection(want_i, want_c, 3))


def _line(x, seed=0):
    """Poses looking along +z at distance x from the origin."""
    bank = np.tile(np.eye(4, dtype=np.float32), (len(x), 1, 1))
    bank[:, 0, 3] = x
    return bank


@pytest.mark.parametrize("N", [1, 63, 64, 65, 255, 256, 257, 1023, 1025, 4095, 4097, 8191, 8192, 8193, 16384, 16385])
@pytest.mark.parametrize("k", [1, 4, 5, 32])
def test_open_gates(N, k):
    rng = np.random.default_rng(N + k)
    bank, query = _line(rng.uniform(0, 9, N)), _line(np.array([0.0, 4.5]))
    _check(bank, query, np.array([N + 9, N // 2], np.int32), k)


@pytest.mark.parametrize("falling", [False, True])
def test_scores_in_order_and_equal(falling):
    """Every entry better than all before it, every entry worse, and all alike."""
    N = 6000
    x = np.arange(N, dtype=np.float32)
    bank = _line(x[::-1] if falling else x)
    _check(bank, _line(np.zeros(1)), np.array([N + 5], np.int32), 32, tau_c=1e9)
    _check(_line(np.ones(N)), _line(np.zeros(1)), np.array([N + 5], np.int32), 32, first=7, delta=20)


@pytest.mark.parametrize("N,step", [(8192, 4096), (20000, 4096), (40000, 4096)])
@pytest.mark.parametrize("k", [3, 9, 32])
def test_best_entries_of_one_lane(N, step, k):
    """The forty best entries sit 64 or 4096 apart, in two lanes: more than a lane keeps."""
    rng = np.random.default_rng(N)
    x = rng.uniform(5, 9, N).astype(np.float32)
    at = np.array([l + 64 * u + step * i for l in (5, 263) for i in range((N - 512) // step + 1) for u in range(4)])[:40]
    x[at] = rng.permutation(len(at)) * 0.01
    _check(_line(x), _line(np.zeros(2)), np.array([N + 3, N + 4], np.int32), k)


def test_distances_at_the_gate():
    """Distances within a few units in the last place of tau_c E, either side."""
    E, tau = np.float32(7.3), np.float32(0.31)
    edge = np.float32(float(E) * float(tau))
    x = np.array([edge], np.float32)
    for _ in range(40):
        x = np.concatenate([[np.nextafter(x[0], np.float32(0))], x, [np.nextafter(x[-1], np.float32(9))]]).astype(np.float32)
    _check(_line(x), _line(np.zeros(1)), np.array([100], np.int32), 32, E=float(E), tau_c=float(tau))
    _check(_line(np.zeros(70)), _line(np.zeros(1)), np.array([100], np.int32), 32, tau_c=0.0)
    _check(_line(x), _line(np.zeros(1)), np.array([100], np.int32), 4, tau_c=-1.0)


@pytest.mark.parametrize("N", [30, 200, 256, 300])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8])
def test_few_and_many_in_reach_of_one_wave(N, k):
    """Around the sizes from which a wave's results come from reductions alone, and its pairs are not
    ranked: 0 to 9, some twenty and thirty, and all entries in reach."""
    rng = np.random.default_rng(N + k)
    x = rng.permutation(N).astype(np.float32) + 1.0
    x[::7] = np.ceil(x[::7] / 4) * 4  # equal scores too
    for reach in (0, 1, 2, 3, 4, 6, 9, 19, 20, 21, 22, 30, 37, 45, 64, 65, 140, N):
        _check(_line(x), _line(np.zeros(1)), np.array([N + 5], np.int32), k, E=1.0, tau_c=reach + 0.5)


@pytest.mark.parametrize("N,Q", [(3000, 300), (3000, 1500), (8192, 2049), (700, 5000)])
@pytest.mark.parametrize("k", [1, 4, 9, 32])
def test_many_queries(N, Q, k):
    """So many queries that each has fewer waves than its bank would fill, or one."""
    rng = np.random.default_rng(Q + k)
    bank, query = _line(rng.uniform(0, 9, N)), _line(rng.uniform(0, 9, Q))
    chunk = rng.integers(0, N + 9, Q).astype(np.int32)
    kw = dict(E=2.0, w_v=0.5, tau_c=0.05, tau_v=1.0, delta=2, first_candidate=1, k=k)
    print(f"N={N} Q={Q} k={k}", flush=True)
    idx, score, count, _ = rv.retrieve_chunks(dev(bank), dev(query), dev(chunk), **kw)
    at = np.r_[0, 1, rng.integers(0, Q, 40), Q - 1]
    want_i, want_s, want_c = ORT.retrieve(bank, query[at], chunk[at], 2.0, 0.5, 0.05, 1.0, 2, 1, k)
    assert np.array_equal(host(count)[at], want_c) and np.array_equal(host(idx)[at], want_i)
    assert same_bits_f32(host(score)[at], want_s.astype(np.float32)).all()


@pytest.mark.parametrize("N,Q,k", [(8193, 256, 4), (8193, 257, 4), (8193, 260, 9), (16385, 129, 1), (16385, 129, 32),
                                   (40000, 90, 4), (40000, 100, 5), (8193, 256, 9)])
@pytest.mark.parametrize("tau_c", [0.02, 1e6])
def test_segments_of_eight_waves(N, Q, k, tau_c):
    """Either side of the number of segments from which each has eight waves, which start at different
    batches of theirs; index ranges that begin and end inside segments."""
    rng = np.random.default_rng(Q + k)
    bank, query = _line(rng.uniform(0, 9, N)), _line(rng.uniform(0, 9, Q))
    chunk = rng.integers(0, N + 9, Q).astype(np.int32)
    chunk[0] = N + 9
    for first in (1, 3000):
        kw = dict(E=2.0, w_v=0.5, tau_c=tau_c, tau_v=1.0, delta=2, first_candidate=first, k=k)
        print(f"N={N} Q={Q} k={k} tau_c={tau_c} first={first}", flush=True)
        idx, score, count, _ = rv.retrieve_chunks(dev(bank), dev(query), dev(chunk), **kw)
        at = np.r_[0, rng.integers(0, Q, 30), Q - 1]
        want_i, want_s, want_c = ORT.retrieve(bank, query[at], chunk[at], 2.0, 0.5, tau_c, 1.0, 2, first, k)
        assert np.array_equal(host(count)[at], want_c) and np.array_equal(host(idx)[at], want_i)
        assert same_bits_f32(host(score)[at], want_s.astype(np.float32)).all()


@pytest.mark.parametrize("N", [128 * 16384, 128 * 16384 + 1, 131 * 16384 - 77])
def test_one_query_of_many_segments(N):
    """One query's segments either side of half the compute units, some in reach in many of them."""
    rng = np.random.default_rng(N)
    x = rng.uniform(1, 9, N).astype(np.float32)
    x[rng.integers(0, N, 500)] = np.float32(0.125) + rng.integers(0, 8, 500).astype(np.float32) / 64
    for k in (1, 4, 9):
        for first, chunk in ((1, N + 9), (1234567, 2000000)):
            _check(_line(x), _line(np.zeros(1)), np.array([chunk], np.int32), k, E=1.0, tau_c=0.2, first=first)
