"""The merge of many key parts (batches of eight, two parts per lane past 32), and the automatic
split of short key ranges, against the fp64 oracle at the bf16 bars (2e-2 on O, 4e-3 on LSE)."""

from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2607_21848_amd as rv
import workloads as W
from oracle import attention as OA
from tests.gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


def _case(Lq, frames, h, w, S, H, seed):
    rng = np.random.default_rng(seed)
    q, k, v = (W.bf16_round(rng.standard_normal((L, H, 128), dtype=np.float32)) for L in (Lq, frames * h * w, frames * h * w))
    k[:40] *= 4.0  # the first part's maxima stand out, the others' sums are scaled down (exact in bf16)
    slot = np.full(frames, -1, np.int32)
    slot[rng.permutation(frames)[:S]] = np.arange(S)
    uv = np.stack([rng.uniform(0, w, (S, Lq)), rng.uniform(0, h, (S, Lq))], -1).astype(np.float32)
    return q, k, v, slot, uv, rng.integers(-4, h * w, size=(S, Lq)).astype(np.int32)


def _check(c, h, w, parts):
    q, k, v, slot, uv, idx = c
    print(f"Lq={q.shape[0]} Lk={k.shape[0]} H={q.shape[1]} parts={parts}", flush=True)
    o, lse = rv.biased_chunk_attention(*(dev(x, torch.bfloat16) for x in (q, k, v)), dev(slot), dev(uv), dev(idx), h=h, w=w,
                                       softmax_scale=128 ** -0.5, lam=1.0, sigma=2.0, key_parts=parts)
    Oo, Lo = OA.biased_attention(q, k, v, slot, uv, idx, h, w, 128 ** -0.5, 1.0, 2.0)
    assert np.abs(host(o) - Oo).max() <= 2e-2 and np.abs(host(lse) - Lo).max() <= 4e-3


@pytest.mark.parametrize("parts", [8, 9, 16, 17, 31, 32, 33, 40, 63, 64])
def test_merge_of_many_parts(parts):
    _check(_case(131, 9, 13, 18, 3, 2, 5), 13, 18, parts)  # 66 key tiles, a ragged last one


@pytest.mark.parametrize("frames", [1, 2, 5, 18])
def test_automatic_split_of_short_ranges(frames):
    _check(_case(60, frames, 9, 16, min(frames, 3), 3, frames), 9, 16, 0)


def test_automatic_split_in_a_smaller_workspace():
    """Short key ranges need no workspace: the split takes what fits (equal to that many forced
    parts, bit for bit). A long range that has always needed one is refused without it."""
    q, k, v, slot, uv, idx = _case(140, 9, 13, 18, 3, 2, 9)
    args = [dev(x, torch.bfloat16) for x in (q, k, v)] + [dev(slot), dev(uv), dev(idx)]
    kw = dict(h=13, w=18, softmax_scale=128 ** -0.5, lam=1.0, sigma=2.0)
    auto = rv.attention_workspace_size(torch.bfloat16, 140, k.shape[0], 2, 128) // (4 * 66560)
    assert auto >= 3
    for nbytes, parts in ((16, 1), (2 * 4 * 66560 - 1, 1), (3 * 4 * 66560, 3), (auto * 4 * 66560, auto)):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        got = rv.biased_chunk_attention(*args, **kw, workspace=ws)
        want = rv.biased_chunk_attention(*args, **kw, key_parts=parts)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (nbytes, parts)
    long = [torch.zeros(n, 1, 128, dtype=torch.bfloat16, device="cuda") for n in (128, 8448, 8448)]
    with pytest.raises(rv.RevisitError):
        rv.biased_chunk_attention(*long, dev(np.full(1, -1, np.int32)), None, None, h=96, w=88, softmax_scale=0.1, lam=1.0,
                                  sigma=1.0, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("parts", [0, 1, 3, 9])
def test_a_part_that_starts_without_a_finite_logit(parts):
    """Keys whose logits are -inf have weight 0 in whichever tile they stand, the first of a part
    (here of every part but the first, and the whole last part) among them, and NaN stays NaN."""
    Lq, frames, h, w, H = 140, 6, 16, 18, 2  # 54 key tiles
    q, k, v, slot, uv, idx = _case(Lq, frames, h, w, 2, H, 21)
    k[:40] /= 4.0
    q[:, :, 0] = 1.0
    q[7, 1, 0] = np.nan
    n = frames * h * w // 32
    dead = np.concatenate([np.arange(32 * (p * n // P), 32 * (p * n // P) + 32) for P in (2, 3, 4, 8, 9, 16) for p in range(1, P)]
                          + [np.arange(32 * (8 * n // 9), 32 * n)])
    k[dead, :, 0] = -np.inf
    args = [dev(x, torch.bfloat16) for x in (q, k, v)] + [dev(slot), dev(uv), dev(idx)]
    o, lse = rv.biased_chunk_attention(*args, h=h, w=w, softmax_scale=128 ** -0.5, lam=1.0, sigma=2.0, key_parts=parts)
    o, lse = host(o), host(lse)
    assert np.isnan(o[7, 1]).all() and np.isnan(lse[1, 7])
    q[7, 1, 0] = 1.0
    k[dead] = 0.0
    k[dead, :, 0] = -2.0 ** 100  # the same weights, in finite numbers
    Oo, Lo = OA.biased_attention(q, k, v, slot, uv, idx, h, w, 128 ** -0.5, 1.0, 2.0)
    rest = np.ones((Lq, H), bool)
    rest[7, 1] = False
    assert np.abs(o - Oo)[rest].max() <= 2e-2 and np.abs(lse - Lo).T[rest].max() <= 4e-3


@pytest.mark.parametrize("parts", [0, 1, 5])
def test_a_row_without_a_finite_logit(parts):
    """Such a row has no weights: its output and its LSE are not numbers, its neighbours' are."""
    q, k, v, slot, uv, idx = _case(60, 5, 9, 16, 2, 2, 22)
    q[:, :, 0] = k[:, :, 0] = 1.0
    q[9, 1, 0] = -np.inf
    args = [dev(x, torch.bfloat16) for x in (q, k, v)] + [dev(slot), dev(uv), dev(idx)]
    o, lse = rv.biased_chunk_attention(*args, h=9, w=16, softmax_scale=128 ** -0.5, lam=1.0, sigma=2.0, key_parts=parts)
    o, lse = host(o), host(lse)
    rest = np.ones((60, 2), bool)
    rest[9, 1] = False
    assert np.isnan(o[9, 1]).all() and np.isnan(lse[1, 9]) and np.isfinite(o[rest]).all() and np.isfinite(lse.T[rest]).all()
