"""fp32 attention at the edges of its 32-query, 32-key tiles and of its W waves per item (wave w takes
key tiles w, w + W, ...; W is 8 from 48 tiles on, and of up to 256 items from 5 on; else 4 from 12
tiles on or of up to 512 items, else 1),
against the fp64 oracle at the fp32 bars (1e-4, as in the targeted tests: sums of at most 1850 fp32
products of N(0, 1) values stay far inside it)."""

from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2607_21848_amd as rv
from oracle import attention as OA
from tests.gpu_helpers import dev, host

pytestmark = pytest.mark.gpu

TOL = 1e-4


def _inputs(seed, Lq, frames, h, w, S, H, D):
    rng = np.random.default_rng(seed)
    hw = h * w
    q, k, v = (rng.standard_normal((L, H, D), dtype=np.float32) for L in (Lq, frames * hw, frames * hw))
    slot = np.full(frames, -1, np.int32)
    slot[rng.permutation(frames)[:S]] = np.arange(S)
    uv = np.stack([rng.uniform(-1, w + 1, (S, Lq)), rng.uniform(-1, h + 1, (S, Lq))], -1).astype(np.float32)
    idx = rng.integers(-5, hw, size=(S, Lq)).astype(np.int32)
    return q, k, v, slot, uv, idx


# (Lq, frames, h, w, S, H, D): one key; one tile less, exactly and more than a key; fewer tiles than
# waves; eight tiles and one key either side; several tiles per wave with a ragged last one; frames
# smaller than a tile, of one token, and of a row of one token; eight waves at 48 and 49 tiles and
# 58 with a ragged last one; one wave for all tiles (over 512 items): one key, 2 tiles and one key, 11;
# eight waves of 256 items, five tiles; four (over 256 items): five, eight and 13 tiles with ragged last ones
@pytest.mark.parametrize("shape", [
    (1, 1, 1, 1, 1, 1, 64), (31, 1, 31, 1, 1, 2, 128), (32, 1, 4, 8, 1, 1, 64), (33, 3, 1, 11, 2, 1, 128),
    (65, 5, 3, 17, 3, 2, 64), (40, 2, 8, 16, 1, 1, 128), (40, 1, 15, 17, 1, 1, 64), (40, 1, 257, 1, 1, 1, 128),
    (70, 9, 7, 13, 4, 3, 128), (20, 40, 1, 1, 12, 1, 64), (50, 33, 2, 3, 5, 1, 128),
    (33, 6, 16, 16, 2, 1, 64), (33, 17, 7, 13, 3, 1, 128), (40, 12, 9, 17, 3, 2, 64), (70, 1, 1, 1, 1, 171, 64),
    (65, 1, 5, 13, 1, 175, 128), (70, 3, 9, 13, 2, 175, 64),
    (33, 1, 10, 13, 1, 128, 64), (33, 1, 10, 13, 1, 129, 64), (70, 2, 9, 13, 1, 90, 64), (40, 3, 9, 15, 2, 130, 128)])
def test_tile_and_wave_edges(shape):
    Lq, frames, h, w, S, H, D = shape
    q, k, v, slot, uv, idx = _inputs(sum(shape), *shape)
    scale = D ** -0.5
    print(f"Lq={Lq} Lk={frames * h * w} grid {h}x{w} S={S} H={H} D={D}", flush=True)
    o, lse = rv.biased_chunk_attention(dev(q), dev(k), dev(v), dev(slot), dev(uv), dev(idx), h=h, w=w,
                                       softmax_scale=scale, lam=1.0, sigma=2.0)
    Oo, Lo = OA.biased_attention(q, k, v, slot, uv, idx, h, w, scale, 1.0, 2.0)
    assert np.abs(host(o) - Oo).max() <= TOL and np.abs(host(lse) - Lo).max() <= TOL


def test_infinities_stay_where_they_belong():
    """An infinite value of the last key reaches its column and no other (rows past the last key
    repeat nothing), and a key whose logits are -inf has weight 0 in whichever tile it stands."""
    Lq, frames, h, w, S, H, D = 33, 9, 7, 5, 2, 1, 64
    q, k, v, slot, uv, idx = _inputs(7, Lq, frames, h, w, S, H, D)
    q[:, :, 0] = 1.0
    k[5, :, 0] = k[40:104, :, 0] = -np.inf  # one key, and whole tiles
    v[-1, 0, 3] = np.inf
    o, lse = rv.biased_chunk_attention(dev(q), dev(k), dev(v), dev(slot), dev(uv), dev(idx), h=h, w=w,
                                       softmax_scale=D ** -0.5, lam=1.0, sigma=2.0)
    o, lse = host(o), host(lse)
    assert np.isposinf(o[:, 0, 3]).all() and np.isfinite(lse).all()
    dead = np.r_[5, 40:104]
    k[dead] = 0.0
    k[dead, :, 0] = -1e30  # the same weights, in finite numbers
    v[-1, 0, 3] = 0.0
    Oo, Lo = OA.biased_attention(q, k, v, slot, uv, idx, h, w, D ** -0.5, 1.0, 2.0)
    rest = np.arange(D) != 3
    assert np.abs(o[:, :, rest] - Oo[:, :, rest]).max() <= TOL and np.abs(lse - Lo).max() <= TOL


def test_no_finite_logit():
    """A row without a finite logit has no weights: its output is not a number, its neighbours' are."""
    Lq, frames, h, w, H, D = 4, 3, 5, 7, 1, 64
    q, k, v, slot, uv, idx = _inputs(11, Lq, frames, h, w, 0, H, D)
    q[:, :, 0], k[:, :, 0] = 0.5, 1.0
    q[2, :, 0] = -np.inf
    o, lse = rv.biased_chunk_attention(dev(q), dev(k), dev(v), dev(slot), None, None, h=h, w=w,
                                       softmax_scale=D ** -0.5, lam=1.0, sigma=2.0)
    o, lse = host(o), host(lse)
    assert np.isnan(o[2]).all() and np.isfinite(o[[0, 1, 3]]).all() and np.isfinite(lse[:, [0, 1, 3]]).all()
    assert np.isnan(lse[:, 2]).all()


@pytest.mark.parametrize("frames,H", [(2, 2), (7, 2), (2, 150), (1, 300)])  # 16, 56, 16 and 8 key tiles: eight waves, eight, four and one
@pytest.mark.parametrize("where", ["query", "tiles of one wave", "one key"])
def test_a_nan_shows_in_the_lse(where, frames, H):
    """A NaN logit makes its rows' sums NaN, and so their LSE, whichever waves hold it."""
    Lq, h, w, D = 35, 16, 16, 64
    q, k, v, slot, uv, idx = _inputs(13, Lq, frames, h, w, 0, H, D)
    bad = np.ones(Lq, bool)
    if where == "query":
        bad[:] = False
        bad[[3, 33]] = True
        q[bad, 0, 5] = np.nan
    elif where == "tiles of one wave":
        k.reshape(-1, 4, 32, H, D)[:, 3, :, 0, 5] = np.nan
    else:
        k[100, 0, 5] = np.nan
    o, lse = rv.biased_chunk_attention(dev(q), dev(k), dev(v), dev(slot), None, None, h=h, w=w,
                                       softmax_scale=D ** -0.5, lam=1.0, sigma=2.0)
    o, lse = host(o), host(lse)
    assert np.isnan(o[bad, 0]).all() and np.isnan(lse[0, bad]).all()
    assert np.isfinite(o[~bad, 0]).all() and np.isfinite(lse[0, ~bad]).all()
    assert np.isfinite(o[:, 1:]).all() and np.isfinite(lse[1:]).all()
