"""The two launches of reproject_rotation (a block for all sources, a block per source) give the same
bits: whole batches against batches of a few problems, which take a block per source, and against
the oracle. Odd grids (pairs that start in the middle of an aligned pair), frames smaller than a
block, empty slots and moved centres, and outputs that are not 16-byte aligned."""

from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2607_21848_amd as rv
import workloads as W
from oracle import reprojection as R

pytestmark = pytest.mark.gpu


def _d(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _bits(t):
    return t.view(torch.int32) if t.dtype == torch.float32 else t


# (B, Tq, S, h, w): more than 512 blocks of all sources, little output; the same with odd frames;
# frames of one partial block; 9.1e6 pairs and few sources (a block per source), odd and even; one
# column of odd height whose blocks take more than 128 pairs, in a small and in a large launch (the
# column of a thread's token is then stepped by 0); frames that end on lines, of three sources (a
# block per source) and of four
@pytest.mark.parametrize("B,Tq,S,h,w", [(60, 3, 6, 30, 52), (40, 3, 9, 45, 35), (600, 1, 3, 5, 7), (650, 3, 3, 30, 52),
                                        (600, 1, 7, 41, 53), (520, 1, 1, 1, 1), (10, 4, 64, 301, 1),
                                        (2600, 1, 7, 513, 1), (2700, 1, 3, 30, 40),
                                        (2000, 1, 4, 30, 40)])
@pytest.mark.parametrize("shift", [0, 1])
def test_launches_agree(B, Tq, S, h, w, shift):
    tc, tk, sc, sk = W.make_rotation_batch(B, Tq=Tq, S=S, h=h, w=w, p=2, distinct=5, seed=B + h)
    sc = sc.copy()
    sc[1, 0, 0, 3] += 0.5  # a moved centre
    sel = np.arange(B * S, dtype=np.int32).reshape(B, S)
    sel[2, S - 1] = -1  # an empty slot
    args = [_d(x) for x in (tc, tk, sc.reshape(B * S, 4, 4), sk.reshape(B * S, 4), sel)]
    Lq = Tq * h * w
    print(f"B={B} Tq={Tq} S={S} {h}x{w} shift={shift}", flush=True)

    def run(b0, b1):
        n = (b1 - b0) * S * Lq
        uv = torch.zeros(2 * n + 2, device="cuda")[2 * shift:2 * shift + 2 * n].view(b1 - b0, S, Lq, 2)
        idx = torch.zeros(n + 1, dtype=torch.int32, device="cuda")[shift:shift + n].view(b1 - b0, S, Lq)
        return rv.reproject_rotation(args[0][b0:b1].contiguous(), args[1][b0:b1].contiguous(), args[2], args[3], h=h, w=w,
                                     p=2, src_sel=args[4][b0:b1].contiguous(), out=(uv, idx))

    uv, idx = run(0, B)
    for b0 in (0, 4, B - 4):
        fu, fi = run(b0, b0 + 4)
        assert torch.equal(_bits(uv[b0:b0 + 4]), _bits(fu)) and torch.equal(idx[b0:b0 + 4], fi)
    for b in (0, 1, 2, B - 1):
        wu, wi = R.reproject_rotation(tc[b], tk[b], sc[b], sk[b], h, w, 2)
        if b == 2:
            wu, wi = wu.copy(), wi.copy()
            wu[S - 1], wi[S - 1] = np.nan, R.NO_SOURCE
        assert np.array_equal(idx[b].cpu().numpy(), wi)
        assert np.array_equal(uv[b].cpu().numpy(), wu.astype(np.float32), equal_nan=True)
