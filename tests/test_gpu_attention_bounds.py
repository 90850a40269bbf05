"""bf16 and fp8 attention over keys that end an allocation: 8.5 key tiles in one part, where the
pipeline's steady steps reach the tile that runs past the last key. Keys fill a whole number of
2 MiB pages, so that a row read past them would belong to nobody."""

from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2607_21848_amd as rv
import workloads as W
from oracle import attention as OA
from tests.gpu_helpers import dev, host
from workloads.synth import fp8e4m3_bits

pytestmark = pytest.mark.gpu

O_TOL, LSE_TOL = 2e-2, 4e-3  # the bf16 bars


@pytest.mark.parametrize("kind,H", [("bf16", 512), ("fp8", 1024)])
@pytest.mark.parametrize("S", [0, 1])
def test_last_key_tile_runs_past_the_keys(kind, H, S):
    Lq, h, w, D = 2, 16, 17, 128
    rng = np.random.default_rng(H + S)
    q, k, v = (rng.standard_normal((L, H, D), dtype=np.float32) for L in (Lq, h * w, h * w))
    slot = np.full(1, 0 if S else -1, np.int32)
    uv = np.stack([rng.uniform(0, w, (S, Lq)), rng.uniform(0, h, (S, Lq))], -1).astype(np.float32)
    idx = rng.integers(-4, h * w, size=(S, Lq)).astype(np.int32)
    v = W.bf16_round(v)
    if kind == "bf16":
        q, k = W.bf16_round(q), W.bf16_round(k)
        tq, tk = dev(q, torch.bfloat16), dev(k, torch.bfloat16)
    else:
        q8, k8 = fp8e4m3_bits(q), fp8e4m3_bits(k)
        q, k = OA.fp8e4m3_values(q8), OA.fp8e4m3_values(k8)
        tq, tk = (torch.from_numpy(x).cuda().view(torch.float8_e4m3fn) for x in (q8, k8))
    assert tk.numel() * tk.element_size() % (2 << 20) == 0
    print(f"{kind} H={H} S={S} Lk={h * w}", flush=True)
    o, lse = rv.biased_chunk_attention(tq, tk, dev(v, torch.bfloat16), dev(slot), dev(uv) if S else None,
                                       dev(idx) if S else None, h=h, w=w, softmax_scale=D ** -0.5, lam=1.0, sigma=2.0,
                                       key_parts=1)
    at = [0, 1, H // 2, H - 1]
    Oo, Lo = OA.biased_attention(*(np.ascontiguousarray(x[:, at]) for x in (q, k, v)), slot, uv, idx, h, w, D ** -0.5, 1.0, 2.0)
    assert np.abs(host(o)[:, at] - Oo).max() <= O_TOL and np.abs(host(lse)[at] - Lo).max() <= LSE_TOL
