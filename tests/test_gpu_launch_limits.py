"""Calls of so many workgroups that one launch of one dimension (2^32 threads) does not hold them."""

from __future__ import annotations

import math

import numpy as np
import pytest
import torch

import paper_2607_21848_amd as rv
from oracle import retrieval as ORT
from tests.gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _give_back():
    torch.cuda.empty_cache()
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def _poses(x, y):
    m = torch.zeros(len(x), 4, 4, device="cuda")
    m[:, range(4), range(4)] = 1.0
    m[:, 0, 3], m[:, 1, 3] = x, y
    return m


@pytest.mark.parametrize("N,Q,k", [(4000, (1 << 22) + 5, 1), (4000, (1 << 22) + 5, 5), (8200, (1 << 23) + 5, 1)])
def test_retrieval_of_many_queries(N, Q, k):
    """2^22 + 5 queries over 4000 entries, which sixteen waves a query would scan; 2^23 + 5 segments of
    eight waves."""
    g = torch.Generator(device="cuda").manual_seed(k)
    r = lambda n: 20 * torch.rand(n, generator=g, device="cuda")  # noqa: E731
    bank, query = _poses(r(N), r(N)), _poses(r(Q), r(Q))
    chunk = torch.full((Q,), N + 3, dtype=torch.int32, device="cuda")
    kw = dict(E=20.0, w_v=0.5, tau_c=0.02, tau_v=1.0, delta=3, first_candidate=1, k=k)
    print(f"N={N} Q={Q} k={k}", flush=True)
    idx, score, count, _ = rv.retrieve_chunks(bank, query, chunk, **kw)
    at = torch.tensor([0, 1, 4095, 1 << 20, (1 << 22) - 1, 1 << 22, Q - 6, Q - 5, Q - 1], device="cuda")
    want_i, want_s, want_c = ORT.retrieve(host(bank), host(query[at]), host(chunk[at]), 20.0, 0.5, 0.02, 1.0, 3, 1, k)
    assert want_c.max() > 0
    assert np.array_equal(host(idx[at]), want_i) and np.array_equal(host(count[at]), want_c)
    assert np.array_equal(host(score[at]), want_s.astype(np.float32))


def test_fp32_attention_of_many_items():
    """2^23 + 1 tiles of 32 queries (one key: every output is that key's value). 137 GB."""
    D, H = 64, 33
    Lq = 32 * ((1 << 23) // H + 1)
    q = torch.ones(Lq, H, D, device="cuda")
    k, v = torch.ones(1, H, D, device="cuda"), torch.randn(1, H, D, device="cuda")
    print(f"Lq={Lq} H={H} D={D}: {Lq // 32 * H} items", flush=True)
    o, lse = rv.biased_chunk_attention(q, k, v, dev(np.full(1, -1, np.int32)), None, None, h=1, w=1,
                                       softmax_scale=D ** -0.5, lam=1.0, sigma=2.0)
    for c in o.split(1 << 20):
        assert torch.equal(c, v.expand_as(c))
    assert (lse - D ** 0.5).abs().max().item() <= 1e-5


def test_stream_of_many_heads_and_layers():
    """bf16, one token a chunk, 256 heads of 65536 layers: 2^24 attention items a step. 104 GB."""
    L, H, D = 1 << 16, 256, 128
    s = rv.StreamDriver(F=1, h=1, w=1, p=1, H=H, D=D, layers=L, dtype=torch.bfloat16, capacity=5, max_chunks=4, E=4.0,
                        w_v=0.5, tau_c=0.1, tau_v=0.7, delta=3, eps=0.05, lam=1.0, sigma=2.0, softmax_scale=D ** -0.5,
                        rope_t_pairs=22, rope_theta=10000.0)
    depth, K = torch.ones(1, 1, 1, device="cuda"), torch.ones(1, 4, device="cuda")
    pose = torch.eye(4, device="cuda")[None].contiguous()
    q = torch.zeros(L, 1, H, D, dtype=torch.bfloat16, device="cuda")
    vs = []
    for n in range(2):
        v = torch.randn(L, 1, H, D, device="cuda", dtype=torch.bfloat16)
        vs.append(v)
        print(f"chunk {n}: {L * H} items", flush=True)
        o, lse = s.step(depth, pose, K, q, q, v)
        # q = 0: the mean of the values so far, rounded to bf16
        for l0 in range(0, L, 4096):
            want = torch.stack([x[l0:l0 + 4096].float() for x in vs]).mean(0)
            assert (o[l0:l0 + 4096].float() - want).abs().max().item() <= 2.0 ** -7 * max(1.0, want.abs().max().item())
        assert (lse - math.log(n + 1)).abs().max().item() <= 1e-5
    s.close()
