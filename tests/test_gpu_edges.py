"""Edges of the kernels' tiles, rows and dispatch rules, against the oracle
(tolerances: tests/parity.py, unless a test states its own)."""
import sys

import numpy as np
import pytest

import oracle
import parity
import tracegen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def L():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2608_08382_amd import llmv
    llmv.load()
    torch.cuda.set_device(0)
    return llmv


def fill(rng, sizes, n_tenants=1, p_prefill=0.3, p_empty=0.0):
    """A trace of the given batch sizes: whole prefill and decode batches and
    a few mixed ones."""
    sizes = np.array(sizes, np.int64)
    if p_empty:
        sizes[rng.random(len(sizes)) < p_empty] = 0
    off = np.zeros(len(sizes) + 1, np.int64)
    off[1:] = np.cumsum(sizes)
    N = int(off[-1])
    pre = np.repeat(rng.random(len(sizes)) < p_prefill, sizes) | (rng.random(N) < 0.002)
    p = np.where(pre, rng.integers(1, 16385, N), 1).astype(np.int32)
    c = np.where(pre, rng.integers(0, 3, N), rng.integers(1, 131073, N)).astype(np.int32)
    t = rng.integers(0, n_tenants, N).astype(np.int32)
    return tracegen.Trace(off, p, c, t, n_tenants, None)


@pytest.mark.parametrize("tail", [0, 1, 2, 3])
def test_feature_rows_at_every_alignment(L, tail):
    """Row k of the feature rows starts at x_req + k*N: N mod 4 decides which
    rows are 16-byte aligned.  Whole tiles, remainders, empty batches and
    batches of two and three tiles; each output also on its own."""
    import torch
    rng = np.random.default_rng(40 + tail)
    sizes = list(rng.integers(0, 300, 180)) + [1792, 1793, 3585, 5000, 1, 0, 7]
    sizes.append((tail - sum(sizes)) % 4 + 8)
    tr = fill(rng, sizes, p_empty=0.1)
    # keep N mod 4 after some batches were emptied
    extra = (tail - tr.n_requests) % 4
    tr = fill(rng, list(tr.sizes()) + [extra])
    assert tr.n_requests % 4 == tail
    shape = tracegen.SHAPES["qwen2.5-32b"]
    dt = L.DeviceTrace.from_host(tr.offsets, tr.p, tr.c)
    rr, rb = oracle.features(tr.offsets, tr.p, tr.c, shape)
    xr, xb = L.features(dt, shape)
    only_r, only_b = torch.full_like(xr, -1.0), torch.full_like(xb, -1.0)
    ws = L.workspace(tr.n_batches, tr.n_requests, 0)
    L.llmv_features(dt, shape, only_r, None, ws)
    L.llmv_features(dt, shape, None, only_b, ws)
    torch.cuda.synchronize()
    say(f"[features] N={tr.n_requests} nB={tr.n_batches}")
    # each value is an fp64 product rounded once to fp32
    assert parity.rel_err(xr.cpu().numpy(), rr).max() <= 2.0 ** -23
    assert parity.rel_err(xb.cpu().numpy(), rb).max() <= 1e-12
    assert torch.equal(only_r, xr) and torch.equal(only_b, xb)
