"""Tenant sums of traces whose tenants do not fit an LDS histogram: the split
by table and log (a workspace of llmv_workspace_size bytes) against the sums
of the shares it wrote, and against the tenant cache (a workspace without the
log), whose latencies, regimes and shares must be the same bits."""
import numpy as np
import pytest
import torch

import tracegen
from paper_2608_08382_amd import llmv

pytestmark = pytest.mark.gpu
MIN = 1 << 20  # shares from which on the split is taken


def _bin0(T):
    """The tenants of the split's first bin."""
    bits = max(13, int(T - 1).bit_length())
    t = np.arange(T, dtype=np.uint64)
    mixed = ((((t >> np.uint64(3)) * np.uint64(0x9E3779B1)) & np.uint64((1 << (bits - 3)) - 1))
             << np.uint64(3)) | (t & np.uint64(7))
    return np.nonzero((mixed >> np.uint64(bits - 8)) == 0)[0]


def _tenants(rng, kind, n, T):
    if kind == "uniform":
        return rng.integers(0, T, n)
    if kind == "one":  # every share on the last tenant
        return np.full(n, T - 1)
    if kind == "bin":  # one bin only: its regions overflow
        return rng.choice(_bin0(T), n)
    return np.minimum((rng.pareto(0.2, n) * 2).astype(np.float64), T - 1).astype(np.int64)


@pytest.mark.parametrize("ext", [False, True])
@pytest.mark.parametrize("kind,n,T", [
    ("uniform", MIN, 4097), ("skew", MIN + 1, 8191), ("one", MIN + 8191, 8193),
    ("uniform", MIN + 4095, 1 << 20), ("skew", 3 * MIN + 3, (1 << 20) + 1),
    ("bin", MIN + 2, 1 << 16), ("bin", 2 * MIN + 5, 1 << 20), ("uniform", MIN + 7, 1 << 22),
    ("uniform", MIN + 7, (1 << 22) + 1), ("uniform", MIN - 1, 1 << 16)])
def test_split_tenant_sums(kind, n, T, ext):
    rng = np.random.default_rng(n + T)
    sizes = rng.integers(0, 300, 2 * n // 300 + 400)
    off = np.concatenate([[0], np.minimum(np.cumsum(sizes), n)])
    off[-1] = n
    t = _tenants(rng, kind, n, T)
    tr = llmv.DeviceTrace.from_host(off, rng.integers(1, 64, n), rng.integers(0, 5000, n), t)
    call = llmv.attribute_ext if ext else llmv.attribute
    co = (tracegen.ext_coeffs if ext else tracegen.base_coeffs)(3)
    ws = llmv.workspace(tr.n_batches, n, T)
    bare = llmv.workspace(tr.n_batches, n, (1 << 22) + 1)
    assert (ws.numel() > bare.numel()) == (n >= MIN and 4096 < T <= 1 << 22)
    got = call(tr, None, co, T, ws=ws)
    old = call(tr, None, co, T, ws=bare)
    for k in ("latency", "regime", "share"):
        assert torch.equal(got[k], old[k])
    share = got["share"].cpu().numpy().astype(np.float64)
    ref = np.bincount(t, weights=share, minlength=T)
    # positive terms added in fp64 in any order: n * 2^-53 relative, on both sides
    tol = 2 * n * 2.0 ** -53
    for out in (got, old):
        ts = out["tenant_sums"].cpu().numpy()
        assert np.all(np.abs(ts - ref) <= tol * ref)
    # again on the same workspace: nothing is left of the first call
    again = call(tr, None, co, T, ws=ws)["tenant_sums"].cpu().numpy()
    assert np.all(np.abs(again - ref) <= tol * ref)
