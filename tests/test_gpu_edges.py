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


# ------------------------------------------------------------ what-if sweep

# A tenant's sum is fp64 sums of features with the groups' integer sums
# rounded to fp32 (2^-24 relative each), times fp64 coefficients: with
# nonnegative terms within 2^-24 of exact plus fp64 rounding; 2^-23 bounds it.
SWEEP_RTOL = 2.0 ** -23


def check_sweep(L, tr, shapes, co, ext, pairs, tag):
    import torch
    dt = L.DeviceTrace.from_host(tr.offsets, tr.p, tr.c, tr.tenant)
    out = L.attribute_sweep(dt, shapes, co, tr.n_tenants, ext=ext)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    attr = oracle.attribute_ext if ext else oracle.attribute
    worst = 0.0
    for s, v in pairs:
        ref = attr(tr.offsets, tr.p, tr.c, tr.tenant, None if shapes is None else shapes[s], co[v],
                   tr.n_tenants, ("tenant_sums",))["tenant_sums"]
        assert np.array_equal(out[s, v][ref == 0], ref[ref == 0]), (tag, s, v)
        worst = max(worst, float(parity.rel_err(out[s, v], ref).max()))
    say(f"[sweep] {tag}: max rel err {worst:.2e}")
    assert worst <= SWEEP_RTOL, (tag, worst)
    return out


def sweep_sets(n, ext, seed=300):
    rng = np.random.default_rng(seed)
    base = tracegen.ext_coeffs(seed) if ext else tracegen.base_coeffs(seed)
    return (base[None, :] * rng.uniform(0.7, 1.4, (n, len(base)))).astype(np.float32)


@pytest.mark.parametrize("ext", [False, True])
@pytest.mark.parametrize("n_shapes,n", [(1, 1), (1, 63), (1, 64), (1, 65), (2, 64), (3, 43), (1, 256),
                                        (1, 257), (2, 256), (1, 513), (4, 256), (3, 342), (1, 1025)])
def test_sweep_settings(L, n_shapes, n, ext):
    """Setting counts around the 64-setting blocks, the blocks per wave (1, 2,
    4, 8), the waves side by side, the 1024-setting rounds, and more
    coefficient vectors than a round holds: the first and last settings of
    blocks and rounds against the oracle."""
    rng = np.random.default_rng(n)
    tr = fill(rng, rng.integers(0, 200, 120), n_tenants=33, p_empty=0.1)
    shapes = [tracegen.SHAPES[k] for k in sorted(tracegen.SHAPES)][:n_shapes]
    co = sweep_sets(n, ext)
    last = n_shapes * n - 1
    at = sorted({min(max(v, 0), last) for e in (0, 64, 512, 1024, last + 1) for v in (e - 1, e, e + 1)})
    check_sweep(L, tr, shapes, co, ext, [(v // n, v % n) for v in at], f"{n_shapes}x{n} ext={ext}")


@pytest.mark.parametrize("ext", [False, True])
@pytest.mark.parametrize("case", ["singles", "few-per-batch", "one-tenant", "hot-tenant", "bins-4096"])
def test_sweep_group_shapes(L, case, ext):
    """Rounds of 64 settings where the masks have no room for more (batches of
    one request), bins of no, one and many groups, chunks that end inside and
    on a bin's end, and both phases of every tenant."""
    rng = np.random.default_rng(sum(map(ord, case)))
    if case == "singles":
        tr = fill(rng, np.ones(5000, np.int64), n_tenants=9, p_empty=0.3)
    elif case == "few-per-batch":
        tr = fill(rng, rng.integers(0, 5, 4000), n_tenants=700)
    elif case == "one-tenant":
        tr = fill(rng, rng.integers(1, 40, 9000), n_tenants=1)
    elif case == "hot-tenant":
        tr = fill(rng, rng.integers(1, 300, 700), n_tenants=200)
        tr.tenant[rng.random(tr.n_requests) < 0.9] = 77
    else:
        tr = fill(rng, rng.integers(1, 900, 60), n_tenants=4096)
    shapes = [tracegen.SHAPES["qwen2.5-14b"], tracegen.SHAPES["70b-like"]]
    co = sweep_sets(70, ext, 400)
    check_sweep(L, tr, shapes, co, ext, [(0, 0), (0, 63), (0, 64), (1, 0), (1, 57), (1, 58), (1, 69)],
                f"{case} ext={ext}")


def test_sweep_under_capture(L):
    """The settings are host arrays: a captured sweep keeps their values, and
    replays after other work give the same sums."""
    import torch
    rng = np.random.default_rng(8)
    tr = fill(rng, rng.integers(0, 200, 300), n_tenants=50)
    dt = L.DeviceTrace.from_host(tr.offsets, tr.p, tr.c, tr.tenant)
    shapes = [tracegen.SHAPES["llama3.1-8b"]]
    co = sweep_sets(100, False)
    ws = L.sweep_workspace(tr.n_batches, tr.n_requests, 50)
    want = L.attribute_sweep(dt, shapes, co, 50).cpu()
    out = torch.empty((1, 100, 50), dtype=torch.float64, device="cuda")
    L.llmv_attribute_sweep(dt, shapes, co, 50, out, ws)  # loads the kernels
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        L.llmv_attribute_sweep(dt, shapes, co, 50, out, ws)
    co[:] = 0.0
    for _ in range(3):
        out.fill_(-1.0)
        ws.zero_()
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_allclose(out.cpu().numpy(), want.numpy(), rtol=1e-12)
        L.attribute(dt, shapes[0], tracegen.base_coeffs(3), 50)
        torch.cuda.synchronize()


# ------------------------------------------------------------ short traces


def sized(rng, N, lo, hi, extra=()):
    """Batch sizes from lo..hi (and the extra ones) adding up to N."""
    sizes = list(extra)
    while sum(sizes) < N:
        sizes.append(int(min(rng.integers(lo, hi + 1), N - sum(sizes))))
    rng.shuffle(sizes)
    assert sum(sizes) == N
    return sizes


@pytest.mark.parametrize("ext", [False, True])
@pytest.mark.parametrize("N,lo,hi,extra,T", [
    (1789, 1, 40, (0, 0), 1),                        # the first of the two-launch traces
    (2048, 0, 9, (508, 509, 512), 7),                # one workgroup; around a 512-slot tile
    (2049, 512, 513, (), 16),                        # every batch about a tile
    (4097, 0, 3, (), 4096),                          # more batches than offsets in a window
    (9000, 505, 520, (0, 1, 2), 300),                # tiles and long batches next to each other
    (14337, 1, 2000, (), 64),
    (40001, 0, 60, (30000,), 1024),                  # one batch over most of the chunks
    (114688, 0, 300, (0, 5000, 1025, 1024), 1000),   # the longest short trace
    (114689, 0, 300, (0, 5000, 1025, 1024), 1000),   # the next path
])
def test_short_trace(L, N, lo, hi, extra, T, ext):
    import torch
    rng = np.random.default_rng(N + T)
    sizes = sized(rng, N, lo, hi, extra)
    tr = fill(rng, [0, 0] + sizes + [0] * 70, n_tenants=T)
    shape = tracegen.SHAPES["llama3.1-8b"]
    co = tracegen.ext_coeffs(5) if ext else tracegen.base_coeffs(5)
    say(f"[short] N={tr.n_requests} nB={tr.n_batches} T={T} ext={ext}")
    dt = L.DeviceTrace.from_host(tr.offsets, tr.p, tr.c, tr.tenant)
    run, orc = ((L.attribute_ext, oracle.attribute_ext) if ext else (L.attribute, oracle.attribute))
    ref = orc(tr.offsets, tr.p, tr.c, tr.tenant, shape, co, T)
    for _ in range(2):  # the second call finds the first one's scratch
        g = {k: v.cpu().numpy() for k, v in run(dt, shape, co, T).items()}
        parity.compare(ref, tr.offsets, g["latency"], g["regime"], g["share"], g["tenant_sums"])
    for outs in (("latency", "tenant_sums"), ("share",), ("regime",)):
        h = run(dt, shape, co, T, outs)
        torch.cuda.synchronize()
        for k in outs:
            if k == "tenant_sums":
                np.testing.assert_allclose(h[k].cpu().numpy(), g[k], rtol=1e-12)
            else:
                assert np.array_equal(h[k].cpu().numpy(), g[k]), (outs, k)
