"""The matvec pair of narrow matrices (up to 1024 columns) that the memory-side
cache does not hold: whole rows per wavefront with non-temporal loads, and the
choice between that form and the one workgroup per row.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def N():
    from paper_2202_11599_amd import nysadmm
    return nysadmm


def pair_fp64(A, D, p, rho):
    """A^T (D o (A p)) + rho p in FP64, 8192 rows at a time"""
    v = rho * p
    for i in range(0, A.shape[0], 8192):
        a = A[i:i + 8192].double()
        s = a @ p
        v = v + a.t().contiguous() @ (s if D is None else D[i:i + 8192] * s)
    return v


# just above 240 MB; every number of chunks per lane (256, 512, 1024 FP32 and
# 128 .. 1024 FP64 columns), whole and ragged rows, padded rows, a first row off
# the 16-byte grid
SHAPES = [
    # n, d, dtype, ld, column offset, weights
    (70001, 1003, torch.float32, 1003, 0, True),
    (130003, 500, torch.float32, 500, 0, True),
    (126000, 513, torch.float32, 515, 1, False),
    (300007, 250, torch.float32, 253, 3, True),
    (64000, 1024, torch.float32, 1024, 0, False),
    (35001, 1001, torch.float64, 1001, 0, True),
    (64003, 511, torch.float64, 512, 1, False),
    (130001, 257, torch.float64, 257, 0, True),
    (270011, 120, torch.float64, 123, 0, True),
]


@pytest.mark.parametrize("plan", ["rows", None])
@pytest.mark.parametrize("n,d,dtype,ld,off,weights", SHAPES)
def test_streaming_pair_parity(N, monkeypatch, n, d, dtype, ld, off, weights, plan):
    """A wavefront's y is a chain of n / 2048 rows at most, then 8 wavefronts
    and 256 workgroups are added, after a dot product of d terms: 700 + d
    roundings, against sums of absolute values some 0.7 sqrt(d) times the
    result (Gaussian A, A^T A p about n p): below 3e-12 relative for d = 1024."""
    if plan is not None:
        monkeypatch.setenv("NYSADMM_GRAM_PLAN", plan)
    g = torch.Generator(device=DEV).manual_seed(n + d)
    A = torch.randn(n, ld, generator=g, device=DEV, dtype=dtype)[:, off:off + d]
    assert n * ld * A.element_size() > 240 * 2 ** 20
    p = torch.randn(d, generator=g, device=DEV, dtype=torch.float64)
    D = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) if weights else None
    ctx = N.Context()
    v, pv = N.nys_hessian_apply(ctx, A, p, rho=1e-3, D=D, want_pv=True)
    torch.cuda.synchronize()
    ref = pair_fp64(A, D, p, 1e-3)
    err = float((v - ref).norm() / ref.norm())
    print(f"[streaming pair] {n} x {d} {dtype} ld={ld} off={off} plan={plan}: {err:.1e}", flush=True)
    assert err < 3e-12
    assert abs(pv - float(p @ ref)) <= 3e-12 * abs(float(p @ ref))
    ctx.close()


@pytest.mark.parametrize("n,d,timed", [(300000, 257, True), (60000, 257, False)])
def test_streaming_pair_is_timed(N, monkeypatch, capfd, n, d, timed):
    """Which form is faster for a streaming A depends on how its columns fill the
    lanes, so the forms are timed; one that the cache holds has one form."""
    monkeypatch.setenv("NYSADMM_VERBOSE", "1")
    monkeypatch.delenv("NYSADMM_TUNE", raising=False)
    ctx = N.Context()
    A = torch.ones(n, d, device=DEV, dtype=torch.float32)
    p = torch.ones(d, device=DEV, dtype=torch.float64)
    v = N.nys_hessian_apply(ctx, A, p, rho=0.0)
    torch.cuda.synchronize()
    assert ("matvec plan for" in capfd.readouterr().err) == timed
    assert bool((v == float(n) * d).all())   # whole numbers: exact
    ctx.close()


def test_first_pair_inside_a_capture(N):
    """A narrow shape that would be timed is captured on its first call too, in
    a workspace (nothing is allocated), and the graph replays."""
    n, d = 300000, 257
    stream = torch.cuda.Stream()
    A = torch.randn(n, d, device=DEV, dtype=torch.float32)
    p = torch.ones(d, device=DEV, dtype=torch.float64)
    out = torch.zeros_like(p)
    ctx = N.Context(stream=stream)
    ctx.set_workspace(torch.empty(ctx.workspace_query(A, 1), dtype=torch.uint8, device=DEV))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        N.nys_hessian_apply(ctx, A, p, rho=0.5, out=out)
    for k in range(4):
        p.copy_(torch.randn(d, device=DEV, dtype=torch.float64))
        out.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        ref = pair_fp64(A, None, p, 0.5)
        assert float((out - ref).norm() / ref.norm()) < 3e-12, k
    ctx.close()
