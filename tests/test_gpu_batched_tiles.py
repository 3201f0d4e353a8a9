"""Batched matvec pair over many tiles: the orders in which tiles are dealt out,
longer tiles for many rows, and batches that the memory-side cache does not hold.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def N():
    from paper_2202_11599_amd import nysadmm
    return nysadmm


def first_step(N, ctx, shapes, seed=23):
    """One ADMM step of the batch and the FP64 solution of its subproblem: with a
    factor whose lambda is 0 the preconditioner is the identity and z stays 0,
    so x = (A^T A + rho I)^-1 A^T b rests on the pair alone."""
    rho = 0.5
    g = torch.Generator(device=DEV).manual_seed(seed)
    probs, opts, facs, keep = [], [], [], []
    for n, d, dt in shapes:
        # ||A|| about 1 + sqrt(d / n) before the scaling by 1/2: condition below 4
        A = (torch.randn(n, d, generator=g, device=DEV, dtype=torch.float64) * 0.5 * n ** -0.5).to(dt)
        b = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
        U = torch.zeros(1, d, dtype=torch.float64, device=DEV)
        U[0, 0] = 1.0
        F = N.nys_factor_import(ctx, U, [0.0])
        facs.append(F)
        keep.append((A, b, U))
        probs.append(N.problem(A, b, 1e9))
        opts.append(N.admm_opts(rho, 1, U, factor=F, max_iter=1,
                                pcg=N.pcg_opts(tol=1e-13, max_iter=200)))
    st = [N.State(k[0].shape[1], DEV) for k in keep]
    N.admm_solve(ctx, probs, opts, st, allow=(N.NYS_OK, N.NYS_ERR_MAXITER))
    errs = []
    for (A, b, _), s in zip(keep, st):
        H = rho * torch.eye(A.shape[1], dtype=torch.float64, device=DEV)
        v = torch.zeros(A.shape[1], dtype=torch.float64, device=DEV)
        for i in range(0, A.shape[0], 16384):
            a = A[i:i + 16384].double()
            at = a.t().contiguous()
            H += at @ a
            v += at @ b[i:i + 16384]
        x = torch.linalg.solve(H.cpu(), v.cpu())
        errs.append(float((s.x.cpu() - x).norm() / x.norm()))
    for f in facs:
        f.close()
    print("[batched tiles]", shapes, ["%.1e" % e for e in errs], flush=True)
    return errs


# condition 4 and a residual of 1e-13 give 4e-13; the reference's own sums of up
# to 3e5 terms add about sqrt(3e5) roundings, 6e-14: within 1e-12
F32, F64 = torch.float32, torch.float64


@pytest.mark.parametrize("shapes", [
    # more tiles of 128 rows than CUs (256) and fewer than twice as many
    [(15000, 40, F32), (14001, 300, F64), (9007, 129, F32)],
    # past 16 tiles per CU: tiles of 256 rows (rows of few columns keep it small)
    [(300001, 24, F32), (299993, 17, F32)],
])
def test_batched_tile_counts(N, shapes):
    ctx = N.Context()
    assert max(first_step(N, ctx, shapes)) < 1e-12
    ctx.close()


# just above 240 MB together
STREAMING = [
    [(70001, 500, F32), (40003, 515, F32), (60000, 129, F64)],
    [(30001, 1300, F32), (20000, 1024, F32), (9001, 700, F64)],
    [(20003, 1900, F32), (150000, 100, F64), (4001, 3000, F32)],
]


@pytest.mark.parametrize("tune", ["0", None])
@pytest.mark.parametrize("shapes", STREAMING)
def test_batched_streaming_parity(N, monkeypatch, shapes, tune):
    if tune is not None:
        monkeypatch.setenv("NYSADMM_TUNE", tune)
    assert sum(n * d * (8 if t == F64 else 4) for n, d, t in shapes) > 240 * 2 ** 20
    ctx = N.Context()
    assert max(first_step(N, ctx, shapes)) < 1e-12
    ctx.close()


@pytest.mark.parametrize("rows,timed", [(140000, True), (20000, False)])
def test_batched_streaming_is_timed(N, monkeypatch, capfd, rows, timed):
    """Which kernel is faster for a streaming batch depends on how its columns
    fill the lanes, so the launch shapes of narrow rows are timed; a batch that
    the cache holds has one launch and nothing to time."""
    monkeypatch.setenv("NYSADMM_VERBOSE", "1")
    ctx = N.Context()
    err = first_step(N, ctx, [(rows, 300, F32), (rows, 300, F32)])
    assert ("batched bucket" in capfd.readouterr().err) == timed
    assert max(err) < 1e-12
    ctx.close()
