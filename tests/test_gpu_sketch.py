"""GPU parity of the randomized Nystrom sketch and its FP64 core against the
oracle (Algorithm RandNysAppx / AdaptiveRandNysAppx), through the C ABI.

U is not unique (signs, rotations inside clusters), so the comparisons use
H_hat = U Lambda U^T, Lambda and the shift nu.  Bars:
  FP64 sketch  ||H_hat - H_hat_oracle|| <= 1e-10 ||H_hat_oracle||
  FP32 sketch  <= 1e-5 (FP32 MFMA, FP64 core)
  BF16 sketch  error reported against the FP64 oracle, sanity bound only.
"""
import numpy as np
import pytest
import torch

from oracle import nystrom as ny
from oracle import pcg as pc
from paper_2202_11599_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def N():
    from paper_2202_11599_amd import nysadmm
    return nysadmm


@pytest.fixture(scope="module")
def ctx(N):
    c = N.Context()
    yield c
    c.close()


def hhat(F, ctx):
    inf = F.info()
    U = F.U(ctx).cpu().numpy().T          # d x r
    lam = np.array(inf["lam"])
    return (U * lam) @ U.T, U, lam, inf


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def test_sketch_fp64_c1_parity(N, ctx):
    p = synth.lasso_c1()
    A = p.A.numpy()
    om = p.omega                                  # (50, 500) rows = columns
    F = N.nys_sketch(ctx, p.A.to(DEV), om.to(DEV), prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A, None, 0.0, om.numpy().T)
    print(f"[sketch fp64 c1] rel(Hhat)={rel(H, f.dense()):.3e} nu={inf['nu']:.3e}/{f.nu:.3e}", flush=True)
    assert rel(H, f.dense()) < 1e-10
    assert np.allclose(lam, f.lam, rtol=1e-10, atol=1e-12 * f.lam[0])
    assert inf["nu"] == f.nu
    assert np.linalg.norm(U.T @ U - np.eye(50)) < 1e-10
    assert inf["rank"] == 50 and inf["lambda_s"] == lam[-1]
    F.close()


def test_sketch_fp64_weights_and_shift(N, ctx):
    # H = A^T diag(D) A + c I (logistic weights, elastic-net shift)
    A64 = synth.decay_matrix(3000, 300, 0.5, seed=21)
    D = torch.rand(3000, dtype=torch.float64, generator=torch.Generator().manual_seed(4)) * 0.25
    om = synth.omega_raw(300, 40, seed=21)
    F = N.nys_sketch(ctx, A64.to(DEV), om.to(DEV), D=D.to(DEV), c=0.3, prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A64.numpy(), D.numpy(), 0.3, om.numpy().T)
    assert rel(H, f.dense()) < 1e-10
    assert inf["nu"] == f.nu
    F.close()


def test_sketch_fp64_rank_deficient_exact(N, ctx):
    # rank(H) = 7 <= r = 12: the approximation is exact (Lemma NysPropLemma)
    g = torch.Generator().manual_seed(5)
    A64 = torch.randn(200, 7, generator=g, dtype=torch.float64) @ torch.randn(7, 60, generator=g, dtype=torch.float64)
    om = synth.omega_raw(60, 12, seed=5)
    F = N.nys_sketch(ctx, A64.to(DEV), om.to(DEV), prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    Ht = A64.numpy().T @ A64.numpy()
    assert rel(H, Ht) < 1e-10
    assert np.all(lam[7:] <= 1e-10 * lam[0])
    F.close()


# the last three run the first pass as full rounds of 16-wavefront workgroups
# plus a launch for the remaining rows (4125, 4376 and 8193 row blocks of 16:
# 29, 280 and 1 block left, the last one holding 5 rows)
@pytest.mark.parametrize("n,d,r", [(20000, 1000, 100), (5003, 517, 37), (30000, 2000, 200),
                                   (66000, 257, 100), (70001, 300, 200), (131077, 257, 200)])
def test_sketch_fp32_parity(N, ctx, n, d, r):
    print(f"[sketch fp32] n={n} d={d} r={r}", flush=True)
    A64 = synth.decay_matrix(n, d, 0.8, seed=n % 97)
    A32 = A64.to(torch.float32)
    om = synth.omega_raw(d, r, seed=3)
    F = N.nys_sketch(ctx, A32.to(DEV), om.to(DEV), prec=N.NYS_F32)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A32.double().numpy(), None, 0.0, om.numpy().T, mantissa_bits=23)
    e = rel(H, f.dense())
    print(f"[sketch fp32] rel(Hhat)={e:.3e} nu={inf['nu']:.3e}/{f.nu:.3e}", flush=True)
    assert e < 1e-5
    assert inf["nu"] == f.nu
    assert np.linalg.norm(U.T @ U - np.eye(r)) < 1e-8
    F.close()


def test_sketch_bf16_reported(N, ctx):
    n, d, r = 20000, 1000, 100
    A32 = synth.decay_matrix(n, d, 0.8, seed=9).to(torch.float32)
    om = synth.omega_raw(d, r, seed=9)
    F = N.nys_sketch(ctx, A32.to(DEV), om.to(DEV), prec=N.NYS_BF16)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A32.double().numpy(), None, 0.0, om.numpy().T, mantissa_bits=23)
    e = rel(H, f.dense())
    el = float(np.max(np.abs(lam[:10] - f.lam[:10]) / f.lam[:10]))
    print(f"[sketch bf16] FP64-oracle error: rel(Hhat)={e:.3e}, top-10 eigenvalue rel err={el:.3e}", flush=True)
    assert e < 3e-2
    assert np.all(np.diff(lam) <= 0) and np.all(lam >= 0)
    F.close()


def test_sketch_append_and_adaptive(N, ctx):
    # Algorithm AdaptiveRandNysAppx: blocks of consecutive omega columns, rank
    # 5, 10, 20, 40 ... until (lambda_s + rho)/rho <= Tol.
    d = 240
    A64 = synth.decay_matrix(2000, d, 1.0, seed=31)
    om = synth.omega_raw(d, 160, seed=31)
    rho, tol = 1e-3, 2.0
    F = N.nys_sketch_adaptive(ctx, A64.to(DEV), om.to(DEV), 5, 160, rho, tol, prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    f, hist = ny.adaptive_rand_nys_appx(A64.numpy(), None, 0.0, om.numpy().T, rho, 5, 160, tol)
    print(f"[adaptive] gpu rank {inf['rank']} oracle ranks {hist}", flush=True)
    assert inf["rank"] == hist[-1][0]
    assert rel(H, f.dense()) < 1e-9
    # explicit append equals the adaptive blocks
    F2 = N.nys_sketch(ctx, A64.to(DEV), om[:5].contiguous().to(DEV), prec=N.NYS_F64)
    F2 = N.nys_sketch(ctx, A64.to(DEV), om[5:10].contiguous().to(DEV), prec=N.NYS_F64, factor=F2)
    H2, _, _, inf2 = hhat(F2, ctx)
    Href = ny.nystrom_definition(A64.numpy().T @ A64.numpy(),
                                 np.concatenate([ny.orthonormalize(om[:5].numpy().T),
                                                 ny.orthonormalize(om[5:10].numpy().T)], axis=1))
    assert inf2["rank"] == 10
    assert rel(H2, Href) < 1e-8
    F.close()
    F2.close()


def test_pcg_with_gpu_factor_matches_oracle_iterations(N, ctx):
    p = synth.lasso_c1()
    A = p.A.numpy()
    F = N.nys_sketch(ctx, p.A.to(DEV), p.omega.to(DEV), prec=N.NYS_F64)
    f = ny.rand_nys_appx(A, None, 0.0, p.omega.numpy().T)
    rhs = A.T @ p.b.numpy()
    ora = pc.nys_pcg(pc.subproblem_matvec(A, None, 0.0, 1.0), rhs, np.zeros(500),
                     pc.nystrom_precond(f, 1.0), 1e-10)
    x = torch.zeros(500, dtype=torch.float64, device=DEV)
    info = N.pcg_solve(ctx, p.A.to(DEV), torch.from_numpy(rhs).to(DEV), x, 1.0, F,
                       opts=N.pcg_opts(tol=1e-10))
    assert abs(info.iters - ora.iters) <= 1
    xs = pc.dense_solve(A, None, 0.0, 1.0, rhs)
    assert np.linalg.norm(x.cpu().numpy() - xs) <= 1e-6 * np.linalg.norm(xs)
    F.close()


def test_sketch_invalid_and_not_spd(N, ctx):
    A = synth.decay_matrix(100, 20, 0.5, seed=1).to(DEV)
    with pytest.raises(N.NysError) as e:
        N.nys_sketch(ctx, A, synth.omega_raw(20, 20, seed=1).to(DEV))     # r >= d
    assert e.value.status == N.NYS_ERR_INVALID
    om = synth.omega_raw(20, 5, seed=1)
    om[2] = 0.0                                                           # zero Gaussian column
    with pytest.raises(N.NysError) as e:
        N.nys_sketch(ctx, A, om.to(DEV))
    assert e.value.status == N.NYS_ERR_NOT_SPD


@pytest.mark.parametrize("prec", ["f32", "bf16"])
def test_sketch_full_size_properties(N, ctx, prec):
    # 100000 x 4000 FP32 with sigma_j = j^-0.8 at rank 200 in the launch
    # configuration of the bench: properties that hold at any size --
    # Lambda descending and >= 0, U orthonormal, x^T H_hat x <= x^T H x
    # (Lemma NysPropLemma, up to the sketch rounding), and the leading Ritz
    # values close to sigma_j^2.
    n, d, r = 100000, 4000, 200
    print(f"[sketch full] {prec} n={n} d={d} r={r}", flush=True)
    A = synth.decay_matrix(n, d, 0.8, seed=0, device=DEV).to(torch.float32)
    om = synth.omega_raw(d, r, seed=0, device=DEV)
    F = N.nys_sketch(ctx, A, om, prec=N.NYS_F32 if prec == "f32" else N.NYS_BF16)
    inf = F.info()
    lam = np.array(inf["lam"])
    U = F.U(ctx)
    assert np.all(np.diff(lam) <= 0) and lam[-1] >= 0
    orth = torch.linalg.norm(U @ U.T - torch.eye(r, dtype=torch.float64, device=DEV)).item()
    assert orth < 1e-6
    g = torch.Generator(device=DEV).manual_seed(2)
    tol = 1e-5 if prec == "f32" else 2e-2
    for _ in range(4):
        x = torch.randn(d, generator=g, device=DEV, dtype=torch.float64)
        xHx = N.nys_hessian_apply(ctx, A, x, want_pv=True)[1]
        c = U @ x
        xHhx = float((c * c * torch.tensor(lam, device=DEV)).sum())
        assert xHhx <= xHx * (1 + tol)
    # interlacing lambda_j(H_hat) <= lambda_j(H) = j^-1.6, and a rank-200
    # sketch of this spectrum captures the leading eigenvalues to ~1e-3
    sig2 = np.arange(1, 6) ** -1.6
    print(f"[sketch full] {prec} top eigs {lam[:5]} vs {sig2}", flush=True)
    assert np.all(lam[:5] <= sig2 * (1 + tol))
    assert np.all(lam[:5] >= sig2 * (1 - 1e-2))
    F.close()


def test_repeated_sketches_reuse_device_blocks(N):
    # Factors built, destroyed and rebuilt in a loop (their device blocks are
    # handed out again by the library's block cache, also while the previous
    # factor's work may still be queued): every rebuild gives bit-for-bit the
    # same factor, on one context and on a second one created and destroyed in
    # between; a factor that outlives its context is still destroyed cleanly.
    d, n = 600, 8000
    A32 = synth.decay_matrix(n, d, 0.8, seed=41).to(torch.float32).to(DEV)
    om = synth.omega_raw(d, 160, seed=41).to(DEV)
    c1 = N.Context()
    ref = None
    for k in range(4):
        c = c1 if k != 2 else N.Context()
        F = N.nys_sketch_adaptive(c, A32, om, 20, 160, 1e-3, 2.0, prec=N.NYS_F32)
        U = F.U(c).clone()
        inf = F.info()
        if ref is None:
            ref = (U, inf["lam"], inf["rank"])
        else:
            assert inf["rank"] == ref[2] and inf["lam"] == ref[1]
            assert torch.equal(U, ref[0])
        F.close()
        if c is not c1:
            c.close()
    F = N.nys_sketch(c1, A32, om[:40].contiguous(), prec=N.NYS_F32)
    c1.close()
    F.close()


@pytest.mark.parametrize("r", [300, 700])
def test_sketch_fp64_large_rank_blocked_cholesky(N, ctx, r):
    # ranks above 256 take the blocked multi-workgroup Cholesky (orthonormal
    # blocks of Omega by CholeskyQR2 and the shifted core), with a ragged last
    # block at r = 300 and 700
    n, d = 4000, 1500
    A64 = synth.decay_matrix(n, d, 0.6, seed=r)
    om = synth.omega_raw(d, r, seed=r + 1)
    print(f"[sketch large rank] r={r}", flush=True)
    F = N.nys_sketch(ctx, A64.to(DEV), om.to(DEV), prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A64.numpy(), None, 0.0, om.numpy().T)
    e = rel(H, f.dense())
    print(f"[sketch large rank] r={r} rel(Hhat)={e:.3e} nu={inf['nu']:.3e}/{f.nu:.3e}", flush=True)
    assert e < 1e-10 and inf["nu"] == f.nu
    # U = B V Sigma^-1 is orthonormal to rounding: ~1e-12 per entry at r = 700
    assert np.linalg.norm(U.T @ U - np.eye(r)) < 1e-11 * r
    F.close()


@pytest.mark.parametrize("r", [1, 15, 16, 17, 31, 32, 33, 64, 65, 96, 255, 256])
def test_sketch_fp64_ranks_at_block_edges(N, ctx, r):
    # ranks at the edges of the Cholesky blocks (32 rows: register diagonal
    # block, MFMA trailing tiles of 16) and of the eigensolver blocks (16,
    # pair blocks of 32, padding to an even block count), FP64 end to end
    n, d = 1200, 300
    A64 = synth.decay_matrix(n, d, 0.6, seed=r)
    om = synth.omega_raw(d, r, seed=r + 1)
    F = N.nys_sketch(ctx, A64.to(DEV), om.to(DEV), prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A64.numpy(), None, 0.0, om.numpy().T)
    e = rel(H, f.dense())
    print(f"[sketch fp64 r={r}] rel(Hhat)={e:.3e} nu={inf['nu']:.3e}/{f.nu:.3e}", flush=True)
    assert e < 1e-10
    assert inf["nu"] == f.nu
    assert np.allclose(lam, f.lam, rtol=1e-9, atol=1e-12 * f.lam[0])
    assert np.linalg.norm(U.T @ U - np.eye(r)) < 1e-10
    F.close()


@pytest.mark.parametrize("n,d,r,dtype,weights", [
    (3, 40, 2, torch.float32, False),        # fewer rows than a tile, one short K step
    (33, 65, 16, torch.float64, True),       # one row past a tile; odd widths
    (1000, 129, 17, torch.float32, True),    # K remainders of 1 and 8, column tile of one block + 1
    (4097, 251, 64, torch.float64, False),   # unaligned rows, a full column tile, split K
    (2049, 513, 65, torch.float32, True),    # one column past a column tile
])
def test_sketch_fp64_product_edges(N, ctx, n, d, r, dtype, weights):
    # edges of the FP64 products' tiles and K steps (16 k, 16 or 32 rows, 64
    # columns); rounding of sums of at most 4097 terms, times the condition
    # that the 1e-10 bar of the other FP64 sketches allows for
    A = synth.decay_matrix(n, d, 0.6, seed=n).to(dtype)
    om = synth.omega_raw(d, r, seed=n + 1)
    D = torch.rand(n, dtype=torch.float64, generator=torch.Generator().manual_seed(n)) + 0.1 \
        if weights else None
    c = 0.2 if n < d else 0.0    # rank(A) < r otherwise
    F = N.nys_sketch(ctx, A.to(DEV), om.to(DEV), D=None if D is None else D.to(DEV), c=c,
                     prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A.double().numpy(), None if D is None else D.numpy(), c, om.numpy().T)
    assert rel(H, f.dense()) < 1e-10
    assert inf["nu"] == f.nu
    F.close()


@pytest.mark.parametrize("r", [1, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("equal", [False, True])
def test_eigensolver_small_ranks(N, ctx, r, equal):
    # ranks at the edges of the one-workgroup eigensolver's padded sizes 32 and
    # 64, with distinct eigenvalues and (equal) with all of them alike; the same
    # bar as the other FP64 sketches
    n, d = 600, 150
    A = torch.linalg.qr(synth.gaussian((n, d), seed=r))[0].contiguous() if equal \
        else synth.decay_matrix(n, d, 0.6, seed=r)
    om = synth.omega_raw(d, r, seed=r + 1)
    F = N.nys_sketch(ctx, A.to(DEV), om.to(DEV), prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A.numpy(), None, 0.0, om.numpy().T)
    assert rel(H, f.dense()) < 1e-10
    assert np.all(np.diff(lam) <= 0.0) and np.allclose(lam, f.lam, rtol=1e-10, atol=0.0)
    assert np.linalg.norm(U.T @ U - np.eye(r)) < 1e-10
    F.close()


@pytest.mark.parametrize("r", [257, 288, 289])
def test_blocked_cholesky_block_edges(N, ctx, r):
    # the blocked Cholesky's blocks of 32: one past its smallest rank, whole
    # blocks, a last block of one; the bars of the large ranks above
    n, d = 2000, 700
    A64 = synth.decay_matrix(n, d, 0.6, seed=r)
    om = synth.omega_raw(d, r, seed=r + 1)
    F = N.nys_sketch(ctx, A64.to(DEV), om.to(DEV), prec=N.NYS_F64)
    H, U, lam, inf = hhat(F, ctx)
    f = ny.rand_nys_appx(A64.numpy(), None, 0.0, om.numpy().T)
    assert rel(H, f.dense()) < 1e-10 and inf["nu"] == f.nu
    assert np.linalg.norm(U.T @ U - np.eye(r)) < 1e-11 * r
    F.close()
