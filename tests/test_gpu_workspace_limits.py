"""A caller's workspace with little room to spare: what is served does not
depend on how the split-K partial sums of the FP64 products are placed.

  * a solve is served in the bytes that its buffers add up to, with no margin
    for scratch that it can do without;
  * a factor has the same bits in every workspace that serves it, and without
    one (the products' K split follows from the sizes alone; a short buffer
    means panels of the result instead).
"""
import pytest
import torch

from paper_2202_11599_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def N():
    from paper_2202_11599_amd import nysadmm
    return nysadmm


def test_lasso_served_without_room_for_more_partial_sums(N):
    # 15900 x 796 FP64 at rank 73: the sizes of the call's buffers and the
    # query's margin of an eighth and 16 MB come to 54.4 MB; 8 MB more of partial
    # sums kept from the sketch on do not fit next to them
    n, d, r, size = 15900, 796, 73, 57035908
    p = synth.lasso_decay(n, d, 0.8, seed=11, device=DEV, dtype=torch.float64, gamma_frac=0.01,
                          rho=1e-3, rank=r, s_max=r, pcg_tol=1e-8)
    ctx = N.Context()
    buf = torch.empty(size, dtype=torch.uint8, device=DEV)
    ctx.set_workspace(buf)
    o = N.admm_opts(p.rho, r, p.omega, pcg=N.pcg_opts(tol=1e-8), max_iter=3)
    st = N.State(d, DEV)
    info = N.admm_solve(ctx, [N.problem(p.A, p.b, p.gamma)], [o], [st])[0]
    assert info.status == N.NYS_OK and info.iters == 3
    assert ctx.workspace_query(p.A, r) <= size
    ctx.close()
    ref = N.Context()
    st0 = N.State(d, DEV)
    N.admm_solve(ref, [N.problem(p.A, p.b, p.gamma)], [o], [st0])
    assert torch.equal(st.z, st0.z) and torch.equal(st.x, st0.x)
    ref.close()


@pytest.mark.parametrize("n,d,r,dtype", [
    (1500, 600, 100, torch.float32),
    (20000, 600, 100, torch.float32),
    (9001, 411, 72, torch.float64),
    (30000, 130, 66, torch.float32),
])
def test_factor_bits_in_every_workspace(N, n, d, r, dtype):
    A = synth.decay_matrix(n, d, 0.6, seed=n).to(dtype).to(DEV)
    om = synth.omega_raw(d, r, seed=n + 1).to(DEV)
    ref = N.Context()
    F = N.nys_sketch(ref, A, om, prec=N.NYS_F64)
    U0, lam0 = F.U(ref).clone(), F.info()["lam"]
    F.close()
    ref.close()
    # down through the sizes without room for the larger partial sums, one by one
    served = []
    for size in range(8 * (n * r + 10 * d * r + 40 * r * r + 256 * d) + (20 << 20), 1 << 19, -(1 << 19)):
        ctx = N.Context()
        buf = torch.empty(size, dtype=torch.uint8, device=DEV)
        ctx.set_workspace(buf)
        try:
            F = N.nys_sketch(ctx, A, om, prec=N.NYS_F64)
        except N.NysError as e:
            assert e.status == N.NYS_ERR_NOMEM
            served.append(False)
        else:
            served.append(True)
            same = torch.equal(F.U(ctx), U0) and list(F.info()["lam"]) == list(lam0)
            F.close()
            assert same, f"{size} bytes"
        ctx.close()
    print(f"[workspace bits] {n} x {d} rank {r}: served {sum(served)} of {len(served)}", flush=True)
    assert served[0] and not served[-1]
    assert served == sorted(served, reverse=True)   # none below the first that is refused


def test_streaming_pair_served_with_the_fewest_partial_sums(N):
    # 300000 x 257 FP32 streams from HBM, so its launch shapes are timed, which
    # takes their partial sums (up to 2048 rows of 320 doubles, 5.2 MB) once for
    # the timing and once to keep; whole rows per wavefront leave 256 rows, 0.7 MB,
    # next to 0.6 MB of vectors
    n, d = 300000, 257
    A = torch.randn(n, d, device=DEV, dtype=torch.float32)
    p = torch.randn(d, device=DEV, dtype=torch.float64)
    ref = A.double().t().contiguous() @ (A.double() @ p) + 0.5 * p
    for size in (3 << 20, 8 << 20, 64 << 20):
        ctx = N.Context()
        buf = torch.empty(size, dtype=torch.uint8, device=DEV)
        ctx.set_workspace(buf)
        for _ in range(2):
            v = N.nys_hessian_apply(ctx, A, p, rho=0.5)
            torch.cuda.synchronize()
            assert float((v - ref).norm() / ref.norm()) < 3e-12, size
        ctx.close()
