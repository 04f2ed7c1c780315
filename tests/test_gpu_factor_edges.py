"""Orthonormalisation at the edges of the Cholesky kernel of the refresh (k_factor_diag): column blocks of 16, halves of 64,
blocks of 128."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 2, 15, 16, 17, 48, 63, 64, 65, 80, 100, 127, 128, 129, 192, 193, 256, 260, 384, 511])
def test_refresh_orthonormalises_at_every_edge_of_the_factor(r):
    """The source is A diag(s) B^T with r equal singular values, so the refreshed subspace is the column space of A; the block is
    a square Gaussian times A, as ill-conditioned as such blocks get, and goes through shifted and unshifted passes."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(r)
    shapes = [(640, 576, r), (1028, 536, max(1, r - 1)), (520, 600, max(1, r // 2))]
    W = [torch.zeros(p, q, device="cuda") for p, q, _ in shapes]
    opt = lordo.Lordo(shapes, lordo.hparams(power_iters=1, seed=1, grad_dtype=lordo.F32), W, torch)
    U, src = [], []
    for p, q, k in shapes:
        a, _ = torch.linalg.qr(torch.randn(p, k, generator=gen, device="cuda", dtype=torch.float64))
        b, _ = torch.linalg.qr(torch.randn(q, k, generator=gen, device="cuda", dtype=torch.float64))
        U.append(a)
        src.append((100.0 * a @ b.T).float())
    opt.refresh_subspace(src)
    opt.poll_status()
    for i, u in enumerate(U):
        got = opt.get_state(i, lordo.STATE_Q).double()
        k = got.shape[1]
        # CholeskyQR2 in fp32: k^2 entries of about 1e-7 (2^-24 times a small factor); a misplaced element is off by 1 / sqrt(p)
        assert float((got.T @ got - torch.eye(k, device="cuda", dtype=torch.float64)).norm()) <= 6e-8 * 8 * k + 1e-6, i
        # rounding of the source and of the products with it, about 1e-7 sqrt(q) of the norm per direction
        assert float((got - u @ (u.T @ got)).norm()) / k ** 0.5 <= 2e-5, i


@pytest.mark.parametrize("r", [1, 16, 63, 64, 65, 72, 100, 128, 130, 200])
@pytest.mark.parametrize("exponent", [-20, 20, 26])
def test_scale_of_the_source_does_not_change_the_factorisation(r, exponent):
    """Every sum, root and quotient of the orthonormalisation scales exactly with a power of two, so the projection of 2^k Src
    (and the initial projection of a block 2^k B) has the same bits as that of Src.  The identity that pads a block of
    the factor does not scale: a column norm of 1e6 made the pivot floor of the block exceed it."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(r)
    p, q = 640, 576
    W = [torch.zeros(p, q, device="cuda")]
    src = 0.1 * torch.randn(p, q, generator=gen, device="cuda")
    block = torch.randn(p, r, generator=gen, device="cuda")
    refreshed, initial = [], []
    for scale in (1.0, 2.0 ** exponent):
        opt = lordo.Lordo([(p, q, r)], lordo.hparams(power_iters=1, seed=1, grad_dtype=lordo.F32), W, torch)
        opt.init_projection([block * scale])
        opt.poll_status()
        initial.append(opt.get_state(0, lordo.STATE_Q))
        opt.refresh_subspace([src * scale])
        opt.poll_status()
        refreshed.append(opt.get_state(0, lordo.STATE_Q))
    assert torch.equal(initial[0], initial[1])
    assert torch.equal(refreshed[0], refreshed[1])


@pytest.mark.parametrize("r", [8, 64, 65])
def test_refresh_of_more_matrices_than_compute_units(r):
    """Several workgroups of the factorisation share a compute unit where no block has a second half (r <= 64), one where it has.
    Without power iterations Q is an orthonormal basis of Src Omega."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(r)
    n, p, q = 700, 96, 80
    src = torch.randn(n, p, q, generator=gen, device="cuda")
    omega = torch.randn(n, q, r, generator=gen, device="cuda")
    opt = lordo.Lordo([(p, q, r)] * n, lordo.hparams(power_iters=0), [torch.zeros(p, q, device="cuda") for _ in range(n)], torch)
    opt.refresh_subspace(list(src.unbind()), list(omega.unbind()))
    opt.poll_status()
    for i in range(n):
        Q, Y = opt.get_state(i, lordo.STATE_Q).double(), src[i].double() @ omega[i].double()
        assert float((Q.T @ Q - torch.eye(r, device="cuda", dtype=torch.float64)).norm()) <= 6e-8 * 8 * r + 1e-6, i
        # fp32 sums over q and the passes of CholeskyQR2: 1e-7 sqrt(r) of a column's norm
        assert float(((Y - Q @ (Q.T @ Y)).norm(dim=0) / Y.norm(dim=0)).max()) <= 2e-5, i
