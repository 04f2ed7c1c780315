"""Products of a tall fp32 matrix with a narrow block on the split-plane kernel (k_gemm_planes): refreshes from an fp32
source at the edges of its tiles (rows 128; columns 64, 128 and 256; k-steps of 16 in pairs) and of its dispatch."""
import pytest

pytestmark = pytest.mark.gpu


# (p, q, r), number of matrices: enough row tiles for the kernel to be taken (128), a lone tall matrix, ranks on both
# sides of each column edge, columns that end inside a 32-column chunk, rows that end inside a row tile, and the shapes
# that stay with the general kernel (q % 4 != 0; few tiles)
@pytest.mark.parametrize("shape, n", [((640, 516, 64), 28), ((520, 1000, 72), 28), ((776, 192, 192), 20), ((2048, 512, 128), 9), ((1100, 260, 132), 16),
                                      ((16500, 384, 256), 1), ((1030, 1028, 260), 16), ((516, 2052, 300), 32), ((640, 518, 64), 28), ((256, 320, 16), 2)])
def test_refresh_from_fp32_source_spans_the_dominant_directions(shape, n):
    """k_gemm_planes in the products Y = Src B, X M^T and the moment rotation.  The source is A diag(s) B^T + noise with k = r
    equal singular values far above the noise, so the refreshed subspace is the column space of A whatever the start block;
    and with an orthonormal Q the rotated first moment is R u."""
    import torch
    from paper_2602_04396_amd import lordo
    p, q, r = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(p + q + r)
    W = [torch.zeros(p, q, device="cuda") for _ in range(n)]
    opt = lordo.Lordo([(p, q, r)] * n, lordo.hparams(power_iters=1, seed=3, grad_dtype=lordo.F32), W, torch)
    opt.init_projection()
    G = [torch.randn(p, q, generator=gen, device="cuda") for _ in range(n)]
    opt.local_step(W, G, 0.0)
    U, src = [], []
    for i in range(n):
        a, _ = torch.linalg.qr(torch.randn(p, r, generator=gen, device="cuda", dtype=torch.float64))
        b, _ = torch.linalg.qr(torch.randn(q, r, generator=gen, device="cuda", dtype=torch.float64))
        U.append(a)
        src.append((100.0 * a @ b.T).float())
    q_old = [opt.get_state(i, lordo.STATE_Q).double() for i in range(n)]
    u_old = [opt.get_state(i, lordo.STATE_U).double() for i in range(n)]
    opt.refresh_subspace(src)
    opt.poll_status()
    for i in range(n):
        Q = opt.get_state(i, lordo.STATE_Q).double()
        # CholeskyQR2 in fp32: r entries of about 1e-7 sqrt(r) per row
        assert float((Q.T @ Q - torch.eye(r, device="cuda", dtype=torch.float64)).norm()) <= 1e-4, i
        # rounding of the source (2^-24 of rank-one entries) and of the products (three-term operands, fp32 sums), both about
        # 1e-7 sqrt(q) of the norm per direction; an element that is lost or in the wrong place is off by 1 / sqrt(p)
        assert float((Q - U[i] @ (U[i].T @ Q)).norm()) / r ** 0.5 <= 2e-5, i
        want = (Q.T @ q_old[i]) @ u_old[i]
        got = opt.get_state(i, lordo.STATE_U).double()
        # R from p products and R u from r products of fp32 values in three-term form: 1e-6 relative
        assert float((got - want).norm() / want.norm()) <= 1e-5, i
        assert float((got - want).abs().max() / want.square().mean().sqrt()) <= 1e-3, i
