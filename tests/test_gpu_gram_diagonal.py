"""The exact diagonal of the Gram matrices: summed on the side by the diagonal tiles of the grouped GEMM, whole or in slices."""
import pytest

pytestmark = pytest.mark.gpu


# tile edges 64 and 128; one slice and up to sixteen; ragged rows and ranks; more tiles than the launch splits
@pytest.mark.parametrize("p, q, r, n", [(100, 96, 4, 1), (191, 200, 33, 1), (193, 260, 64, 2), (3000, 130, 65, 1), (9000, 256, 128, 1), (8191, 300, 131, 2),
                                        (1024, 768, 256, 2), (700, 640, 500, 80), (20000, 64, 60, 1)])
def test_columns_of_the_basis_have_unit_length(p, q, r, n):
    """||q_k||^2 - 1 carries the error of the diagonal alone.  Around an exact diagonal it is the rounding of S_kk, of the factor and
    of X M^T: a few 2^-24 per step of a chain of r / 16 sums, which average out; a diagonal out of the three-term products
    is too small by 2e-6 and more at these heights, a column or slice that is missing by per cents."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(p + q + r)
    W = [torch.zeros(p, q, device="cuda") for _ in range(n)]
    opt = lordo.Lordo([(p, q, r)] * n, lordo.hparams(power_iters=1, seed=3), W, torch)
    src = [torch.randn(p, q, generator=gen, device="cuda") for _ in range(min(n, 2))]
    opt.refresh_subspace([src[i % len(src)] for i in range(n)])
    opt.poll_status()
    for i in (0, n - 1):
        Q = opt.get_state(i, lordo.STATE_Q).double()
        off = (Q * Q).sum(0) - 1
        assert float(off.abs().max()) <= 1.5e-6, float(off.abs().max())
        assert abs(float(off.mean())) <= 5e-7, float(off.mean())
        assert float((Q.T @ Q - torch.eye(r, device="cuda", dtype=torch.float64)).norm()) <= 1e-4
