"""Orthonormalisation at the edges of the Cholesky kernel (k_factor_diag): column blocks of 16, halves of 64, blocks of 128."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 2, 15, 16, 17, 48, 63, 64, 65, 80, 100, 127, 128, 129, 192, 193, 256, 260, 384, 511])
@pytest.mark.parametrize("spread", [1.0, 30.0])
def test_initial_projection_is_the_q_factor_of_the_block(r, spread):
    """init_projection(Block): the thin QR factor with a positive diagonal of R is unique, so every element is compared with
    float64.  The block has columns of very different lengths (`spread` per half) and a common direction that correlates them."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(r)
    shapes = [(640, 64, r), (1028, 36, max(1, r - 1)), (520, 96, max(1, r // 2))]
    W = [torch.zeros(p, q, device="cuda") for p, q, _ in shapes]
    blocks = []
    for p, q, k in shapes:
        b = torch.randn(p, k, generator=gen, device="cuda") + 0.5 * torch.randn(p, 1, generator=gen, device="cuda")
        blocks.append(b * spread ** torch.linspace(-1, 1, k, device="cuda"))
    opt = lordo.Lordo(shapes, lordo.hparams(seed=1, grad_dtype=lordo.F32), W, torch)
    opt.init_projection(blocks)
    opt.poll_status()
    for i, b in enumerate(blocks):
        q64, r64 = torch.linalg.qr(b.double())
        want = q64 * torch.sign(torch.diagonal(r64))
        got = opt.get_state(i, lordo.STATE_Q).double()
        k = got.shape[1]
        # fp32 QR: 2^-24 times the condition number with the columns scaled to unit length (here up to about 15 at r = 511 of
        # 520 .. 640 rows, sqrt(r) from the common direction), sqrt(r) columns: below 5e-5 of the norm; a misplaced element is off by 1 / sqrt(p)
        cond = float(torch.linalg.cond(b.double() / b.double().norm(dim=0)))
        assert float((got - want).norm()) <= 6e-8 * 8 * cond * k ** 0.5, (i, cond)
        assert float((got.T @ got - torch.eye(k, device="cuda", dtype=torch.float64)).norm()) <= 6e-8 * 8 * k, i
