"""Products of a tall fp32 matrix with a narrow block on the split-plane kernel (k_gemm_planes): refreshes from an fp32
source at the edges of its tiles (rows 128; columns 64, 128 and 256; k-steps of 16 in pairs) and of its dispatch."""
import pytest

pytestmark = pytest.mark.gpu


# (p, q, r), number of matrices: column tiles of 64, then of 128 and of 256 (512 tiles of that width), a lone tall matrix, columns
# that end inside a 32-column chunk, rows that end inside a row tile, and the shapes that stay with the general kernel
# (r <= 64; q % 4 != 0; few tiles)
@pytest.mark.parametrize("shape, n", [((640, 516, 64), 28), ((520, 1000, 72), 28), ((776, 192, 192), 20), ((2048, 512, 128), 9), ((1100, 260, 132), 16),
                                      ((16500, 384, 256), 1), ((1030, 1028, 260), 16), ((516, 2052, 300), 32), ((1100, 1028, 256), 32), ((1030, 640, 500), 32),
                                      ((640, 518, 64), 28), ((640, 518, 100), 28), ((256, 320, 16), 2)])
def test_refresh_from_fp32_source_spans_the_dominant_directions(shape, n):
    """k_gemm_planes in the products Y = Src B, X M^T and the moment rotation.  The source is 100 A B^T with orthonormal A and B of
    r columns: exactly rank r up to fp32 rounding, all r singular values equal, so the refreshed subspace is the column space
    of A whatever the start block; and with an orthonormal Q the rotated moments follow from R = Q^T Q_old.  A local step behind
    the refresh finds the operand planes of N and the array g, which the products used as scratch, rewritten in full."""
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
    opt.local_step(W, [torch.randn(p, q, generator=gen, device="cuda") for _ in range(n)], 0.0)     # (a second one, so that v - u^2 is a variance)
    U, src = [], []
    for i in range(n):
        a, _ = torch.linalg.qr(torch.randn(p, r, generator=gen, device="cuda", dtype=torch.float64))
        b, _ = torch.linalg.qr(torch.randn(q, r, generator=gen, device="cuda", dtype=torch.float64))
        U.append(a)
        src.append((100.0 * a @ b.T).float())
    q_old = [opt.get_state(i, lordo.STATE_Q).double() for i in range(n)]
    u_old = [opt.get_state(i, lordo.STATE_U).double() for i in range(n)]
    v_old = [opt.get_state(i, lordo.STATE_V).double() for i in range(n)]
    opt.refresh_subspace(src)
    opt.poll_status()
    b1, b2, eps = opt.hp.beta1, opt.hp.beta2, opt.hp.eps
    c1, c2 = 1 - b1 ** 2, 1 - b2 ** 2
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
        R = Q.T @ q_old[i]
        want = c2 * ((R * R) @ (v_old[i] / c2 - (u_old[i] / c1) ** 2) + (R @ u_old[i] / c1) ** 2).abs()
        got = opt.get_state(i, lordo.STATE_V).double()
        assert float((got - want).norm() / want.norm()) <= 1e-5, i
        assert float((got - want).abs().max() / want.square().mean().sqrt()) <= 1e-3, i
    u_old = [opt.get_state(i, lordo.STATE_U).double() for i in range(n)]
    v_old = [opt.get_state(i, lordo.STATE_V).double() for i in range(n)]
    opt.local_step(W, G, 1.0)
    for i in range(n):
        Q = opt.get_state(i, lordo.STATE_Q).double()
        g = Q.T @ G[i].double()
        u, v = opt.get_state(i, lordo.STATE_U).double(), opt.get_state(i, lordo.STATE_V).double()
        # sums over p of fp32 values in three-term form
        assert float((u - (b1 * u_old[i] + (1 - b1) * g)).norm() / u.norm()) <= 1e-5, i
        assert float((v - (b2 * v_old[i] + (1 - b2) * g * g)).norm() / v.norm()) <= 1e-5, i
        dW = Q @ (u / (1 - b1 ** 3) / ((v / (1 - b2 ** 3)).sqrt() + eps))
        # two-term operands of Q and N, 2^-17 each
        assert float((W[i].double() + dW).norm() / dW.norm()) <= 3e-5, i
        assert float((W[i].double() + dW).abs().max() / dW.square().mean().sqrt()) <= 1e-3, i


# every way the fallback reads the tile table: entries of 128 x 64 as two 64 x 64 tiles, of 128 x 128 as one tile, of 128 x 256 as two
# 128 x 128 tiles; and a set that takes k_gemm32 in the first place
@pytest.mark.parametrize("shape, n", [((640, 516, 100), 28), ((1028, 516, 100), 64), ((516, 516, 200), 52), ((516, 516, 500), 52), ((640, 516, 64), 28)])
@pytest.mark.parametrize("source", ["fp32", "fp32 off by 4 bytes", "bf16"])
def test_source_product_spans_src_times_start_block(shape, n, source):
    """Y = Src Omega where the source is read by k_gemm_planes (aligned fp32) and where it falls back to k_gemm32 on the
    same tile table (q % 32 != 0 in bf16, fp32 rows that are not 16-byte aligned).  Without power iterations Q spans Y: nothing
    of any column of the product lies outside.  Matrices that are left out keep their projection."""
    import torch
    from paper_2602_04396_amd import lordo
    p, q, r = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(p + 3 * q + r)
    W = [torch.zeros(p, q, device="cuda") for _ in range(n)]
    opt = lordo.Lordo([(p, q, r)] * n, lordo.hparams(power_iters=0, seed=3), W, torch)
    del W
    dtype = torch.bfloat16 if source == "bf16" else torch.float32
    src = []
    for _ in range(n):
        flat = torch.randn(p * q + 1, generator=gen, device="cuda").to(dtype)
        src.append(flat[1:].view(p, q) if "off" in source else flat[:p * q].view(p, q))
    omega = [torch.randn(q, r, generator=gen, device="cuda") for _ in range(n)]
    left_out = n // 2
    q_before = opt.get_state(left_out, lordo.STATE_Q)
    opt.refresh_subspace([None if i == left_out else s for i, s in enumerate(src)], omega)
    opt.poll_status()
    assert torch.equal(opt.get_state(left_out, lordo.STATE_Q), q_before)
    for i in range(n):
        if i == left_out:
            continue
        Q = opt.get_state(i, lordo.STATE_Q).double()
        Y = src[i].double() @ omega[i].double()
        out = Y - Q @ (Q.T @ Y)
        # fp32 sums over q (three-term operands: the same) and the passes of CholeskyQR2, 1e-7 sqrt(r) of a column's norm;
        # a wrong tile leaves a share of the column of the order of one
        assert float((out.norm(dim=0) / Y.norm(dim=0)).max()) <= 2e-5, i


@pytest.mark.parametrize("n, p, q, r", [(64, 640, 516, 512), (256, 260, 260, 256), (256, 260, 260, 192)])      # edges 256, 128, 64
def test_split_planes_give_the_bits_of_the_general_kernel(n, p, q, r):
    """The same matrices and inputs in two sets: alone, where Y = Src B, X M^T and the rotation products run on k_gemm_planes, and
    with one more matrix whose columns and rank are no multiples of four, which sends those products of the whole
    set to k_gemm32.  (At least 1024 tiles of 128 x 128 in the Gram product: no K slices in either set.)"""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    src = [torch.randn(p, q, generator=gen, device="cuda") for _ in range(n)]
    q0 = torch.linalg.qr(torch.randn(p, r, generator=gen, device="cuda"))[0].contiguous()
    u0 = torch.randn(r, q, generator=gen, device="cuda")
    v0 = u0 * u0 + torch.rand(r, q, generator=gen, device="cuda")
    results = []
    for extra in ([], [(p, q + 2, r - 2)]):
        shapes = [(p, q, r)] * n + extra
        opt = lordo.Lordo(shapes, lordo.hparams(power_iters=0, seed=3), [torch.zeros(s[0], s[1], device="cuda") for s in shapes], torch)
        for i in range(n):
            opt.set_state(i, lordo.STATE_Q, q0)
            opt.set_state(i, lordo.STATE_U, u0)
            opt.set_state(i, lordo.STATE_V, v0)
        opt.step = 5
        opt.refresh_subspace(src + [torch.randn(s[0], s[1], generator=gen, device="cuda") for s in extra])
        opt.poll_status()
        results.append([opt.get_state(i, which) for i in range(n) for which in (lordo.STATE_Q, lordo.STATE_U, lordo.STATE_V)])
        del opt
    assert all(torch.equal(a, b) for a, b in zip(*results))


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("shape, n", [((640, 516, 64), 28), ((1100, 260, 132), 16)])
def test_breakdown_leaves_projection_and_moments(shape, n, bad):
    """One element of one source that is not finite: the refresh latches LORDO_ENUMERIC and every matrix keeps Q, u and v; the
    next refresh, after the poll, is one of a context that never saw it."""
    import torch
    from paper_2602_04396_amd import lordo
    p, q, r = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    src = [torch.randn(p, q, generator=gen, device="cuda") for _ in range(n)]
    omega = [torch.randn(q, r, generator=gen, device="cuda") for _ in range(n)]
    G = [torch.randn(p, q, generator=gen, device="cuda") for _ in range(n)]
    states = (lordo.STATE_Q, lordo.STATE_U, lordo.STATE_V)
    after = []
    for broken in (True, False):
        W = [torch.zeros(p, q, device="cuda") for _ in range(n)]
        opt = lordo.Lordo([(p, q, r)] * n, lordo.hparams(power_iters=1, seed=3, grad_dtype=lordo.F32), W, torch)
        opt.init_projection()
        opt.local_step(W, G, 1.0)
        if broken:
            before = [opt.get_state(i, which) for i in range(n) for which in states]
            spoiled = list(src)
            spoiled[n // 2] = src[n // 2].clone()
            spoiled[n // 2][p - 1, q - 1] = bad
            opt.refresh_subspace(spoiled, omega)
            with pytest.raises(lordo.LordoError):
                opt.poll_status()
            assert all(torch.equal(a, b) for a, b in zip(before, [opt.get_state(i, which) for i in range(n) for which in states]))
        opt.refresh_subspace(src, omega)
        opt.poll_status()
        opt.local_step(W, G, 1.0)
        after.append([opt.get_state(i, which) for i in range(n) for which in states] + W)
    assert all(torch.equal(a, b) for a, b in zip(*after))
