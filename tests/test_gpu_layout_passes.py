"""Layout passes of the refresh (k_pack_q and its modes, k_glow_to_z, k_rot_pre, k_rot_post) at ragged rows, columns and ranks."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p, q, r", [(64, 64, 32), (65, 96, 33), (31, 40, 8), (33, 64, 30), (200, 136, 100), (257, 320, 36), (640, 512, 128), (515, 1000, 130)])
@pytest.mark.parametrize("source", ["bf16", "fp32"])
def test_refresh_and_step_keep_projection_planes_and_moments_consistent(p, q, r, source):
    """After a refresh from an equal-valued low-rank source: Q spans it, u and v are those of before, rotated, and the next step's
    moments and weights follow from the Q that get_state returns, i.e. the operand planes hold the same Q in both orientations."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 * p + q + r)
    n = 3
    W = [torch.randn(p, q, generator=gen, device="cuda") for _ in range(n)]
    beta1, lr = 0.9, 0.5
    opt = lordo.Lordo([(p, q, r)] * n, lordo.hparams(beta1=beta1, power_iters=1, seed=3), W, torch)
    opt.init_projection()
    G = [torch.randn(p, q, generator=gen, device="cuda").bfloat16() for _ in range(n)]
    opt.local_step(W, G, lr)
    opt.local_step(W, [torch.randn(p, q, generator=gen, device="cuda").bfloat16() for _ in range(n)], lr)      # (so that v - u^2 is a variance)
    q_old = [opt.get_state(i, lordo.STATE_Q).double() for i in range(n)]
    u_old = [opt.get_state(i, lordo.STATE_U).double() for i in range(n)]
    v_old = [opt.get_state(i, lordo.STATE_V).double() for i in range(n)]
    c1, c2 = 1 - beta1 ** 2, 1 - opt.hp.beta2 ** 2
    src, U = [], []
    for i in range(n):
        k = min(p, q, r)
        a, _ = torch.linalg.qr(torch.randn(p, k, generator=gen, device="cuda", dtype=torch.float64))
        b, _ = torch.linalg.qr(torch.randn(q, k, generator=gen, device="cuda", dtype=torch.float64))
        s = 100.0 * a @ b.T
        s = s.bfloat16() if source == "bf16" else s.float()
        src.append(s)
        U.append(torch.linalg.svd(s.double(), full_matrices=False)[0][:, :k])
    opt.refresh_subspace(src)
    opt.poll_status()
    Q = [opt.get_state(i, lordo.STATE_Q).double() for i in range(n)]
    for i in range(n):
        k = U[i].shape[1]
        if source == "fp32":      # (a bf16 source has rounding noise: its trailing directions depend on the start block)
            assert float((U[i] - Q[i] @ (Q[i].T @ U[i])).norm()) / k ** 0.5 <= 5e-5, i
        want = (Q[i].T @ q_old[i]) @ u_old[i]
        got = opt.get_state(i, lordo.STATE_U).double()
        assert float((got - want).norm() / want.norm()) <= 1e-5, i              # fp32 sums over p and r
        R = Q[i].T @ q_old[i]
        want = c2 * ((R * R) @ (v_old[i] / c2 - (u_old[i] / c1) ** 2) + (R @ u_old[i] / c1) ** 2).abs()
        got = opt.get_state(i, lordo.STATE_V).double()
        assert float((got - want).norm() / want.norm()) <= 1e-5, i              # the same, on terms of one size
    u1 = [opt.get_state(i, lordo.STATE_U).double() for i in range(n)]
    before = [w.double() for w in W]
    opt.local_step(W, G, lr)
    for i in range(n):
        want = beta1 * u1[i] + (1 - beta1) * (Q[i].T @ G[i].double())
        got = opt.get_state(i, lordo.STATE_U).double()
        assert float((got - want).norm() / want.norm()) <= 3e-5, i              # two-term planes of Q: 2^-17 each
        step = W[i].double() - before[i]
        inside = Q[i] @ (Q[i].T @ step)
        # the update is -lr Q N: nothing of it lies outside span(Q) but the planes' 2^-17 and the rounding of W (2^-24 |W| / |step|)
        assert float((step - inside).norm()) <= 3e-5 * float(step.norm()) + 1.2e-7 * float(W[i].double().norm()), i
