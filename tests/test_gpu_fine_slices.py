"""Small sets split the contraction of the down-projection into slices below 256 rows."""
import pytest

pytestmark = pytest.mark.gpu


# one slice doubled and quadrupled, matrices of unequal height, heights that leave empty slices, ranks of every tile
@pytest.mark.parametrize("shapes", [[(256, 96, 16)], [(260, 300, 200)], [(640, 640, 12)], [(128, 256, 24), (256, 128, 24), (128, 128, 24)], [(384, 384, 64)] * 12,
                                    [(400, 264, 300), (300, 520, 260)], [(2048, 64, 33), (129, 40, 5), (520, 72, 100)], [(33, 256, 8), (1030, 256, 8)]])
@pytest.mark.parametrize("update", ["plain", "ef_full"])
def test_sliced_step_follows_the_formulas(shapes, update):
    """u, v and the residual or weights of one step from given moments against float64 at the library's own Q; and the packed payload
    keeps its order: where no matrix is higher than the shortest (or 256 rows) they stand in it by their index, however finely they are split."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(shapes) + shapes[0][0])
    W = [torch.randn(p, q, generator=gen, device="cuda") for p, q, r in shapes]
    G = [torch.randn(p, q, generator=gen, device="cuda").bfloat16() for p, q, r in shapes]
    ef = update == "ef_full"
    opt = lordo.Lordo(shapes, lordo.hparams(seed=4, error_feedback=ef, qhm_mode=2 if ef else 0, omega=0.9), W, torch)
    opt.init_projection()
    for i, (p, q, r) in enumerate(shapes):
        opt.set_state(i, lordo.STATE_U, torch.randn(r, q, generator=gen, device="cuda"))
        opt.set_state(i, lordo.STATE_V, 1.0 + torch.rand(r, q, generator=gen, device="cuda"))
    u0 = [opt.get_state(i, lordo.STATE_U).double() for i in range(len(shapes))]
    v0 = [opt.get_state(i, lordo.STATE_V).double() for i in range(len(shapes))]
    W0 = [w.double() for w in W]
    lr, om = 0.25, 0.9
    opt.local_step(W, G, lr)
    opt.poll_status()
    b1, b2, eps = opt.hp.beta1, opt.hp.beta2, opt.hp.eps
    payload, moments = opt.sync_payload()
    for i, (p, q, r) in enumerate(shapes):
        Q = opt.get_state(i, lordo.STATE_Q).double()
        g = Q.T @ G[i].double()
        u, v = b1 * u0[i] + (1 - b1) * g, b2 * v0[i] + (1 - b2) * g * g
        # two-term planes of Q (2^-17) over fp32 sums
        assert float((opt.get_state(i, lordo.STATE_U).double() - u).norm() / u.norm()) <= 2e-5, i
        assert float((opt.get_state(i, lordo.STATE_V).double() - v).norm() / v.norm()) <= 2e-5, i
        den = (v / (1 - b2)).sqrt() + eps
        N = (u / (1 - b1)) / den
        if ef:
            E = G[i].double() - Q @ g
            assert float((opt.get_state(i, lordo.STATE_ERR).double() - E).norm() / G[i].double().norm()) <= 2e-5, i
            want = W0[i] - lr * (om * Q @ N + (1 - om) * G[i].double() / den.mean(0))
        else:
            want = W0[i] - lr * Q @ N
        assert float((W[i].double() - want).abs().max()) <= 3e-5 * float(want.abs().max()), i
    padded = [(q + 31) // 32 * 32 * ((r + 31) // 32 * 32) for p, q, r in shapes]
    assert moments == 2 * sum(padded)
    heights = [p for p, q, r in shapes]
    if max(heights) <= max(256, min(heights)):
        for i in range(len(shapes)):            # the first element of a matrix's block is rank 0 of column 0
            at = sum(padded[:i])
            assert float(payload[at]) == float(opt.get_state(i, lordo.STATE_U)[0, 0]), i
            assert float(payload[sum(padded) + at]) == float(opt.get_state(i, lordo.STATE_V)[0, 0]), i
