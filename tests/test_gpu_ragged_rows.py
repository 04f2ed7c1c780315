"""Matrices whose rows start at any element: odd numbers of columns, ranks that are no multiple of four, arrays that begin in the middle
of a vector.  The step reads and writes them in vectors at element alignment, the grouped GEMM reads them so."""
import pytest

pytestmark = pytest.mark.gpu


def _window(torch, p, q, dtype, offset, gen, scale=1.0):
    """(flat buffer, p x q view that starts `offset` elements into its middle): what lies around the view must stay as it is."""
    pad = 512
    flat = (scale * torch.randn(p * q + 2 * pad, generator=gen, device="cuda")).to(dtype)
    return flat, flat[pad + offset:pad + offset + p * q].view(p, q)


@pytest.mark.parametrize("p, q, r", [(9, 1, 1), (1, 7, 1), (33, 2, 2), (40, 3, 3), (130, 5, 4), (31, 63, 20), (129, 65, 33), (64, 127, 64), (128, 129, 100), (257, 131, 96),
                                     (131, 255, 128), (100, 257, 61), (300, 259, 130), (270, 1023, 256), (515, 190, 300), (1000, 321, 5)])
@pytest.mark.parametrize("store", ["f32", "bf16"])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_step_on_rows_at_any_element(p, q, r, store, offset):
    """One plain step from given moments: u, v and the weights against the formulas in float64 at the library's own Q, and nothing
    written outside the matrix.  v >= 1 keeps N = u_hat / sqrt(v_hat) smooth in g."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 * p + q + r)
    wt = torch.bfloat16 if store == "bf16" else torch.float32
    shapes = [(p, q, r), (q, p, min(r, q))]
    bufs = [_window(torch, a, b, wt, offset, gen) for a, b, _ in shapes]
    grads = [_window(torch, a, b, torch.bfloat16, offset, gen) for a, b, _ in shapes]
    W, G = [v for _, v in bufs], [v for _, v in grads]
    opt = lordo.Lordo(shapes, lordo.hparams(seed=5, param_dtype=lordo.BF16 if store == "bf16" else lordo.F32), W, torch)
    opt.init_projection()
    lr = 0.25
    for i, (a, b, k) in enumerate(shapes):
        opt.set_state(i, lordo.STATE_U, torch.randn(k, b, generator=gen, device="cuda"))
        opt.set_state(i, lordo.STATE_V, 1.0 + torch.rand(k, b, generator=gen, device="cuda"))
    u0 = [opt.get_state(i, lordo.STATE_U).double() for i in range(2)]
    v0 = [opt.get_state(i, lordo.STATE_V).double() for i in range(2)]
    before = [f.clone() for f, _ in bufs]
    opt.local_step(W, G, lr)
    opt.poll_status()
    b1, b2, eps = opt.hp.beta1, opt.hp.beta2, opt.hp.eps
    for i, (a, b, k) in enumerate(shapes):
        Q = opt.get_state(i, lordo.STATE_Q).double()
        g = Q.T @ G[i].double()
        u, v = b1 * u0[i] + (1 - b1) * g, b2 * v0[i] + (1 - b2) * g * g
        # g: two-term planes of Q (2^-17) over fp32 sums
        assert float((opt.get_state(i, lordo.STATE_U).double() - u).norm() / u.norm()) <= 2e-5, i
        assert float((opt.get_state(i, lordo.STATE_V).double() - v).norm() / v.norm()) <= 2e-5, i
        N = (u / (1 - b1)) / ((v / (1 - b2)).sqrt() + eps)
        flat0, start = before[i], 512 + offset
        want = flat0[start:start + a * b].view(a, b).double() - lr * Q @ N
        got = bufs[i][0].clone()
        if store == "f32":       # |Q N| of the order of the weights: planes' 2^-17 of it, and the rounding of the sum
            assert float((W[i].double() - want).abs().max()) <= 3e-5 * float(want.abs().max()), i
        else:                    # rounded once: half a bf16 unit of the value, and the same 2^-17 ahead of it
            assert float(((W[i].double() - want).abs() - 2.0 ** -8 * want.abs()).max()) <= 3e-5 * float(want.abs().max()), i
        got[start:start + a * b] = flat0[start:start + a * b]
        assert torch.equal(got, flat0), i
