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


# ranks and sides around the edges of tiles (32, 64, 128) and of vectors (remainders 1 to 3), and sides too short for a vector
@pytest.mark.parametrize("p, q, r", [(5, 3, 2), (3, 9, 3), (37, 70, 5), (67, 41, 4), (65, 129, 39), (131, 258, 63), (130, 97, 66), (200, 301, 127), (389, 514, 130), (257, 515, 171)])
@pytest.mark.parametrize("source", ["bf16", "fp32"])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_refresh_at_any_element(p, q, r, source, offset):
    """Refresh from a source of r equal singular values, source and start block at any element of a buffer: Q is orthonormal and
    spans the source's columns, and u and v are those of before, rotated."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7 * p + q + r)
    n = 2
    W = [torch.randn(p, q, generator=gen, device="cuda") for _ in range(n)]
    beta1 = 0.9
    opt = lordo.Lordo([(p, q, r)] * n, lordo.hparams(beta1=beta1, power_iters=1, seed=3), W, torch)
    opt.init_projection()
    for _ in range(2):
        opt.local_step(W, [torch.randn(p, q, generator=gen, device="cuda").bfloat16() for _ in range(n)], 0.5)
    q_old = [opt.get_state(i, lordo.STATE_Q).double() for i in range(n)]
    u_old = [opt.get_state(i, lordo.STATE_U).double() for i in range(n)]
    v_old = [opt.get_state(i, lordo.STATE_V).double() for i in range(n)]
    dt = torch.bfloat16 if source == "bf16" else torch.float32
    src, om, U = [], [], []
    for i in range(n):
        a, _ = torch.linalg.qr(torch.randn(p, r, generator=gen, device="cuda", dtype=torch.float64))
        b, _ = torch.linalg.qr(torch.randn(q, r, generator=gen, device="cuda", dtype=torch.float64))
        s = _window(torch, p, q, dt, offset, gen)[1]
        s.copy_(100.0 * a @ b.T)
        o = _window(torch, q, r, torch.float32, offset, gen)[1]
        src.append(s)
        om.append(o)
        U.append(a)
    opt.refresh_subspace(src, om)
    opt.poll_status()
    c1, c2 = 1 - beta1 ** 2, 1 - opt.hp.beta2 ** 2
    for i in range(n):
        Q = opt.get_state(i, lordo.STATE_Q).double()
        assert float((Q.T @ Q - torch.eye(r, device="cuda", dtype=torch.float64)).norm()) <= 1e-4, i      # CholeskyQR2 in fp32
        if source == "fp32":      # (a bf16 source has rounding noise: its trailing directions depend on the start block)
            assert float((U[i] - Q @ (Q.T @ U[i])).norm()) / r ** 0.5 <= 5e-5, i
        R = Q.T @ q_old[i]
        want = R @ u_old[i]
        assert float((opt.get_state(i, lordo.STATE_U).double() - want).norm() / want.norm()) <= 1e-5, i   # fp32 sums over p and r
        want = c2 * ((R * R) @ (v_old[i] / c2 - (u_old[i] / c1) ** 2) + (R @ u_old[i] / c1) ** 2).abs()
        assert float((opt.get_state(i, lordo.STATE_V).double() - want).norm() / want.norm()) <= 1e-5, i


@pytest.mark.parametrize("p, q, r", [(256, 320, 64), (384, 256, 128), (512, 384, 192)])
def test_aligned_source_at_an_odd_address_gives_the_same_bits(p, q, r):
    """An fp32 source whose rows are whole vectors, once on the grid of 16-byte vectors and once 4 bytes off it: the kernel for
    operands at any element sums the same values in the same order."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(p + q + r)
    data = torch.randn(p, q, generator=gen, device="cuda")
    om = torch.randn(q, r, generator=gen, device="cuda")
    got = []
    for offset in (0, 1):
        W = [torch.zeros(p, q, device="cuda")]
        opt = lordo.Lordo([(p, q, r)], lordo.hparams(power_iters=0, seed=3), W, torch)
        s = _window(torch, p, q, torch.float32, offset, gen)[1]
        s.copy_(data)
        opt.refresh_subspace([s], [om])
        got.append(opt.get_state(0, lordo.STATE_Q))
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("p, q, r", [(33, 65, 7), (130, 259, 37), (301, 77, 66)])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("offset", [0, 1])
def test_fp32_gradients_at_any_element(p, q, r, side, offset):
    """fp32 gradients run in the grouped GEMM, on either side: u of one step against float64 at the library's own Q."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(p + 3 * q + r)
    W = [torch.randn(p, q, generator=gen, device="cuda")]
    G = [_window(torch, p, q, torch.float32, offset, gen)[1]]
    opt = lordo.Lordo([(p, q, r, side)], lordo.hparams(seed=2, grad_dtype=lordo.F32), W, torch)
    opt.init_projection()
    opt.local_step(W, G, 0.1)
    opt.poll_status()
    Q = opt.get_state(0, lordo.STATE_Q).double()
    g = Q.T @ (G[0].double().T if side else G[0].double())
    u = (1 - opt.hp.beta1) * g
    assert float((opt.get_state(0, lordo.STATE_U).double() - u).norm() / u.norm()) <= 2e-6       # fp32 products and sums over 300 terms


# one element, one stage of rows and a bit, K slices, ranks of every tile of the down-projection
@pytest.mark.parametrize("p, r", [(1, 1), (2, 2), (33, 20), (300, 130), (700, 40), (520, 300), (4096, 4)])
@pytest.mark.parametrize("offset", [0, 1])
def test_one_column_beside_a_wide_matrix(p, r, offset):
    """A matrix of one column (a bias, a norm's scale) is read element by element and leaves the route of its neighbours alone: the
    wide matrix has the bits it has beside a matrix of two columns, and the column follows the formulas."""
    import torch
    from paper_2602_04396_amd import lordo
    got = []
    for cols in (1, 2):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(p + r)
        wide = (max(p, 256), 515 if offset else 512, max(r, 4))
        shapes = [wide, (p, cols, r)]
        G = [_window(torch, wide[0], wide[1], torch.bfloat16, offset, gen)[1]]
        W = [torch.randn(wide[0], wide[1], generator=gen, device="cuda")]
        flat, w = _window(torch, p, cols, torch.float32, offset, gen)
        G.append(_window(torch, p, cols, torch.bfloat16, offset, gen)[1])
        before = flat.clone()
        opt = lordo.Lordo(shapes, lordo.hparams(seed=7), W + [w], torch)
        opt.init_projection()
        opt.set_state(1, lordo.STATE_V, 1.0 + torch.rand(r, cols, generator=gen, device="cuda"))
        v0 = opt.get_state(1, lordo.STATE_V).double()
        opt.local_step(W + [w], G, 0.25)
        opt.poll_status()
        got.append((opt.get_state(0, lordo.STATE_U), opt.get_state(0, lordo.STATE_V), W[0]))
        b1, b2, eps = opt.hp.beta1, opt.hp.beta2, opt.hp.eps
        Q = opt.get_state(1, lordo.STATE_Q).double()
        g = Q.T @ G[1].double()
        u, v = (1 - b1) * g, b2 * v0 + (1 - b2) * g * g
        # g: two-term planes of Q (2^-17) over fp32 sums
        assert float((opt.get_state(1, lordo.STATE_U).double() - u).norm() / u.norm()) <= 2e-5
        N = (u / (1 - b1)) / ((v / (1 - b2)).sqrt() + eps)
        want = before[512 + offset:512 + offset + p * cols].view(p, cols).double() - 0.25 * Q @ N
        assert float((w.double() - want).abs().max()) <= 3e-5 * float(want.abs().max())
        flat[512 + offset:512 + offset + p * cols] = before[512 + offset:512 + offset + p * cols]
        assert torch.equal(flat, before)
    for one, two in zip(*got):
        assert torch.equal(one, two)


# plain update on 128-wide and on 256-wide tiles, last tiles of every size
@pytest.mark.parametrize("r", [40, 128, 256])
@pytest.mark.parametrize("store", ["f32", "bf16"])
def test_whole_rows_beside_ragged_ones(r, store):
    """Matrices of whole aligned quads beside others (streamed there): the same bits, and nothing outside, as with every array at an odd
    element, where no row is whole."""
    import torch
    from paper_2602_04396_amd import lordo
    wt = torch.bfloat16 if store == "bf16" else torch.float32
    shapes = [(260, 512, r), (300, 259, r), (513, 68, r), (256, 4, r)]
    results = []
    for offset in (0, 1):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(r)
        bufs = [_window(torch, p, q, wt, offset, gen) for p, q, _ in shapes]
        G = [torch.randn(p, q, generator=gen, device="cuda").bfloat16() for p, q, _ in shapes]
        data = [torch.randn(p, q, generator=gen, device="cuda").to(wt) for p, q, _ in shapes]
        for (_, view), x in zip(bufs, data):
            view.copy_(x)
        W = [view for _, view in bufs]
        before = [flat.clone() for flat, _ in bufs]
        opt = lordo.Lordo(shapes, lordo.hparams(seed=5, param_dtype=lordo.BF16 if store == "bf16" else lordo.F32), W, torch)
        opt.init_projection()
        for _ in range(2):
            opt.local_step(W, G, 0.25)
        opt.poll_status()
        results.append([w.clone() for w in W])
        for (flat, view), old, x in zip(bufs, before, data):
            assert not torch.equal(view, x)
            view.copy_(x)
            assert torch.equal(flat, old)
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("shape", [(128, 256, 64), (384, 132, 16), (260, 512, 130)])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_fp32_gradients_of_an_aligned_shape_have_the_same_bits_beside_a_ragged_one(shape, side, offset):
    """fp32 gradients whose rows are whole vectors, at any element: their step runs on the fp32 matrix cores where the pointer is off the
    grid of 16-byte vectors, as that of ragged shapes does, whatever else the set holds; g against float64 at the library's own Q."""
    import torch
    from paper_2602_04396_amd import lordo
    p, q, r = shape
    got = []
    for rest in ([], [(33, 65, 7, side)]):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(p + q)
        shapes = [(p, q, r, side)] + rest
        G = [_window(torch, s[0], s[1], torch.float32, offset, gen)[1] for s in shapes]
        W = [torch.zeros(s[0], s[1], device="cuda") for s in shapes]
        opt = lordo.Lordo(shapes, lordo.hparams(seed=2, grad_dtype=lordo.F32), W, torch)
        k = q if side else p
        block, _ = torch.linalg.qr(torch.randn(k, r, generator=torch.Generator().manual_seed(1), dtype=torch.float64))
        opt.set_state(0, lordo.STATE_Q, block.float().cuda().contiguous())
        opt.local_step(W, G, 0.1)
        opt.poll_status()
        u = opt.get_state(0, lordo.STATE_U)
        Q = opt.get_state(0, lordo.STATE_Q).double()
        want = (1 - opt.hp.beta1) * (Q.T @ (G[0].double().T if side else G[0].double()))
        assert float((u.double() - want).norm() / want.norm()) <= 2e-6       # fp32 products and sums over 500 terms
        got.append(u)
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("store", ["f32", "bf16"])
@pytest.mark.parametrize("offset", [0, 1])
def test_many_wide_tiles_on_rows_at_any_element(store, offset):
    """Enough tiles of 256 x 128 for the kernel that takes ranks from 256 up on them: one ragged matrix beside one of whole quads (offset 0), and
    both ragged.  Weights against float64 at the library's own Q and N, nothing written outside."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(offset)
    wt = torch.bfloat16 if store == "bf16" else torch.float32
    shapes = [(3050, 16385, 256), (520, 512, 300)]
    bufs = [_window(torch, p, q, wt, offset, gen) for p, q, _ in shapes]
    G = [torch.randn(p, q, generator=gen, device="cuda").bfloat16() for p, q, _ in shapes]
    W = [view for _, view in bufs]
    before = [flat.clone() for flat, _ in bufs]
    opt = lordo.Lordo(shapes, lordo.hparams(seed=5, param_dtype=lordo.BF16 if store == "bf16" else lordo.F32), W, torch)
    opt.init_projection()
    lr = 0.25
    opt.local_step(W, G, lr)
    opt.poll_status()
    for i, (p, q, r) in enumerate(shapes):
        start = 512 + offset
        old = before[i][start:start + p * q].view(p, q).double()
        want = old - lr * opt.get_state(i, lordo.STATE_Q).double() @ opt.get_state(i, lordo.STATE_NUPD).double()
        ulp = 0.0 if store == "f32" else 2.0 ** -8                # rounded once; ahead of it the planes' 2^-17 of Q N, and fp32 sums
        assert float(((W[i].double() - want).abs() - ulp * want.abs()).max()) <= 3e-5 * float(want.abs().max()), i
        got = bufs[i][0].clone()
        got[start:start + p * q] = before[i][start:start + p * q]
        assert torch.equal(got, before[i]), i


@pytest.mark.parametrize("p, q, r", [(128, 200, 64), (130, 67, 33), (40, 3, 3), (96, 260, 5)])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("grad", ["f32", "bf16"])
def test_an_infinity_stays_in_its_column(p, q, r, side, grad):
    """Rows that an edge tile of the grouped GEMM reads in the place of absent ones end in no element that is stored: infinities in the
    first and last element of G reach the moments of their own columns (rows, projected on the right) alone."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(p + q)
    if side:
        p, q = q, p
    G = torch.randn(p, q, generator=gen, device="cuda")
    G[0, 0] = G[-1, -1] = float("inf")
    G = G if grad == "f32" else G.bfloat16()
    W = [torch.zeros(p, q, device="cuda")]
    r = min(r, q if side else p)
    opt = lordo.Lordo([(p, q, r, side)], lordo.hparams(seed=2, grad_dtype=lordo.F32 if grad == "f32" else lordo.BF16), W, torch)
    opt.init_projection()
    opt.local_step(W, [G], 0.1)
    u = opt.get_state(0, lordo.STATE_U)
    bad = ~torch.isfinite(u).all(0)
    assert bad[0] and bad[-1] and int(bad.sum()) == 2
    payload, moments = opt.sync_payload()
    cols = p if side else q
    v = payload[:moments // 2].view((cols + 31) // 32, -1, 32, 8)          # column block, rank group, column, rank
    assert bool((v[-1, :, cols % 32:] == 0).all()) or cols % 32 == 0
    if r % 32:
        pad = v.permute(1, 3, 0, 2).reshape(-1, v.shape[0] * 32)[r:]          # ranks past the last one
        assert bool(torch.isfinite(pad[:, 1:cols - 1]).all())


@pytest.mark.parametrize("source", ["bf16", "fp32"])
@pytest.mark.parametrize("offset", [0, 1])
def test_refresh_of_a_set_of_every_kind(source, offset):
    """Aligned, ragged and too-short operands in one launch (ranks and sides below four beside large matrices): every basis is orthonormal,
    spans its source's columns, and the moments are those of before, rotated."""
    import torch
    from paper_2602_04396_amd import lordo
    gen = torch.Generator(device="cuda")
    gen.manual_seed(offset)
    shapes = [(256, 320, 64), (389, 515, 131), (130, 97, 2), (300, 3, 3), (96, 1, 1), (68, 256, 3), (257, 129, 66)]
    W = [torch.randn(p, q, generator=gen, device="cuda") for p, q, r in shapes]
    opt = lordo.Lordo(shapes, lordo.hparams(power_iters=1, seed=3), W, torch)
    opt.init_projection()
    for _ in range(2):
        opt.local_step(W, [torch.randn(p, q, generator=gen, device="cuda").bfloat16() for p, q, r in shapes], 0.5)
    q_old = [opt.get_state(i, lordo.STATE_Q).double() for i in range(len(shapes))]
    u_old = [opt.get_state(i, lordo.STATE_U).double() for i in range(len(shapes))]
    dt = torch.bfloat16 if source == "bf16" else torch.float32
    src, om, U = [], [], []
    for p, q, r in shapes:
        a, _ = torch.linalg.qr(torch.randn(p, r, generator=gen, device="cuda", dtype=torch.float64))
        b, _ = torch.linalg.qr(torch.randn(q, r, generator=gen, device="cuda", dtype=torch.float64))
        src.append(_window(torch, p, q, dt, offset, gen)[1])
        src[-1].copy_(100.0 * a @ b.T)
        om.append(_window(torch, q, r, torch.float32, offset, gen)[1])
        U.append(a)
    opt.refresh_subspace(src, om)
    opt.poll_status()
    for i, (p, q, r) in enumerate(shapes):
        Q = opt.get_state(i, lordo.STATE_Q).double()
        assert float((Q.T @ Q - torch.eye(r, device="cuda", dtype=torch.float64)).norm()) <= 1e-4, i      # CholeskyQR2 in fp32
        if source == "fp32":      # (a bf16 source has rounding noise: its trailing directions depend on the start block)
            assert float((U[i] - Q @ (Q.T @ U[i])).norm()) / r ** 0.5 <= 5e-5, i
        want = (Q.T @ q_old[i]) @ u_old[i]
        assert float((opt.get_state(i, lordo.STATE_U).double() - want).norm() / want.norm()) <= 1e-5, i   # fp32 sums over p and r
