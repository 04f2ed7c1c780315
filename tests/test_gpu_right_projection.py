"""Projection on the right (`side = 1` of a shape): Sec. 2 applied to the transposed matrix, on the caller's row-major
arrays.  The library's two products of the step and its refresh against the oracle's explicit right-side formulas."""
import numpy as np
import pytest

from oracle import lordo_oracle as orc
from paper_2602_04396_amd import synth
from tests.harness import Pair, rel_l2

pytestmark = pytest.mark.gpu

TOL, TOL_SUBSPACE, TOL_ORTH = 1e-4, 1e-3, 1e-4


def lowrank_dims(sh):
    """(rows of Q, columns of the moments) of a shape: those of the transposed problem for side 1."""
    p, q, r = sh[:3]
    return (q, p) if len(sh) > 3 and sh[3] else (p, q)


SHAPE_SETS = {
    "mixed": [(300, 96, 24, 1), (128, 256, 32, 0), (517, 130, 33, 1)],            # ragged, odd rank, both sides in one context
    "right_only": [(1024, 256, 64, 1), (768, 128, 128, 1)],                       # tall matrices, rank = short side included
    "aligned_mixed": [(520, 128, 36, 1), (256, 384, 64, 0), (3072, 768, 128, 1)], # shapes the streaming kernel takes, beside a left-projected one
}


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "fp32"])
@pytest.mark.parametrize("qhm", ["none", "low", "low_ef", "full", "full_ef"])
@pytest.mark.parametrize("name", list(SHAPE_SETS))
def test_right_projection_steps_refresh_outer(name, qhm, bf16):
    import torch
    from paper_2602_04396_amd import lordo
    shapes = SHAPE_SETS[name]
    ef = qhm.endswith("_ef")             # error feedback (Alg. 1): the residual of a right-projected matrix, E <- s G + E - g Q^T
    qhm = qhm.split("_")[0]              # full: Sec. 3.2 on the transposed problem, the gradient term scaled per row of W
    n = len(shapes)
    omega = 0.8 if qhm != "none" else 1.0
    common = dict(omega=omega, outer_lr=0.7, outer_momentum=0.9, outer_nesterov=True, power_iters=1, error_feedback=ef)
    ohp = orc.Hyper(qhm_mode=qhm, **common)
    ghp = lordo.hparams(qhm_mode={"none": 0, "low": 1, "full": 2}[qhm], grad_dtype=lordo.BF16 if bf16 else lordo.F32, **common)
    W0 = [synth.weights(np.random.default_rng(synth.seed_for(80, i)), sh[0], sh[1]) for i, sh in enumerate(shapes)]
    Q0 = [synth.orthonormal(np.random.default_rng(synth.seed_for(81, i)), lowrank_dims(sh)[0], sh[2]).astype(np.float32)
          for i, sh in enumerate(shapes)]
    pair = Pair(torch, shapes, W0, ohp, ghp, Q0)
    gens = [synth.SpikedGradient(sh[0], sh[1], 4, synth.seed_for(82, i), bf16=bf16) for i, sh in enumerate(shapes)]
    if (ef or qhm == "full") and name == "mixed":
        # the gradient-term epilogue of the up-projection kernel needs rows of W of a multiple of 4 floats: 130 columns are refused
        W_before = [w.clone() for w in pair.W_gpu]
        with pytest.raises(lordo.LordoError) as e:
            pair.opt.local_step(pair.W_gpu, pair.to_dev([g.draw(0) for g in gens], bf16), 1e-3)
        assert e.value.code == lordo.EINVAL and pair.opt.step == 0
        assert all(torch.equal(a, b) for a, b in zip(W_before, pair.W_gpu))
        return
    for t in range(3):
        pair.local_step([g.draw(t) for g in gens], lr=1e-3 * (1 + t), grad_scale=0.9, bf16=bf16, first_step_patch=(t == 0))
        pair.compare_local(TOL)
    # outer step (elementwise on the caller's arrays; the oracle state of a right-projected matrix holds transposes)
    pair.opt.outer_step(pair.W_gpu, None)
    for i in range(n):
        st = pair.st[i]
        Wt = pair.W_orc[i].T if pair.side[i] else pair.W_orc[i]
        Wt = orc.outer_step(st, orc.pseudo_gradient(st, Wt), ohp)
        pair.W_orc[i] = Wt.T.copy() if pair.side[i] else Wt
        got = pair.W_gpu[i].cpu().numpy().astype(np.float64)
        assert rel_l2(got - pair.W0[i], pair.W_orc[i] - pair.W0[i]) <= TOL, f"outer step, matrix {i}"
    # refresh from a fresh source: Omega has as many rows as the moments have columns
    Src = [g.draw(100) for g in gens]
    Om = [synth.omega(np.random.default_rng(synth.seed_for(83, i)), lowrank_dims(sh)[1], sh[2]) for i, sh in enumerate(shapes)]
    dists, orths = pair.refresh(Src, Om, bf16=bf16)
    assert max(orths) <= TOL_ORTH and max(dists) <= TOL_SUBSPACE, f"orth {orths} dist {dists}"
    for i, sh in enumerate(shapes):                     # the basis of a right-projected matrix lives on the columns
        assert pair.get(i, lordo.STATE_Q).shape == (lowrank_dims(sh)[0], sh[2])
    for t in range(2):
        pair.local_step([g.draw(5 + t) for g in gens], lr=1e-3, bf16=bf16)
        pair.compare_local(TOL)


def test_right_projection_rayleigh_ritz_and_metrics():
    """Rayleigh-Ritz refresh on a right-projected matrix: ordered right singular vectors, Ritz values, stable rank."""
    import torch
    from paper_2602_04396_amd import lordo
    shapes = [(640, 160, 32, 1)]
    p, q, r = shapes[0][:3]
    ghp = lordo.hparams(power_iters=2, rayleigh_ritz=True, grad_dtype=lordo.F32)
    W0 = [synth.weights(np.random.default_rng(synth.seed_for(84, 0)), p, q)]
    pair = Pair(torch, shapes, W0, orc.Hyper(power_iters=2, rayleigh_ritz=True), ghp)
    Src = [synth.SpikedGradient(p, q, 12, synth.seed_for(85, 0), bf16=False).draw(0)]
    Om = [synth.omega(np.random.default_rng(synth.seed_for(86, 0)), p, r)]
    dists, orths = pair.refresh(Src, Om, bf16=False)
    assert max(orths) <= TOL_ORTH
    A = np.asarray(Src[0], dtype=np.float64)
    Qg = pair.get(0, lordo.STATE_Q)                      # q x r
    ritz = pair.get(0, lordo.STATE_RITZ)
    sv = np.linalg.svd(A, compute_uv=False)
    assert np.all(np.diff(ritz) <= 1e-6 * ritz[0])
    np.testing.assert_allclose(ritz[:12], sv[:12], rtol=1e-4)            # the spikes are found exactly
    B = A @ Qg                                           # columns: A q_i, orthogonal with norms = Ritz values
    gram = B.T @ B
    off = gram - np.diag(np.diag(gram))
    assert np.linalg.norm(off) <= 1e-4 * np.linalg.norm(gram)
    np.testing.assert_allclose(np.sqrt(np.diag(gram)), ritz, rtol=1e-4, atol=1e-6 * ritz[0])
    sr = float(pair.opt.stable_rank().cpu().numpy()[0])
    assert abs(sr - orc.stable_rank(A)) <= 1e-4 * orc.stable_rank(A)
    # spectral gap (Sec. 5.1): the estimate of sigma_(r+1) against the oracle's iteration on the transposed source with
    # the library's basis, and against the exact norm of the deflated source; the basis is left alone
    Om2 = synth.omega(np.random.default_rng(synth.seed_for(86, 1)), p, r)
    Q_before = pair.opt.get_state(0, lordo.STATE_Q)
    gap = float(pair.opt.spectral_gap(pair.to_dev(Src, False), pair.to_dev([Om2], False)).cpu().numpy()[0])
    pair.opt.poll_status()
    assert torch.equal(pair.opt.get_state(0, lordo.STATE_Q), Q_before)
    est_gpu = ritz[-1] - gap
    est_orc = orc.next_singular_value_estimate(A.T, Qg, np.asarray(Om2, dtype=np.float64), 2)
    deflated = np.linalg.svd(A.T - Qg @ (Qg.T @ A.T), compute_uv=False)[0]
    assert abs(est_gpu - est_orc) <= 1e-4 * est_orc
    assert 0.85 * deflated <= est_gpu <= (1 + 1e-4) * deflated


@pytest.mark.parametrize("mom", [0.0, 0.9])
@pytest.mark.parametrize("name", ["mixed", "aligned_mixed"])
def test_right_projection_uplink_buffer_and_lowrank_outer_step(name, mom):
    """Up-link buffer (App. A.5.1) with right-projected matrices: A accumulates lr * N in the layout of the transposed
    problem (r x rows), and the outer step forms Delta = (Q A)^T in the up-projection kernel on the caller's rows."""
    import torch
    from paper_2602_04396_amd import lordo
    shapes = SHAPE_SETS[name]
    common = dict(uplink_buffer=True, outer_lr=0.7, outer_momentum=mom, outer_nesterov=True, power_iters=1)
    ohp = orc.Hyper(**common)
    ghp = lordo.hparams(grad_dtype=lordo.BF16, **common)
    W0 = [synth.weights(np.random.default_rng(synth.seed_for(87, i)), sh[0], sh[1]) for i, sh in enumerate(shapes)]
    Q0 = [synth.orthonormal(np.random.default_rng(synth.seed_for(88, i)), lowrank_dims(sh)[0], sh[2]).astype(np.float32)
          for i, sh in enumerate(shapes)]
    pair = Pair(torch, shapes, W0, ohp, ghp, Q0)
    gens = [synth.SpikedGradient(sh[0], sh[1], 4, synth.seed_for(89, i), bf16=True) for i, sh in enumerate(shapes)]
    for window in range(2):
        for t in range(3):
            pair.local_step([g.draw(10 * window + t) for g in gens], lr=1e-3 * (1 + t), bf16=True, first_step_patch=(window == 0 and t == 0))
        pair.compare_local(TOL)                          # includes the buffer A
        out = [torch.empty(sh[2], lowrank_dims(sh)[1], dtype=torch.float32, device="cuda") for sh in shapes]
        pair.opt.export_uplink(out)
        avg = [0.5 * o.cpu().numpy() for o in out]       # stand-in for the mean over workers
        pair.opt.outer_step_lowrank(pair.W_gpu, pair.to_dev(avg, False))
        for i in range(len(shapes)):
            Wt = orc.outer_step_lowrank(pair.st[i], np.asarray(avg[i], dtype=np.float64), ohp)
            pair.W_orc[i] = Wt.T.copy() if pair.side[i] else Wt
            got = pair.W_gpu[i].cpu().numpy().astype(np.float64)
            assert rel_l2(got - pair.W0[i], pair.W_orc[i] - pair.W0[i]) <= TOL, f"window {window}, matrix {i}"
            assert np.array_equal(pair.get(i, lordo.STATE_ANCHOR), got.astype(np.float32).astype(np.float64))


@pytest.mark.parametrize("name", ["right_only", "aligned_mixed"])
def test_right_projection_local_variant(name):
    """Alg. 2 with right-projected matrices: identity columns as Q_0, projection from s G + E of the step's own gradient,
    low-rank QHM with error feedback; two refreshes with steps between."""
    import torch
    from paper_2602_04396_amd import lordo
    shapes = SHAPE_SETS[name]
    common = dict(omega=0.8, error_feedback=True, power_iters=1)
    ohp = orc.Hyper(qhm_mode="low", **common)
    ghp = lordo.hparams(qhm_mode=1, grad_dtype=lordo.BF16, **common)
    W0 = [synth.weights(np.random.default_rng(synth.seed_for(90, i)), sh[0], sh[1]) for i, sh in enumerate(shapes)]
    pair = Pair(torch, shapes, W0, ohp, ghp)
    gens = [synth.SpikedGradient(sh[0], sh[1], 4, synth.seed_for(91, i), bf16=True) for i, sh in enumerate(shapes)]
    t = 0
    for window in range(2):
        G = [g.draw(t) for g in gens]
        Om = [synth.omega(np.random.default_rng(synth.seed_for(92, 10 * window + i)), lowrank_dims(sh)[1], sh[2]) for i, sh in enumerate(shapes)]
        dists, orths = pair.refresh_local(G, Om, grad_scale=0.9, bf16=True)
        assert max(orths) <= TOL_ORTH and max(dists) <= TOL_SUBSPACE, f"window {window}: orth {orths} dist {dists}"
        pair.local_step(G, lr=1e-3, grad_scale=0.9, bf16=True, first_step_patch=(window == 0))
        pair.compare_local(TOL)
        t += 1
        for _ in range(2):
            pair.local_step([g.draw(t) for g in gens], lr=1e-3, grad_scale=0.9, bf16=True)
            t += 1
        pair.compare_local(TOL)


@pytest.mark.parametrize("shape", [(64, 96, 20, 1), (160, 64, 4, 1), (40, 160, 100, 1)])
def test_padding_of_the_payload_stays_zero_beside_an_infinity(shape):
    """The packed payload is padded with zeros (lordo_sync_payload), also where a gradient holds an infinity: the streaming kernel stores the
    product of absent rank planes as zero, not as 0 * inf."""
    import torch
    from paper_2602_04396_amd import lordo
    p, q, r, side = shape
    G = torch.randn(p, q, generator=torch.Generator().manual_seed(p)).bfloat16().cuda()
    G[p - 1, 3] = float("inf")
    W = [torch.zeros(p, q, device="cuda")]
    opt = lordo.Lordo([shape], lordo.hparams(seed=2), W, torch)
    opt.init_projection()
    opt.local_step(W, [G], 0.1)
    payload, moments = opt.sync_payload()
    u = payload[:moments // 2].view((p + 31) // 32, -1, 32, 8).permute(0, 2, 1, 3).reshape((p + 31) // 32 * 32, -1)      # state column, rank
    assert not bool(torch.isfinite(u[p - 1, :r]).all()) and bool(torch.isfinite(u[:p - 1]).all())
    assert bool((u[:, r:] == 0).all()) and bool((u[p:] == 0).all())
