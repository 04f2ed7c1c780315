"""Products whose every element is checked: a value lost or overwritten on its way out of a kernel is a single element of
millions and moves no norm."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q, r, repeats", [(2048, 256, 4), (768, 128, 4)])
def test_source_times_block_leaves_no_element_behind(q, r, repeats):
    """k_src_times_block, seen through the low-rank gradient g = G Q of right-projected matrices: the store of a tile's last
    rows was overtaken by the next instruction, about once in a thousand tiles."""
    import torch
    from paper_2602_04396_amd import lordo
    n, p = 24, 2048
    gen = torch.Generator(device="cuda")
    gen.manual_seed(q + r)
    G = [torch.randn(p, q, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(n)]
    W = [torch.zeros(p, q, device="cuda") for _ in range(n)]
    opt = lordo.Lordo([(p, q, r, 1)] * n, lordo.hparams(power_iters=0, seed=5), W, torch)
    opt.init_projection()
    ref = [G[i].float() @ opt.get_state(i, lordo.STATE_Q) for i in range(n)]
    for _ in range(repeats):
        opt.local_step(W, G, 0.0)
        for i in range(n):
            g = opt.get_state(i, lordo.STATE_GLOW).T
            # q products of exact bf16 values with Q in two bf16 planes (2^-17 each, random): 8e-6 of the rms, five sigma
            # over half a million elements 4e-5; a lost element is off by itself
            worst = float((g - ref[i]).abs().max() / ref[i].square().mean().sqrt())
            assert worst <= 1e-3, f"matrix {i}: an element is off by {worst:.2e} of the rms"
