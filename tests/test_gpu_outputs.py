"""rt_hit_outputs: hit records split into (t, u, v), prim and hit flags."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 100_001])
def test_hit_outputs(n):
    import torch
    from paper_1912_12786_amd import rtx
    rtx.load_library()
    print(f"[gpu-case] hit outputs n={n}", flush=True)
    g = torch.Generator().manual_seed(n)
    hits = torch.randn(n, 4, generator=g)
    prim = torch.randint(0, 2**29 - 1, (n,), generator=g, dtype=torch.int32)
    prim[torch.rand(n, generator=g) < 0.3] = -1
    hits[:, 1] = prim.view(torch.float32)
    hits[prim == -1, 0] = float("inf")
    h = hits.cuda()
    # one element more of each, which stays as it is
    tuv = torch.full((n + 1, 3), 7.0, device="cuda")
    out = torch.full((n + 1,), 7, dtype=torch.int32, device="cuda")
    flag = torch.full((n + 1,), 7, dtype=torch.uint8, device="cuda")
    rtx.rt_hit_outputs(h.data_ptr(), n, tuv.data_ptr(), out.data_ptr(), flag.data_ptr(),
                       torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    want = torch.where((prim == -1)[:, None], torch.zeros(1), hits[:, [0, 2, 3]])
    assert torch.equal(tuv[:n].cpu().view(torch.int32), want.view(torch.int32))
    assert torch.equal(out[:n].cpu(), prim)
    assert torch.equal(flag[:n].cpu(), (prim != -1).to(torch.uint8))
    assert (tuv[n] == 7).all() and out[n] == 7 and flag[n] == 7


def test_only_prim_used():
    """A loss without t, u, v gives zero gradients rather than an error."""
    import numpy as np
    import torch
    from paper_1912_12786_amd import diff
    print("[gpu-case] differentiable hit, gradient of a zero weight", flush=True)
    v = torch.tensor([[0., 0, 0], [1, 0, 0], [0, 1, 0]], device="cuda", requires_grad=True)
    r = torch.tensor([[.2, .2, -1, 0, 0, 0, 1, np.inf]], dtype=torch.float32, device="cuda",
                     requires_grad=True)
    tuv, prim, hit = diff.DifferentiableHit.apply(r, v, torch.tensor([[0, 1, 2]]), None, None, None)
    assert prim.dtype == torch.int32 and hit.dtype == torch.bool and bool(hit[0]) and int(prim[0]) == 0
    gr, gv = torch.autograd.grad((tuv * 0).sum(), (r, v))
    assert torch.equal(gr, torch.zeros_like(r)) and torch.equal(gv, torch.zeros_like(v))


def test_no_gradient_of_tuv(monkeypatch):
    """An operation after the hit that has no gradient of its own: the rays and
    vertices still get zeros, without a run of the adjoint."""
    import numpy as np
    import torch
    from paper_1912_12786_amd import diff, rtx

    class Stops(torch.autograd.Function):
        @staticmethod
        def forward(ctx, x):
            return x.sum()

        @staticmethod
        def backward(ctx, g):
            return None

    def refuse(*a):
        raise AssertionError("the adjoint ran")

    monkeypatch.setattr(rtx, "rt_hit_backward", refuse)
    print("[gpu-case] differentiable hit, no gradient of t, u, v", flush=True)
    v = torch.tensor([[0., 0, 0], [1, 0, 0], [0, 1, 0]], device="cuda", requires_grad=True)
    r = torch.tensor([[.2, .2, -1, 0, 0, 0, 1, np.inf]], dtype=torch.float32, device="cuda",
                     requires_grad=True)
    tuv, _, hit = diff.DifferentiableHit.apply(r, v, torch.tensor([[0, 1, 2]]), None, None, None)
    assert bool(hit[0])
    # and a path of its own for each input, so that the loss depends on both
    gr, gv = torch.autograd.grad(Stops.apply(tuv) + (r[:, :3] + v[:1]).sum(), (r, v))
    assert gr.tolist() == [[1, 1, 1, 0, 0, 0, 0, 0]] and gv.tolist() == [[1, 1, 1], [0, 0, 0], [0, 0, 0]]
    gr, gv = torch.autograd.grad(Stops.apply(
        diff.DifferentiableHit.apply(r, v, torch.tensor([[0, 1, 2]]), None, None, None)[0]), (r, v))
    assert torch.equal(gr, torch.zeros_like(r)) and torch.equal(gv, torch.zeros_like(v))
