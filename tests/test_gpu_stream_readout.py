"""The streamed last launch that reads out both colours (no final state wanted)
against one launch per half-sweep and a readout pass.

The arithmetic is the same, so labels and soft-argmin disparities must agree bit
for bit: tolerance 0.  Each lane split and last launch (two and three pairs), the
forms of the transform, strips and segments that do not divide the grid, labels
alone and soft disparities alone, replays with other inputs in between (nothing
of the last call's state may show), and batches.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("L,H,W,levels,K,fmt,tau", [
    (64, 653, 96, 1, 4, "f32", 2.0),
    (64, 251, 263, 2, 10, "f32", 2.6),
    (64, 500, 517, 2, 12, "f32", 2.0),     # three pairs at the end
    (64, 499, 503, 1, 8, "f32", 5.0),
    (32, 707, 723, 1, 6, "f32", 2.0),
    (16, 1001, 1009, 1, 6, "f32", 2.0),
    (16, 1001, 1009, 1, 4, "f32", 5.0),
    (96, 211, 203, 2, 6, "f32", 2.6),
    (96, 400, 421, 1, 6, "f32", 2.0),
    (128, 353, 360, 1, 6, "f32", 2.0),
    (128, 401, 347, 2, 4, "f32", 2.6),
    (128, 353, 367, 1, 4, "f32", 5.0),
    (64, 251, 263, 2, 8, "f16", 2.0),
    (128, 353, 367, 3, 12, "bf16", 2.0),
    (128, 505, 512, 3, 12, "bf16", 2.6),
])
def test_both_colours_read_out(dev, L, H, W, levels, K, fmt, tau):
    import paper_1902_09733_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(L + H + W + K)
    costs = [20.0 * torch.rand((L, H, W), generator=g, device=dev) for _ in range(2)]
    p = [bp.BPParams(levels=levels, iters=K, lam=7.3, tau=tau, msg_dtype=fmt, variant=v, temperature=0.7) for v in (0, 1)]
    ref = [bp.run(c, p[1], want_soft=True, want_msgs=True) for c in costs]
    for i, (d, s) in ((0, (True, True)), (1, (True, False)), (0, (False, True)), (1, (True, True))):
        o = bp.run(costs[i], p[0], want_disp=d, want_soft=s)
        torch.cuda.synchronize()
        assert not d or torch.equal(o["disp"], ref[i]["disp"])
        assert not s or torch.equal(o["soft"], ref[i]["soft"])


@pytest.mark.parametrize("fmt", ["f32", "f16"])
def test_batch(dev, fmt):
    import paper_1902_09733_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    pairs = []
    for L, h, w in [(64, 260, 420), (64, 40, 53), (128, 200, 331), (32, 31, 40)]:
        img = torch.randint(0, 256, (2, h, w, 3), generator=g, device=dev, dtype=torch.uint8)
        pairs.append(bp.Pair(img[0].contiguous(), img[1].contiguous(), L, 20.0))
    outs = bp.run(pairs, bp.BPParams(levels=2, iters=8, msg_dtype=fmt), want_soft=True)
    for p, o in zip(pairs, outs):
        cost = bp.cost_volume(p.left, p.right, p.num_labels, 20.0)
        r = bp.run(cost, bp.BPParams(levels=2, iters=8, msg_dtype=fmt, variant=1), want_soft=True)
        torch.cuda.synchronize()
        assert torch.equal(o["disp"], r["disp"]) and torch.equal(o["soft"], r["soft"]), p.shape
