"""The data term's kernels: every absolute-difference sum of three channels, and
the pair route (frames read directly, or packed after averaging) against the
volume route.

Tolerances: none.  The rounded mean is an integer; the exact mean is the
correctly rounded quotient sum / 3, which FP32 division gives too; the routes
run the same arithmetic on the same costs.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("mode", [0, 1])
def test_every_sum(dev, mode):
    import paper_1902_09733_amd as bp
    s = np.arange(766)
    left = np.zeros((4, 766, 3), np.uint8)
    for c in range(3):
        left[:2, :, c] = np.clip(s - 255 * c, 0, 255)
    right = left[[2, 3, 0, 1]].copy()
    cost = bp.cost_volume(torch.from_numpy(left).to(dev), torch.from_numpy(right).to(dev), 1, 1000.0, rgb_mode=mode)
    want = ((s + 1) // 3).astype(np.float32) if mode == 0 else s.astype(np.float32) / np.float32(3)
    assert np.array_equal(cost.cpu().numpy()[0], np.broadcast_to(want, (4, 766)))


@pytest.mark.parametrize("w,h,L,levels,ds,ch,mode", [
    (161, 67, 33, 1, 1, 1, 0), (161, 67, 33, 1, 1, 3, 1), (97, 41, 16, 2, 1, 3, 0), (131, 35, 64, 3, 1, 3, 1),
    (64, 33, 5, 2, 1, 1, 0), (75, 30, 128, 2, 1, 3, 0), (70, 31, 100, 1, 1, 3, 0), (129, 64, 64, 2, 2, 3, 0),
    (130, 33, 20, 1, 3, 3, 1), (128, 33, 48, 2, 4, 1, 0), (40, 9, 64, 2, 1, 3, 1),
])
def test_pair_route_equals_volume_route(dev, w, h, L, levels, ds, ch, mode):
    import paper_1902_09733_amd as bp
    print(f"pair route {w}x{h} L={L} levels={levels} ds={ds} ch={ch} mode={mode}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(w + h + L)
    shape = (2, h * ds, w * ds) + ((3,) if ch == 3 else ())
    img = torch.randint(0, 256, shape, generator=g, device=dev, dtype=torch.uint8)
    left, right = img[0].contiguous(), img[1].contiguous()
    for trunc in (20.0, 33.3):
        cost = bp.cost_volume(left, right, L, trunc, downsample=ds, rgb_mode=mode)
        for K in (2, 5):
            p = bp.BPParams(levels=levels, iters=K, lam=7.0, tau=2.5)
            a = bp.run(bp.Pair(left, right, L, trunc, downsample=ds, rgb_mode=mode), p, want_soft=True, want_msgs=True)
            b = bp.run(cost, p, want_soft=True, want_msgs=True)
            torch.cuda.synchronize()
            for k in ("disp", "soft", "msgs"):
                assert torch.equal(a[k], b[k]), (trunc, K, k)
