"""Several pairs of half-sweeps per launch (streamed down strips of columns)
against one launch per half-sweep.

Levels of at least 4 M values (width * height * stored labels), 64 rows and two
blocks' columns run two pairs per launch, from 16 M values three.  Variant 1 is
the one-half-sweep kernel with the same per-message arithmetic, so labels,
soft-argmin disparities and final messages must agree bit for bit on
real-valued costs: tolerance 0.  Shapes: each lane split, the smallest widths and
heights the rule takes, strips and segments that do not divide the grid, odd
and even K (schedules of one, two and three pairs), each form of the transform
(tau 2, 2.6 and 5), a pyramid under a streamed finest level, and the storage
formats (16-bit levels under the FP32 coarsest level need an even number of
launches).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1902_09733_amd as bp
    bp.stereo._abi.lib()
    return torch.device("cuda:0")


CASES = [
    # (L, H, W, levels, K, fmt, tau)
    (64, 653, 96, 1, 4, "f32", 2.0),       # two columns more than a strip with its edges, many segments
    (64, 64, 978, 1, 5, "f32", 2.6),       # the lowest grid
    (64, 251, 263, 2, 10, "f32", 2.0),     # 1 + 2 + 2 pairs
    (64, 401, 641, 2, 10, "f32", 2.0),     # 3 + 2 pairs
    (64, 499, 503, 1, 8, "f32", 5.0),      # 2 + 2 pairs of three-pair size, scans
    (64, 500, 517, 1, 12, "f32", 2.6),     # 3 + 3
    (32, 411, 307, 2, 7, "f32", 2.6),
    (32, 707, 723, 1, 6, "f32", 2.0),
    (16, 640, 401, 1, 6, "f32", 2.0),
    (16, 1001, 1009, 1, 6, "f32", 5.0),
    (96, 211, 203, 2, 6, "f32", 2.6),
    (96, 400, 421, 1, 6, "f32", 2.0),
    (128, 505, 65, 1, 4, "f32", 2.0),
    (128, 181, 190, 2, 12, "f32", 2.6),
    (128, 353, 360, 1, 6, "f32", 2.0),
    (64, 251, 263, 2, 12, "f16", 2.0),     # an even number of launches: 2 + 2 + 1 + 1
    (64, 500, 517, 2, 10, "f16", 2.6),     # 3 + 2
    (64, 500, 517, 2, 6, "bf16", 2.0),     # 3 as 1 + 2
    (96, 400, 421, 2, 8, "f16", 2.0),
    (128, 353, 360, 2, 12, "bf16", 2.6),
    (128, 353, 367, 3, 8, "f16", 2.0),
]


@pytest.mark.parametrize("L,H,W,levels,K,fmt,tau", CASES)
def test_streamed_equal_single_half_sweeps(dev, L, H, W, levels, K, fmt, tau):
    import paper_1902_09733_amd as bp
    print(f"streamed vs single: L={L} {W}x{H} levels={levels} K={K} {fmt} tau={tau}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(L * 1000 + H + W + K)
    cost = 20.0 * torch.rand((L, H, W), generator=g, device=dev)
    outs = []
    for variant in (0, 1):
        p = bp.BPParams(levels=levels, iters=K, lam=7.3, tau=tau, msg_dtype=fmt, variant=variant, temperature=0.7)
        outs.append(bp.run(cost, p, want_soft=True, want_msgs=True))
    torch.cuda.synchronize()
    for k in ("disp", "soft", "msgs"):
        assert torch.equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("L,rgb_mode,K", [(64, 0, 10), (96, 0, 8), (128, 0, 8), (64, 1, 8)])
def test_streamed_pair_route_equals_volume_route(dev, L, rgb_mode, K):
    """Byte and FP16 costs of the pair route (FP32 with the exact mean) against the FP32 volume route."""
    import paper_1902_09733_amd as bp
    print(f"streamed pair route: L={L} rgb_mode={rgb_mode} K={K}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(L + K)
    left = torch.randint(0, 256, (341, 547, 3), generator=g, device=dev, dtype=torch.uint8)
    right = torch.randint(0, 256, (341, 547, 3), generator=g, device=dev, dtype=torch.uint8)
    p = bp.BPParams(levels=3, iters=K)
    a = bp.run(bp.Pair(left, right, L, 20.0, rgb_mode=rgb_mode), p, want_msgs=True)
    cost = bp.cost_volume(left, right, L, 20.0, rgb_mode=rgb_mode)
    b = bp.run(cost, bp.BPParams(levels=3, iters=K, variant=1), want_msgs=True)
    torch.cuda.synchronize()
    assert torch.equal(a["disp"], b["disp"]) and torch.equal(a["msgs"], b["msgs"])


@pytest.mark.parametrize("fmt,K,levels", [("f32", 6, 2), ("f16", 8, 3)])
def test_batch_with_streamed_problems(dev, fmt, K, levels):
    """A batch in which some problems stream (a group of their own) and the small ones share launches, in
    byte, FP16 and FP32 finest-level costs, against each problem alone with one launch per half-sweep."""
    import paper_1902_09733_amd as bp
    shapes = [(64, 260, 420), (64, 40, 53), (96, 250, 301), (32, 31, 40), (64, 39, 50), (128, 200, 331)]
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    pairs = []
    for L, h, w in shapes:
        img = torch.randint(0, 256, (2, h, w, 3), generator=g, device=dev, dtype=torch.uint8)
        pairs.append(bp.Pair(img[0].contiguous(), img[1].contiguous(), L, 20.0))
    outs = bp.run(pairs, bp.BPParams(levels=levels, iters=K, msg_dtype=fmt), want_msgs=True)
    for p, o in zip(pairs, outs):
        cost = bp.cost_volume(p.left, p.right, p.num_labels, 20.0)
        r = bp.run(cost, bp.BPParams(levels=levels, iters=K, msg_dtype=fmt, variant=1), want_msgs=True)
        torch.cuda.synchronize()
        assert torch.equal(o["disp"], r["disp"]) and torch.equal(o["msgs"], r["msgs"]), p.shape
