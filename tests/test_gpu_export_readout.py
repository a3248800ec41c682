"""Final messages and the readout in one pass, against each asked for alone.

Same rows, same arithmetic: tolerance 0.  Every lane split and tile width, grids
narrower than a tile and one pixel past it, odd and even K (which colours are
still to read out), the cost formats of the pair route, 16-bit messages, a batch.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


def check(bp, what, p):
    both = bp.run(what, p, want_soft=True, want_msgs=True)
    read = bp.run(what, p, want_soft=True)
    msgs = bp.run(what, p, want_disp=False, want_msgs=True)
    torch.cuda.synchronize()
    one = lambda o: o if isinstance(o, list) else [o]
    for b, r, m in zip(one(both), one(read), one(msgs)):
        assert torch.equal(b["disp"], r["disp"]) and torch.equal(b["soft"], r["soft"])
        assert torch.equal(b["msgs"], m["msgs"])


@pytest.mark.parametrize("L,w,h", [(5, 3, 2), (16, 65, 9), (20, 64, 7), (64, 129, 5), (48, 63, 33), (96, 33, 8),
                                   (100, 31, 6), (128, 32, 5), (130, 33, 4), (256, 40, 3)])
@pytest.mark.parametrize("K,fmt", [(2, "f32"), (3, "f32"), (4, "f16")])
def test_volume(dev, L, w, h, K, fmt):
    import paper_1902_09733_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(L + w)
    cost = 20.0 * torch.rand((L, h, w), generator=g, device=dev)
    check(bp, cost, bp.BPParams(levels=2, iters=K, lam=7.3, tau=2.6, msg_dtype=fmt, temperature=0.7))


@pytest.mark.parametrize("L", [64, 96])
def test_pairs_and_batch(dev, L):
    import paper_1902_09733_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    pairs = []
    for h, w in ((40, 70), (33, 65)):
        img = torch.randint(0, 256, (2, h, w, 3), generator=g, device=dev, dtype=torch.uint8)
        pairs.append(bp.Pair(img[0].contiguous(), img[1].contiguous(), L, 20.0))
    p = bp.BPParams(levels=2, iters=6)
    check(bp, pairs[0], p)
    check(bp, pairs, p)
