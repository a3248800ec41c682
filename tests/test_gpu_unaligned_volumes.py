"""Cost volumes and cost gradients whose rows are not 16-byte aligned (widths off
multiples of four, bases off 16 bytes) against the same numbers in aligned
rows: a transpose moves values, so tolerance 0."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("L,w,h", [(5, 1, 3), (16, 3, 2), (48, 62, 5), (64, 65, 4), (33, 127, 3), (100, 66, 3), (130, 67, 2)])
def test_split(dev, L, w, h):
    """A volume at an offset of one float against its aligned copy, and label 0 .. L - 1 of each pixel
    through one half-sweep without smoothness (messages are the costs less their minimum)."""
    import paper_1902_09733_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(L + w)
    buf = torch.randint(0, 50, (L * h * w + 4,), generator=g, device=dev).float()
    p = bp.BPParams(levels=1, iters=3, lam=4.0, tau=2.0)
    ref = None
    for off in (0, 1, 2, 3):
        c = buf[off:off + L * h * w].view(L, h, w)
        c.copy_(torch.randint(0, 50, (L, h, w), generator=torch.Generator(device="cuda").manual_seed(7), device=dev).float())
        o = bp.run(c, p, want_msgs=True)
        b = bp.run(c, bp.BPParams(levels=1, iters=3, lam=4.0, tau=2.0, pm_from=1), want_msgs=True)
        torch.cuda.synchronize()
        assert torch.equal(o["disp"], b["disp"]) and torch.equal(o["msgs"], b["msgs"])
        ref = ref or o
        assert torch.equal(o["disp"], ref["disp"]) and torch.equal(o["msgs"], ref["msgs"])


@pytest.mark.parametrize("L,w,h", [(5, 3, 2), (16, 65, 3), (64, 66, 4), (33, 63, 3), (100, 67, 2)])
def test_gradient(dev, L, w, h):
    """Two problems in one call: the second's gradient starts off 16 bytes."""
    import paper_1902_09733_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(L + w)
    cost = [20.0 * torch.rand((L, h, w), generator=g, device=dev) for _ in range(2)]
    gs = [torch.randn((h, w), generator=g, device=dev) for _ in range(2)]
    p = bp.BPParams(levels=1, iters=4, lam=3.0, tau=2.5, temperature=0.5, checkpoint_every=2)

    def grads(ids):
        vols = [cost[i] for i in ids]
        ck = torch.empty(bp.checkpoint_bytes(vols, p), dtype=torch.uint8, device=dev)
        bp.run(vols, p, want_disp=False, want_soft=True, checkpoints=ck)
        return bp.backward(vols, p, ck, [gs[i] for i in ids])[0]

    both, one, two = grads([0, 1]), grads([0]), grads([1])
    torch.cuda.synchronize()
    assert torch.equal(both[0], one[0]) and torch.equal(both[1], two[0])
    assert all(x.abs().sum() > 0 for x in both)
