"""The pixel-major reverse half-sweep on both sides of its window rule (an
untruncated winner within four labels takes the form without LDS), at label
counts that end inside a lane, one-pixel and one-row grids, a single half-sweep
(its readout adjoint read from the cost adjoint), and more problems than one
launch carries; against the FP64 oracle adjoint.

Tolerances: entries agree to FP32 rounding unless FP32 and FP64 pick different
winners at a near-tie, which moves single entries; up to 127 labels, 8
half-sweeps and gradients of unit scale leave rounding below 1e-3 of the largest
entry, and 99.9% of entries must be within it.  tau lies off the integers: at an
integer the truncation meets the minimum's cone exactly, and which of the two a
label takes (all that tau's derivative counts) is rounding."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


def check(shapes, K, every, lam, tau, dev, T=0.5):
    import paper_1902_09733_amd as bp
    rng = np.random.default_rng(sum(shapes[0]) + K)
    costs = [(rng.integers(0, 20, size=s) + rng.uniform(0.0, 0.5, size=s)).astype(np.float32) for s in shapes]
    g = [rng.normal(size=s[1:]).astype(np.float32) for s in shapes]
    p = bp.BPParams(levels=1, iters=K, lam=lam, tau=tau, temperature=T, checkpoint_every=every)
    vols = [torch.from_numpy(c).to(dev) for c in costs]
    ck = torch.empty(bp.checkpoint_bytes(vols, p), dtype=torch.uint8, device=dev)
    bp.run(vols, p, want_disp=False, want_soft=True, checkpoints=ck)
    gc, gl, gt = bp.backward(vols, p, ck, [torch.from_numpy(x).to(dev) for x in g])
    ol = ot = 0.0
    for i, c in enumerate(costs):
        _, gc_o, gl_o, gt_o = oracle.backward(c.astype(np.float64), K, lam, tau, T, g[i].astype(np.float64))
        ol += gl_o
        ot += gt_o
        close = np.abs(gc[i].cpu().numpy() - gc_o) <= 1e-3 * np.abs(gc_o).max() + 1e-5
        assert close.mean() >= 0.999, (i, shapes[i], close.mean())
    assert abs(float(gl) - ol) <= 1e-3 * max(1.0, abs(ol)), (float(gl), ol)
    assert abs(float(gt) - ot) <= 1e-3 * max(1.0, abs(ot)), (float(gt), ot)


@pytest.mark.parametrize("L", [3, 17, 62, 65, 97, 127])
@pytest.mark.parametrize("tau", [0.4, 2.99, 3.01])
def test_window_rule(dev, L, tau):
    check([(L, 7, 9), (L, 6, 8)], 5, 2, 2.0, tau, dev)


@pytest.mark.parametrize("shape", [(20, 1, 1), (64, 1, 2), (32, 2, 1), (64, 3, 3), (16, 1, 35)])
@pytest.mark.parametrize("K", [1, 2, 8])
def test_small_grids(dev, shape, K):
    check([shape], K, 1, 3.0, 2.5, dev)


def test_more_problems_than_a_launch(dev):
    check([(32 if i % 3 else 64, 4 + i % 2, 5 + i % 4) for i in range(35)], 3, 2, 3.0, 2.5, dev)
