"""Which launches stream, and that every form of the streamed kernel equals one
launch per half-sweep.

Each case names the pairs of half-sweeps of the finest level's launches, in order,
and the launch records (bp_run_profiled: a launch of n pairs covers 2 n w h L
updates) must show them, so a case that stops reaching its kernel fails.  The
kernels: each form of the transform (tau 2: three labels, 2.6: five, 2.9: five up
to four labels per lane and the scans above, 5: scans) at each lane split and
storage, with two and three pairs, sizes just above the rule's lines, and one
pair just below them.

The arithmetic per message is variant 1's, so labels, soft-argmin disparities and
final messages agree bit for bit on real-valued costs: tolerance 0; with messages
out (the last launch stores the state) and without (it reads out both colours).

Where lambda is below h / 2^18 the five-label form above four labels per lane may
differ from the scans by roundings of h: there its messages' largest error against
the FP64 oracle is at most the scans', and the mean within a thousandth of theirs.
"""
import ctypes

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


CASES = [
    # (L, H, W, levels, K, fmt, tau, pairs of each launch of the finest level)
    (16, 701, 733, 1, 6, "f32", 2.6, [1, 2]),
    (16, 1001, 1003, 1, 10, "f32", 2.0, [3, 2]),
    (16, 1009, 1021, 2, 12, "f16", 2.0, [3, 3]),
    (32, 509, 521, 1, 8, "f32", 2.6, [2, 2]),
    (32, 511, 519, 2, 8, "f16", 2.6, [2, 2]),
    (32, 731, 719, 1, 12, "f32", 2.0, [3, 3]),
    (64, 341, 389, 1, 4, "f32", 2.9, [2]),
    (64, 499, 521, 2, 10, "bf16", 2.0, [3, 2]),
    (64, 701, 733, 2, 8, "f16", 5.0, [2, 2]),
    (96, 293, 301, 1, 6, "f32", 2.6, [1, 2]),
    (96, 293, 301, 1, 8, "f32", 2.9, [2, 2]),
    (96, 331, 389, 1, 6, "f32", 2.75, [1, 2]),
    (96, 487, 523, 1, 10, "f32", 2.0, [3, 2]),
    (96, 487, 523, 2, 10, "f16", 2.0, [3, 2]),
    (96, 487, 523, 2, 12, "bf16", 2.0, [3, 3]),
    (96, 331, 367, 2, 8, "bf16", 2.6, [2, 2]),
    (96, 571, 601, 2, 8, "f16", 5.0, [2, 2]),
    (96, 571, 601, 2, 8, "bf16", 2.9, [2, 2]),
    (128, 241, 289, 1, 8, "f32", 2.6, [2, 2]),
    (128, 251, 257, 1, 6, "f32", 5.0, [1, 2]),
    (128, 431, 443, 2, 10, "f16", 2.0, [3, 2]),
    (128, 431, 443, 2, 12, "bf16", 2.0, [3, 3]),
    (128, 283, 307, 2, 8, "f16", 2.6, [2, 2]),
    (128, 499, 509, 2, 8, "bf16", 5.0, [2, 2]),
    (128, 499, 509, 2, 8, "f16", 2.9, [2, 2]),
    # One pair per launch below the lines.
    (64, 241, 257, 1, 4, "f32", 2.0, [1, 1]),
    (64, 241, 257, 2, 8, "f16", 2.0, [1, 1, 1, 1]),
    (96, 269, 281, 2, 8, "f16", 2.0, [1, 1, 1, 1]),
    (96, 289, 341, 2, 8, "bf16", 2.6, [1, 1, 1, 1]),
    (96, 271, 301, 1, 4, "f32", 2.9, [1, 1]),
    (96, 451, 461, 2, 8, "f16", 2.9, [1, 1, 1, 1]),
    (128, 241, 257, 1, 4, "f32", 2.9, [1, 1]),
    (128, 431, 443, 2, 8, "bf16", 2.9, [1, 1, 1, 1]),
]


def launches(cost, params, dev):
    """Pairs of half-sweeps of each launch of the finest level, from the launch records."""
    from paper_1902_09733_amd import _abi, stereo
    L, h, w = cost.shape
    disp = torch.empty((h, w), dtype=torch.int32, device=dev)
    probs, p = stereo._problems([cost], [disp], [None], [None]), params.c()
    lib = _abi.lib()
    nb = lib.bp_workspace_size(probs, 1, ctypes.byref(p))
    ws = stereo.Workspace().get(nb, dev)
    rec, n = (_abi.BpLaunchRecord * 256)(), ctypes.c_int32()
    _abi.check("bp_run_profiled",
               lib.bp_run_profiled(probs, 1, ctypes.byref(p), ctypes.c_void_p(ws.data_ptr()), nb,
                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), 0, rec, 256,
                                   ctypes.byref(n)))
    return [rec[i].units / (2.0 * w * h * L) for i in range(n.value) if rec[i].level == 0]


@pytest.mark.parametrize("L,H,W,levels,K,fmt,tau,pairs", CASES)
def test_forms(dev, L, H, W, levels, K, fmt, tau, pairs):
    import paper_1902_09733_amd as bp
    print(f"streamed forms: L={L} {W}x{H} levels={levels} K={K} {fmt} tau={tau}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(L * 1000 + H + W + K)
    cost = 20.0 * torch.rand((L, H, W), generator=g, device=dev)
    p = [bp.BPParams(levels=levels, iters=K, lam=7.3, tau=tau, msg_dtype=fmt, variant=v, temperature=0.7) for v in (0, 1)]
    assert launches(cost, p[0], dev) == pairs
    if max(pairs) == 1:
        return
    ref = bp.run(cost, p[1], want_soft=True, want_msgs=True)
    out = bp.run(cost, p[0], want_soft=True, want_msgs=True)
    torch.cuda.synchronize()
    for k in ("disp", "soft", "msgs"):
        assert torch.equal(out[k], ref[k]), k
    out = bp.run(cost, p[0], want_soft=True)
    torch.cuda.synchronize()
    for k in ("disp", "soft"):
        assert torch.equal(out[k], ref[k]), k


@pytest.mark.parametrize("L,H,W", [(96, 293, 301), (128, 241, 289)])
@pytest.mark.parametrize("low,span,lam", [(0.0, 20.0, 1e-7), (0.0, 20.0, 1e-5), (15.0, 0.05, 1e-6), (15.0, 0.05, 2e-5),
                                          (15.0, 0.05, 1e-3)])
def test_five_labels_at_small_lambda(dev, L, H, W, low, span, lam):
    import paper_1902_09733_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(L + H)
    cost = low + span * torch.rand((L, H, W), generator=g, device=dev)
    p = [bp.BPParams(levels=1, iters=4, lam=lam, tau=2.6, variant=v) for v in (0, 1)]
    assert launches(cost, p[0], dev) == [2]
    out = [bp.run(cost, q, want_msgs=True)["msgs"].cpu().numpy() for q in p]
    ref = oracle.run(cost.cpu().numpy().astype(np.float64), 1, 4, float(np.float32(lam)), float(np.float32(2.6)),
                     want_msgs=True)["msgs"]
    e = [np.abs(o - ref) for o in out]
    print(f"L={L} lam={lam}: largest error {e[0].max():.3e} / {e[1].max():.3e}, mean {e[0].mean():.4e} / {e[1].mean():.4e}",
          flush=True)
    assert e[0].max() <= e[1].max() and e[0].mean() <= 1.001 * e[1].mean()


def test_batch_on_both_sides_of_the_shared_line(dev):
    """16-bit problems of 4 to 6 M values: neighbours of one lane split that share tiled launches, one whose
    neighbours are of other splits (streamed), and one above the line, against each alone with single half-sweeps."""
    import paper_1902_09733_amd as bp
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    costs = [20.0 * torch.rand((L, h, w), generator=g, device=dev)
             for L, h, w in [(64, 241, 281), (64, 239, 277), (96, 100, 120), (64, 251, 263), (128, 90, 111), (64, 311, 331)]]
    p = [bp.BPParams(levels=2, iters=8, lam=7.3, tau=2.0, msg_dtype="f16", variant=v, temperature=0.7) for v in (0, 1)]
    outs = bp.run(costs, p[0], want_soft=True, want_msgs=True)
    for c, o in zip(costs, outs):
        r = bp.run(c, p[1], want_soft=True, want_msgs=True)
        torch.cuda.synchronize()
        assert all(torch.equal(o[k], r[k]) for k in ("disp", "soft", "msgs")), tuple(c.shape)
