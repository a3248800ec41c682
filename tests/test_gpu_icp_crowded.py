"""ICP on clouds whose points crowd into few cells, and on clouds with many
holes (NaN points, as the triangulation writes them where there is no
disparity).

Ordering the source by cell takes time linear in the points however they fall:
a call on four times the points of one cell takes less than eight times as long
(comparing a cell's points with each other takes sixteen), and a cloud with
100 000 holes less than three times as long as one with none.  Pairings stay the
exhaustive ones, index for index, and repeated calls give identical bits.
"""
import time

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

EYE = [1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


def cloud(n, seed, half):
    rng = np.random.default_rng(seed)
    xy = rng.uniform(-half, half, size=(n, 2))
    return np.column_stack([xy, 0.1 * np.sin(xy[:, 0])]).astype(np.float32)


def call(src, dst, dev, iters=5, dmax=1.0):
    import paper_1902_09733_amd as bp
    s, d = torch.from_numpy(src).to(dev), torch.from_numpy(dst).to(dev)
    pose, ws = torch.tensor(EYE, dtype=torch.float64, device=dev), bp.Workspace()
    return lambda: bp.icp(s, d, pose, iters, dmax, want_corr=True, workspace=ws)


def seconds(f):
    f()
    torch.cuda.synchronize()
    best = np.inf
    for _ in range(7):
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def check(src, dst, dev, dmax=1.0, sample=2000):
    f = call(src, dst, dev, 1, dmax)
    a, b = f(), f()
    torch.cuda.synchronize()
    assert all(torch.equal(a[k], b[k]) for k in a)
    pick = np.random.default_rng(3).choice(len(src), min(sample, len(src)), replace=False)
    _, corr, _ = oracle.icp_correspond(src[pick], dst, np.eye(3, dtype=np.float32), np.zeros(3, np.float32), dmax)
    got = a["corr"].cpu().numpy()
    np.testing.assert_array_equal(got[pick], corr)
    assert int(a["pairs"][0]) == (got >= 0).sum()
    return a


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2048, 9000, 70_001])
@pytest.mark.parametrize("kind", ["one", "few", "runs"])
def test_crowded_cells_exact_and_repeatable(dev, n, kind):
    """One cell; a few of them, indices mixed; and long runs of indices per cell (whole slices full)."""
    src = cloud(n, n, 0.3)
    if kind == "few":
        src[:, 0] += np.arange(n) % 5
    elif kind == "runs":
        src[:, 1] += 2 * (np.arange(n) * 7 // n)
    dst = np.concatenate([cloud(60, 5, 0.4), cloud(40, 6, 6.0)])
    check(src, dst, dev)
    again = call(src, dst, dev)
    a, b = again(), again()
    torch.cuda.synchronize()
    assert all(torch.equal(a[k], b[k]) for k in a)


def test_holes_exact(dev):
    """Holes of every kind among the points leave the others' pairings and sums as they are without them."""
    n = 50_000
    src = cloud(n, 8, 20.0)
    dst = cloud(n, 9, 20.0)
    full = check(src, dst, dev)
    holes = np.random.default_rng(1).choice(n, 20_000, replace=False)
    src[holes[:10_000]] = np.nan
    src[holes[10_000:15_000], 1] = np.inf
    src[holes[15_000:], 2] = -np.inf
    out = check(src, dst, dev)
    corr, ref = out["corr"].cpu().numpy(), full["corr"].cpu().numpy()
    assert (corr[holes] == -1).all()
    keep = np.setdiff1d(np.arange(n), holes)
    np.testing.assert_array_equal(corr[keep], ref[keep])
    # The same points without the holes: FP64 sums of the same pairs in another order.
    alone = call(src[keep], dst, dev, 1)()
    np.testing.assert_allclose(out["pose"].cpu().numpy(), alone["pose"].cpu().numpy(), rtol=0, atol=1e-11)


def test_holes_only(dev):
    src = np.full((3000, 3), np.nan, np.float32)
    out = call(src, cloud(100, 2, 1.0), dev, 3)()
    assert (out["corr"] == -1).all() and (out["pairs"] == 0).all()
    assert out["pose"].cpu().tolist() == EYE


def test_time_is_linear_in_a_crowded_cell(dev):
    dst = cloud(100, 4, 0.4)
    t = [seconds(call(cloud(n, n, 0.3), dst, dev)) for n in (64_000, 256_000)]
    print(f"one cell: {t[0] * 1e6:.0f} us, four times the points {t[1] * 1e6:.0f} us", flush=True)
    assert t[1] < 8 * t[0]


def test_time_with_holes(dev):
    n = 256_000
    src, dst = cloud(n, 8, 100.0), cloud(n, 9, 100.0)
    whole = seconds(call(src, dst, dev))
    src[np.random.default_rng(1).choice(n, 100_000, replace=False)] = np.nan
    holes = seconds(call(src, dst, dev))
    print(f"no holes: {whole * 1e6:.0f} us, 100 000 holes {holes * 1e6:.0f} us", flush=True)
    assert holes < 3 * whole
