"""ICP pairings after the first iteration, where the search starts from the
previous iteration's target: the pairing of iteration k is the exhaustive one
at the pose after k - 1 iterations, index for index (FP32 decisions on both
sides), and repeated calls give identical bits (the queries' order does not
depend on the sort's atomics).  Block edges, clouds of different sizes,
duplicated points (ties to the lowest index) and crowded buckets."""
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


def cloud(n, seed, half, copies=1):
    rng = np.random.default_rng(seed)
    xy = rng.uniform(-half, half, size=((n + copies - 1) // copies, 2))
    p = np.column_stack([xy, np.sin(0.7 * xy[:, 0]) * np.cos(0.5 * xy[:, 1])])
    return np.ascontiguousarray(np.repeat(p, copies, axis=0)[:n].astype(np.float32))


@pytest.mark.parametrize("n,m,half,copies,dmax", [
    (1, 1, 1.0, 1, 1.0), (3, 700, 3.0, 1, 0.6), (255, 256, 4.0, 1, 1.0), (257, 4100, 8.0, 1, 0.7),
    (2048, 1300, 8.0, 4, 0.8),        # every point four times
    (1500, 1500, 0.4, 1, 2.0),        # every point in a few buckets
    (300_000, 900, 30.0, 1, 1.0),     # more than 1024 blocks of queries
])
def test_later_pairings_exact_and_repeatable(dev, n, m, half, copies, dmax):
    import paper_1902_09733_amd as bp
    src = cloud(n, n + m, half, copies)
    dst = cloud(m, m, half, copies) + np.float32([0.11, -0.07, 0.05])
    s, d = torch.from_numpy(src).to(dev), torch.from_numpy(dst).to(dev)
    eye = torch.tensor([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], dtype=torch.float64, device=dev)
    for k in (2, 5):
        before = bp.icp(s, d, eye, k - 1, dmax)["pose"].cpu().numpy()
        out = bp.icp(s, d, eye, k, dmax, want_corr=True)
        again = bp.icp(s, d, eye, k, dmax, want_corr=True)
        torch.cuda.synchronize()
        for key in ("pose", "rms", "pairs", "corr"):
            assert torch.equal(out[key], again[key]), key
        pick = np.arange(n) if n <= 5000 else np.random.default_rng(1).choice(n, 3000, replace=False)
        _, corr, _ = oracle.icp_correspond(src[pick], dst, before[:9].reshape(3, 3).astype(np.float32),
                                           before[9:].astype(np.float32), dmax)
        np.testing.assert_array_equal(out["corr"].cpu().numpy()[pick], corr)
        if n <= 5000:
            assert int(out["pairs"][k - 1]) == (corr >= 0).sum()
