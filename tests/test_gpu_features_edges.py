"""Edges of the Harris and ZSSD kernels against the integer oracle, bit for bit:
frames narrower than one 8-byte load, column and row tails of the response
tiles, cells whose largest response has a larger neighbour outside the cell (or
equal ones inside), patches of every word count with odd search ranges, and
corners whose search region leaves the frame."""
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


@pytest.mark.parametrize("w,h,g", [(1, 1, 1), (5, 9, 2), (7, 7, 1), (7, 40, 3), (8, 8, 1), (9, 70, 4), (64, 16, 2),
                                   (63, 17, 3), (65, 65, 2), (71, 64, 9), (200, 131, 64), (600, 23, 1), (259, 40, 1)])
@pytest.mark.parametrize("kind", ["noise", "ramp", "blocks"])
def test_harris_edges(dev, w, h, g, kind):
    import paper_1902_09733_amd as bp
    rng = np.random.default_rng(w * h + g)
    yy, xx = np.mgrid[0:h, 0:w]
    if kind == "noise":
        img = rng.integers(0, 256, size=(h, w))
    elif kind == "ramp":                        # responses grow across cell borders
        img = ((xx * xx + 3 * xx * yy + yy * yy) // 7) % 256
    else:                                       # many equal responses
        img = ((xx // 4 + yy // 4) % 2) * 255
    img = np.ascontiguousarray(img.astype(np.uint8))
    r = oracle.harris_response(img)
    for thr in (0, -10 ** 12, 10 ** 9):
        out = bp.harris(torch.from_numpy(img).to(dev), grid=g, threshold=thr)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out["response"].cpu().numpy(), r)
        got = np.stack([out[k].cpu().numpy() for k in ("x", "y", "corner_response")], axis=1).astype(np.int64)
        np.testing.assert_array_equal(got, oracle.harris_cells(r, g, thr))


@pytest.mark.parametrize("pr,sr", [(0, 3), (1, 1), (1, 32), (3, 8), (4, 2), (5, 16), (6, 9), (9, 4), (10, 7), (13, 5),
                                   (15, 32)])
@pytest.mark.parametrize("flat", [False, True])
def test_zssd_words_and_borders(dev, pr, sr, flat):
    import paper_1902_09733_amd as bp
    rng = np.random.default_rng(pr * 50 + sr)
    h, w = 83, 101
    a = rng.integers(0, 256, size=(h, w), dtype=np.uint8)
    b = np.roll(a, (1, 2), axis=(0, 1))
    if flat:                                    # ties everywhere: the first shift in row-major order
        a[:], b[:] = 90, 17
    pts = [(50, 41), (pr, pr), (w - 1 - pr, h - 1 - pr), (pr, h - 1 - pr), (w - 1 - pr, pr), (pr + 1, 40), (w - 2 - pr, 40),
           (50, pr + 2), (-1, -1), (pr - 1, 30)]
    corners = np.array([(x, y, 0) for x, y in pts], dtype=np.int64)
    raw = np.zeros((len(pts), 2), dtype=np.int64)
    raw[:, 0] = (corners[:, 0] & 0xffffffff) | (corners[:, 1] << 32)
    m = bp.zssd_match(torch.from_numpy(a).to(dev), torch.from_numpy(b).to(dev), torch.from_numpy(raw).to(dev),
                      patch_radius=pr, search_radius=sr)
    torch.cuda.synchronize()
    got = np.stack([m[k].cpu().numpy() for k in ("x", "y", "cost")], axis=1)
    np.testing.assert_array_equal(got, oracle.zssd_match(a, b, corners, pr, sr))
