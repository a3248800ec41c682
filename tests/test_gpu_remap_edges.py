"""The undistortion's row tails, addresses and frame ends against the oracle,
bit for bit (FP32 decisions on both sides, as in test_gpu_remap.py)."""
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


@pytest.mark.parametrize("w,h,C,off,pad", [
    (1, 1, 3, 0, 0), (2, 1, 3, 1, 0), (1, 7, 1, 3, 0), (2, 4, 1, 0, 0),   # one load of the frame or less
    (3, 1, 3, 0, 0), (3, 2, 3, 2, 1),
    (64, 16, 3, 0, 0), (63, 17, 3, 1, 5), (65, 33, 3, 3, 2), (66, 15, 1, 1, 3), (67, 16, 1, 2, 0),
])
def test_undistort_tails_and_addresses(dev, w, h, C, off, pad):
    """Row tails of every length, odd addresses and padded rows, samples on the
    frame's last row and column (zero distortion) and outside it; what lies
    beyond the frame's last byte is never needed."""
    import paper_1902_09733_amd as bp
    from paper_1902_09733_amd import _abi
    rng = np.random.default_rng(w * 100 + h + C)
    img = rng.integers(0, 256, size=(h, w) + ((3,) if C == 3 else ()), dtype=np.uint8)
    stride = w * C + pad
    rows = np.zeros((h, stride), dtype=np.uint8)
    rows[:, :w * C] = img.reshape(h, w * C)
    src = torch.empty(off + rows.size, dtype=torch.uint8, device=dev)
    src[off:] = torch.from_numpy(rows.reshape(-1)).to(dev)
    for K in ((1.0 * w, 1.0 * h, 0.5 * w, 0.5 * h, 0.0, 0.0, 0.0), (0.6 * w, 0.7 * w, 0.4 * w, 0.6 * h, 0.3, -0.1, 0.02)):
        dst = torch.full((off + h * stride,), 7, dtype=torch.uint8, device=dev)
        k = bp.Intrinsics(*K).c()
        st = _abi.lib().bp_undistort(ctypes.c_void_p(src.data_ptr() + off), w, h, C, stride, ctypes.byref(k),
                                     ctypes.c_void_p(dst.data_ptr() + off), stride, None)
        assert st == 0
        torch.cuda.synchronize()
        got = dst.cpu().numpy()[off:].reshape(h, stride)
        np.testing.assert_array_equal(got[:, :w * C].reshape(img.shape), oracle.undistort(img, *K))
        assert (got[:, w * C:] == 7).all()           # row padding is left alone
