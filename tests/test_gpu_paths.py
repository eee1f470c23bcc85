"""Edges of the kernels' work splits, on the GPU, against the FP64 oracle or plain references."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2603_09277_amd import gsr, scenes

from gpu_helpers import DEV, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = gsr.Rasterizer(max_views=8)
    yield r
    r.close()


def _cam(w, h):
    return scenes.Camera(w, h, float(w), float(w), w / 2, h / 2, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))


# D-SSIM: bands of 64 pixels, segments of 12 to 124 rows, 32 views a launch.  Tolerances as
# for the plain parity test: FP32 window sums against FP64 (loss absolute, gradient relative L2).
@pytest.mark.parametrize("sizes", [[(63, 12)], [(64, 13), (65, 11)], [(128, 125), (129, 44)], [(1, 130), (200, 1)],
                                   [(7, 9)] * 33 + [(66, 29)]])
@pytest.mark.parametrize("with_grad", [True, False])
def test_dssim_bands_and_segments(R, sizes, with_grad):
    rng = np.random.default_rng(len(sizes) * 100 + sizes[0][0])
    xs = [rng.uniform(0, 1, (h, w, 3)).astype(np.float32) for w, h in sizes]
    ys = [np.clip(x + rng.normal(0, 0.1, x.shape), 0, 1).astype(np.float32) for x in xs]
    x = torch.from_numpy(np.concatenate([a.reshape(-1, 3) for a in xs])).to(DEV)
    y = torch.from_numpy(np.concatenate([a.reshape(-1, 3) for a in ys])).to(DEV)
    grad = torch.zeros_like(x) if with_grad else None
    loss = R.dssim([_cam(w, h) for w, h in sizes], x, y, 0.2, grad).cpu().numpy()
    at = 0
    for v, (w, h) in enumerate(sizes):
        s, gs = orc.ssim(xs[v], ys[v])
        assert abs(loss[v] - 0.2 * (1.0 - s)) <= 2e-5, (v, w, h)
        if with_grad:
            g = grad[at:at + w * h].cpu().numpy().reshape(h, w, 3).astype(np.float64)
            assert np.linalg.norm(g + 0.2 * gs) <= 1e-4 * np.linalg.norm(0.2 * gs), (v, w, h)
        at += w * h
