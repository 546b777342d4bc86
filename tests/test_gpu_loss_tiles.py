"""The L1 + SSIM loss at the edges of its tiles (32 columns, 32 rows,
16-byte and ragged rows, images smaller than the window) vs the FP64 oracle,
on the GPU: gradients within 1e-3 relative (floor 1e-2 x rms), the loss
value within 1e-5 relative, the bounds of the other loss tests."""
import numpy as np
import pytest
import torch

from oracle import loss as LOSS
from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from tests import gpu_common as GC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[(1, 1), (3, 40)], [(31, 33), (32, 32), (33, 31)], [(40, 48), (72, 49)],
                                   [(73, 100), (128, 7)], [(1001, 700)], [(704, 993)]])
def test_loss_tiles(sizes):
    print(f"loss tiles sizes={sizes}", flush=True)
    rng = np.random.default_rng(sum(w + h for w, h in sizes))
    n = sum(3 * w * h for w, h in sizes)
    rgb = np.clip(rng.uniform(0.2, 0.8, size=n) + 0.05 * rng.normal(size=n), 0, 1).astype(np.float32)
    target = np.clip(rgb + 0.1 * rng.normal(size=n), 0, 1).astype(np.float32)
    cams = L.cameras([scenes.make_camera(np.eye(3, 4, dtype=np.float32), w, h) for w, h in sizes])
    ws = torch.empty(L.linprim_loss_workspace_size(cams), dtype=torch.uint8, device="cuda")
    x, y = torch.as_tensor(rgb, device="cuda"), torch.as_tensor(target, device="cuda")
    g = torch.empty_like(x)
    L.linprim_loss_grad(x, y, cams, ws, g)
    val = L.linprim_loss_value(ws, cams)
    ref_val, ref = LOSS.loss_and_grad(rgb, target, sizes)
    assert abs(val - ref_val) <= 1e-5 * abs(ref_val)
    rms = float(np.sqrt(np.mean(ref ** 2)))
    err = np.abs(g.cpu().numpy().astype(np.float64) - ref) / np.maximum(np.abs(ref), 1e-2 * rms)
    print(f"  gradient worst rel err {err.max():.2e}", flush=True)
    assert err.max() <= GC.GRAD_TOL
