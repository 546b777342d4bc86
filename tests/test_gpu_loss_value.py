"""Rounding of the loss value's block sums.  Pixels are multiples of 2^-20, so
|x - y| is exact, and without the SSIM term the value's only rounding is that of
the three blocks' sums of a 32 x 32 image.  Over many images it is to stay below
that of a tree in float over 256 threads of four pixels of a column, formed here
of the same pixels.  (In units of 2^-24, rms, of one block, from the orders of
the additions: 0.69 the tree, 0.52 four-pixel sums by waves of 512 threads with
the waves added in double, 0.78 everything in float one after the other; 400
images tell values 5% apart.)"""
import numpy as np
import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes

pytestmark = pytest.mark.gpu
SIZE, IMAGES = 32, 400


def _tree(d):
    """Sums of [..., 32, 32] float32 images."""
    cols = d.reshape(d.shape[:-2] + (8, 4, 32))
    s = cols[..., 0, :]
    for k in range(1, 4):
        s = s + cols[..., k, :]
    s = s.reshape(d.shape[:-2] + (256,))
    while s.shape[-1] > 1:
        h = s.shape[-1] // 2
        s = s[..., :h] + s[..., h:]
    return s[..., 0]


def test_block_sums():
    print(f"loss value, {IMAGES} images {SIZE}x{SIZE}", flush=True)
    rng = np.random.default_rng(0)
    shape = (IMAGES, 3, SIZE, SIZE)
    grid = lambda a: (np.round(a * 2 ** 20) / 2 ** 20).astype(np.float32)
    y = grid(rng.random(shape))
    x = grid(y + 0.1 * rng.standard_normal(shape))
    d = np.abs(x - y)
    exact = d.astype(np.float64).mean((1, 2, 3))
    tree = _tree(d).astype(np.float64).sum(1) / (3 * SIZE * SIZE)
    cams = L.cameras([scenes.look_at((8, 0, 0), (0, 0, 0), SIZE, SIZE)])
    ws = torch.empty(L.linprim_loss_workspace_size(cams), dtype=torch.uint8, device="cuda")
    grad = torch.empty(3 * SIZE * SIZE, device="cuda")
    xd, yd = torch.as_tensor(x, device="cuda"), torch.as_tensor(y, device="cuda")
    got = np.empty(IMAGES)
    for k in range(IMAGES):
        L.linprim_loss_grad(xd[k], yd[k], cams, ws, grad, lam=0.0)
        got[k] = L.linprim_loss_value(ws, cams, lam=0.0)
    rms = lambda v: float(np.sqrt(np.mean(((v - exact) / exact) ** 2)))
    print(f"relative error {rms(got):.2e} rms, of the tree {rms(tree):.2e}", flush=True)
    assert rms(got) <= rms(tree)
