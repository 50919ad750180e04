"""The weight gradient's sums over pixels against float64 sums of the same
stored values: the bfloat16 activations and gradients that a training pass
leaves in its workspace (network input, five 32-channel activations, then the
gradients of the last layer and of layers 0 and 1).

Products of bfloat16 values are exact in float32, so only the additions round:
16 in a matrix product, four such products per row of a strip of 64 pixels, the
four waves of a workgroup, and one per workgroup.  The bar for every weight is
that count times 2^-24 times the sum of the products' magnitudes, and the CPU
test shows that it is far below what one column beside a strip, or one row
beside a group of four, contributes."""
import sys

import numpy as np
import pytest

STRIP, ROWS, GROUPS = 64, 4, 512       # pixels along i1, rows staged together, workgroups aimed at


def plan(N, I1, I2):
    """(rows, workgroups) of the kernel's split."""
    strips, steps = N * -(-I1 // STRIP), -(-I2 // ROWS)
    rows = ROWS * min(steps, -(-strips * steps // GROUPS))
    return rows, strips * -(-I2 // rows)


def bar(N, I1, I2):
    rows, groups = plan(N, I1, I2)
    return (16 * 4 * rows // ROWS + 4 + groups) * 2.0 ** -24


def sums(g, x, lost=None):
    """dW[co, t1, t2, ci] = sum of g[n, i2, i1, co] x[n, i2 + t2 - 1, i1 + t1 - 1, ci]
    in float64; lost(i1 of g, i1 of x, i2 of g, i2 of x) drops products."""
    N, I2, I1, Co = g.shape
    out = np.zeros((Co, 3, 3, x.shape[3]))
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    i1, i2 = np.arange(I1)[None, :], np.arange(I2)[:, None]
    for t1 in range(3):
        for t2 in range(3):
            keep = np.ones((I2, I1), bool) if lost is None else ~(lost(i1, i1 + t1 - 1, i2, i2 + t2 - 1) | np.zeros((I2, I1), bool))
            a = (g * keep[None, :, :, None]).reshape(-1, Co)
            out[:, t1, t2] = a.T @ xp[:, t2:t2 + I2, t1:t1 + I1].reshape(-1, x.shape[3])
    return out


SEAMS = {
    "column to the left of a strip": lambda g1, x1, g2, x2: (x1 // STRIP != g1 // STRIP) & (x1 < g1),
    "column to the right of a strip": lambda g1, x1, g2, x2: (x1 // STRIP != g1 // STRIP) & (x1 > g1),
    "row above a group": lambda g1, x1, g2, x2: (x2 // ROWS != g2 // ROWS) & (x2 < g2),
    "row below a group": lambda g1, x1, g2, x2: (x2 // ROWS != g2 // ROWS) & (x2 > g2),
}
SHAPES = [(1, 64, 4), (2, 72, 5), (1, 136, 9), (3, 24, 37), (40, 72, 34), (1, 200, 1), (2, 256, 67)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("channels", [(32, 3), (32, 32), (3, 32)], ids=str)
def test_bar_is_below_every_seam(shape, channels):
    N, I1, I2 = shape
    rng = np.random.default_rng(I1 + I2)
    g = rng.standard_normal((N, I2, I1, channels[0]))
    x = np.maximum(rng.standard_normal((N, I2, I1, channels[1])), 0.0)
    want, size = sums(g, x), sums(np.abs(g), np.abs(x))
    for name, lost in SEAMS.items():
        if I1 <= STRIP and "column" in name or I2 <= ROWS and "row" in name:
            continue
        err = (np.abs(sums(g, x, lost) - want) / np.maximum(size, 1e-300)).max()
        assert err > 10 * bar(*shape), name


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_weight_gradient_sums(shape):
    import torch
    from paper_2603_00839_amd import rtg
    from test_gpu_cnn import flat, images, random_params, unflat
    N, I1, I2 = shape
    net = rtg.WarmStartNet(flat(random_params(14, last_scale=1.0)))
    C = images(15, N, I1, I2)
    Y = C + images(16, N, I1, I2) - 0.5
    net.gradients(torch.from_numpy(C).cuda(), torch.from_numpy(Y).cuda())
    got = unflat(net.read_gradients())
    px, at, stored = N * I1 * I2, 0, []
    for ch in [8] + 5 * [32] + [8, 32, 32]:
        raw = net._ws[at:at + px * ch * 2].view(torch.bfloat16).double().cpu().numpy()
        stored.append(raw.reshape(N, I2, I1, ch))
        at += -(-px * ch * 2 // 256) * 256
    x0, a1, a5, g5, g0, g1 = stored[0], stored[1], stored[5], stored[6], stored[7], stored[8]
    for l, g, x in ((5, g5[..., :3], a5), (1, g1, a1), (0, g0, x0[..., :3])):
        assert np.abs(g).max() > 0 and np.abs(x).max() > 0
        size = sums(np.abs(g), np.abs(x))
        err = (np.abs(got[l]["w"] - sums(g, x)) / np.maximum(size, 1e-300)).max()
        gs = np.abs(g).sum(axis=(0, 1, 2))
        errb = (np.abs(got[l]["b"] - g.sum(axis=(0, 1, 2))) / np.maximum(gs, 1e-300)).max()
        print(f"{shape} layer {l}: w {err:.1e} b {errb:.1e} bar {bar(*shape):.1e}", file=sys.stderr, flush=True)
        assert err <= bar(*shape) and errb <= bar(*shape)
