"""The stand-alone sketch where its finish changes form: few channels of many
column tiles (one pass, more tiles than one round of loads, ragged last
workgroups, with and without a third factor), one channel more (two passes).

Against the oracle's float64 sketch of the same values, in bfloat16 with Om_1
rounded as the library rounds it: 2e-5 of its norm in float32 (as for the stored
sketches of the Gram step), 2^-8 in bfloat16."""
import sys

import numpy as np
import pytest

from paper_2603_00839_amd import synth
from oracle.sketch import Sketch
import _util as U

pytestmark = pytest.mark.gpu

# I1, I2, J, l1, l2, l3
SHAPES = [
    (48, 994, 3, 33, 16, 3),      # 32 tiles in three channels, 528 pairs: a half-full last workgroup
    (40, 994, 8, 33, 16, 3),      # eight channels, Om3
    (16, 1600, 1, 9, 7, 1),       # 50 tiles in one channel, 63 pairs
    (24, 1050, 2, 8, 9, 1),       # 33 tiles: one in the second round; Om3 to one value
    (32, 250, 8, 16, 16, 8),      # identity on mode 3
    (32, 250, 8, 12, 11, 7),
    (32, 250, 9, 12, 11, 7),      # nine channels: two passes
    (16, 1700, 1, 1, 1, 1),       # one pair
]


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sketch_matches_oracle(shape, dtype):
    import torch
    from paper_2603_00839_amd import rtg
    I1, I2, J, l1, l2, l3 = shape
    p = synth.small_problem(3, I1, I2, J, 1, 1, 0, l1, l2, l3, 1)
    _, sk = U.gpu_pair(p)
    om1 = U.bf16_round(p.om1) if dtype == "bf16" else p.om1
    X = np.random.default_rng(4).standard_normal((I1, I2, J)).astype(np.float32)
    Xd = U.to_dev(X, torch.bfloat16 if dtype == "bf16" else None)
    got = U.from_dev(rtg.sketch(sk, Xd).reshape(l3, l2, l1))
    want = np.asarray(Sketch(om1, p.om2, p.om3)(U.from_dev(Xd)))
    err = U.rel(got, want)
    print(f"{shape} {dtype}: {err:.2e}", file=sys.stderr, flush=True)
    assert err <= (2e-5 if dtype == "f32" else 2.0 ** -8)
