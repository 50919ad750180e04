"""The sketched Gram step's finish of the partial sketches and its float64
tail at the sizes where their branches change: pairs that allow 16-byte, 8-byte
and single loads, one and several workgroups, channels beyond one LDS chunk
with and without the sliced sums, mode 3 in LDS and from memory.

H against the oracle's (float64) Arnoldi process: the bar of the float32 path
(1e-4 of the largest entry), as in test_gpu_parity.py."""
import sys

import numpy as np
import pytest

from paper_2603_00839_amd import synth
from oracle.arnoldi import sketched_global_arnoldi
import _util as U

pytestmark = pytest.mark.gpu

# I1, I2, J, rB, l1, l2, l3, m
SHAPES = [
    (32, 40, 3, 2, 16, 16, 3, 6),      # 256 pairs: four workgroups of 64, 16-byte loads
    (32, 40, 3, 2, 13, 14, 3, 6),      # 182 pairs: 8-byte loads, a ragged last workgroup
    (32, 40, 3, 2, 13, 15, 3, 6),      # 195 pairs: single loads
    (40, 300, 2, 1, 9, 7, 2, 5),       # ten column tiles, 63 pairs: one workgroup
    (16, 24, 136, 1, 8, 9, 16, 4),     # one tile a channel, 136 channels: sliced sums in two chunks
    (16, 24, 45, 2, 8, 8, 45, 4),      # identity on mode 3, 45 finished values a pair
    (16, 20, 47, 1, 12, 11, 15, 4),    # Om3 without slices, ragged groups of finished values
    (16, 40, 33, 1, 7, 7, 5, 4),       # sliced sums, slices of five, the last one of three
]


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
@pytest.mark.parametrize("basis", ["f32", "bf16"])
def test_gram_finish_matches_oracle(shape, basis):
    from paper_2603_00839_amd import rtg
    I1, I2, J, rB, l1, l2, l3, m = shape
    p = synth.small_problem(21, I1, I2, J, 3, 3, rB, l1, l2, l3, m, random_bands=True)
    op_o, sk_o = U.oracle_pair(p)
    op, sk = U.gpu_pair(p)
    C, _ = U.observation(p)
    bt, m = (rtg.F32, m) if basis == "f32" else (rtg.BF16, 1)
    d = rtg.arnoldi(op, sk, U.to_dev(C), m, bt)
    assert int(d["m_done"].item()) == m
    H, S = d["H"].cpu().numpy(), d["SV"].cpu().numpy().astype(np.float64)
    ref = sketched_global_arnoldi(op_o, sk_o, C.astype(np.float64), m)
    err = np.abs(H - ref.H).max() / np.abs(ref.H).max()
    # the stored sketch of V_1 (internal order (a l2 + b) l3 + c), of the stored V_1
    V1 = U.from_dev(d["V"][0])
    want = np.asarray(sk_o(V1)).reshape(-1)
    es = np.linalg.norm(S[0] - want) / np.linalg.norm(want)
    print(f"{shape} {basis}: H {err:.2e} S(V_1) {es:.2e}", file=sys.stderr, flush=True)
    # bfloat16: V_1 and Om_1 rounded (2^-9 each) before every product
    assert err <= (1e-4 if basis == "f32" else 1e-2)
    assert es <= (2e-5 if basis == "f32" else 2.0 ** -8)
