"""The tile kernel's blocks and row parts: columns of one short block, of a
block and a remainder, of whole blocks, cut in two parts (few column tiles) or
not, with every count of sketch column tiles a wave can have.

The Arnoldi process against the oracle's: H within 1e-4 of its largest entry,
the stored basis V_{j+1} within 1e-4 of the relation that forms it (the bars of
the float32 path, as in test_gpu_parity.py); a batch and its problems alone
(other row parts: the partial sums are added in another order) within 1e-5."""
import sys

import numpy as np
import pytest

from paper_2603_00839_amd import synth
from oracle.arnoldi import sketched_global_arnoldi
import _util as U

pytestmark = pytest.mark.gpu

# I1, I2, J, l1, l2
SHAPES = [(8, 33, 1, 8, 20), (64, 40, 3, 16, 17), (72, 31, 2, 30, 16), (128, 65, 3, 33, 65), (200, 64, 2, 100, 64),
          (256, 40, 3, 64, 40), (264, 70, 1, 128, 70), (520, 130, 1, 40, 128)]


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_blocks_and_parts_match_oracle(shape):
    from paper_2603_00839_amd import rtg
    I1, I2, J, l1, l2 = shape
    m = 5
    p = synth.small_problem(31, I1, I2, J, 3, 3, min(1, J - 1), l1, l2, J, m, random_bands=True)
    op_o, sk_o = U.oracle_pair(p)
    op, sk = U.gpu_pair(p)
    C, delta = U.observation(p)
    d = rtg.arnoldi(op, sk, U.to_dev(C), m)
    assert int(d["m_done"].item()) == m
    H = d["H"].cpu().numpy()
    ref = sketched_global_arnoldi(op_o, sk_o, C.astype(np.float64), m)
    V = [U.from_dev(d["V"][i]) for i in range(m + 1)]
    rel = max(U.rel(H[j + 1, j] * V[j + 1], op_o(V[j]) - sum(H[i, j] * V[i] for i in range(j + 1))) for j in range(m))
    print(f"{shape}: H {U.maxrel(H, ref.H):.2e} relation {rel:.2e}", file=sys.stderr, flush=True)
    assert U.maxrel(H, ref.H) < 1e-4
    assert rel < 1e-4


def test_batch_of_many_tiles_equals_its_problems():
    """Past the column tiles up to which columns are cut in parts: the batch
    takes whole columns, its first problem alone two parts."""
    import torch
    from paper_2603_00839_amd import rtg
    ps = [synth.small_problem(60 + k, 200, 200, 3, 3, 3, 1, 24, 24, 3, 8) for k in range(8)]   # 8 x 21 column tiles
    ops, sks, Cs, prms = [], [], [], []
    for p in ps:
        o, s = U.gpu_pair(p)
        C, delta = U.observation(p)
        ops.append(o)
        sks.append(s)
        Cs.append(U.to_dev(C))
        prms.append(rtg.make_params(8, rtg.F32, delta=delta, eta=1.01))
    plan = rtg.BatchPlan(ops, sks, Cs, [None] * len(ps), prms)
    plan.run()
    infos = plan.infos()
    for k in (0, 7):
        X, ib = rtg.solve(ops[k], sks[k], Cs[k], None, prms[k])
        one = rtg.read_info(ib)
        err = float(torch.linalg.vector_norm((X - plan.outs[k]).double()) / torch.linalg.vector_norm(X.double()))
        print(f"problem {k}: {err:.2e}", file=sys.stderr, flush=True)
        assert err < 1e-5 and one.iters == infos[k].iters and one.flags == infos[k].flags
