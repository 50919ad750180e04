"""Which form of the tile kernel a batch takes: in passes over few terms 64 rows
per block where that saves a round of workgroups over the chip (513 to 768
column tiles), and two, three or four sketch tiles of 16 rows per wave.

Rows per block only cut the loop over a column: the same problem in batches on
both sides of the rule has to give the same bits.  Sketch tiles per wave:
against the oracle's Arnoldi process with the bars of the float32 path (H
within 1e-4 of its largest entry, as in test_gpu_tile.py)."""
import sys

import numpy as np
import pytest

from paper_2603_00839_amd import synth
from oracle.arnoldi import sketched_global_arnoldi
from oracle.operator import PSFOperator, make_observation
from oracle.sketch import Sketch
import _util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("I1", [136, 264])
@pytest.mark.parametrize("form", ["golub_kahan", "golub_kahan_bf16", "golub_kahan_bf16_wide", "psf", "psf_mixed", "mixed",
                                  "mixed_wide", "f32"])
def test_rows_per_block_leave_the_bits(form, I1):
    import torch
    from paper_2603_00839_amd import rtg
    I2, J, l1, l2, m = 232, 3, 72 if form.endswith("wide") else 16, 16, 10    # 24 column tiles; steps on both sides of 8 terms
    rng = np.random.default_rng(I1)
    if form.startswith("psf"):
        p = synth.psf_problem(9, I1, I2, J, r=3, l1=l1, l2=l2, m=m)
        op = rtg.setup_operator_psf(I1, I2, J, p.psf, p.b_band)
        sk = rtg.setup_sketch(I1, I2, J, p.om1, p.om2, p.om3)
    else:
        p = synth.small_problem(9, I1, I2, J, 3, 3, 1, l1, l2, J, m)
        op, sk = U.gpu_pair(p)
    Cs = [U.to_dev(rng.standard_normal((I1, I2, J))) for _ in range(26)]
    basis = rtg.F32_BF16 if "mixed" in form else (rtg.BF16 if "bf16" in form else rtg.F32)
    method = rtg.METHOD_GOLUB_KAHAN if form.startswith("golub_kahan") else rtg.METHOD_GMRES

    def solve(n):
        plan = rtg.BatchPlan([op] * n, [sk] * n, Cs[:n], [None] * n,
                             [rtg.make_params(m, basis, mu=1e-2, method=method)] * n)
        plan.run()
        return [x.clone() for x in plan.outs]

    # 144 and 240 column tiles (one round in any form), 528 and 624
    runs = {n: solve(n) for n in (6, 10, 22, 26)}
    assert all(bool(torch.isfinite(x).all()) and float(x.abs().max()) > 0 for x in runs[6])
    for n in (10, 22, 26):
        for a, b in zip(runs[6], runs[n]):
            assert torch.equal(a, b), n


@pytest.mark.parametrize("l1", [64, 65, 80, 96, 97, 128])
@pytest.mark.parametrize("psf", [False, True])
def test_sketch_tiles_per_wave_match_oracle(l1, psf):
    from paper_2603_00839_amd import rtg
    I1, I2, J, l2, m = 200, 72, 2, 40, 4
    if psf:
        p = synth.psf_problem(5, I1, I2, J, r=3, l1=l1, l2=l2, m=m)
        op_o, sk_o = PSFOperator(p.psf, p.b_band, p.dims), Sketch(p.om1, p.om2, p.om3)
        op = rtg.setup_operator_psf(I1, I2, J, p.psf, p.b_band)
        sk = rtg.setup_sketch(I1, I2, J, p.om1, p.om2, p.om3)
        C = make_observation(op_o, p.x_true, p.noise_dir, p.nu)[0].astype(np.float32)
    else:
        p = synth.small_problem(5, I1, I2, J, 3, 3, 1, l1, l2, J, m, random_bands=True)
        (op_o, sk_o), (op, sk) = U.oracle_pair(p), U.gpu_pair(p)
        C, _ = U.observation(p)
    H = rtg.arnoldi(op, sk, U.to_dev(C), m)["H"].cpu().numpy()
    err = U.maxrel(H, sketched_global_arnoldi(op_o, sk_o, C.astype(np.float64), m).H)
    print(f"l1 {l1} psf {psf}: H {err:.2e}", file=sys.stderr, flush=True)
    assert err < 1e-4
