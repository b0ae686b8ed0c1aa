"""Gram products of at most half a round of tiles with a long k: on either side of the lengths where they go from small tiles (64 x 64,
128 x 128 with eight stages, with three) to the large kernel cut along k, from X and from X^T, and as the first product of merged steps.
Against the oracle, Delta W to 3e-2 (bf16 operands), momentum to 1e-6."""
import numpy as np
import pytest

from oracle import muon as OM
from paper_2602_06079_amd import workloads as W
from tests.gpu_harness import DeviceGroup, oracle_hparams, rel_fro, run_step, widen

pytestmark = pytest.mark.gpu

# (count, rows, cols, steps); k is cols rounded up to 256
SHAPES = [
    (1, 100, 196300, 5),     # 6136 k-steps of 32: 64 x 64 tiles
    (1, 100, 196400, 5),     # 6144: split, from X
    (9, 130, 196613, 5),     # 2304 padded rows in all: from X^T, nine tiles in eight slices
    (28, 40, 45056, 2),      # 1408 k-steps, 280 blocks of 64 x 64 would share the CUs: split in eight
    (56, 40, 44800, 2),      # 1400 k-steps, 168 blocks of 128 x 128 with eight stages
    (56, 40, 45100, 2),      # 1416: split in four
    (1, 2830, 19300, 3),     # 78 tiles of merged steps (the first two of three) in three slices, then alone
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%dx%d" % s[:3])
def test_against_the_oracle(canz, shape):
    n, rows, cols, steps = shape
    two = [W.gen_grad(99, i, rows, cols)[0] for i in range(min(n, 2))]
    grads = [two[i % len(two)] for i in range(n)]
    zeros = [np.zeros((rows, cols), np.float32)] * n
    hp = canz.Hparams(out_mode=canz.OUT_DELTA, ns_steps=steps)
    dg = DeviceGroup(canz, rows, cols, grads, zeros)
    run_step(canz, [dg], hp)
    for i in sorted({0, n - 1}):
        ref = OM.muon_step(widen(grads[i]), widen(zeros[i]), oracle_hparams(hp))
        assert rel_fro(dg.mom_host(i), ref["mom"]) <= 1e-6
        assert rel_fro(dg.out_host(i), ref["delta"]) <= 3e-2
