"""Muon steps whose Newton-Schulz steps are merged (two or three at a time among the m x m matrices): parity with the
oracle at the edges of the rule that selects them, for every split of the step count into stages, and the workspace."""
import numpy as np
import pytest

from oracle import muon as OM
from paper_2602_06079_amd import workloads as W
from tests.gpu_harness import DeviceGroup, log, oracle_hparams, rel_fro, run_step, widen

pytestmark = pytest.mark.gpu

# The bound of single steps (each stored operand rounded once per step, 2^-9 relative, slope of the map at most 1.7: about
# 1e-2 for Gaussian inputs) holds for merged ones, whose operands are rounded less often.
TOL = 1.0e-2


@pytest.fixture(scope="module")
def canz():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_06079_amd import binding
    return binding


def _inputs(seed, rows, cols, n):
    grads = [W.gen_grad(seed, i, rows, cols)[0] for i in range(n)]
    moms = [W.gen_normal_f32(seed, i, 5, rows, cols, 0.01) for i in range(n)]
    params = [W.gen_param(seed, i, rows, cols) for i in range(n)]
    return grads, moms, params


def _check(dg, ins, hp, name):
    ohp = oracle_hparams(hp)
    for i, (g, m, p) in enumerate(zip(*ins)):
        ref = OM.muon_step(widen(g), widen(m), ohp, widen(p))
        got = dg.out_host(i) - (widen(p) * (1.0 - ohp.lr * ohp.weight_decay))
        err = rel_fro(got, ref["delta"])
        log("%s matrix %d: %.3g" % (name, i, err))
        assert err <= TOL, "%s matrix %d: error %.3g" % (name, i, err)
        assert rel_fro(dg.mom_host(i), ref["mom"]) <= 1e-6


@pytest.mark.parametrize("rows,cols,steps", [
    (1536, 3072, 5),   # the smallest, whole tiles
    (1535, 3072, 5),   # just below: single steps
    (3075, 1537, 5),   # odd, tall: padding in every matrix, the swapped last product
    (1536, 3071, 5),   # just too square: single steps
    (2560, 3840, 5),   # the spare arrays would just not fit: single steps
    (2560, 3900, 5),   # the wider rule from 2560 rows on, the spare arrays just fit
    (1600, 3300, 3),   # stages 2 + 1
    (1600, 3300, 4),   # stages 3 + 1
    (1600, 3300, 6),   # stages 3 + 2 + 1
    (1600, 3300, 2),   # not merged
])
def test_merged_steps(canz, rows, cols, steps):
    ins = _inputs(81, rows, cols, 2)
    hp = canz.Hparams(ns_steps=steps, nesterov=True, weight_decay=0.1)
    dg = DeviceGroup(canz, rows, cols, ins[0], ins[1], outs=ins[2])
    run_step(canz, [dg], hp)
    _check(dg, ins, hp, "%dx%d, %d steps" % (rows, cols, steps))


def test_merged_steps_share_launches(canz):
    """Wide and tall matrices of one class, a second merged class and one with single steps in one call: parity, and the
    same bits as each group alone."""
    shapes = [(1536, 3328, 2), (3328, 1536, 1), (1792, 3584, 1), (512, 768, 2)]
    hp = canz.Hparams(weight_decay=0.1)
    ins = [_inputs(90 + k, *s) for k, s in enumerate(shapes)]
    make = lambda k: DeviceGroup(canz, shapes[k][0], shapes[k][1], ins[k][0], ins[k][1], outs=ins[k][2])  # noqa: E731
    together = [make(k) for k in range(len(shapes))]
    run_step(canz, together, hp)
    for k, s in enumerate(shapes):
        _check(together[k], ins[k], hp, "group %d" % k)
        alone = make(k)
        run_step(canz, [alone], hp)
        for i in range(s[2]):
            assert np.array_equal(alone.out_host(i), together[k].out_host(i))


def test_cubic_and_expanding_coefficients_keep_single_steps(canz):
    rows, cols = 1536, 3072
    ins = _inputs(83, rows, cols, 1)
    for co in ((1.5, -0.5, 0.0), (3.6, -4.9, 2.05)):
        hp = canz.Hparams(a=co[0], b=co[1], c=co[2])
        dg = DeviceGroup(canz, rows, cols, ins[0], ins[1], outs=ins[2])
        groups = [dg.group()]
        # three X arrays, two m x m arrays and the k-split scratch: none of the merged steps' arrays
        assert canz.canz_muon_workspace_bytes(groups, hp) < 2 * (3 * rows * cols + 2 * rows * rows) + (64 << 20) + (1 << 20)
        run_step(canz, [dg], hp)
        ohp = oracle_hparams(hp)
        ref = OM.muon_step(widen(ins[0][0]), widen(ins[1][0]), ohp, widen(ins[2][0]))
        assert rel_fro(dg.out_host(0) - widen(ins[2][0]), ref["delta"]) <= 2 * TOL


def test_workspace_of_small_merged_batches_is_unchanged(canz):
    """The merged steps' arrays lie in X and the X^T that is not in use: no more is asked for than for single steps."""
    one = canz.Group(rows=1536, cols=3072, mom=[], n_mats=1)
    rows, cols = 1536, 3072
    need = canz.canz_muon_workspace_bytes([one], canz.Hparams())
    assert need < 2 * (3 * rows * cols + 2 * rows * rows) + (64 << 20) + (1 << 20)
