"""The refresh of both sides in the same launches: one side ends before the other, at and around the numbers of remaining rows where the
panel kernel changes (512, 1024, 2048) and the blocks of 128 columns, three matrices, every kind of rotation (which place the statistic
and Q^T differently).  Against the oracle, with the tolerances of the SOAP tests."""
import pytest

from paper_2602_06079_amd import workloads as W
from tests.test_gpu_soap import SoapDevice, TOL16_UPDATE, TOL16_VAR, check, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16_rot", [False, True], ids=["terms", "bf16"])
@pytest.mark.parametrize("shape", [(640, 130), (130, 1025), (513, 512), (1153, 1000)], ids=lambda s: "%dx%d" % s)
def test_refresh_of_two_sides(canz, shape, bf16_rot):
    rows, cols = shape
    n = 3 if rows * cols < 1 << 19 else 1
    grads = [W.gen_grad(97, i, rows, cols)[0] for i in range(n)]
    states = [W.gen_soap_state(97, i, rows, cols) for i in range(n)]
    hp = canz.SoapHparams(lr=0.01, eps=1e-8, step=10, refresh=True, out_mode=canz.OUT_DELTA, bf16_rotations=bf16_rot)
    dev = SoapDevice(canz, rows, cols, grads, states)
    run(canz, [dev], hp)
    tol = dict(tol_update=TOL16_UPDATE, tol_var=TOL16_VAR) if bf16_rot else {}
    check(dev, grads, states, None, hp, "refresh of two sides %dx%d" % shape, **tol)


@pytest.mark.parametrize("shape", [(3201, 2060), (2060, 3201)], ids=lambda s: "%dx%d" % s)
def test_refresh_of_two_long_sides(canz, shape):
    """Both sides beyond the 2048 rows of the shorter panel kernels: panels that stream their rows beyond the registers (3328 and 2176
    remaining rows in one launch, then 3200 beside 2048, a launch each), panels of up to 3072 rows beside short ones of the other side,
    in either order of the sides."""
    rows, cols = shape
    grads = [W.gen_grad(99, 0, rows, cols)[0]]
    states = [W.gen_soap_state(99, 0, rows, cols)]
    hp = canz.SoapHparams(lr=0.01, eps=1e-8, step=10, refresh=True, out_mode=canz.OUT_DELTA)
    dev = SoapDevice(canz, rows, cols, grads, states)
    run(canz, [dev], hp)
    check(dev, grads, states, None, hp, "refresh of two long sides %dx%d" % shape)
