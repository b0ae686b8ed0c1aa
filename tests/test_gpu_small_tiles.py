"""GPU parity of the small-product kernel's variants (64 x 64 and 128 x 128 tiles, three or eight stages) and of the last
product's epilogue on rows of any length: shapes on either side of the numbers of blocks where the launcher changes variant,
column remainders 1 to 3, in-place fp32 and bf16 parameters and Delta W.  The tolerance of Delta W is 3e-2 relative (bf16
operands, five iterations); bf16 results are rounded once more (2^-8 of the largest value).  What lies behind a matrix in
memory stays as it was."""
import numpy as np
import pytest

from oracle import muon as OM
from paper_2602_06079_amd import workloads as W
from tests.gpu_harness import DeviceGroup, oracle_hparams, rel_fro, run_step, to_host64, widen

pytestmark = pytest.mark.gpu

TOL = 3e-2
# (count, rows, cols): blocks of the Gram and of the update product on 256 CUs
SHAPES = [
    (1, 5, 9), (2, 63, 65), (3, 130, 258),   # one tile of 64 x 64 or a few
    (1, 259, 12801),                         # k = 13056: four hundred steps on a handful of tiles
    (4, 515, 1537),                          # Gram 60 blocks of 128, update 280
    (9, 777, 1022),                          # Gram 324 blocks: three stages
    (3, 1029, 1283),                         # Gram 135 blocks, k = 1536: eight stages of 128
    (1, 2050, 2563),                         # update 99 tiles, k = 2304: 256 x 128
]
OUTS = ["param_f32", "param_bf16", "delta_f32", "delta_bf16"]


@pytest.mark.parametrize("out", OUTS)
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%dx%d" % s)
def test_variants_against_the_oracle(canz, shape, out):
    import torch
    n, rows, cols = shape
    check = sorted({0, n - 1})                       # the oracle runs on the first and the last matrix
    grads = [W.gen_grad(95, i, rows, cols)[0] for i in range(n)]
    moms = [W.gen_normal_f32(95, i, 3, rows, cols, 0.01) for i in range(n)]
    bf16, in_place = out.endswith("bf16"), out.startswith("param")
    params = None
    if in_place:
        params = [W.gen_param(95, i, rows, cols, std=0.5) for i in range(n)]
        if bf16:
            params = [W.f32_to_bf16_bits(p) for p in params]
    hp = canz.Hparams(out_mode=canz.OUT_PARAM if in_place else canz.OUT_DELTA, weight_decay=0.1, lr=0.5)
    dg = DeviceGroup(canz, rows, cols, grads, moms, outs=params, out_np_dtype=np.uint16 if bf16 else np.float32)
    # the results in buffers with a guard behind them
    guard, whole = 64, []
    for i, t in enumerate(dg.out_t):
        buf = torch.full((t.numel() + guard,), 7.0, dtype=t.dtype, device="cuda")
        buf[:t.numel()] = t.reshape(-1)
        whole.append(buf)
        dg.out_t[i] = buf[:t.numel()].view(rows, cols)
    run_step(canz, [dg], hp)
    for buf in whole:
        assert bool((buf[-guard:] == 7.0).all()), "written behind the matrix"
    for i in check:
        ref = OM.muon_step(widen(grads[i]), widen(moms[i]), oracle_hparams(hp), param=None if params is None else widen(params[i]))
        assert rel_fro(dg.mom_host(i), ref["mom"]) <= 1e-6
        got, want = dg.out_host(i), ref["param" if in_place else "delta"]
        if bf16:
            assert np.max(np.abs(got - want)) <= 2.0 ** -8 * np.max(np.abs(want)) + TOL * np.max(np.abs(ref["delta"])) * 4
        else:
            assert np.linalg.norm(got - want) <= TOL * np.linalg.norm(ref["delta"])


@pytest.mark.parametrize("shape", [(256, 512), (300, 77), (640, 1100)], ids=lambda s: "%dx%d" % s)
def test_variants_agree_bit_for_bit(canz, shape):
    """A matrix on its own (64 x 64 tiles) and among 40 alike (128 x 128 tiles): the same products in the same order."""
    rows, cols = shape
    n = 40
    grads = [W.gen_grad(96, i, rows, cols)[0] for i in range(n)]
    zeros = [np.zeros((rows, cols), np.float32)] * n
    hp = canz.Hparams(out_mode=canz.OUT_DELTA)
    many = DeviceGroup(canz, rows, cols, grads, zeros)
    run_step(canz, [many], hp)
    for i in (0, n // 2, n - 1):
        one = DeviceGroup(canz, rows, cols, grads[i:i + 1], zeros[:1])
        run_step(canz, [one], hp)
        assert np.array_equal(to_host64(one.out_t[0]), to_host64(many.out_t[i]))


@pytest.mark.parametrize("shapes", [[(2, 432, 640), (2, 181, 192)], [(3, 64, 520), (1, 130, 66), (5, 97, 257)],
                                    [(2, 1024, 1024), (1, 700, 1300)]],
                         ids=lambda s: "+".join("%dx%dx%d" % x for x in s))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_classes_of_a_call_as_each_alone(canz, shapes, dtype):
    """Classes that share their launches (momentum, norm, last product; the Gram product from X^T once the rows together
    reach 1536): every matrix has the bits that it has in a call of its own."""
    hp = canz.Hparams(out_mode=canz.OUT_DELTA)
    made = []
    for c, (n, rows, cols) in enumerate(shapes):
        grads = [W.gen_grad(97, 16 * c + i, rows, cols)[0] for i in range(n)]
        if dtype == "bf16":
            grads = [W.f32_to_bf16_bits(widen(g).astype(np.float32)) for g in grads]
        else:
            grads = [widen(g).astype(np.float32) for g in grads]
        made.append((rows, cols, grads, [W.gen_normal_f32(97, 16 * c + i, 3, rows, cols, 0.01) for i in range(n)]))
    together = [DeviceGroup(canz, r, k, g, m) for r, k, g, m in made]
    run_step(canz, together, hp)
    for dg, (rows, cols, grads, moms) in zip(together, made):
        for i in range(len(grads)):
            one = DeviceGroup(canz, rows, cols, grads[i:i + 1], moms[i:i + 1])
            run_step(canz, [one], hp)
            assert np.array_equal(to_host64(one.out_t[0]), to_host64(dg.out_t[i]))
            assert np.array_equal(one.mom_host(0), dg.mom_host(i))


@pytest.mark.parametrize("n,rows,cols", [(31, 2047, 1023), (32, 2047, 1023), (27, 1024, 2043)], ids=lambda x: str(x))
@pytest.mark.parametrize("out", ["param_f32", "delta_bf16"])
def test_last_products_of_a_few_rounds(canz, n, rows, cols, out):
    """992, 1024 and 864 tiles of 256 x 256: on either side of where the last product of parameters, and that of Delta W, goes from small
    tiles to large ones for the full rounds.  Every matrix checked has the bits that it has alone."""
    delta = out.startswith("delta")
    two = [W.gen_grad(94, i, rows, cols)[0] for i in range(2)]
    zeros = [np.zeros((rows, cols), np.float32)] * n
    params = None if delta else [W.gen_param(94, i % 2, rows, cols, std=0.5) for i in range(n)]
    hp = canz.Hparams(out_mode=canz.OUT_DELTA if delta else canz.OUT_PARAM, weight_decay=0.1, lr=0.5)
    dtype = np.uint16 if out.endswith("bf16") else np.float32
    many = DeviceGroup(canz, rows, cols, [two[i % 2] for i in range(n)], zeros, outs=params, out_np_dtype=dtype)
    run_step(canz, [many], hp)
    for i in (0, n - 1):
        one = DeviceGroup(canz, rows, cols, [two[i % 2]], zeros[:1], outs=None if delta else [params[i]], out_np_dtype=dtype)
        run_step(canz, [one], hp)
        assert np.array_equal(to_host64(one.out_t[0]), to_host64(many.out_t[i]))
