"""Calls whose groups differ in everything a group may differ in - column fragments, row length, gradient and output type - share the
launches of momentum, norm and last product as long as their buffers fit one table.  Every matrix must have the bits that it has when
its group is run alone, its momentum must agree with the oracle (1e-6), nothing is read behind a gradient fragment (NaNs lie there)
and nothing written behind a result."""
import numpy as np
import pytest

from paper_2602_06079_amd import workloads as W
from tests.gpu_harness import DeviceGroup, oracle_hparams, rel_fro, run_step, to_host64, widen

pytestmark = pytest.mark.gpu

GUARD = 2048
# (count, rows, cols, tp, bf16 gradients, bf16 results)
CALLS = {
    "tp2+ragged": [(2, 256, 512, 2, True, True), (1, 300, 77, 1, True, True)],
    "ragged+tp4": [(1, 333, 129, 1, False, True), (2, 96, 768, 4, True, False)],
    "tp4+ragged+tp2": [(2, 320, 768, 4, False, False), (3, 130, 66, 1, True, True), (2, 97, 144, 2, True, False)],
    "one orientation each": [(1, 192, 640, 4, True, False), (1, 640, 191, 1, False, False), (2, 640, 192, 2, True, True)],
    # 2304 > 2048: the last products run one by one, from the shifted table
    "last products apart": [(1, 2304, 2320, 2, True, True), (2, 77, 301, 1, False, False), (1, 301, 80, 2, True, False)],
    # 128 + 3 gradient buffers: no shared table
    "too many buffers": [(16, 64, 128, 8, True, True), (3, 33, 77, 1, True, False)],
}


def _guarded(t, fill):
    import torch
    buf = torch.full((t.numel() + GUARD,), fill, dtype=t.dtype, device="cuda")
    buf[:t.numel()] = t.reshape(-1)
    return buf, buf[:t.numel()].view(t.shape)


def _make(canz, c, spec, delta):
    n, rows, cols, tp, grad16, out16 = spec
    whole = [widen(W.gen_grad(98, 32 * c + i, rows, cols)[0]).astype(np.float32) for i in range(n)]
    whole = [W.f32_to_bf16_bits(g) for g in whole] if grad16 else whole
    moms = [W.gen_normal_f32(98, 32 * c + i, 3, rows, cols, 0.01) for i in range(n)]
    params = None
    if not delta:
        params = [W.gen_param(98, 32 * c + i, rows, cols, std=0.5) for i in range(n)]
        params = [W.f32_to_bf16_bits(p) for p in params] if out16 else params
    dg = DeviceGroup(canz, rows, cols, [W.split_columns(g, tp) for g in whole] if tp > 1 else whole, moms, outs=params, tp=tp,
                     out_np_dtype=np.uint16 if out16 else np.float32)
    dg.grad_t = [_guarded(t, float("nan"))[1] for t in dg.grad_t]
    bufs = [_guarded(t, 7.0) for t in dg.out_t]
    dg.out_t = [view for _, view in bufs]
    return dg, whole, moms, [buf for buf, _ in bufs]


@pytest.mark.parametrize("delta", [False, True], ids=["param", "delta"])
@pytest.mark.parametrize("call", CALLS)
def test_each_group_as_alone(canz, call, delta):
    hp = canz.Hparams(out_mode=canz.OUT_DELTA if delta else canz.OUT_PARAM, nesterov=1, weight_decay=0.1, lr=0.5)
    together = [_make(canz, c, spec, delta) for c, spec in enumerate(CALLS[call])]
    run_step(canz, [t[0] for t in together], hp)
    ohp = oracle_hparams(hp)
    for c, (dg, whole, moms, bufs) in enumerate(together):
        for buf in bufs:
            assert bool((buf[-GUARD:] == 7.0).all()), "written behind a result"
        for i in range(dg.n):
            want = ohp.beta * widen(moms[i]) + widen(whole[i])
            assert rel_fro(dg.mom_host(i), want) <= 1e-6, "momentum of matrix %d of group %d" % (i, c)
        alone = _make(canz, c, CALLS[call][c], delta)[0]
        run_step(canz, [alone], hp)
        for i in range(dg.n):
            assert np.array_equal(alone.mom_host(i), dg.mom_host(i)), "momentum of matrix %d of group %d" % (i, c)
        for k, (a, b) in enumerate(zip(alone.out_t, dg.out_t)):
            assert np.isfinite(to_host64(b)).all()
            assert np.array_equal(to_host64(a), to_host64(b)), "result %d of group %d" % (k, c)
