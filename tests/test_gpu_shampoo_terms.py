"""The Shampoo root iteration on matrices of three bf16 terms: sizes around its 256-wide tiles, shares of the work between
the large and the small kernel, few and many rounds, the padding, sides that take turns, and statistics of mixed scale."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def canz():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_06079_amd import binding
    return binding


def _newton(torch, s, eps, rounds, dtype=None):
    """The same rounds in 64 bits: what exact arithmetic would give after so many."""
    d = s.shape[0]
    dtype = dtype or torch.float64
    eye = torch.eye(d, device=s.device, dtype=dtype)
    a = s.to(dtype) + eps * eye
    nrm = a.norm()
    ap = a / nrm
    a2 = ap @ ap
    z = 2.5 / (a2 @ a2).norm() ** 0.25
    m, x = z * ap, eye * (z / nrm) ** 0.25
    del a2, a
    for _ in range(rounds):
        t = 1.25 * eye - 0.25 * m
        x = x @ t
        t2 = t @ t
        m = t2 @ t2 @ m
    return x


GUARD = 1 << 16   # bytes behind the workspace that must stay as they are


def _step(torch, canz, rows, cols, n, rounds, grad_dtype, eps, level=0.02, beta=1.0, least=False):
    g = torch.Generator(device="cuda").manual_seed(rows * 10007 + cols)
    draw = lambda r, c: torch.randn(r, c, generator=g, device="cuda")  # noqa: E731
    grads = [(draw(rows, cols) * level).to(grad_dtype) for _ in range(n)]
    left = [torch.zeros(rows, rows, device="cuda") for _ in range(n)]
    right = [torch.zeros(cols, cols, device="cuda") for _ in range(n)]
    lroot, rroot = [torch.empty_like(x) for x in left], [torch.empty_like(x) for x in right]
    out = [torch.zeros(rows, cols, device="cuda") for _ in range(n)]
    grp = canz.ShampooGroup(rows=rows, cols=cols, grad=grads, left=left, right=right, out=out, lroot=lroot, rroot=rroot,
                            grad_dtype=canz.DT_BF16 if grad_dtype == torch.bfloat16 else canz.DT_F32)
    hp = canz.ShampooHparams(beta=beta, lr=1.0, eps=eps, root_iters=rounds, out_mode=canz.OUT_DELTA)
    need = canz.canz_shampoo_workspace_bytes([grp], hp)
    if least:   # the size of fp32 matrices padded to 128 is accepted as well
        rp, cp = (rows + 127) // 128 * 128, (cols + 127) // 128 * 128
        need = n * 4 * (3 * rp * cp + rp * rp + cp * cp + 8 * max(rp, cp) ** 2 + 128)
    ws = torch.full((need + GUARD,), 0xFF, dtype=torch.uint8, device="cuda")   # every byte a NaN: nothing may be read unwritten
    canz.canz_shampoo_step([grp], hp, ws, need, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xFF).all())
    return grads, left, right, lroot, rroot, out


@pytest.mark.parametrize("rows,cols,n,rounds,bf16", [
    (256, 256, 1, 22, True),     # one tile
    (255, 257, 2, 22, True),     # one short of a tile, one past it
    (96, 520, 3, 22, False),     # fp32 gradients, odd padding
    (1024, 2048, 5, 22, True),   # enough tiles for the large kernel, and left-over ones for the small kernel
    (2304, 1280, 3, 22, False),
    (300, 700, 1, 1, True),      # the first round is the last
    (300, 700, 1, 2, True),
    (300, 700, 1, 36, True),     # converged long ago: nothing drifts ...
    (300, 700, 1, 60, True),     # ... however many rounds are asked for, and the padding does not overflow
])
def test_roots_against_the_same_rounds_in_64_bits(canz, rows, cols, n, rounds, bf16):
    import torch
    eps = 1e-3
    step = _step(torch, canz, rows, cols, n, rounds, torch.bfloat16 if bf16 else torch.float32, eps)
    _check(torch, rows, cols, n, rounds, eps, *step)


def _check(torch, rows, cols, n, rounds, eps, grads, left, right, lroot, rroot, out):
    for i in range(n):
        g = grads[i].double()
        for got, want in ((left[i], g @ g.t()), (right[i], g.t() @ g)):
            assert float((got.double() - want).norm() / want.norm()) <= 1e-6
            assert torch.equal(got, got.t())
        for s, got in ((left[i], lroot[i]), (right[i], rroot[i])):
            want = _newton(torch, s, float(np.float32(eps)), min(rounds, 36))
            # matrices held to about 24 bits: an eigenvalue near eps is off by up to an fp32 ulp of the largest one
            # (of a Gaussian matrix's statistic: (sqrt(rows) + sqrt(cols))^2 entries), the well-conditioned rest by rounding
            largest = 0.02 ** 2 * (rows ** 0.5 + cols ** 0.5) ** 2
            assert float((got.double() - want).norm() / want.norm()) <= 2.0 ** -24 * largest / eps + 2e-6
        want = -(lroot[i].double() @ g @ rroot[i].double())
        # two fp32 products: each rounds relative to the norms of its factors (a root's is at most eps^(-1/4)), not to
        # the result, in which G's own directions meet the small end of the roots' spectra
        assert float((out[i].double() - want).norm()) <= 1e-6 * eps ** -0.5 * float(g.norm())


@pytest.mark.parametrize("rows,cols,n,bf16", [
    (96, 128, 3, True),      # fp32 matrices: padding to 256 is four times the size
    (640, 600, 1, False),    # ... 1.44 times, and only one matrix
    (300, 380, 4, True),     # 1.78 times: smaller batches, both sides side by side
    (512, 500, 2, True),     # the sides take turns
    (760, 700, 1, False),
    (1024, 300, 2, True),    # all that is asked for
])
def test_least_workspace(canz, rows, cols, n, bf16):
    import torch
    step = _step(torch, canz, rows, cols, n, 22, torch.bfloat16 if bf16 else torch.float32, 1e-3, least=True)
    _check(torch, rows, cols, n, 22, 1e-3, *step)


@pytest.mark.parametrize("level", [1e-6, 1e6])
def test_scale_of_the_gradients_does_not_matter(canz, level):
    """The terms hold A / ||A||: tiny and huge statistics give the same iteration as those of order one."""
    import torch
    eps = 2.5 * level * level
    _, left, _, lroot, _, _ = _step(torch, canz, 200, 300, 1, 22, torch.float32, eps, level=level)
    want = _newton(torch, left[0], float(np.float32(eps)), 22)
    assert float((lroot[0].double() - want).norm() / want.norm()) <= 3e-5


def test_zero_gradient_zero_statistics(canz):
    import torch
    _, left, right, lroot, _, out = _step(torch, canz, 300, 200, 1, 40, torch.bfloat16, 0.0, level=0.0, beta=0.0)
    assert not left[0].any() and not right[0].any() and not out[0].any()
    assert torch.isfinite(lroot[0]).all()


def test_sides_that_take_turns(canz):
    """One matrix whose two sides would not fit the batch memory together: the sides share one set of buffers."""
    import torch
    rows, cols, eps = 16640, 24, 1e-3
    _, left, right, lroot, rroot, _ = _step(torch, canz, rows, cols, 1, 2, torch.bfloat16, eps)
    for s, got in ((left[0], lroot[0]), (right[0], rroot[0])):
        want = _newton(torch, s, float(np.float32(eps)), 2)
        want -= got.double()
        assert float(want.norm() / got.double().norm()) <= 3e-5


def _statistic(torch, kind, d):
    """Symmetric d x d fp32 statistics whose elements differ by many orders of magnitude, largest eigenvalue about 1."""
    g = torch.Generator(device="cuda").manual_seed(d)
    h = torch.randn(d, 2 * d, generator=g, device="cuda", dtype=torch.float64)
    decades = torch.arange(d, device="cuda", dtype=torch.float64) / (d - 1)
    if kind == "empty":                      # half of the rows have seen no gradient
        h[d // 2:] = 0
    elif kind.startswith("rows"):            # row scales 1 .. 10^-n
        h *= (10.0 ** (-float(kind[4:]) * decades))[:, None]
    s = torch.diag(10.0 ** (-float(kind[4:]) * decades)) if kind.startswith("diag") else h @ h.t() / (6 * d)
    s = s.float()
    return torch.triu(s) + torch.triu(s, 1).t()


@pytest.mark.parametrize("kind,d,eps,rounds", [
    ("empty", 300, 1e-6, 34),
    ("empty", 300, 1e-8, 25),
    ("empty", 513, 1e-10, 34),
    ("rows4", 300, 0.0, 30),
    ("rows4", 500, 0.0, 30),
    ("rows5", 256, 0.0, 30),
    ("rows6", 300, 0.0, 36),
    ("diag12", 300, 0.0, 36),
    ("diag12", 1000, 0.0, 45),   # the bound of the largest eigenvalue is loose: more rounds
])
def test_statistics_of_mixed_scale(canz, kind, d, eps, rounds):
    """What is small against ||A|| makes up the root.  As long as the matrix is well conditioned once its rows and columns
    are scaled to one size, relative rounding per element (fp32) moves the root by what the products round and no more: 4
    products a round, each a sum that is rounded up to d / 2 times (fp32 MFMA; small shapes run on it), 2^-24 each time, all
    adding up like random errors: 2^-24 sqrt(d / 2) sqrt(4 rounds), 8e-6 at d = 300.  An absolute resolution of 2^-38 ||A||
    is off by 1e-4 to 1 here."""
    import torch
    s = _statistic(torch, kind, d)
    cols = 40
    left, right = [s.clone()], [torch.eye(cols, device="cuda")]
    lroot, rroot = [torch.empty_like(s)], [torch.empty_like(right[0])]
    grp = canz.ShampooGroup(rows=d, cols=cols, grad=[torch.zeros(d, cols, device="cuda")], left=left, right=right,
                            out=[torch.zeros(d, cols, device="cuda")], lroot=lroot, rroot=rroot, grad_dtype=canz.DT_F32)
    hp = canz.ShampooHparams(beta=1.0, lr=1.0, eps=eps, root_iters=rounds, out_mode=canz.OUT_DELTA)
    need = canz.canz_shampoo_workspace_bytes([grp], hp)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    canz.canz_shampoo_step([grp], hp, ws, need, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(left[0], s)
    want = _newton(torch, s, float(np.float32(eps)), rounds)
    err = float((lroot[0].double() - want).norm() / want.norm())
    print("%s d %d eps %g rounds %d: %.3g" % (kind, d, eps, rounds, err))
    assert err <= 2.0 ** -24 * (d / 2 * 4 * rounds) ** 0.5


@pytest.mark.parametrize("d,rank,eps,rounds", [(512, 64, 1e-5, 22), (512, 64, 1e-6, 25), (1000, 300, 1e-6, 25), (300, 1, 1e-6, 25), (96, 8, 1e-5, 22)])
def test_rank_deficient_statistics(canz, d, rank, eps, rounds):
    """S = H H^T of few columns, down to the eps of 1e-6 of the largest eigenvalue that is called safe: the rounds are no further
    from 64 bits than the same rounds in fp32 (within half, the scatter where few products dominate)."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(d + rank)
    h = torch.randn(d, rank, generator=g, device="cuda", dtype=torch.float64)
    s = h @ h.t()
    s = (s / torch.linalg.matrix_norm(s.cpu(), 2).to(s.device)).float()
    s = torch.triu(s) + torch.triu(s, 1).t()
    left, right = [s.clone()], [torch.eye(32, device="cuda")]
    lroot, rroot = [torch.empty_like(s)], [torch.empty_like(right[0])]
    grp = canz.ShampooGroup(rows=d, cols=32, grad=[torch.zeros(d, 32, device="cuda")], left=left, right=right,
                            out=[torch.zeros(d, 32, device="cuda")], lroot=lroot, rroot=rroot, grad_dtype=canz.DT_F32)
    hp = canz.ShampooHparams(beta=1.0, lr=1.0, eps=eps, root_iters=rounds, out_mode=canz.OUT_DELTA)
    need = canz.canz_shampoo_workspace_bytes([grp], hp)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    canz.canz_shampoo_step([grp], hp, ws, need, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    want = _newton(torch, s, float(np.float32(eps)), rounds)
    err = float((lroot[0].double() - want).norm() / want.norm())
    fp32 = float((_newton(torch, s, float(np.float32(eps)), rounds, torch.float32).double() - want).norm() / want.norm())
    print("d %d rank %d eps %g: %.3g, in fp32 %.3g" % (d, rank, eps, err, fp32))
    assert err <= 1.5 * fp32
