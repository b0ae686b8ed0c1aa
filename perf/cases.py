"""Performance cases: one optimizer step of one rank, through the public entry points.

A case is one call of canz_muon_step, canz_shampoo_step or canz_soap_step (paper_2602_06079_amd.binding)
on the matrices one rank owns, as a training program issues it once per iteration: the buffers, the
micro-groups and the workspace are made once and kept, the step updates momentum, statistics and
parameters in place (or writes the Delta W fragments of a tensor-parallel rank).

Shapes are those of this repository's workloads (paper_2602_06079_amd/workloads.py: the tiny set, the
Qwen3 0.6B / 8B / 32B shaped layers, the 8B set as column fragments) and generic odd ones.  A case is a
dict of plain values:

  op        "muon" | "shampoo" | "soap"
  shapes    "<count>x<rows>x<cols>+...": the micro-groups of the call, in order
  grad      "bf16" | "f32"
  out       "param_f32" | "param_bf16" (updated in place) | "delta_bf16" | "delta_f32" (fragments, overwritten)
  tp        column fragments each gradient (and Delta W) arrives in
  muon:     nesterov, wd, scale (0 none, 1 aspect, 2 rms)
  shampoo:  iters (root rounds), keep (1: roots of an earlier step, kept by the caller)
  soap:     bf16rot, refresh
"""
import math

import torch

from paper_2602_06079_amd import binding as canz

DEV = "cuda"
NS = (3.4445, -4.7750, 2.0315)   # the quintic of the Muon step
NS_STEPS = 5
BETA = 0.95
LR = 0.02
SOAP_LR = 3e-3
SOAP_STEP = 20                   # t of the bias correction: a run that is under way
MAX_PRECOND_DIM = 10000


def listed():
    return [
        # the tiny workload: 8 x 256 x 512, fp32 gradients.  Launches, host work and latency.
        dict(name="muon_tiny", op="muon", shapes="8x256x512", grad="f32", out="param_f32", tp=1, nesterov=0, wd=0.0, scale=2),
        # 0.6B-shaped set over 8 ranks: the share of rank 0 (26 matrices of one shape)
        dict(name="muon_0p6b_share", op="muon", shapes="26x2048x1024", grad="bf16", out="param_f32", tp=1, nesterov=0, wd=0.0,
             scale=2),
        # the seven matrices of one 0.6B-shaped layer: a rank that owns whole layers; four shape classes in one call,
        # bf16 parameters, Nesterov momentum, weight decay
        dict(name="muon_layer_mixed", op="muon", shapes="2x3072x1024+1x1024x3072+1x2048x1024+1x1024x2048+2x1024x1024", grad="bf16",
             out="param_bf16", tp=1, nesterov=1, wd=0.1, scale=2),
        # odd extents: rows that are no multiple of any vector or tile, two classes
        dict(name="muon_ragged", op="muon", shapes="3x1000x1531+2x777x333", grad="bf16", out="param_f32", tp=1, nesterov=1, wd=0.01,
             scale=1),
        # 8B-shaped set over 32 ranks, balanced by FLOPs: the share of the slowest rank
        dict(name="muon_8b_share", op="muon", shapes="5x4096x12288", grad="bf16", out="param_f32", tp=1, nesterov=0, wd=0.0, scale=2),
        # the square projections of the 8B-shaped set as a tensor-parallel host rank sees them: four column fragments
        # per gradient, Delta W fragments out
        dict(name="muon_tp4_square", op="muon", shapes="6x4096x4096", grad="bf16", out="delta_bf16", tp=4, nesterov=0, wd=0.0, scale=2),
        # 32B-shaped set over 64 ranks: the share of the heaviest rank (the benchmark's default)
        dict(name="muon_32b_share", op="muon", shapes="4x25600x5120", grad="bf16", out="param_f32", tp=1, nesterov=0, wd=0.0, scale=2),
        # Shampoo as published: roots computed on the step (and handed to the caller, who keeps them)
        dict(name="shampoo_roots", op="shampoo", shapes="4x3072x1024", grad="bf16", out="param_f32", tp=1, iters=22, keep=0),
        # Shampoo between two root computations: the 0.6B-shaped share on kept roots
        dict(name="shampoo_kept", op="shampoo", shapes="8x3072x1024+6x3072x1024", grad="bf16", out="param_f32", tp=1, iters=22, keep=1),
        # SOAP between two refreshes, everything in fp32: 0.6B-shaped matrices
        dict(name="soap_plain", op="soap", shapes="8x3072x1024", grad="bf16", out="param_f32", tp=1, bf16rot=0, refresh=0),
        # SOAP refresh step (QR of both sides)
        dict(name="soap_refresh", op="soap", shapes="4x2048x1024", grad="bf16", out="param_f32", tp=1, bf16rot=0, refresh=1),
        # SOAP on the 32B-shaped set with the rotations on bf16 operands
        dict(name="soap_32b_bf16rot", op="soap", shapes="2x8192x5120", grad="bf16", out="param_f32", tp=1, bf16rot=1, refresh=0),
    ]


def draw(rng):
    """One more case of the same ranges: sizes spread over their logarithm, odd ones among them."""
    op = rng.choice(["muon", "muon", "muon", "shampoo", "soap"])

    def extent(lo, hi):
        x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        kind = rng.random()
        if kind < 0.4:
            x = max(1, round(x / 128)) * 128
        elif kind < 0.7:
            x = max(1, round(x / 8)) * 8
        return max(lo, min(hi, x))

    grad = rng.choice(["bf16", "bf16", "f32"])
    if op == "muon":
        groups, flops = [], 0.0
        for _ in range(rng.choice([1, 1, 2, 3])):
            rows, cols = extent(96, 25600), extent(96, 12288)
            if min(rows, cols) > 5120:
                cols = extent(96, 5120)
            one = _muon_flops(rows, cols)
            most = int(min(10, max(1, (1.5e13 - flops) / one)))
            if flops + one > 1.5e13:
                continue
            count = int(round(math.exp(rng.uniform(0, math.log(most))))) if most > 1 else 1
            groups.append((count, rows, cols))
            flops += count * one
        if not groups:
            groups = [(2, extent(96, 1024), extent(96, 1024))]
        tp, out = 1, rng.choice(["param_f32", "param_f32", "param_bf16"])
        if rng.random() < 0.25:
            tp, out = rng.choice([2, 4]), "delta_bf16"
            groups = [(min(c, 4), r, max(1, round(k / (8 * tp))) * 8 * tp) for c, r, k in groups]
        return dict(op="muon", shapes=_text(groups), grad=grad, out=out, tp=tp, nesterov=rng.choice([0, 1]),
                    wd=rng.choice([0.0, 0.1]), scale=rng.choice([1, 2]))
    if op == "shampoo":
        rows, cols = extent(96, 3072), extent(96, 2048)
        keep = rng.choice([0, 1])
        most = 8 if max(rows, cols) <= 1024 else 3
        return dict(op="shampoo", shapes=_text([(rng.randint(1, most), rows, cols)]), grad=grad, out="param_f32", tp=1, iters=22,
                    keep=keep)
    refresh = 1 if rng.random() < 0.3 else 0
    rows, cols = (extent(96, 2048), extent(96, 1536)) if refresh else (extent(96, 8192), extent(96, 4096))
    most = 8 if max(rows, cols) <= 1024 else 2
    return dict(op="soap", shapes=_text([(rng.randint(1, most), rows, cols)]), grad=grad, out="param_f32", tp=1,
                bf16rot=rng.choice([0, 1]), refresh=refresh)


# ------------------------------------------------------------------ inputs

def _text(groups):
    return "+".join("%dx%dx%d" % g for g in groups)


def _groups(case):
    return [tuple(int(x) for x in part.split("x")) for part in case["shapes"].split("+")]


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(20260206 + int(seed))
    return g


def _normal(g, rows, cols, std):
    return torch.randn(rows, cols, generator=g, device=DEV, dtype=torch.float32).mul_(std)


def _gradient(g, rows, cols, std=0.02):
    """Noise plus a rank-8 part with geometrically decaying weights, as gradients of a layer have: small and large
    singular values together."""
    x = _normal(g, rows, cols, std)
    left, right = _normal(g, rows, 8, 1.0), _normal(g, 8, cols, 1.0)
    weights = (0.5 ** torch.arange(8, device=DEV, dtype=torch.float32)).mul_(std * 0.5)
    return x.addmm_(left * weights, right)


def _spd(g, d, level, aspect):
    """A statistic under way: level * H H^T / n of a Gaussian d x n factor (rank deficient where n < d)."""
    n = max(8, int(aspect * d))
    h = _normal(g, d, n, 1.0)
    s = (h @ h.t()).mul_(level / n)
    return torch.triu(s) + torch.triu(s, 1).t()


def _basis(g, d):
    """A dense orthogonal d x d matrix: the cosine basis with its rows and columns permuted and signed at random."""
    i = torch.arange(d, device=DEV)
    arg = (i[:, None] * (2 * i[None, :] + 1)) % (4 * d)
    q = torch.cos(arg.to(torch.float64).mul_(math.pi / (2 * d))).mul_(math.sqrt(2.0 / d))
    q[0].mul_(math.sqrt(0.5))
    sign = lambda: torch.randint(0, 2, (d,), generator=g, device=DEV).to(torch.float64).mul_(2).sub_(1)  # noqa: E731
    q = q[torch.randperm(d, generator=g, device=DEV)] * sign()[:, None] * sign()[None, :]
    return q.to(torch.float32).contiguous()


def _young_basis(g, d):
    """The basis of a run whose first refreshes are just behind it: still close to the identity it started from (two
    reflections), so the signs of the next QR factor are far from any tie."""
    q = torch.eye(d, device=DEV, dtype=torch.float64)
    for _ in range(2):
        v = torch.randn(d, 1, generator=g, device=DEV, dtype=torch.float64)
        v /= v.norm()
        q = q - 2.0 * v @ (v.t() @ q)
    return q.to(torch.float32).contiguous()


def _matrices(case, seed):
    """Per micro-group, per matrix: a dict of device tensors (gradient whole, before it is cut into fragments)."""
    g = _generator(seed)
    gdt = torch.bfloat16 if case["grad"] == "bf16" else torch.float32
    odt = torch.bfloat16 if case["out"].endswith("bf16") else torch.float32
    param = case["out"].startswith("param")
    all_groups = []
    for count, rows, cols in _groups(case):
        mats = []
        for _ in range(count):
            m = {"grad": _gradient(g, rows, cols).to(gdt)}
            if param:
                m["param"] = _normal(g, rows, cols, 0.02).to(odt)
            if case["op"] == "muon":
                m["mom"] = _gradient(g, rows, cols, 0.05)
            elif case["op"] == "shampoo":
                m["left"] = _spd(g, rows, 4e-4 * cols, 0.5)
                m["right"] = _spd(g, cols, 4e-4 * rows, 0.5)
                if case["keep"]:
                    # symmetric positive definite, of the size inverse fourth roots of such statistics have
                    m["lroot"] = _spd(g, rows, (4e-4 * cols) ** -0.25, 4)
                    m["rroot"] = _spd(g, cols, (4e-4 * rows) ** -0.25, 4)
                else:
                    m["lroot"] = torch.zeros(rows, rows, device=DEV)
                    m["rroot"] = torch.zeros(cols, cols, device=DEV)
            else:
                basis = _young_basis if case["refresh"] else _basis
                m["mom"] = _normal(g, rows, cols, 0.02)
                m["var"] = sum(_normal(g, rows, cols, 0.02).square_() for _ in range(4)).mul_(0.25)
                if rows <= MAX_PRECOND_DIM:
                    m["left"], m["qleft"] = _spd(g, rows, 4e-4 * cols, 2), basis(g, rows)
                if cols <= MAX_PRECOND_DIM:
                    m["right"], m["qright"] = _spd(g, cols, 4e-4 * rows, 2), basis(g, cols)
                rot = m["mom"]
                if "qleft" in m:
                    rot = m["qleft"].t() @ rot
                if "qright" in m:
                    rot = rot @ m["qright"]
                m["mom_rot"] = rot.contiguous()
            mats.append(m)
        all_groups.append((rows, cols, mats))
    return all_groups


def _fragments(x, tp):
    w = x.shape[1] // tp
    return [x[:, f * w:(f + 1) * w].contiguous() for f in range(tp)]


def _shampoo_eps(case):
    """About 1e-4 of the largest eigenvalue of the statistics such gradients give: the noise and the strongest of the
    rank-8 part (see _gradient)."""
    return 1e-4 * max(2.4e-3 * max(r, c) + 1e-4 * r * c for _, r, c in _groups(case))


def _hparams(case):
    out_mode = canz.OUT_PARAM if case["out"].startswith("param") else canz.OUT_DELTA
    if case["op"] == "muon":
        return canz.Hparams(beta=BETA, lr=LR, weight_decay=case["wd"], nesterov=bool(case["nesterov"]), ns_steps=NS_STEPS,
                            scale_mode=case["scale"], out_mode=out_mode)
    if case["op"] == "shampoo":
        return canz.ShampooHparams(beta=BETA, lr=LR, eps=_shampoo_eps(case), root_iters=case["iters"], out_mode=out_mode,
                                   keep_roots=bool(case["keep"]))
    return canz.SoapHparams(beta1=BETA, beta2=BETA, lr=SOAP_LR, step=SOAP_STEP, refresh=bool(case["refresh"]),
                            max_precond_dim=MAX_PRECOND_DIM, out_mode=out_mode, mom_rot_valid=True,
                            bf16_rotations=bool(case["bf16rot"]))


def prepare(case, seed):
    tp = case["tp"]
    gdt = canz.DT_BF16 if case["grad"] == "bf16" else canz.DT_F32
    odt = canz.DT_BF16 if case["out"].endswith("bf16") else canz.DT_F32
    groups, outputs = [], []
    for rows, cols, mats in _matrices(case, seed):
        grad, out = [], []
        for m in mats:
            grad += _fragments(m["grad"], tp) if tp > 1 else [m["grad"]]
            if "param" in m:
                out.append(m["param"])
            else:
                dt = torch.bfloat16 if odt == canz.DT_BF16 else torch.float32
                out += [torch.zeros(rows, cols // tp, device=DEV, dtype=dt) for _ in range(tp)]
        tab = lambda key: [m[key] for m in mats if key in m]  # noqa: E731
        common = dict(rows=rows, cols=cols, grad=grad, out=out, tp=tp, grad_dtype=gdt, out_dtype=odt)
        if case["op"] == "muon":
            groups.append(canz.Group(mom=tab("mom"), **common))
            outputs.append({"mom": tab("mom"), "out": out})
        elif case["op"] == "shampoo":
            groups.append(canz.ShampooGroup(left=tab("left"), right=tab("right"), lroot=tab("lroot"), rroot=tab("rroot"), **common))
            outputs.append({"left": tab("left"), "right": tab("right"), "out": out})
            if not case["keep"]:
                outputs[-1].update(lroot=tab("lroot"), rroot=tab("rroot"))
        else:
            keys = ("mom", "var", "left", "right", "qleft", "qright", "mom_rot")
            groups.append(canz.SoapGroup(**{k: tab(k) for k in keys}, **common))
            outputs.append({k: tab(k) for k in keys if case["refresh"] or k not in ("qleft", "qright")})
            outputs[-1]["out"] = out
    hp = _hparams(case)
    need = {"muon": canz.canz_muon_workspace_bytes, "shampoo": canz.canz_shampoo_workspace_bytes,
            "soap": canz.canz_soap_workspace_bytes}[case["op"]](groups, hp)
    step = {"muon": canz.canz_muon_step, "shampoo": canz.canz_shampoo_step, "soap": canz.canz_soap_step}[case["op"]]
    return {"step": step, "groups": groups, "hp": hp, "ws": torch.empty(need, dtype=torch.uint8, device=DEV), "ws_bytes": need,
            "outputs": outputs}


def run(state):
    state["step"](state["groups"], state["hp"], state["ws"], state["ws_bytes"], torch.cuda.current_stream().cuda_stream)
    return state["outputs"]


# ------------------------------------------------------------------ work

def _muon_flops(rows, cols):
    m, n = min(rows, cols), max(rows, cols)
    # per Newton-Schulz step: Gram (symmetric: half of 2 m^2 n), its square (symmetric: half of 2 m^3), B X
    return NS_STEPS * (1.0 * m * m * n + 1.0 * m * m * m + 2.0 * m * m * n)


def work(case):
    gb = 2 if case["grad"] == "bf16" else 4
    ob = (2 if case["out"].endswith("bf16") else 4) * (2 if case["out"].startswith("param") else 1)
    nbytes = flops = 0.0
    for count, r, c in _groups(case):
        el = float(r * c)
        if case["op"] == "muon":
            nbytes += count * el * (gb + 8 + ob)
            flops += count * _muon_flops(r, c)
        elif case["op"] == "shampoo":
            # statistics (symmetric), two preconditioning products; a root: four symmetric products per round
            sides = float(r * r + c * c)
            nbytes += count * (el * (gb + ob) + sides * (8 + 4))
            flops += count * (el * (r + c) + 2.0 * el * (r + c))
            if not case["keep"]:
                flops += count * (4.0 * case["iters"] - 3.0) * (float(r) ** 3 + float(c) ** 3)
        else:
            dims = [d for d in (r, c) if d <= MAX_PRECOND_DIM]
            sides = float(sum(d * d for d in dims))
            # gradient, momentum, its rotation, second moment, parameter; statistics and bases
            nbytes += count * (el * (gb + 8 + 8 + 8 + ob) + sides * (8 + 4 + (4 if case["refresh"] else 0)))
            # G into the bases, N' back, statistics (symmetric); refresh: S Q, QR, accumulation of Q, M into the new bases
            flops += count * sum(5.0 * el * d for d in dims)
            if case["refresh"]:
                flops += count * sum((2.0 + 8.0 / 3.0) * float(d) ** 3 + 2.0 * el * d for d in dims)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the path shows against 64 bits."""
    if case["op"] == "muon":
        # bf16 operands through five iterations: 1e-2 of the update; a parameter is several times the update
        return {"rel": 0.03, "max": 0.3} if case["out"].startswith("delta") else {"rel": 0.01, "max": 0.1}
    if case["op"] == "shampoo":
        # fp32 statistics: their rounding, 6e-8 of the largest eigenvalue, against eps in the root; exact roots otherwise
        return {"rel": 2e-6, "max": 1e-4} if case["keep"] else {"rel": 1e-3, "max": 2e-2}
    if case["bf16rot"]:
        return {"rel": 1.3e-2, "max": 0.1} if case["refresh"] else {"rel": 3e-3, "max": 0.05}
    return {"rel": 1e-5, "max": 1e-3} if case["refresh"] else {"rel": 2e-6, "max": 1e-4}


# ------------------------------------------------------------------ 64 bits

def _f32(x):
    """The value a C float carries."""
    return float(torch.tensor(x, dtype=torch.float32))


def _inverse_fourth_root(s, eps):
    """(S + eps I)^(-1/4) in 64 bits: the coupled Newton iteration until it stands still (M -> I)."""
    d = s.shape[0]
    eye = torch.eye(d, device=s.device, dtype=s.dtype)
    a = 0.5 * (s + s.t()) + eps * eye
    z = 2.5 / float(torch.linalg.matrix_norm(a))
    m, x = z * a, z ** 0.25 * eye
    for _ in range(100):
        t = 1.25 * eye - 0.25 * m
        x = x @ t
        t2 = t @ t
        m = (t2 @ t2) @ m
        m = 0.5 * (m + m.t())
        if float((m - eye).abs().max()) < 1e-12:
            break
    return 0.5 * (x + x.t())


def _qr(s):
    return torch.linalg.qr(s.cpu())[0].to(s.device)


def _put(case, tp, m, delta, decay):
    if "param" in m:
        return [m["param"].double() * decay + delta]
    return _fragments(delta, tp)


def exact(case, seed):
    tp = case["tp"]
    if case["op"] == "soap" and case["refresh"] and any(max(r, c) > 2048 for _, r, c in _groups(case)):
        return None   # the QR factors on the host would take too long
    outputs = []
    for rows, cols, mats in _matrices(case, seed):
        got = {}
        add = lambda key, v: got.setdefault(key, []).append(v)  # noqa: E731
        for m in mats:
            g = m["grad"].double()
            if case["op"] == "muon":
                beta, lr = _f32(BETA), _f32(LR)
                mom = beta * m["mom"].double() + g
                u = g + beta * mom if case["nesterov"] else mom
                x = u / (torch.linalg.vector_norm(u) + _f32(1e-7))
                a, b, c = (_f32(v) for v in NS)
                x = x.t().contiguous() if rows > cols else x
                for _ in range(NS_STEPS):
                    gram = x @ x.t()
                    x = a * x + (b * gram + c * (gram @ gram)) @ x
                x = x.t() if rows > cols else x
                scale = 0.2 * math.sqrt(max(rows, cols)) if case["scale"] == 2 else math.sqrt(max(1.0, rows / cols))
                add("mom", mom)
                got.setdefault("out", []).extend(_put(case, tp, m, -lr * scale * x, 1.0 - lr * _f32(case["wd"])))
            elif case["op"] == "shampoo":
                beta, lr, eps = _f32(BETA), _f32(LR), _f32(_shampoo_eps(case))
                left = beta * m["left"].double() + g @ g.t()
                right = beta * m["right"].double() + g.t() @ g
                lroot = m["lroot"].double() if case["keep"] else _inverse_fourth_root(left, eps)
                rroot = m["rroot"].double() if case["keep"] else _inverse_fourth_root(right, eps)
                add("left", left)
                add("right", right)
                if not case["keep"]:
                    add("lroot", lroot)
                    add("rroot", rroot)
                got.setdefault("out", []).extend(_put(case, tp, m, -lr * (lroot @ g @ rroot), 1.0))
            else:
                b1, lr, eps = _f32(BETA), _f32(SOAP_LR), _f32(1e-8)
                ql = m["qleft"].double() if "qleft" in m else None
                qr = m["qright"].double() if "qright" in m else None

                def into(x, ql_, qr_):
                    x = x if ql_ is None else ql_.t() @ x
                    return x if qr_ is None else x @ qr_

                mom = b1 * m["mom"].double() + (1.0 - b1) * g
                g_rot = into(g, ql, qr)
                m_rot = b1 * m["mom_rot"].double() + (1.0 - b1) * g_rot
                var = b1 * m["var"].double() + (1.0 - b1) * g_rot * g_rot
                c = 1.0 / (1.0 - b1 ** SOAP_STEP)
                n = (c * m_rot) / ((c * var).sqrt() + eps)
                n = n if qr is None else n @ qr.t()
                n = n if ql is None else ql @ n
                add("mom", mom)
                add("var", var)
                if ql is not None:
                    left = b1 * m["left"].double() + (1.0 - b1) * (g @ g.t())
                    add("left", left)
                if qr is not None:
                    right = b1 * m["right"].double() + (1.0 - b1) * (g.t() @ g)
                    add("right", right)
                if case["refresh"]:
                    if ql is not None:
                        ql = _qr(left @ ql)
                        add("qleft", ql)
                    if qr is not None:
                        qr = _qr(right @ qr)
                        add("qright", qr)
                    m_rot = into(mom, ql, qr)
                add("mom_rot", m_rot)
                got.setdefault("out", []).extend(_put(case, tp, m, -lr * n, 1.0))
        outputs.append(got)
    return outputs
