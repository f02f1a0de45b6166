"""What users have this library do, as cases that can be timed and compared.

A case is one pass through the public entry points on one problem.  Four families of problems,
the ones the method is used on: small dense instances, FIR filter design (dense, fp64), discrete
tomography (CSR) and weight quantisation (a batch of rows that share the calibration matrix); and
the calls users make on them: the descent, the outer loop (destroy, repair, local search), the swap
search, the l2 changes, and the same iteration taken one entry point at a time.

All inputs are made on the GPU from the seed alone and do not depend on the order of a floating-point
sum: targets are sums of fixed-point numbers that fit their accumulator exactly.

    listed()            the cases, smallest to largest problem of each family among them
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs and handle, on the GPU
    run(state)          one pass, its outputs whole
    work(case)          bytes and flops one pass cannot do without
    tolerance(case)     every output is fixed bit for bit by the library's arithmetic contract
    exact(case, seed)   the computed numbers in 64 bits with plain torch, where they are functions of
                        the inputs alone (a descent's are functions of the moves it took)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2508_13437_amd import dmmv

DEVICE = "cuda:0"


# --------------------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------------------
def listed():
    return [
        # a small dense instance from a random start: latency of a call and of an iteration
        dict(name="dense_small_descent", family="dense", call="descent", dtype="f64", m=256, n=64, nd=16,
             iters=200, prune=False),
        # FIR low-pass with 10-bit coefficients, from a window design rounded to 7 bits
        dict(name="fir_descent", family="fir", call="descent", dtype="f64", m=4096, n=32, nd=1024,
             iters=500, prune=False),
        # a long filter (order 500: 251 free coefficients, 16 grid points per tap) with 8-bit
        # coefficients, under the outer loop
        dict(name="fir_long_alns", family="fir", call="alns", dtype="f64", m=8016, n=251, nd=256,
             iters=12, moves=8, prune=False),
        # tomography 256 x 256, 180 angles x 363 bins, three levels: descent with default options
        dict(name="tomo_descent", family="tomo", call="descent", dtype="f32", size=256, angles=180, bins=363,
             levels=3, iters=300, prune=False),
        # tomography 128 x 128, 64 angles x 128 bins, four grey levels: ten outer iterations
        dict(name="tomo_alns", family="tomo", call="alns", dtype="f32", size=128, angles=64, bins=128,
             levels=4, iters=10, moves=8, prune=True),
        # one iteration of the method taken call by call, fp64, odd sizes
        dict(name="tomo_f64_step", family="tomo", call="step", dtype="f64", size=187, angles=101, bins=265,
             levels=3, prune=False),
        # 20 rows of a small layer (768 features), 3 bits, under the outer loop: few instances
        # at a time
        dict(name="llm_rows_alns", family="llm", call="alns", dtype="f32", m=2048, n=768, R=20, bits=3,
             iters=10, moves=8, prune=True),
        # a whole linear layer, 4 bits: every row to its local optimum
        dict(name="llm_layer_descent", family="llm", call="descent", dtype="f32", m=2048, n=4096, R=4096, bits=4,
             iters=100, prune=True),
        # part of the layer under the outer loop
        dict(name="llm_layer_alns", family="llm", call="alns", dtype="f32", m=2048, n=4096, R=1024, bits=4,
             iters=4, moves=4, prune=True),
        # one iteration call by call with the whole score table, a ragged number of rows, 4 bits
        dict(name="llm_step", family="llm", call="step", dtype="f32", m=2048, n=4096, R=500, bits=4, prune=False),
        # MLP-shaped, 3 bits: residual, l2 changes and the best move that keeps the l2 norm down
        dict(name="llm_mlp_guarded", family="llm", call="guarded", dtype="f32", m=4096, n=4096, R=1376, bits=3,
             prune=False),
        # best exchange of two variables' values, every row of part of a layer
        dict(name="llm_swap", family="llm", call="swap", dtype="f32", m=2048, n=4096, R=512, bits=4, prune=False),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["dense", "fir", "tomo", "tomo", "llm", "llm", "llm"])
    if family == "dense":
        return dict(family=family, call=rng.choice(["descent", "alns", "step", "swap"]),
                    dtype=rng.choice(["f64", "f32"]), m=_log_uniform(rng, 64, 2048), n=_log_uniform(rng, 16, 512),
                    nd=_log_uniform(rng, 2, 64), iters=rng.randint(20, 200), moves=rng.randint(1, 8),
                    prune=rng.random() < 0.5)
    if family == "fir":
        n = _log_uniform(rng, 8, 251)
        call = rng.choice(["descent", "alns", "step"])
        return dict(family=family, call=call, dtype="f64", m=max(256, min(8192, n * rng.randint(32, 128))), n=n,
                    nd=2 ** rng.randint(4, 10 if n <= 64 else 8),
                    iters=rng.randint(50, 300) if call == "descent" else rng.randint(4, 12),
                    moves=rng.randint(1, 8), prune=False)
    if family == "tomo":
        size = _log_uniform(rng, 24, 256)
        call = rng.choice(["descent", "alns", "step"])
        dtype = "f32" if rng.random() < 0.75 else "f64"
        return dict(family=family, call=call, dtype=dtype, size=size,
                    angles=rng.randint(max(8, size // 4), max(12, (7 * size) // 10)),
                    bins=rng.randint(size, int(1.42 * size) + 1), levels=rng.choice([2, 3, 4]),
                    iters=rng.randint(20, 200) if call == "descent" else rng.randint(4, 10),
                    moves=rng.randint(1, 8), prune=rng.random() < 0.5)
    call = rng.choice(["descent", "alns", "step", "guarded", "swap"])
    m, n, bits = _log_uniform(rng, 256, 4096), _log_uniform(rng, 128, 4096), rng.choice([2, 3, 4])
    top = {"descent": 4096, "alns": 1024, "step": 500, "guarded": 1376, "swap": 512}[call]
    size = n * n if call == "swap" else m * n                # as much work as the listed case at most
    room = {"descent": 2048, "alns": 2048, "step": 2048, "guarded": 4096, "swap": 4096}[call] * 4096 * top // size
    return dict(family=family, call=call, dtype="f32", m=m, n=n, R=max(4, min(_log_uniform(rng, 8, top), room)),
                bits=bits, iters=rng.randint(20, 100) if call == "descent" else rng.randint(2, 4),
                moves=rng.randint(1, 4), prune=call in ("descent", "alns"))


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _levels(case):
    """The value set D, ascending."""
    if case["family"] == "tomo":
        return {2: [0.0, 1.0], 3: [0.0, 0.5, 1.0], 4: [0.0, 85.0, 170.0, 255.0]}[case["levels"]]
    nd = 2 ** case["bits"] if case["family"] == "llm" else case["nd"]
    return [float(v - nd // 2) for v in range(nd)]


# --------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------
def _fixed(v, bits):
    """v rounded to a multiple of 2^-bits (sums of products of such numbers are exact in fp64)."""
    return torch.round(v * 2.0 ** bits) * 2.0 ** -bits


def _dense_inputs(case, g):
    m, n, nd = case["m"], case["n"], case["nd"]
    A = _fixed(torch.randn(n, m, generator=g, device=DEVICE, dtype=torch.float64), 18)
    lo = -(nd // 2)
    xs = torch.randint(lo, lo + nd, (n,), generator=g, device=DEVICE).double()
    noise = _fixed(torch.rand(m, generator=g, device=DEVICE, dtype=torch.float64) - 0.5, 18)
    b = xs @ A + noise
    x0 = torch.randint(lo, lo + nd, (n,), generator=g, device=DEVICE).double()
    return A, b, x0


def _fir_inputs(case, g):
    """Low-pass of random band edges: A_kj = 2 cos(w_k j), target D_max on the passband and 0 on the
    stopband, starting from the window design rounded to 7 bits (a coarse filter being refined)."""
    m, n, half = case["m"], case["n"], case["nd"] // 2
    u = torch.rand(2, generator=g, device=DEVICE, dtype=torch.float64).tolist()
    w_pass = (0.15 + 0.15 * u[0]) * math.pi
    w_stop = w_pass + (1.0 + u[1]) * 2.0 * math.pi / (2 * n)
    m_pass = int(round(m * w_pass / (w_pass + math.pi - w_stop)))
    w = torch.cat([torch.linspace(0.0, w_pass, m_pass, dtype=torch.float64),
                   torch.linspace(w_stop, math.pi, m - m_pass, dtype=torch.float64)]).to(DEVICE)
    j = torch.arange(n, device=DEVICE, dtype=torch.float64)
    A = 2.0 * torch.cos(torch.outer(j, w))                        # row j = column j of the matrix
    b = torch.cat([torch.full((m_pass,), float(half)), torch.zeros(m - m_pass)]).double().to(DEVICE)
    wc = 0.5 * (w_pass + w_stop)
    jj = np.arange(1, n, dtype=np.float64)
    h = np.concatenate([[wc / (2.0 * math.pi)], np.sin(wc * jj) / (math.pi * jj)])
    h *= 0.54 + 0.46 * np.cos(math.pi * np.arange(n) / n)
    coarse = max(1, case["nd"] // 128)
    x0 = torch.from_numpy(np.clip(np.rint(half * h / coarse) * coarse, -half, half - 1)).to(DEVICE)
    return A, b, x0


def _phantom(case, g):
    """Eight random ellipses of random grey levels, as level indices."""
    size, nl = case["size"], case["levels"]
    u = torch.rand(8, 6, generator=g, device=DEVICE, dtype=torch.float64).tolist()
    c = (size - 1) / 2.0
    ax = torch.arange(size, device=DEVICE, dtype=torch.float64)
    yy, xx = ax[:, None], ax[None, :]
    img = torch.zeros(size, size, device=DEVICE, dtype=torch.int64)
    for e, (u0, u1, u2, u3, u4, u5) in enumerate(u):
        rad, ang, th = u0 * 0.55 * size / 2.0, u1 * 2 * math.pi, u4 * math.pi
        cx, cy = c + rad * math.cos(ang), c + rad * math.sin(ang)
        sx, sy = (10 + 35 * u2) * size / 256.0, (10 + 35 * u3) * size / 256.0
        p = (xx - cx) * math.cos(th) + (yy - cy) * math.sin(th)
        q = -(xx - cx) * math.sin(th) + (yy - cy) * math.cos(th)
        img = torch.where((p / sx) ** 2 + (q / sy) ** 2 <= 1.0, 1 + (e + int(u5 * 8)) % (nl - 1), img)
    return img


def _tomo_matrix(case, first_angle):
    """Parallel-beam projection matrix as CSR: row = angle * bins + bin, column = pixel, entry = exact
    chord length of a unit-spaced ray through a unit pixel (a trapezoid in the ray's offset)."""
    size, angles, bins = case["size"], case["angles"], case["bins"]
    c0, mid = (size - 1) / 2.0, (bins - 1) // 2
    pix = torch.arange(size * size, device=DEVICE)
    px, py = (pix % size).double() - c0, (pix // size).double() - c0
    keys, vals = [], []
    for a in range(angles):
        t = first_angle + a * math.pi / angles
        ac, sn = abs(math.cos(t)), abs(math.sin(t))
        w1, w2, top = 0.5 * (ac + sn), 0.5 * abs(ac - sn), 1.0 / max(ac, sn)
        p = px * math.cos(t) + py * math.sin(t)
        base = torch.floor(p).long()
        for off in (-1, 0, 1, 2):
            s = base + off
            d = (s.double() - p).abs()
            ln = (top * ((w1 - d) / max(w1 - w2, 1e-12)).clamp(0.0, 1.0)).to(_dtype(case))
            ok = (ln > 0) & (s + mid >= 0) & (s + mid < bins)
            keys.append(((a * bins + s + mid)[ok]) * (size * size) + pix[ok])
            vals.append(ln[ok])
    key, order = torch.sort(torch.cat(keys))
    val = torch.cat(vals)[order].contiguous()
    m, n = angles * bins, size * size
    row = torch.div(key, n, rounding_mode="floor")
    col = (key - row * n).to(torch.int32)
    rowptr = torch.zeros(m + 1, dtype=torch.int64, device=DEVICE)
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=m), 0)
    return rowptr, col, val, row


def _tomo_inputs(case, g):
    size = case["size"]
    first = float(torch.rand(1, generator=g, device=DEVICE, dtype=torch.float64)) * math.pi / case["angles"]
    rowptr, col, val, row = _tomo_matrix(case, first)
    img = _phantom(case, g)
    D = torch.tensor(_levels(case), device=DEVICE, dtype=torch.float64)
    # A x* in integers (entries to 2^-30, levels to 2^-1): the sum does not depend on its order
    iv = torch.round(val.double() * 2.0 ** 30).long() * torch.round(D * 2).long()[img.reshape(-1)][col.long()]
    m = case["angles"] * case["bins"]
    clean = torch.zeros(m, dtype=torch.int64, device=DEVICE).index_add_(0, row, iv).double() * 2.0 ** -31
    noise = (torch.rand(m, generator=g, device=DEVICE, dtype=torch.float64) * 2 - 1) * 0.02
    b = clean + noise * clean.max()
    # starting image: the blurred phantom with some noise, rounded to the levels (as a rounded
    # reconstruction has them, the errors sit along the edges)
    blur = torch.nn.functional.avg_pool2d(D[img][None, None], 5, 1, 2, count_include_pad=False)[0, 0]
    blur = blur + D[-1] * 0.08 * torch.randn(size, size, generator=g, device=DEVICE, dtype=torch.float64)
    x0 = D[(blur.reshape(-1, 1) - D[None, :]).abs().argmin(1)]
    return (rowptr, col, val), b, x0


def _llm_inputs(case, g):
    """Calibration activations with heavy tails and 1 % of outlier channels, normal weights, absmax
    scales, round-to-nearest start."""
    m, n, R = case["m"], case["n"], case["R"]
    half = 2 ** (case["bits"] - 1)
    z = torch.randn(n, m, generator=g, device=DEVICE, dtype=torch.float64)
    u = torch.rand(2, n, m, generator=g, device=DEVICE, dtype=torch.float64).clamp_min(1e-12)
    X = z * torch.rsqrt(-(torch.log(u[0]) + torch.log(u[1])) * 0.5)          # Student t, 4 degrees of freedom
    hot = torch.randperm(n, generator=g, device=DEVICE)[:max(1, round(0.01 * n))]
    X[hot] *= 20.0
    X = _fixed(X, 10)                                                         # row j = column j of the matrix
    W = _fixed(torch.randn(R, n, generator=g, device=DEVICE, dtype=torch.float64) * 0.02, 20)
    scale = (W.abs().amax(1) / max(half - 1, 1)).float()
    x0 = torch.round(W / scale.double()[:, None]).clamp(-half, half - 1)
    b = W @ X
    return X, b, x0, scale


def prepare(case, seed):
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    dt = _dtype(case)
    kw = dict(D=_levels(case), prune=bool(case["prune"]))
    if case["family"] == "tomo":
        csr, b, x0 = _tomo_inputs(case, g)
        kw.update(csr=csr, m=case["angles"] * case["bins"], n=case["size"] ** 2, device=DEVICE)
    elif case["family"] == "llm":
        X, b, x0, scale = _llm_inputs(case, g)
        kw.update(A=X.to(dt).t(), scale=scale.cpu().numpy(), alns=case["call"] == "alns")
        if case["call"] == "guarded":
            kw["l2_rule"] = 2
    else:
        A, b, x0 = (_dense_inputs if case["family"] == "dense" else _fir_inputs)(case, g)
        kw["A"] = A.to(dt).t()
    h = dmmv.Handle(b=b.to(dt).contiguous(), **kw)
    state = dict(case=case, seed=seed, h=h, x0=x0.to(dt).contiguous())
    if case["call"] == "swap":                       # the search starts from a residual that is there
        dmmv.dmmv_set_x(h, state["x0"])
        dmmv.dmmv_residual(h)
    return state


# --------------------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------------------
def run(state):
    case, h, x0 = state["case"], state["h"], state["x0"]
    if case["call"] == "descent":
        res = dmmv.dmmv_solve(h, x0, case["iters"], trace=True)
        return {"x": res.x, "r": dmmv.dmmv_get_state(h)[1], "t": res.max_violation, "moves": res.iters_done,
                "trace": res.trace, "trace_t": res.trace_t}
    if case["call"] == "alns":
        res = dmmv.dmmv_alns(h, x0, case["iters"], ls_moves=case["moves"], seed=1 + state["seed"] % 1000)
        x, r, t = dmmv.dmmv_get_state(h)
        return {"x_best": res.x_best, "t_best": res.t_best, "trace": res.trace, "trace_t": res.trace_t,
                "x": x, "r": r, "t": t}
    if case["call"] == "swap":
        sw = dmmv.dmmv_swap_move(h, apply=False)
        return {"i": sw.i, "j": sw.j, "t": sw.t}
    dmmv.dmmv_set_x(h, x0)
    r = dmmv.dmmv_residual(h)
    if case["call"] == "guarded":
        dq = dmmv.dmmv_l2_changes(h)
        best, best_s = dmmv.dmmv_argmin_move(h)
        return {"r": r, "dq": dq, "best": best, "best_score": best_s}
    scores = dmmv.dmmv_eval_moves(h)
    best, best_s = dmmv.dmmv_argmin_move(h, scores)
    dmmv.dmmv_apply_move(h, best)
    x, r_new, t = dmmv.dmmv_get_state(h)
    return {"r": r, "scores": scores, "best": best, "best_score": best_s, "x": x, "r_new": r_new, "t": t}


# --------------------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------------------
def work(case):
    w = 8 if case["dtype"] == "f64" else 4
    R, nd = case.get("R", 1), len(_levels(case))
    if case["family"] == "tomo":
        m, n = case["angles"] * case["bins"], case["size"] ** 2
        # about 1.27 rays of an angle meet a pixel; detectors narrower than the image miss its corners
        entries = 1.27 * case["angles"] * n * min(1.0, case["bins"] / (1.2 * case["size"]))
        matrix = entries * (w + 4) + 8 * (m + 1)
    else:
        m, n = case["m"], case["n"]
        entries = float(m) * n
        matrix = entries * w
    table = R * n * nd * w
    data = matrix + R * (m + 2 * n) * w               # matrix, targets, start, result
    flops = 2.0 * entries * R                         # the residual
    if case["call"] in ("step", "guarded"):
        # a result for every candidate move: each is a maximum (a sum) over all rows
        data += table + R * m * w
        flops += 3.0 * entries * (nd - 1) * R if case["call"] == "step" else 2.0 * entries * R
    elif case["call"] == "swap":
        data, flops = matrix + R * (m + n) * w, 2.0 * R * n * (n - 1)
    elif case["call"] == "alns":
        data += case["iters"] * R * m * w
        flops += 4.0 * case["iters"] * R * (0.005 * entries + m)
    return {"bytes": float(data), "flops": float(flops)}


def tolerance(case):
    # every rounding is fixed (order of the residual's sum, one fused multiply-add per row and move,
    # exact maxima, lowest index among equals), for scores, moves, x, r and the l2 changes alike
    return "exact"


# --------------------------------------------------------------------------------------
# the same numbers in 64 bits
# --------------------------------------------------------------------------------------
def exact(case, seed):
    if case["call"] not in ("step", "guarded"):
        return None                                   # what comes out depends on the moves taken on the way
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    dt = _dtype(case)
    D = torch.tensor(_levels(case), device=DEVICE, dtype=torch.float64)
    if case["family"] == "tomo":
        (rowptr, col, val), b, x0 = _tomo_inputs(case, g)
        return _exact_sparse(case, D, rowptr, col.long(), val.double(), b.to(dt).double(), x0.double())
    if case["family"] == "llm":
        X, b, x0, scale = _llm_inputs(case, g)
        At, s = X.to(dt).double(), scale.double()
    else:
        At, b, x0 = (_dense_inputs if case["family"] == "dense" else _fir_inputs)(case, g)
        At, s = At.to(dt).double(), torch.ones(1, device=DEVICE, dtype=torch.float64)
    b, x0 = b.to(dt).double().reshape(len(s), -1), x0.reshape(len(s), -1)
    r = (x0 @ At) * s[:, None] - b                    # [R][m]
    step = s[:, None, None] * (D[None, None, :] - x0[:, :, None])      # [R][n][nd]
    squeeze = (lambda v: v.reshape(v.shape[0], -1)) if case["family"] == "llm" else (lambda v: v.reshape(-1))
    if case["call"] == "guarded":
        gq = r @ At.t()                               # [R][n]
        dq = step * (2.0 * gq[:, :, None] + step * (At * At).sum(1)[None, :, None])
        return {"r": squeeze(r), "dq": squeeze(dq), "best": None, "best_score": None}
    if float(r.numel()) * At.shape[0] * D.numel() > 2.0e11:
        return None
    scores = torch.zeros_like(step)
    rows = max(1, int(2 ** 27 // max(step.numel(), 1)))
    for i0 in range(0, r.shape[1], rows):
        a = At[:, i0:i0 + rows].t()[None]             # [1][rows][n]
        v = torch.addcmul(r[:, i0:i0 + rows, None, None], a[..., None], step[:, None])
        scores = torch.maximum(scores, v.abs_().amax(1))
    best = scores.reshape(len(s), -1).amin(1)
    return {"r": squeeze(r), "scores": squeeze(scores), "best": None, "best_score": best, "x": None,
            "r_new": None, "t": best}


def _exact_sparse(case, D, rowptr, col, val, b, x0):
    m, n = b.numel(), x0.numel()
    row = torch.repeat_interleave(torch.arange(m, device=DEVICE), rowptr[1:] - rowptr[:-1])
    r = torch.zeros(m, device=DEVICE, dtype=torch.float64).index_add_(0, row, val * x0[col]) - b
    # largest |r| among the rows without an entry in a column: the largest |r| it does not hold
    top = torch.topk(r.abs(), min(m, 4096))
    rank = torch.full((m,), m, device=DEVICE, dtype=torch.int64)
    rank[top.indices] = torch.arange(top.indices.numel(), device=DEVICE)
    order = torch.argsort(col * (m + 1) + rank[row])
    c, k = col[order], rank[row][order]
    first = torch.searchsorted(c, torch.arange(n, device=DEVICE))
    held = (k == torch.arange(c.numel(), device=DEVICE) - first[c]) & (k < top.indices.numel())
    # a column holds the ranks 0 .. p - 1 exactly when its p smallest ranks are 0 .. p - 1
    count = torch.zeros(n, device=DEVICE, dtype=torch.int64).index_add_(0, c, held.long())
    if int(count.max()) >= top.indices.numel():
        return None
    outside = top.values[count]
    scores = torch.empty(n, D.numel(), device=DEVICE, dtype=torch.float64)
    for q in range(D.numel()):
        v = (r[row] + (D[q] - x0[col]) * val).abs()
        scores[:, q] = torch.maximum(outside, torch.zeros(n, device=DEVICE, dtype=torch.float64)
                                     .scatter_reduce(0, col, v, "amax"))
    best = scores.min().reshape(1)
    return {"r": r, "scores": scores.reshape(-1), "best": None, "best_score": best, "x": None, "r_new": None,
            "t": best}
