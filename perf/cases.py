"""The work that a user of this library has it do, as cases that can be timed.

Every case goes through the package's public entry points on seeded inputs of
the kind the synthetic workloads draw (T_ij ~ CN(0, 1)/sqrt(m), noise variances
in [0.5, 2], an eighth of the coefficients foreground with variance 1e4, theta
uniform in the prior box [-1, 3]).

  listed()             the cases, smallest to largest of each path
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  inputs on the GPU (host arrays for the out-of-core path)
                       and the handles a program keeps: the precomputed
                       context, the group, the surrogate
  run(state)           one pass; returns the outputs whole
  work(case)           bytes and operations a pass cannot do without
  exact(case, seed)    the outputs in 64 bits by plain torch, where that takes
                       seconds

Kinds of case, and what they stand for:
  loglike    theta batches of one dataset: from one theta of a chain or an audit,
             through the remainder of a batch, to the sampler's full batches
  group      uneven sub-bands evaluated in one call
  precompute a new dataset: A, dbar and the scalars, in FP64 or a reduced
             precision of the A product
  step       loss and gradient of one training minibatch of the ensemble
  gate       the ensemble's prediction for proposals, as the sampler asks for it
  forward    T from a beam, baselines and a Fourier basis
  ooc        logL with A in host memory and a bounded device window
"""
import math

import numpy as np
import torch

import paper_2501_12928_amd as eor

LO, HI = -1.0, 3.0   # prior box
FG_VAR = 1.0e4       # prior variance of the foreground coefficients
C_LIGHT = 299792458.0


def listed():
    return [
        # one step of a chain on the smallest workload (480 x 200): latency
        {"name": "chain_n200", "kind": "loglike", "m": 480, "n": 200, "n_k": 3, "B": 1},
        # a few theta of a ragged medium problem: what a shrinking batch or an audit leaves
        {"name": "few_n1003_B24", "kind": "loglike", "m": 3000, "n": 1003, "n_k": 6, "B": 24},
        # one theta at the full size: a chain step or a check of a single point
        {"name": "one_n4096", "kind": "loglike", "m": 20000, "n": 4096, "n_k": 12, "B": 1},
        # the plain batched workload
        {"name": "batch_n2048_B256", "kind": "loglike", "m": 8000, "n": 2048, "n_k": 8, "B": 256},
        # the headline batch of the sampler
        {"name": "batch_n4096_B512", "kind": "loglike", "m": 20000, "n": 4096, "n_k": 12, "B": 512},
        # uneven sub-bands in one call
        {"name": "group_12", "kind": "group", "n_inst": 12, "n_lo": 256, "n_hi": 2048, "th_lo": 16, "th_hi": 64,
         "shape_seed": 1002},
        # a new dataset at the full size, and the split-BF16 product at the plain batched size
        {"name": "pre_fp64_20000x4096", "kind": "precompute", "m": 20000, "n": 4096, "n_k": 12, "prec": "fp64"},
        {"name": "pre_bf16x3_8000x2048", "kind": "precompute", "m": 8000, "n": 2048, "n_k": 8, "prec": "bf16x3"},
        # one minibatch of the surrogate's training
        {"name": "step_nb512", "kind": "step", "nb": 512, "n_in": 12, "H": 256, "M": 5},
        # screening a million proposals
        {"name": "gate_1e6", "kind": "gate", "B": 1000000, "n_in": 12, "H": 256, "M": 5},
        # T of the synthetic instrument, 20000 x 4096
        {"name": "forward_20000x4096", "kind": "forward", "F": 32, "n_bl": 625, "n_side": 64, "kx": 16, "ky": 8,
         "n_eta": 32},
        # Sigma through a bounded device window, A in host memory
        {"name": "ooc_n3000_B4", "kind": "ooc", "n": 3000, "n_k": 8, "B": 4, "mib": 128},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["loglike", "loglike", "loglike", "loglike", "group", "precompute", "precompute", "step", "gate",
                       "forward", "ooc"])
    if kind == "loglike":
        n = _log_int(rng, 64, 4096)
        B = min(_log_int(rng, 1, 512), int(512 * (4096 / n) ** 2))
        return {"kind": kind, "m": int(n * rng.uniform(2.0, 4.8)), "n": n, "n_k": rng.randint(1, 12), "B": B}
    if kind == "group":
        return {"kind": kind, "n_inst": rng.randint(2, 16), "n_lo": 256, "n_hi": _log_int(rng, 600, 2500),
                "th_lo": 4, "th_hi": rng.randint(16, 64), "shape_seed": rng.randrange(1 << 30)}
    if kind == "precompute":
        n = _log_int(rng, 200, 4096)
        return {"kind": kind, "m": min(20000, int(n * rng.uniform(2.0, 8.0))), "n": n, "n_k": rng.randint(1, 12),
                "prec": rng.choice(["fp64", "fp64", "fp32", "bf16x3", "bf16x2"])}
    if kind == "step":
        return {"kind": kind, "nb": _log_int(rng, 64, 2048), "n_in": rng.randint(4, 16),
                "H": 4 * rng.randint(16, 96), "M": rng.randint(3, 8)}
    if kind == "gate":
        return {"kind": kind, "B": _log_int(rng, 256, 1000000), "n_in": rng.randint(4, 16),
                "H": 4 * rng.randint(16, 96), "M": rng.randint(3, 8)}
    if kind == "forward":
        return {"kind": kind, "F": rng.randint(2, 32), "n_bl": _log_int(rng, 40, 625), "n_side": rng.randint(16, 64),
                "kx": rng.randint(4, 16), "ky": rng.randint(4, 9), "n_eta": rng.randint(4, 32)}
    n = _log_int(rng, 400, 4096)
    N = (n + 63) // 64
    return {"kind": kind, "n": n, "n_k": rng.randint(1, 12), "B": rng.randint(1, 6),
            "mib": max(24, N * rng.randint(2, 6))}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _cn(g, *shape):
    return torch.randn(*shape, dtype=torch.complex128, device="cuda", generator=g)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)


def _bins(n, n_k):
    """Contiguous balanced bins over the EoR coefficients, -1 for the foreground."""
    n_eor = n - n // 8
    j = np.arange(n, dtype=np.int64)
    b = (j * n_k) // n_eor
    b[j >= n_eor] = -1
    b = b.astype(np.int32)
    return b, np.where(b < 0, FG_VAR, 0.0)


def _dataset(g, m, n, n_k):
    T = _cn(g, m, n) / math.sqrt(m)
    nv = _uniform(g, 0.5, 2.0, m)
    bins, fixed = _bins(n, n_k)
    star = np.linspace(0.5, 1.5, n_k)
    phi = torch.from_numpy(np.where(bins >= 0, 10.0 ** star[np.maximum(bins, 0)], fixed)).cuda()
    a = _cn(g, n) * phi.sqrt()
    d = T @ a + _cn(g, m) * nv.sqrt()
    return T, nv, d, bins, fixed


def _group_shapes(case):
    r = np.random.default_rng(case["shape_seed"])
    return [(int(r.integers(case["n_lo"], case["n_hi"] + 1)), int(r.integers(case["th_lo"], case["th_hi"] + 1)),
             int(r.integers(4, 13))) for _ in range(case["n_inst"])]


def _weights(g, case, spread):
    """Ensemble weights as training leaves them: He-normal scale, members near
    a common network (relative distance `spread`)."""
    n_in, H, M = case["n_in"], case["H"], case["M"]
    P = H * n_in + H + H * H + H + H + 1
    sd = torch.full((P,), 0.05, device="cuda")
    o = H * n_in
    sd[:o] = math.sqrt(2.0 / n_in)
    sd[o + H:o + H + H * H] = math.sqrt(2.0 / H)
    sd[o + 2 * H + H * H:o + 3 * H + H * H] = math.sqrt(2.0 / H)
    base = torch.randn(1, P, device="cuda", generator=g)
    own = torch.randn(M, P, device="cuda", generator=g)
    return ((base + spread * own) / math.sqrt(1.0 + spread * spread) * sd).contiguous()


def _instrument(case, g):
    F, n_bl, side = case["F"], case["n_bl"], case["n_side"]
    freq = 150e6 + 100e3 * torch.arange(F, dtype=torch.float64, device="cuda")
    r = 60.0 * torch.sqrt(_uniform(g, (14.6 / 60.0) ** 2, 1.0, n_bl))
    ang = _uniform(g, 0.0, 2.0 * math.pi, n_bl)
    bl = torch.stack([r * torch.cos(ang), r * torch.sin(ang)], dim=1).contiguous()
    delta = 0.3 / side
    x = (torch.arange(side, dtype=torch.float64, device="cuda") - side // 2) * delta
    lm = torch.stack([x.repeat(side), x.repeat_interleave(side)], dim=1).contiguous()
    sigma = 1.03 * (C_LIGHT / freq) / 14.0 / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    beam = torch.exp(-(lm ** 2).sum(1)[None, :] / (2.0 * sigma[:, None] ** 2)).contiguous()
    du = 1.0 / (side * delta)
    ix = torch.arange(case["kx"], dtype=torch.float64, device="cuda") - case["kx"] // 2
    iy = torch.arange(case["ky"], dtype=torch.float64, device="cuda") - case["ky"] // 2
    uv = torch.stack([ix.repeat_interleave(case["ky"]) * du, iy.repeat(case["kx"]) * du], dim=1).contiguous()
    e = torch.arange(case["n_eta"], dtype=torch.float64, device="cuda") - case["n_eta"] // 2
    ph = 2.0 * math.pi * torch.arange(F, dtype=torch.float64, device="cuda")[:, None] * e[None, :] / F
    Z = torch.complex(torch.cos(ph), torch.sin(ph)).contiguous()
    return freq, bl, lm, beam, uv, Z, 1.0 / (side * side)


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = {"case": case}
    if kind == "loglike":
        T, nv, d, bins, fixed = _dataset(g, case["m"], case["n"], case["n_k"])
        s["ctx"] = eor.Context(0).precompute(T, nv, d, case["n_k"], bins, fixed)
        s["theta"] = _uniform(g, LO, HI, case["B"], case["n_k"])
    elif kind == "group":
        s["ctx"], s["theta"], s["outs"] = [], [], (None, None)
        for n, B, n_k in _group_shapes(case):
            T, nv, d, bins, fixed = _dataset(g, 4 * n, n, n_k)
            s["ctx"].append(eor.Context(0).precompute(T, nv, d, n_k, bins, fixed))
            s["theta"].append(_uniform(g, LO, HI, B, n_k))
        s["group"] = eor.Group(s["ctx"])
    elif kind == "precompute":
        s["data"] = _dataset(g, case["m"], case["n"], case["n_k"])
        s["ctx"] = eor.Context(0)
    elif kind == "step":
        s["net"] = eor.Surrogate(case["n_in"], LO, HI, n_members=case["M"], hidden=case["H"], seed=1)
        s["net"].set_params(_weights(g, case, 1.0))
        s["x"] = 2.0 * torch.rand(case["M"], case["nb"], case["n_in"], device="cuda", generator=g) - 1.0
        s["y"] = torch.randn(case["M"], case["nb"], device="cuda", generator=g)
    elif kind == "gate":
        s["net"] = eor.Surrogate(case["n_in"], LO, HI, n_members=case["M"], hidden=case["H"], seed=1)
        s["net"].set_params(_weights(g, case, 0.02))
        s["net"].standardisation((0.25, 0.5))
        s["theta"] = _uniform(g, LO, HI, case["B"], case["n_in"])
    elif kind == "forward":
        s["args"] = _instrument(case, g)
        F, n_bl = case["F"], case["n_bl"]
        s["T"] = torch.empty((F * n_bl, case["n_eta"] * case["kx"] * case["ky"]), dtype=torch.complex128, device="cuda")
    else:
        n, n_k = case["n"], case["n_k"]
        T, nv, d, bins, fixed = _dataset(g, 2 * n, n, n_k)
        A, dbar, c, K0 = _products(T, nv, d)
        s["host"] = (A.cpu().numpy(), dbar.cpu().numpy(), float(c), float(K0), n_k, bins, fixed, None,
                     _uniform(g, LO, HI, case["B"], n_k).cpu().numpy(), case["mib"] << 20)
    return s


def run(state):
    kind = state["case"]["kind"]
    if kind == "loglike":
        return state["ctx"].loglike_batch(state["theta"])
    if kind == "group":
        state["outs"] = state["group"].loglike(state["theta"], outs=state["outs"][0], infos=state["outs"][1])
        return state["outs"]
    if kind == "precompute":
        T, nv, d, bins, fixed = state["data"]
        ctx = state["ctx"].precompute(T, nv, d, state["case"]["n_k"], bins, fixed, prec=state["case"]["prec"])
        return ctx.export_precompute()
    if kind == "step":
        return state["net"].loss_grad(state["x"], state["y"])
    if kind == "gate":
        return state["net"].gate(state["theta"], -math.inf, 0.05)
    if kind == "forward":
        return eor.forward_model(*state["args"], out=state["T"])
    return eor.loglike_host(*state["host"])


# ------------------------------------------------------- work and 64 bits

def _like_work(n, B, n_k):
    return {"bytes": 8 * n * (n + 1) + 16 * n + 8 * B * (n_k + 1) + 4 * B, "flops": B * (4.0 / 3.0 * n ** 3 + 4.0 * n * n)}


def _net_params(case):
    n_in, H = case["n_in"], case["H"]
    return H * n_in + H + H * H + H + H + 1


def work(case):
    kind = case["kind"]
    if kind == "loglike":
        return _like_work(case["n"], case["B"], case["n_k"])
    if kind == "group":
        w = [_like_work(n, B, n_k) for n, B, n_k in _group_shapes(case)]
        return {"bytes": sum(x["bytes"] for x in w), "flops": sum(x["flops"] for x in w)}
    if kind == "precompute":
        m, n = case["m"], case["n"]
        return {"bytes": 16 * m * n + 24 * m + 16 * n * n + 16 * n, "flops": 4.0 * m * n * n + 8.0 * m * n}
    if kind == "step":
        M, nb, P = case["M"], case["nb"], _net_params(case)
        return {"bytes": 4 * M * (2 * P + nb * (case["n_in"] + 1)), "flops": 6.0 * M * nb * P}
    if kind == "gate":
        M, B, P = case["M"], case["B"], _net_params(case)
        return {"bytes": 4 * M * P + 8 * B * case["n_in"] + 20 * B, "flops": 2.0 * M * B * P}
    if kind == "forward":
        F, n_bl, n_pix, n_uv = case["F"], case["n_bl"], case["n_side"] ** 2, case["kx"] * case["ky"]
        rows = F * n_bl
        return {"bytes": 16 * rows * n_uv * case["n_eta"] + 8 * (F * n_pix + 2 * n_pix),
                "flops": 8.0 * rows * n_pix * n_uv + 8.0 * rows * n_uv * case["n_eta"]}
    return _like_work(case["n"], case["B"], case["n_k"])


def _products(T, nv, d):
    W = T.conj() / nv[:, None]
    A = W.t() @ T
    dbar = (W.t() @ d[:, None])[:, 0]
    c = ((d.conj() * d).real / nv).sum()
    K0 = -T.shape[0] * math.log(math.pi) - nv.log().sum()
    A = 0.5 * (A + A.conj().t())
    return A, dbar, c, K0


def _loglike(A, dbar, c, K0, bins, fixed, theta):
    b = torch.from_numpy(bins.astype(np.int64)).cuda()
    fv = torch.from_numpy(fixed).cuda()
    out = []
    for th in theta:
        phi = torch.where(b >= 0, 10.0 ** th[b.clamp(min=0)], fv)
        S = A + torch.diag((1.0 / phi).to(torch.complex128))
        L = torch.linalg.cholesky(S)
        y = torch.linalg.solve_triangular(L, dbar[:, None], upper=False)
        out.append(K0 - phi.log().sum() - 2.0 * torch.diagonal(L).real.log().sum() - (c - (y.conj() * y).real.sum()))
    return torch.stack(out)


def _net(p, case, x):
    """Outputs [nb] of one member (flat parameters p, 64 bits) at x [nb, n_in]."""
    n_in, H = case["n_in"], case["H"]
    W1, b1, W2, b2, W3, b3 = torch.split(p, [H * n_in, H, H * H, H, H, 1])
    h = torch.nn.functional.gelu(x @ W1.view(H, n_in).t() + b1)
    h = torch.nn.functional.gelu(h @ W2.view(H, H).t() + b2)
    return h @ W3 + b3


def exact(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind in ("loglike", "ooc"):
        n, B, n_k = case["n"], case["B"], case["n_k"]
        if B * n ** 3 > 64 * 4096 ** 3:
            return None
        T, nv, d, bins, fixed = _dataset(g, case.get("m", 2 * n), n, n_k)
        theta = _uniform(g, LO, HI, B, n_k)
        return [_loglike(*_products(T, nv, d), bins, fixed, theta), None]
    if kind == "group":
        outs = []
        for n, B, n_k in _group_shapes(case):
            T, nv, d, bins, fixed = _dataset(g, 4 * n, n, n_k)
            outs.append(_loglike(*_products(T, nv, d), bins, fixed, _uniform(g, LO, HI, B, n_k)))
        return [outs, [None for _ in outs]]
    if kind == "precompute":
        T, nv, d, bins, fixed = _dataset(g, case["m"], case["n"], case["n_k"])
        A, dbar, c, K0 = _products(T, nv, d)
        return [A, dbar, float(c), float(K0)]
    if kind == "step":
        M, nb = case["M"], case["nb"]
        w = _weights(g, case, 1.0).double()
        x = (2.0 * torch.rand(M, nb, case["n_in"], device="cuda", generator=g) - 1.0).double()
        y = torch.randn(M, nb, device="cuda", generator=g).double()
        loss, grad = [], []
        for z in range(M):
            p = w[z].clone().requires_grad_(True)
            v = ((_net(p, case, x[z]) - y[z]) ** 2).mean()
            v.backward()
            loss.append(v.detach())
            grad.append(p.grad)
        return [torch.stack(loss), torch.stack(grad)]
    if kind == "gate":
        w = _weights(g, case, 0.02).double()
        theta = _uniform(g, LO, HI, case["B"], case["n_in"])
        x = 2.0 * (theta - LO) / (HI - LO) - 1.0
        mean, spread = [], []
        for x0 in torch.split(x, 65536):
            f = 0.25 + 0.5 * torch.stack([_net(w[z], case, x0) for z in range(case["M"])])
            mean.append(f.mean(0))
            spread.append(f.std(0, unbiased=False))
        return [torch.cat(mean), torch.cat(spread), None]
    freq, bl, lm, beam, uv, Z, norm = _instrument(case, g)
    S = 2.0 * math.pi * (lm @ uv.t())
    S = torch.complex(torch.cos(S), torch.sin(S))
    rows = []
    for f in range(case["F"]):
        ph = -2.0 * math.pi * (freq[f] / C_LIGHT) * (bl @ lm.t())
        G = (torch.complex(torch.cos(ph), torch.sin(ph)) * beam[f][None, :]) @ S
        rows.append((norm * Z[f][None, :, None] * G[:, None, :]).reshape(case["n_bl"], -1))
    return torch.cat(rows)
