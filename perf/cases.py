"""Performance cases: what programs that sample the determinantal weight have
this library do, with the inputs they come with.

Every case is one call of the Python binding (paper_2003_05286_amd.binding)
over a batch of Markov chains of the half-filled Hubbard model (U = 4,
dtau = 0.1), the model of the package's own workloads.  `n` is the number of
sites: an L x L square lattice where n is a square, else a ring of n sites.

  kind         call                             stands for
  greens       Context.greens                   measurements at equal time
  uneven       Context.greens, mixed sizes      many lattices and temperatures at once
  tdisp        Context.greens_tdisp             G(tau, 0) for spectra
  grad         LogDet1pB forward and backward   training on / differentiating the weight
  langevin     Context.langevin                 gradient-driven updates of a continuous field
  local        Context.local_sweep              single-site updates, two spin flavours
  dense        Context.greens_tdisp_dense       models whose slices are not E diag(v)
  complex      Context.greens_complex           complex slices (phase problems)
  udt_complex  Context.udt_complex              the factorization on its own
"""
import math

import numpy as np
import torch

from paper_2003_05286_amd import binding as sdq
from paper_2003_05286_amd import workloads as wl

U, DTAU = 4.0, 0.1
LAMBDA = wl.hirsch_lambda(U, DTAU)
# Sampled fields of the half-filled model are mostly antiferromagnetic; a
# quarter of the spins against that order gives fields with the sampled ones'
# well-conditioned Green's functions (independent random spins do not: the
# weight suppresses the fields with a nearly singular 1 + B).
FLIPPED = 0.25
UNEVEN_NS, UNEVEN_MS = (36, 64, 100, 144), (100, 200, 400)


def listed():
    return [
        # one small chain per call: latency of a program that runs a single Markov chain
        {"name": "greens n16 single", "kind": "greens", "n": 16, "m": 100, "k": 10, "count": 1},
        # a modest batch of a ragged size, tiles not full
        {"name": "greens n49 batch 96", "kind": "greens", "n": 49, "m": 160, "k": 10, "count": 96},
        # lattices and temperatures of a phase diagram in one call
        {"name": "greens uneven batch 512", "kind": "uneven", "n": 144, "m": 400, "k": 10, "count": 512},
        # the standard production size: equal-time and 40 time-displaced functions of 512 chains
        {"name": "tdisp n64 batch 512", "kind": "tdisp", "n": 64, "m": 400, "k": 10, "count": 512, "lstep": 10},
        # a larger lattice, few chains, slices between the stabilization points too
        {"name": "tdisp n121 batch 24", "kind": "tdisp", "n": 121, "m": 120, "k": 8, "count": 24, "lstep": 6},
        # 16 x 16 sites: a chain is spread over several compute units
        {"name": "tdisp n256 batch 64", "kind": "tdisp", "n": 256, "m": 400, "k": 10, "count": 64, "lstep": 10},
        # 32 x 32 sites, one chain
        {"name": "tdisp n1024 single", "kind": "tdisp", "n": 1024, "m": 200, "k": 10, "count": 1, "lstep": 20},
        # log det and its gradient with respect to a continuous field
        {"name": "grad n64 batch 128", "kind": "grad", "n": 64, "m": 200, "k": 10, "count": 128},
        # one Langevin step of a batch on a smaller lattice
        {"name": "langevin n36 batch 200", "kind": "langevin", "n": 36, "m": 100, "k": 10, "count": 200},
        # a sweep of single-site flips, both spin flavours
        {"name": "local n64 batch 128", "kind": "local", "n": 64, "m": 200, "k": 10, "count": 128},
        # dense slices
        {"name": "dense n64 batch 128", "kind": "dense", "n": 64, "m": 200, "k": 10, "count": 128, "lstep": 10},
        # complex slices
        {"name": "complex n64 batch 128", "kind": "complex", "n": 64, "m": 200, "k": 10, "count": 128},
    ]


def _flops(case):
    n, m, k, c, kind = case["n"], case["m"], case["k"], case["count"], case["kind"]
    nb = -(-m // k)
    sweep = (2.0 * m + nb * 11.0 / 3.0) * n ** 3
    if kind == "uneven":
        return sum((2.0 * mm + -(-mm // k) * 11.0 / 3.0 + 6.3) * nn ** 3 for nn, mm in _uneven_shapes(case))
    if kind == "greens":
        return c * (sweep + 6.3 * n ** 3)
    if kind in ("tdisp", "dense"):
        return c * (2 * sweep + 6.3 * n ** 3 + 8.7 * n ** 3 * (m // case["lstep"]))
    if kind in ("grad", "langevin"):
        return c * (2 * sweep + nb * 16.0 * n ** 3 + 4.0 * m * n ** 3)
    if kind == "local":
        return 2 * c * (2 * sweep + nb * 20.0 * n ** 3 + 4.0 * m * n ** 3 + m * n * n * n)
    if kind == "complex":
        return c * (8.0 * m + nb * 44.0 / 3.0 + 32.0 / 3.0) * n ** 3
    return c * 32.0 / 3.0 * n ** 3


def work(case):
    n, m, c, kind = case["n"], case["m"], case["count"], case["kind"]
    mat = 8.0 * n * n
    if kind == "uneven":
        b = sum(8.0 * (nn * nn + mm * nn) for nn, mm in _uneven_shapes(case))
    elif kind == "greens":
        b = c * (mat + 8.0 * m * n)
    elif kind == "tdisp":
        b = c * (mat * (1 + m // case["lstep"]) + 8.0 * m * n)
    elif kind == "grad":
        b = c * 16.0 * m * n
    elif kind == "langevin":
        b = c * 32.0 * m * n
    elif kind == "local":
        b = c * 24.0 * m * n
    elif kind == "dense":
        b = c * (mat * m + mat * (1 + m // case["lstep"]))
    elif kind == "complex":
        b = c * 2 * mat * (m + 1)
    else:
        b = c * (6 * mat + 8.0 * n)
    return {"bytes": b, "flops": _flops(case)}


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(("greens", "greens", "uneven", "tdisp", "tdisp", "grad", "langevin", "local", "dense",
                       "complex", "udt_complex"))
    case = {"kind": kind, "n": log(9, 144), "m": log(10, 400), "k": rng.choice((5, 7, 8, 10)),
            "count": log(1, 512)}
    if kind in ("greens", "tdisp") and rng.random() < 0.2:  # a chain over several compute units
        case.update(n=log(145, 400), m=log(10, 100), count=log(1, 32))
    if kind == "uneven":
        case.update(n=144, count=log(20, 512))
    elif kind == "local":
        case.update(n=log(9, 100), m=log(10, 200), count=log(1, 128))
    elif kind in ("dense", "complex", "udt_complex"):
        case["n"] = log(9, 64 if kind != "dense" else 80)
        case["count"] = log(1, 128) if kind != "udt_complex" else log(16, 4096)
    if kind in ("tdisp", "dense"):
        case["lstep"] = min(case["m"], rng.choice((case["k"], case["k"], 3, 10, 20)))
    case["k"] = min(case["k"], case["m"])
    while case["count"] > 1 and _flops(case) > 1.5e12:
        case["count"] //= 2
    return case


# ---------------------------------------------------------------------------
# inputs


def _hopping(n):
    side = math.isqrt(n)
    return wl.hopping_matrix(side) if side * side == n and side > 1 else wl.chain_hopping_matrix(n)


def _staggered(n):
    side = math.isqrt(n)
    i = torch.arange(n, device="cuda")
    odd = (i % side + i // side) % 2 if side * side == n else i % 2
    return 1.0 - 2.0 * odd.double()


def _uneven_shapes(case):
    rng = np.random.default_rng(case["count"])
    return [(int(rng.choice(UNEVEN_NS)), int(rng.choice(UNEVEN_MS))) for _ in range(case["count"])]


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _inputs(case, seed):
    """The tensors of a case, all on the GPU."""
    n, m, c, kind = case["n"], case["m"], case["count"], case["kind"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    f64 = {"dtype": torch.float64, "device": "cuda", "generator": gen}

    def ising(*shape):
        flipped = torch.rand(*shape, **f64) < FLIPPED
        return _staggered(shape[-1]) * (1.0 - 2.0 * flipped.double())

    if kind == "udt_complex":  # column scales over 30 decades in random order
        x = torch.complex(torch.randn(c, n, n, **f64), torch.randn(c, n, n, **f64))
        order = torch.rand(c, n, **f64).argsort(1).double()
        return {"w": x * torch.pow(10.0, -30.0 * order / max(n - 1, 1))[:, None, :]}
    if kind == "uneven":
        shapes = _uneven_shapes(case)
        es = {nn: _dev(wl.expk_pair(_hopping(nn), DTAU)[0]) for nn, _ in set(shapes)}
        return {"shapes": shapes, "es": es, "fields": [ising(mm, nn) for nn, mm in shapes]}
    e, ei = (_dev(x) for x in wl.expk_pair(_hopping(n), DTAU))
    d = {"e": e, "ei": ei}
    if kind in ("grad", "langevin"):
        d["field"] = torch.randn(c, m, n, **f64)
        if kind == "langevin":
            d["noise"] = torch.randn(c, m, n, **f64)
        return d
    d["field"] = ising(c, m, n)
    if kind == "local":
        d["unif"] = torch.rand(c, m, n, **f64)
    elif kind == "dense":
        d["slices"] = e[None, None] * torch.exp(LAMBDA * d["field"])[:, :, None, :]
    elif kind == "complex":
        phase = 0.6 * torch.rand(c, m, n, **f64) - 0.3
        d["slices"] = e[None, None] * torch.exp(torch.complex(LAMBDA * d["field"], phase))[:, :, None, :]
    return d


def prepare(case, seed):
    x = _inputs(case, seed)
    s = {"case": case, "x": x, "ctx": sdq.context()}
    kind, k = case["kind"], case["k"]
    if kind == "uneven":
        s["chains"] = [sdq.Chain(x["es"][nn], f, LAMBDA, k) for (nn, _), f in zip(x["shapes"], x["fields"])]
    elif kind == "local":
        s["chains"] = [sdq.Chain(x["e"], f, a, k, x["ei"]) for f in x["field"] for a in (LAMBDA, -LAMBDA)]
    elif kind == "langevin":
        s["chains"] = [sdq.Chain(x["e"], f, DTAU, k, x["ei"]) for f in x["field"]]
    elif kind in ("greens", "tdisp"):
        s["chains"] = [sdq.Chain(x["e"], f, LAMBDA if i % 2 == 0 else -LAMBDA, k)
                       for i, f in enumerate(x["field"])]
    elif kind == "grad":
        x["field"].requires_grad_()
    elif kind in ("dense", "complex"):
        s["slices"] = list(x["slices"])
    if "lstep" in case:
        s["ls"] = _l_list(case)
    return s


def _l_list(case):
    return list(range(case["lstep"], case["m"] + 1, case["lstep"]))


def _whole(ts):
    """A batch's matrices as one tensor (a short list stays as it is)."""
    return ts if len(ts) <= 8 else torch.cat([t.reshape(-1) for t in ts])


def run(s):
    ctx, case, x = s["ctx"], s["case"], s["x"]
    kind = case["kind"]
    if kind in ("greens", "uneven"):
        gs, ld, sg, st = ctx.greens(s["chains"])
        return {"g": _whole(gs), "ld": ld, "sg": sg, "st": st}
    if kind == "tdisp":
        gts, gs, ld, sg, st = ctx.greens_tdisp(s["chains"], s["ls"])
        return {"gt": _whole(gts), "g": _whole(gs), "ld": ld, "sg": sg, "st": st}
    if kind == "grad":
        ld, sg = sdq.LogDet1pB.apply(x["field"], x["e"], x["ei"], DTAU, case["k"])
        (grad,) = torch.autograd.grad(ld.sum(), x["field"])
        return {"grad": grad, "ld": ld.detach(), "sg": sg}
    if kind == "langevin":
        force, ld, sg, st = ctx.langevin(s["chains"], 1, 1e-3, 1.0, x["noise"])
        return {"field": x["field"], "force": force, "ld": ld, "sg": sg, "st": st}
    if kind == "local":
        acc, st = ctx.local_sweep(s["chains"], 2, x["unif"])
        return {"acc": acc, "field": x["field"], "st": st}
    if kind == "dense":
        gts, gs, ld, sg, st = ctx.greens_tdisp_dense(s["slices"], case["k"], s["ls"])
        return {"gt": _whole(gts), "g": _whole(gs), "ld": ld, "sg": sg, "st": st}
    if kind == "complex":
        gs, ld, ph, st = ctx.greens_complex(s["slices"], case["k"])
        return {"g": _whole(gs), "ld": ld, "ph": ph, "st": st}
    u, d, t = ctx.udt_complex(x["w"])
    return {"u": u, "d": d, "t": t}


# ---------------------------------------------------------------------------
# the same results from plain torch / numpy in 64 bits


def _qr(a, pivot=False):
    """Householder QR of a batch (diag R real): q, r, perm, a[:, :, perm] = q r.  With `pivot` the column of
    largest remaining norm at every step, else the columns as they stand."""
    a = a.clone()
    c, n, _ = a.shape
    perm = torch.arange(n, device="cuda").repeat(c, 1)
    rows = torch.arange(c, device="cuda")
    q = torch.eye(n, dtype=a.dtype, device="cuda").repeat(c, 1, 1)
    for j in range(n):
        if pivot:
            p = j + torch.linalg.vector_norm(a[:, j:, j:], dim=1).argmax(1)
            col, held = a[:, :, j].clone(), perm[:, j].clone()
            a[:, :, j] = a[rows, :, p]
            a[rows, :, p] = col
            perm[:, j] = perm[rows, p]
            perm[rows, p] = held
        v = a[:, j:, j].clone()
        if j == n - 1 and not a.is_complex():
            break
        alpha = v[:, 0].clone()
        beta = -torch.where(alpha.real < 0, -1.0, 1.0) * torch.linalg.vector_norm(v, dim=1)
        tau = (beta - alpha) / beta
        if j == n - 1:  # one entry: nothing to do where it is real already
            tau = torch.where(alpha.imag == 0, 0.0, tau)
        v[:, 0] -= beta
        v /= (alpha - beta)[:, None]
        h = v.conj()[:, None, :]
        a[:, j:, j:] -= (tau.conj()[:, None] * v)[:, :, None] * torch.matmul(h, a[:, j:, j:])
        q[:, :, j:] -= torch.matmul(q[:, :, j:], (tau[:, None] * v)[:, :, None]) * h
    return q, torch.triu(a), perm


def _udt(w, t):
    """w = u d t' with the columns sorted by norm before the QR; t' applied to t."""
    order = torch.linalg.vector_norm(w, dim=1).argsort(1, descending=True)
    q, r, _ = _qr(torch.gather(w, 2, order[:, None, :].expand_as(w)))
    d = torch.diagonal(r, dim1=1, dim2=2).abs()
    tp = torch.gather(t, 1, order[:, :, None].expand_as(t))
    return q, d, torch.matmul(r / d[:, :, None], tp)


def _stages(mult, n, batch, dtype, m, stops, k, reverse=False):
    """{l: (u, d, t)} at the slices `stops` of the product of the slices, which mult(l, w) applies from the
    left: slices 1..l, or (reverse) m..l+1 of the transposes."""
    u = torch.eye(n, dtype=dtype, device="cuda").expand(batch, n, n).contiguous()
    d = torch.ones(batch, n, dtype=torch.float64, device="cuda")
    t, got, since = u.clone(), {}, 0
    want = set(stops)
    at = m if reverse else 0
    if at in want:
        got[at] = (u, d, t)
    w = u * d[:, None, :]
    for step in range(m):
        l = m - step if reverse else step + 1
        w, since = mult(l, w), since + 1
        at = l - 1 if reverse else l
        if since == k or at in want or step == m - 1:
            u, d, t = _udt(w, t)
            w, since = u * d[:, None, :], 0
            if at in want:
                got[at] = (u, d, t)
    return got


def _equal(udt):
    u, d, t = udt
    dp, dm = d.clamp(min=1.0), d.clamp(max=1.0)
    rhs = u.conj().transpose(1, 2).contiguous() / dp[:, :, None]
    mid = rhs + dm[:, :, None] * t
    sm, lm = torch.linalg.slogdet(mid)
    su, _ = torch.linalg.slogdet(u)
    return torch.linalg.solve(mid, rhs), lm + dp.log().sum(1), su * sm


def _pair(f, b):
    """(B(tau,0)^-1 + B(beta,tau))^-1 from the two factorizations around tau."""
    (u1, d1, t1), (u2, d2, t2) = f, b
    lm, lpi = 1.0 / d1.clamp(min=1.0), d1.clamp(max=1.0)
    rpi, rm = 1.0 / d2.clamp(min=1.0), d2.clamp(max=1.0)
    h1, t2t = u1.transpose(1, 2).contiguous(), t2.transpose(1, 2).contiguous()
    mid = lm[:, :, None] * torch.matmul(h1, u2) * rpi[:, None, :] + lpi[:, :, None] * torch.matmul(t1, t2t) * rm[:, None, :]
    return torch.matmul(u2 * rpi[:, None, :], torch.linalg.solve(mid, lpi[:, :, None] * t1))


def _mults(case, x):
    """mult(l, w) of the chain and of its transposes."""
    if "slices" in x:
        sl = x["slices"]
        return (lambda l, w: torch.matmul(sl[:, l - 1], w),
                lambda l, w: torch.matmul(sl[:, l - 1].transpose(1, 2).contiguous(), w))
    alpha = torch.full((x["field"].shape[0], 1, 1), DTAU if case["kind"] in ("grad", "langevin") else LAMBDA,
                       dtype=torch.float64, device="cuda")
    if case["kind"] == "tdisp" or case["kind"] == "greens":
        alpha[1::2] *= -1.0
    v = torch.exp(alpha * x["field"].detach())
    e = x["e"]
    return (lambda l, w: torch.matmul(e, v[:, l - 1, :, None] * w),
            lambda l, w: v[:, l - 1, :, None] * torch.matmul(e.T.contiguous(), w))


def _exact_gradient(case, x):
    n, m, c = case["n"], case["m"], case["count"]
    fwd, bwd = _mults(case, x)
    stops = list(range(0, m, 5))
    f = _stages(fwd, n, c, torch.float64, m, stops + [m], 5)
    b = _stages(bwd, n, c, torch.float64, m, stops, 5, reverse=True)
    _, ld, sg = _equal(f[m])
    v = torch.exp(DTAU * x["field"].detach())
    diag = torch.empty(c, m, n, dtype=torch.float64, device="cuda")
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    for s in stops:
        # G_l = (1 + B(l-1, 0) B(beta, l-1))^-1 at l = s + 1
        (u1, d1, t1), (u2, d2, t2) = f[s], b[s]
        ip, im = 1.0 / d1.clamp(min=1.0), d1.clamp(max=1.0)
        jp, jm = 1.0 / d2.clamp(min=1.0), d2.clamp(max=1.0)
        h1, t2t = u1.transpose(1, 2).contiguous(), t2.transpose(1, 2).contiguous()
        mid = ip[:, :, None] * torch.matmul(h1, u2) * jp[:, None, :] + im[:, :, None] * torch.matmul(t1, t2t) * jm[:, None, :]
        g = torch.matmul(u2 * jp[:, None, :], torch.linalg.solve(mid, ip[:, :, None] * h1))
        for l in range(s + 1, min(s + 5, m) + 1):
            diag[:, l - 1] = torch.diagonal(g, dim1=1, dim2=2)
            g = torch.matmul(torch.matmul(x["e"], v[:, l - 1, :, None] * g / v[:, l - 1, None, :]), x["ei"])
    return DTAU * (1.0 - diag), ld, sg


def _exact_udt_complex(w):
    q, r, perm = _qr(w, pivot=True)
    d = torch.diagonal(r, dim1=1, dim2=2).abs()
    t = torch.empty_like(r).scatter_(2, perm[:, None, :].expand_as(r), r / d[:, :, None])
    return {"u": q, "d": d, "t": t}


def exact(case, seed):
    kind, n, m, c = case["kind"], case["n"], case["m"], case["count"]
    if kind == "local":
        return None
    x = _inputs(case, seed)
    if kind == "udt_complex":
        return _exact_udt_complex(x["w"])
    if kind == "uneven":
        g, ld, sg = [None] * c, torch.empty(c, dtype=torch.float64), torch.empty(c, dtype=torch.float64)
        for nn, mm in sorted(set(x["shapes"])):
            at = [i for i, sh in enumerate(x["shapes"]) if sh == (nn, mm)]
            v = torch.exp(LAMBDA * torch.stack([x["fields"][i] for i in at]))
            e = x["es"][nn]
            f = _stages(lambda l, w: torch.matmul(e, v[:, l - 1, :, None] * w), nn, len(at), torch.float64, mm, [mm], 5)
            gg, l1, s1 = _equal(f[mm])
            ld[at], sg[at] = l1.cpu(), s1.cpu()
            for i, one in zip(at, gg):
                g[i] = one
        return {"g": _whole(g), "ld": ld, "sg": sg, "st": None}
    if kind == "grad":
        grad, ld, sg = _exact_gradient(case, x)
        return {"grad": grad, "ld": ld, "sg": sg}
    if kind == "langevin":
        grad, ld, sg = _exact_gradient(case, x)
        force = x["field"] - grad
        field = x["field"] - 1e-3 * force + math.sqrt(2e-3) * x["noise"]
        return {"field": field, "force": force, "ld": ld, "sg": sg, "st": None}
    fwd, bwd = _mults(case, x)
    dtype = torch.complex128 if kind == "complex" else torch.float64
    ls = _l_list(case) if "lstep" in case else []
    f = _stages(fwd, n, c, dtype, m, ls + [m], 5)
    g, ld, sg = _equal(f[m])
    if kind == "complex":
        return {"g": _whole(list(g)), "ld": ld, "ph": sg, "st": None}
    got = {"g": _whole(list(g)), "ld": ld, "sg": sg, "st": None}
    if ls:
        b = _stages(bwd, n, c, dtype, m, ls, 5, reverse=True)
        gt = torch.stack([_pair(f[l], b[l]) for l in ls], 1)
        got["gt"] = _whole(list(gt))
    return got
