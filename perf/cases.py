"""Performance cases: what a program that builds diffusion maps with this
library asks of it, through the binding's public functions.

A case is a dict of plain values.  ``op`` names the call:

* ``product``  one fused product diag(sl) K diag(sr) V (``fd_kernel_matmul``),
  square (``rows`` = 0) or of ``rows`` new points against ``n`` columns;
* ``noalloc``  the same through ``fd_kernel_matmul_noalloc``;
* ``degree``   the normalisation vectors at one bandwidth (``fd_degree``);
* ``dyadic``   the normalisation vectors of a ladder of ``levels`` bandwidths;
* ``step``     ``fd_degree`` and one product normalised with its s: the whole
  path of one application of M = diag(s) K diag(s);
* ``solve``    the leading ``k`` eigenpairs (``fd_block_lanczos``);
* ``ladder``   warm-started eigensolves over two nested prefixes and two
  bandwidths (``fd_continuation``, with a Nystrom extension between them).

``points`` names the point set (drawn on the device from the seed): a flat
torus (``angles`` angles, radii of the six-torus set-up where ``paper``, noise
``noise``, zero-padded to ``d``), the molecule-like set (von Mises angles
through a small tanh network), or Gaussian data near an 8-dimensional subspace.
``beta`` = 0 stands for 1 / median squared distance.
"""
import math

import torch

from paper_2609_38198_amd import _lib as fd
from paper_2609_38198_amd.inputs import T6_RADII

BASE = {"points": "torus", "angles": 6, "paper": False, "noise": 0.0, "d": 12, "n": 65536,
        "rows": 0, "dtype": "f32", "beta": 2.0, "alpha": 0.5, "b": 16, "scaled": True, "k": 0,
        "levels": 0, "time": 0}
LANDMARKS = 64  # points whose diffusion affinities a solve returns


def _case(name=None, **kw):
    c = dict(BASE, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the 2-torus operator at its own size: the call an eigensolver or a
        # serving loop makes thousands of times; launches and latency
        _case("product_torus2", op="product", angles=2, d=4, n=2048, beta=8.0, b=8),
        # a ragged small set in the molecule-like width, without a workspace
        # (callers under graph capture or that must not allocate)
        _case("product_noalloc_ragged", op="noalloc", points="molecule", d=30, n=5003, beta=0.0,
              b=5),
        # the 6-torus product of the bandwidth sweep, middle bandwidth
        _case("product_torus6", op="product"),
        # Nystrom extension: 64 vectors from 16,384 points to 30,011 others
        _case("product_nystrom", op="product", noise=0.01, n=16384, rows=30011, beta=0.5, b=64,
              scaled=False),
        # raw K v on the six-torus set-up padded to 32 features, one column
        _case("product_one_column", op="product", paper=True, d=32, n=65536, beta=1.0, b=1,
              scaled=False),
        # normalisation alone, small and ragged (one probe of a bandwidth scan)
        _case("degree_small", op="degree", noise=0.01, n=4099, beta=1.0),
        # normalisation alone, a ragged molecule-like set
        _case("degree_molecule", op="degree", points="molecule", d=30, n=200003, beta=0.0),
        # the bandwidth sweep's five normalisations
        _case("dyadic_torus6", op="dyadic", beta=0.5, levels=5),
        # bfloat16 data with wide blocks: normalisation and product
        _case("step_bf16", op="step", points="gauss", d=64, n=131072, dtype="bf16", beta=0.0, b=64),
        # the headline step at its full size: the largest case
        _case("step_molecule", op="step", points="molecule", d=30, n=1 << 20, beta=0.0, b=32),
        # a small eigensolve: many short calls in a row
        _case("solve_torus2", op="solve", angles=2, d=4, n=2048, beta=8.0, b=8, k=16, time=16),
        # a warm-started ladder: prefixes n / 4 and n, bandwidths beta and 2 beta
        _case("ladder_torus6", op="ladder", noise=0.01, n=16384, beta=0.5, b=32, k=64, time=8),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _points(rng):
    """A point set of any feature width, and a bandwidth that suits it."""
    kind = rng.choice(["torus", "torus", "molecule", "gauss"])
    if kind == "torus":
        angles = rng.randint(1, 6)
        return {"points": "torus", "angles": angles, "paper": rng.random() < 0.3,
                "d": 2 * angles if rng.random() < 0.7 else rng.randint(2 * angles, 64),
                "noise": rng.choice([0.0, 0.01]), "beta": rng.choice([0.5, 1.0, 2.0, 4.0, 8.0])}
    return {"points": kind, "d": rng.randint(2, 64), "beta": 0.0}


def draw(rng):
    op = rng.choice(["product", "product", "product", "noalloc", "degree", "dyadic", "step", "step",
                     "solve", "ladder"])
    if op == "solve":
        return _case(op=op, angles=2, d=4, n=_size(rng, 1200, 9000), beta=rng.choice([4.0, 8.0]),
                     b=rng.choice([4, 8, 16]), k=rng.randint(8, 20), time=16)
    if op == "ladder":
        return _case(op=op, noise=0.01, n=_size(rng, 6000, 30000), beta=0.5,
                     b=rng.choice([16, 32]), k=rng.choice([32, 64]), time=8)
    kw = _points(rng)
    kw["dtype"] = rng.choice(["f32", "f32", "f32", "bf16"])
    if op == "noalloc":
        return _case(op=op, n=_size(rng, 300, 30000), b=_size(rng, 1, 32), **kw)
    if op == "product":
        kw["rows"] = rng.choice([0, 0, 0, _size(rng, 300, 200000)])
        kw["scaled"] = rng.random() < 0.7
        return _case(op=op, n=_size(rng, 300, 300000), b=_size(rng, 1, 64), **kw)
    kw["alpha"] = rng.choice([0.5, 0.5, 1.0, 0.0])
    if op == "dyadic":
        kw["beta"] = 0.0 if kw["beta"] == 0.0 else 0.5
        return _case(op=op, n=_size(rng, 1000, 200000), levels=rng.randint(2, 5), **kw)
    return _case(op=op, n=_size(rng, 1000, 300000), b=_size(rng, 2, 64), **kw)


# ------------------------------------------------------------------ inputs


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _cloud(c, seed):
    """The points (float32 or bfloat16, centred before the cast) and beta."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    n, d = c["n"] + c["rows"], c["d"]
    if c["points"] == "torus":
        th = 2 * math.pi * _uniform(g, n, c["angles"])
        r = torch.ones(c["angles"], device="cuda", dtype=torch.float64)
        if c["paper"]:
            r = torch.tensor(T6_RADII[: c["angles"]], device="cuda", dtype=torch.float64)
        x = torch.stack([r * th.cos(), r * th.sin()], dim=2).reshape(n, 2 * c["angles"])
        if c["noise"] > 0:
            x = x + c["noise"] * _normal(g, *x.shape)
        x = torch.nn.functional.pad(x, (0, d - x.shape[1]))
    elif c["points"] == "molecule":
        with torch.random.fork_rng(devices=[torch.cuda.current_device()]):
            torch.manual_seed(int(seed))
            means = 2 * math.pi * _uniform(g, 2) + math.pi * torch.randint(
                0, 2, (n, 2), generator=g, device="cuda")
            kappa = torch.full_like(means, 4.0)
            ang = torch.distributions.VonMises(
                torch.remainder(means + math.pi, 2 * math.pi) - math.pi, kappa,
                validate_args=False).sample()
        f = torch.cat([ang.cos(), ang.sin()], dim=1)
        x = torch.tanh(f @ (0.5 * _normal(g, 4, 64))) @ (0.125 * _normal(g, 64, d))
        x = x + 0.05 * _normal(g, n, d)
    else:
        u, _ = torch.linalg.qr(_normal(g, d, min(8, d)).cpu())
        x = _normal(g, n, min(8, d)) @ u.cuda().T.contiguous() + 0.1 * _normal(g, n, d)
    x = (x - x.mean(dim=0)).to(torch.float32 if c["dtype"] == "f32" else torch.bfloat16)
    beta = c["beta"]
    if beta == 0.0:
        sub = x[:: max(1, n // 2048)][:2048].double()
        dist = torch.cdist(sub, sub, compute_mode="donot_use_mm_for_euclid_dist")
        i, j = torch.triu_indices(len(sub), len(sub), 1, device="cuda")
        beta = 1.0 / float(dist[i, j].square().median())
    # the entry points take beta as float32
    return x.contiguous(), float(torch.tensor(beta, dtype=torch.float32)), g


def _inputs(c, seed):
    x, beta, g = _cloud(c, seed)
    s = {"case": c, "beta": beta, "X": x}
    if c["op"] in ("product", "noalloc", "step"):
        s["V"] = torch.randn(c["n"], c["b"], generator=g, device="cuda")
        s["R"] = x[c["n"]:] if c["rows"] else x
        s["C"] = x[: c["n"]] if c["rows"] else None
        s["sl"] = s["sr"] = None
        if c["scaled"] and c["op"] != "step":
            # like a normalisation: about n^-1/2, spread by the density
            size = c["n"] ** -0.5
            s["sr"] = (size * (0.2 * _normal(g, c["n"])).exp()).float()
            s["sl"] = (size * (0.2 * _normal(g, c["rows"])).exp()).float() if c["rows"] else s["sr"]
    return s


def _ladder(c, beta):
    """Prefix sizes and bandwidths of a ladder's four solves."""
    small = c["n"] // 4
    return [small, small, c["n"], c["n"]], [beta, 2 * beta, beta, 2 * beta]


def _workspace(op, nr, nc, d, b=1, k=1):
    return torch.empty(fd.fd_workspace_size(op, nr, nc, d, b, k), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    c = dict(BASE, **case)
    s = _inputs(c, seed)
    n, d, b, k = c["n"], c["d"], c["b"], c["k"]
    if c["op"] in ("product", "step"):
        s["ws"] = _workspace(fd.FD_OP_KERNEL_MATMUL, c["rows"] or n, n, d, b)
    if c["op"] in ("product", "noalloc"):
        s["Y"] = torch.empty(c["rows"] or n, b, device="cuda")
    if c["op"] in ("degree", "step"):
        s["ws_degree"] = _workspace(fd.FD_OP_DEGREE, n, n, d)
    elif c["op"] == "dyadic":
        s["ws"] = _workspace(fd.FD_OP_DEGREE_DYADIC, n, n, d)
    elif c["op"] == "solve":
        s["ws"] = _workspace(fd.FD_OP_BLOCK_LANCZOS, n, n, d, b, k)
    elif c["op"] == "ladder":
        s["ws"] = _workspace(fd.FD_OP_CONTINUATION, n, 4, d, b, k)
    return s


# ------------------------------------------------------------------ one pass


def _vectors(deg):
    return {"q": deg.q, "d": deg.d, "s": deg.s, "s_off": deg.s_off}


def _affinity(c, evals, phi):
    """Diffusion affinities (M^time restricted to the eigenpairs) of every
    point to the first LANDMARKS points: what a diffusion map is used for, and
    free of the eigenvectors' signs and of rotations inside a cluster."""
    lam = torch.tensor(evals, dtype=phi.dtype, device=phi.device).pow(c["time"])
    return (phi * lam) @ phi[:LANDMARKS].T.contiguous()


def run(state):
    c, x, beta = state["case"], state["X"], state["beta"]
    op = c["op"]
    if op == "product":
        return fd.fd_kernel_matmul(state["R"], state["C"], beta, state["V"], sl=state["sl"],
                                   sr=state["sr"], Y=state["Y"], ws=state["ws"])
    if op == "noalloc":
        return fd.fd_kernel_matmul_noalloc(state["R"], state["C"], beta, state["V"], state["Y"],
                                           sl=state["sl"], sr=state["sr"])
    if op == "degree":
        return _vectors(fd.fd_degree(x, beta, c["alpha"], ws=state["ws_degree"]))
    if op == "dyadic":
        return _vectors(fd.fd_degree_dyadic(x, beta, c["levels"], c["alpha"], ws=state["ws"]))
    if op == "step":
        deg = fd.fd_degree(x, beta, c["alpha"], ws=state["ws_degree"])
        y = fd.fd_kernel_matmul(x, None, beta, state["V"], sl=deg.s, sr=deg.s, ws=state["ws"])
        return dict(_vectors(deg), Y=y)
    if op == "solve":
        e = fd.fd_block_lanczos(x, beta, c["k"], c["b"], alpha=c["alpha"], ws=state["ws"])
        return {"evals": e.evals[: c["k"]], "affinity": _affinity(c, e.evals, e.evecs)}
    ns, betas = _ladder(c, beta)
    lad = fd.fd_continuation(x, ns, betas, c["k"], c["b"], alpha=c["alpha"], ws=state["ws"])
    return {"evals": torch.tensor(lad.evals, dtype=torch.float64),
            "affinity": _affinity(c, lad.evals[-1], lad.evecs)}


# ------------------------------------------------------------------ work


def work(case):
    c = dict(BASE, **case)
    n, d, b, k = c["n"], c["d"], c["b"], c["k"]
    nr = c["rows"] or n
    size = 4 if c["dtype"] == "f32" else 2
    x = (n + c["rows"]) * d * size
    product = {"bytes": x + 4 * b * (n + nr) + 8 * n * c["scaled"], "flops": 2.0 * n * nr * (d + b)}
    # K is symmetric: one evaluation of an entry serves two row sums
    sums = 1.0 * n * n * (d + 2)
    degree = {"bytes": x + 12 * n, "flops": sums * (1 if c["alpha"] == 0 else 2)}
    if c["op"] in ("product", "noalloc"):
        return product
    if c["op"] == "degree":
        return degree
    if c["op"] == "dyadic":
        return {"bytes": x + 12 * n * c["levels"],
                "flops": sums * (c["levels"] + (0 if c["alpha"] == 0 else 1))}
    if c["op"] == "step":
        return {"bytes": degree["bytes"] + product["bytes"],
                "flops": degree["flops"] + product["flops"]}
    # a solve: at least one product per block of the wanted vectors and the
    # kept ones, and their orthogonalisation
    blocks = -(-2 * k // b)
    solve = {"bytes": x + 4 * n * k,
             "flops": degree["flops"] + blocks * product["flops"] + 8.0 * n * k * k}
    if c["op"] == "solve":
        return solve
    return {"bytes": x + 4 * n * k, "flops": 2 * solve["flops"] * (1 + 1 / 16)}


def tolerance(case):
    """Another correct implementation at the same precision; each about four
    times the distance measured from a float64 evaluation, or for the solves
    between two random starts."""
    c = dict(BASE, **case)
    if c["op"] == "solve":
        return {"rel": 1e-3, "max": 2e-2}
    if c["op"] == "ladder":
        return {"rel": 2e-3, "max": 4e-2}
    if c["dtype"] == "bf16" and c["op"] in ("product", "noalloc", "step"):
        return {"rel": 1e-3, "max": 1e-2}
    # float32 sums of kernel entries whose exponent carries a few units of
    # 2^-22 of beta |x|^2
    return {"rel": 1e-5, "max": 4e-4}


# ------------------------------------------------------------------ in 64 bits


def _blocks(xr, xc, beta, same):
    """Row blocks (i0, K[i0:i1]) of the kernel in float64, difference-exact to
    rounding (Gram form in float64 on centred data), unit diagonal."""
    rows = max(1, min(len(xr), (1 << 27) // len(xc)))
    rc = xc.square().sum(dim=1)
    xt = xc.T.contiguous()
    for i in range(0, len(xr), rows):
        a = xr[i:i + rows]
        h = torch.addmm(rc + a.square().sum(dim=1, keepdim=True), a, xt, alpha=-2.0)
        h = h.clamp_(min=0.0)
        if same:
            m = torch.arange(len(a), device=a.device)
            h[m, m + i] = 0.0
        yield i, h.mul_(-beta).exp_()


def _apply(xr, xc, beta, v, same):
    return torch.cat([kb @ v for _, kb in _blocks(xr, xc, beta, same)])


def _degree(x, beta, alpha):
    one = torch.ones(len(x), 1, device=x.device, dtype=torch.float64)
    q = _apply(x, x, beta, one, True)
    w = q.pow(-alpha)
    d = w * _apply(x, x, beta, w, True) if alpha else q
    s = w / d.sqrt()
    return {"q": q[:, 0], "d": d[:, 0], "s": s[:, 0], "s_off": q.sum().reshape(1) - len(x)}


def exact(case, seed):
    c = dict(BASE, **case)
    # above this a float64 evaluation takes too long
    if c["op"] == "ladder" or c["n"] > (4096 if c["op"] == "solve" else 400000):
        return None
    s = _inputs(c, seed)
    x, beta = s["X"].double(), s["beta"]
    if c["op"] in ("product", "noalloc"):
        v = s["V"].double()
        if s["sr"] is not None:
            v = v * s["sr"].double()[:, None]
        xc = x[: c["n"]]
        xr = x[c["n"]:] if c["rows"] else x
        y = _apply(xr, xc, beta, v, not c["rows"])
        return y if s["sl"] is None else y * s["sl"].double()[:, None]
    if c["op"] == "dyadic":
        lev = [_degree(x, beta * 2.0 ** i, c["alpha"]) for i in range(c["levels"])]
        return {m: torch.stack([v[m] for v in lev]) if m != "s_off"
                else torch.cat([v[m] for v in lev]) for m in ("q", "d", "s", "s_off")}
    deg = _degree(x, beta, c["alpha"])
    if c["op"] == "degree":
        return deg
    if c["op"] == "step":
        sv = deg["s"][:, None]
        return dict(deg, Y=sv * _apply(x, x, beta, sv * s["V"].double(), True))
    m = torch.cat([kb for _, kb in _blocks(x, x, beta, True)])
    m = (deg["s"][:, None] * m * deg["s"][None, :]).cpu()
    lam, phi = torch.linalg.eigh(m)
    lam, phi = lam.flip(0)[: c["k"]], phi.flip(1)[:, : c["k"]].contiguous()
    return {"evals": lam.tolist(), "affinity": _affinity(c, lam.tolist(), phi)}
