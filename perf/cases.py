"""Performance cases: what a user of this library has it do.

Each case is one call, or one short sequence of calls, of the public entry
points (paper_1201_4060_amd.Field / Batch / Server) on a synthetic turbulent
field: a Kolmogorov spectrum |k|^(-11/6) with random phases, cut off at |k| =
n/3, divergence free for three components.  Kinds:

  step     a new spectrum is prefiltered and evaluated at the particles: one
           time step of a pseudo-spectral simulation with tracers (the
           coefficient grid stays inside the field, as it does for a program:
           the outputs are what the particles read from it)
  eval     the particles alone, on a field that is already prefiltered: every
           further Runge-Kutta stage, and post-processing of a stored field
  hessian  u, grad u and the second derivatives (strain-rate statistics)
  batch    many fields with uneven particle sets as one planned unit, replayed
           from a HIP graph
  serve    requests from host memory to resident fields, all in flight at once
"""
import math
import weakref
from fractions import Fraction

import torch

import paper_1201_4060_amd as bsi

TWO_PI = 2.0 * math.pi
COEF = {"f64": bsi.BSI_F64, "f32": bsi.BSI_F32, "bf16": bsi.BSI_BF16}
BASIS = {"bspline": bsi.BSI_BASIS_BSPLINE, "lagrange": bsi.BSI_BASIS_LAGRANGE,
         "hermite": bsi.BSI_BASIS_HERMITE}
PREFILTER = {"l2opt": bsi.BSI_PREFILTER_L2OPT, "interp": bsi.BSI_PREFILTER_INTERP,
             "none": bsi.BSI_PREFILTER_NONE}
COEF_BYTES = {"f64": 8, "f32": 4, "bf16": 2}
# axis lengths the library transforms
SIZES = [16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512]


def _case(name, kind, n, ncomp, order, P, coef="f32", spectrum="c128", basis="bspline", prefilter="l2opt",
          cloud="uniform", grad=True):
    c = {"kind": kind, "n0": n[0], "n1": n[1], "n2": n[2], "ncomp": ncomp, "order": order, "P": P, "coef": coef,
         "spectrum": spectrum, "basis": basis, "prefilter": prefilter, "cloud": cloud, "grad": grad}
    if name is not None:
        c["name"] = name
    return c


def _many(name, kind, count, nmax, pmin, pmax, pick):
    c = {"kind": kind, "count": count, "nmax": nmax, "pmin": pmin, "pmax": pmax, "pick": pick}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest whole step: a scalar in double precision, launches count
        _case("step_32_scalar_f64", "step", (32, 32, 32), 1, 4, 10000, coef="f64"),
        # a thousand tracers on a small velocity field: latency of one evaluation
        _case("eval_64_1e3", "eval", (64, 64, 64), 3, 6, 1000),
        # the plain method at its usual size: 256^3 velocity, 10^6 tracers, cubic
        _case("step_256_o4_1e6", "step", (256, 256, 256), 3, 4, 1000000),
        # the same field, the evaluation of one Runge-Kutta stage, quintic, a ragged count
        _case("eval_256_o6_1e6", "eval", (256, 256, 256), 3, 6, 1000003),
        # the headline: 512^3 velocity, 10^7 particles half in clusters, quintic
        _case("step_512_o6_1e7", "step", (512, 512, 512), 3, 6, 10000000, cloud="clustered"),
        # the same particles on a grid stored in BF16
        _case("eval_512_bf16_1e7", "eval", (512, 512, 512), 3, 6, 10000000, coef="bf16", cloud="clustered"),
        # a double-precision step on a ragged grid, values at grid nodes kept (INTERP)
        _case("step_ragged_f64", "step", (192, 128, 256), 3, 6, 300007, coef="f64", prefilter="interp",
              cloud="clustered"),
        # second derivatives of the plain field
        _case("hessian_256_o6_1e6", "hessian", (256, 256, 256), 3, 6, 1000000),
        # the comparison method with eight derivative fields, complex64 spectrum
        _case("step_hermite_128", "step", (128, 128, 128), 3, 4, 200000, spectrum="c64", basis="hermite",
              prefilter="none"),
        # the largest axis: a 1024^3 scalar from a complex64 spectrum, particles far apart
        _case("step_1024_scalar_bf16", "step", (1024, 1024, 1024), 1, 6, 4000000, coef="bf16", spectrum="c64"),
        # 24 fields of 64^3 .. 192^3, 10^3 .. 10^6 particles each, one graph
        _many("batch_24_fields", "batch", 24, 192, 1000, 1000000, 7),
        # 24 host requests of 10^3 .. 3*10^5 particles to four resident 128^3 / 256^3 snapshots
        _many("serve_24_requests", "serve", 24, 256, 1000, 300000, 11),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "eval", "eval", "hessian", "batch", "serve"])
    if kind == "batch":
        return _many(None, kind, rng.randint(6, 32), rng.choice([96, 128, 192]), 1000, _log_int(rng, 50000, 1000000),
                     rng.randrange(1 << 20))
    if kind == "serve":
        return _many(None, kind, rng.randint(6, 32), rng.choice([96, 128, 256]), 1000, _log_int(rng, 30000, 300000),
                     rng.randrange(1 << 20))
    coef = rng.choice(["f32", "f32", "f32", "bf16", "f64"])
    basis, order, prefilter = "bspline", rng.choice([4, 6]), rng.choice(["l2opt", "l2opt", "interp"])
    if kind != "hessian":
        other = rng.random()
        if other < 0.1:
            basis, order, prefilter = "lagrange", rng.choice([2, 4, 6]), "none"
        elif other < 0.2:
            basis, order, prefilter = "hermite", 4, "none"
    heavy = basis == "hermite" or coef == "f64" or kind == "hessian"
    top = 7 if basis == "hermite" else 9 if heavy else 11
    at = rng.randrange(top)
    if rng.random() < 0.4:  # a box of unequal sides
        n = tuple(SIZES[min(top - 1, max(0, at + rng.choice([-1, 0, 0, 1])))] for _ in range(3))
    else:
        n = (SIZES[at],) * 3
    # a step carries at least one particle per 6^3 cells, a later look at a field may have few
    least = max(1000, n[0] * n[1] * n[2] // 216) if kind == "step" else 1000
    P = _log_int(rng, least, 1000000 if heavy else 5000000)
    grad = kind == "hessian" or rng.random() < 0.8
    return _case(None, kind, n, rng.choice([1, 3, 3]), order, P, coef, rng.choice(["c128", "c128", "c64"]), basis,
                 prefilter, rng.choice(["uniform", "clustered"]), grad)


# ---- inputs ------------------------------------------------------------------

def _gen(seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    return g


def _wavenumbers(n, device="cuda"):
    k = [torch.fft.fftfreq(m, 1.0 / m, dtype=torch.float64, device=device) for m in n[:2]]
    k.append(torch.arange(n[2] // 2 + 1, dtype=torch.float64, device=device))
    return k[0][:, None, None], k[1][None, :, None], k[2][None, None, :]


def _spectrum(n, C, seed, kind):
    """Kolmogorov half spectrum [C][n0][n1][n2/2+1], Hermitian, variance about 1."""
    g = _gen(seed)
    k = _wavenumbers(n)
    kk = (k[0] * k[0] + k[1] * k[1]) + k[2] * k[2]
    cut = min(n) / 3.0
    amp = torch.where((kk > 0) & (kk <= cut * cut), kk.clamp_min(1.0) ** (-11.0 / 12.0), torch.zeros_like(kk))
    # sum of |k|^(-11/3) over the shells 4 pi k^2 dk up to the cut
    amp *= 1.0 / math.sqrt(4.0 * math.pi * 1.5 * (1.0 - max(cut, 2.0) ** (-2.0 / 3.0)) + 6.0)
    out = torch.empty((C,) + tuple(kk.shape), dtype=torch.complex128, device="cuda")
    for c in range(C):
        r = torch.randn(out.shape[1:] + (2,), dtype=torch.float64, device="cuda", generator=g)
        z = torch.view_as_complex(r) * math.sqrt(0.5)
        p = z[:, :, 0]
        z[:, :, 0] = (p + torch.roll(torch.flip(p, (0, 1)), (1, 1), (0, 1)).conj()) * math.sqrt(0.5)
        torch.mul(z, amp, out=out[c])
        del r, z, p
    if C == 3:
        dot = (out[0] * k[0] + out[1] * k[1]) + out[2] * k[2]
        dot /= kk.clamp_min(1.0)
        for c in range(3):
            out[c] -= dot * k[c]
    return out if kind == "c128" else out.to(torch.complex64)


def _positions(P, cloud, seed):
    """[P][3] in [0, 2 pi): uniform, or half of it in Gaussian blobs, in random order."""
    g = _gen(seed + 1000003)
    x = torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=g) * TWO_PI
    if cloud == "clustered":
        m = P // 2
        blobs = max(1, min(100, m // 500))
        centre = torch.rand((blobs, 3), dtype=torch.float64, device="cuda", generator=g) * TWO_PI
        owner = torch.randint(0, blobs, (m,), device="cuda", generator=g)
        at = centre[owner] + 0.1 * torch.randn((m, 3), dtype=torch.float64, device="cuda", generator=g)
        x[:m] = torch.remainder(at, TWO_PI)
        x = x[torch.randperm(P, device="cuda", generator=g)]
    return x.contiguous()


def _members(case):
    """The fields and particle counts of a batch or serve case: (field spec, P, field index)."""
    import random
    rng = random.Random(case["pick"])
    sizes = [n for n in (64, 96, 128, 192, 256) if n <= case["nmax"]]
    out = []
    if case["kind"] == "batch":
        for i in range(case["count"]):
            n = rng.choice(sizes)
            f = {"n": (n, n, n), "ncomp": 3, "order": rng.choice([4, 6]), "coef": "f32"}
            out.append((f, _log_int(rng, case["pmin"], case["pmax"]), i))
        return out
    fields = [{"n": (n, n, n), "ncomp": 3, "order": order, "coef": "f32"}
              for n in (max(case["nmax"] // 2, 48), case["nmax"]) for order in (4, 6)]
    for _ in range(case["count"]):
        i = rng.randrange(len(fields))
        out.append((fields[i], _log_int(rng, case["pmin"], case["pmax"]), i))
    return out


def _field_seed(seed, i):
    return seed * 1009 + 17 * i + 5


def _positions_seed(seed, i):
    return seed * 2003 + 31 * i + 9


def _n(case):
    return (case["n0"], case["n1"], case["n2"])


# ---- states ------------------------------------------------------------------

class _State(dict):
    """What a program holds between calls; its handles are closed with it."""

    def own(self, *handles):
        weakref.finalize(self, _close, handles)
        return self


def _close(handles):
    for h in handles:
        h.close()


def prepare(case, seed):
    ctx = bsi.Context(0)
    if case["kind"] == "batch":
        fields, items = [], []
        for f, P, i in _members(case):
            fl = bsi.Field(ctx, f["n"], f["ncomp"], f["order"], COEF[f["coef"]])
            fl.set_spectrum(_spectrum(f["n"], f["ncomp"], _field_seed(seed, i), "c128"))
            pos = _positions(P, "uniform", _positions_seed(seed, i))
            u = torch.empty((P, f["ncomp"]), dtype=fl.out_dtype, device="cuda")
            g = torch.empty((P, f["ncomp"], 3), dtype=fl.out_dtype, device="cuda")
            fields.append(fl)
            items.append((fl, pos, u, g))
        batch = bsi.Batch(ctx, items)
        return _State(kind="batch", batch=batch, items=items).own(batch, *fields, ctx)
    if case["kind"] == "serve":
        fields, requests = {}, []
        for i, (f, P, key) in enumerate(_members(case)):
            if key not in fields:
                fl = bsi.Field(ctx, f["n"], f["ncomp"], f["order"], COEF[f["coef"]])
                fl.set_spectrum(_spectrum(f["n"], f["ncomp"], _field_seed(seed, key), "c128"))
                fields[key] = fl
            cloud = "clustered" if i % 2 else "uniform"
            pos = _positions(P, cloud, _positions_seed(seed, i)).cpu().pin_memory()
            u = torch.empty((P, f["ncomp"]), dtype=torch.float32, pin_memory=True)
            g = torch.empty((P, f["ncomp"], 3), dtype=torch.float32, pin_memory=True)
            requests.append((key, pos, u, g))
        torch.cuda.synchronize()
        server = bsi.Server(ctx, hbm_budget=1 << 30, max_slots=8)
        for key, fl in fields.items():
            server.add_field(key, fl)
        return _State(kind="serve", server=server, requests=requests).own(server, *fields.values(), ctx)
    field = bsi.Field(ctx, _n(case), case["ncomp"], case["order"], COEF[case["coef"]],
                      PREFILTER[case["prefilter"]], basis=BASIS[case["basis"]])
    uhat = _spectrum(_n(case), case["ncomp"], seed, case["spectrum"])
    pos = _positions(case["P"], case["cloud"], seed)
    if case["kind"] != "step":
        field.set_spectrum(uhat)
        uhat = None
    return _State(kind=case["kind"], field=field, uhat=uhat, pos=pos, grad=case["grad"]).own(field, ctx)


def run(state):
    kind = state["kind"]
    if kind == "batch":
        state["batch"].run(use_graph=True)
        return [(u, g) for _, _, u, g in state["items"]]
    if kind == "serve":
        server = state["server"]
        tickets = [server.submit(key, pos, u, g) for key, pos, u, g in state["requests"]]
        for t in tickets:
            server.wait(t)
        return [(u, g) for _, _, u, g in state["requests"]]
    field = state["field"]
    if kind == "hessian":
        return field.eval_hessian(state["pos"])
    if kind == "step":
        field.set_spectrum(state["uhat"])
    u, g = field.eval(state["pos"], grad=state["grad"])
    return (u, g) if state["grad"] else (u,)


# ---- the work that cannot be avoided ---------------------------------------------

def _eval_work(n, C, N, P, coef, grad, hess=False, basis="bspline"):
    size = n[0] * n[1] * n[2]
    per = 8 if basis == "hermite" else 1
    wide = 2 if basis == "hermite" else N
    touched = size * -math.expm1(-P * float(wide ** 3) / size)
    out = 8 if coef == "f64" else 4
    values = C * (1 + (3 if grad else 0) + (6 if hess else 0))
    # each row of N points along axis 2, then axis 1, then axis 0, one set of sums per derivative
    a, b, c = (3, 6, 10) if hess else (2, 3, 4) if grad else (1, 1, 1)
    fma = C * (a * N ** 3 + b * N ** 2 + c * N) + 3 * N * (N + (N - 1 if grad else 0))
    grid = touched * per * C * COEF_BYTES[coef]
    return {"grid": grid, "particles": P * (24 + values * out), "flops": 2 * fma * P}


def work(case):
    if case["kind"] in ("batch", "serve"):
        total = {"bytes": 0.0, "flops": 0.0}
        seen = {}
        for f, P, key in _members(case):
            w = _eval_work(f["n"], f["ncomp"], f["order"], P, f["coef"], True)
            total["bytes"] += w["particles"]
            total["flops"] += w["flops"]
            seen[key] = (f, seen.get(key, (f, 0))[1] + P)
        for f, P in seen.values():
            total["bytes"] += _eval_work(f["n"], f["ncomp"], f["order"], P, f["coef"], True)["grid"]
        return total
    n, C = _n(case), case["ncomp"]
    size = n[0] * n[1] * n[2]
    w = _eval_work(n, C, case["order"], case["P"], case["coef"], case["grad"], case["kind"] == "hessian",
                   case["basis"])
    total = {"bytes": w["particles"], "flops": w["flops"]}
    if case["kind"] == "step":
        # the spectrum is read, the field's grid is written; the particles can read it from there
        per = 8 if case["basis"] == "hermite" else 1
        total["bytes"] += C * n[0] * n[1] * (n[2] // 2 + 1) * (16 if case["spectrum"] == "c128" else 8)
        total["bytes"] += per * C * size * COEF_BYTES[case["coef"]]
        total["flops"] += per * C * 2.5 * size * math.log2(size)
    else:
        total["bytes"] += w["grid"]
    return total


# ---- the same in 64 bits, in plain torch ---------------------------------------

def _integer_sample(M, s):
    """The centred B-spline of order M at the integer s, exactly."""
    acc = Fraction(0)
    for k in range(M + 1):
        x = Fraction(M, 2) + s - k
        if x > 0:
            acc += (-1) ** k * math.comb(M, k) * x ** (M - 1)
    return acc / math.factorial(M - 1)


def _symbol(n, N, prefilter):
    """c(k) for the n indices of one axis."""
    if prefilter == "none":
        return torch.ones(n, dtype=torch.float64)
    kappa = torch.fft.fftfreq(n, dtype=torch.float64)

    def lattice(M):  # sum over i of sinc(kappa + i)^M
        total = torch.full((n,), float(_integer_sample(M, 0)), dtype=torch.float64)
        for s in range(1, M // 2):
            total += 2.0 * float(_integer_sample(M, s)) * torch.cos(TWO_PI * s * kappa)
        return total
    if prefilter == "interp":
        return 1.0 / lattice(N)
    return torch.sinc(kappa) ** N / lattice(2 * N)


def _exact_grid(uhat, n, N, prefilter, basis):
    uhat = uhat.to(torch.complex128)
    if basis != "hermite":
        c = [_symbol(m, N, prefilter).cuda() for m in n]
        h = (c[0][:, None, None] * c[1][None, :, None]) * c[2][None, None, : n[2] // 2 + 1]
        return torch.stack([torch.fft.irfftn(u * h, s=n, dim=(0, 1, 2), norm="forward") for u in uhat])
    k = _wavenumbers(n)
    d = []  # i 2 pi k'/n per axis, nothing at the Nyquist index
    for ax in range(3):
        v = k[ax] * (TWO_PI / n[ax])
        d.append(1j * torch.where(k[ax].abs() * 2 == n[ax], torch.zeros_like(v), v))
    out = torch.empty((uhat.shape[0],) + tuple(2 * m for m in n), dtype=torch.float64, device="cuda")
    for a in range(8):
        o = ((a >> 2) & 1, (a >> 1) & 1, a & 1)
        for c in range(uhat.shape[0]):
            z = uhat[c]
            for ax in range(3):
                z = z * d[ax] if o[ax] else z
            out[c, o[0]::2, o[1]::2, o[2]::2] = torch.fft.irfftn(z, s=n, dim=(0, 1, 2), norm="forward")
    return out


def _bspline_values(t, N):
    """Order-N uniform B-spline pieces at t in [0, 1): [N][P]."""
    b = [torch.ones_like(t)]
    for j in range(1, N):
        saved, nb = torch.zeros_like(t), []
        for r in range(j):
            q = b[r] / j
            nb.append(saved + (r + 1 - t) * q)
            saved = (t + (j - r - 1)) * q
        b = nb + [saved]
    return torch.stack(b)


def _difference(b):
    z = torch.zeros_like(b[:1])
    return torch.cat([z, b]) - torch.cat([b, z])


def _weights(t, N, basis):
    """w, w', w'' (grid units) of the N stencil points: [N][P] each."""
    if basis == "bspline":
        w = _bspline_values(t, N)
        d = _difference(_bspline_values(t, N - 1)) if N > 1 else torch.zeros_like(w)
        h = _difference(_difference(_bspline_values(t, N - 2))) if N > 2 else torch.zeros_like(w)
        return w, d, h
    if basis == "hermite":
        t2, t3 = t * t, t * t * t
        w = [1 - 3 * t2 + 2 * t3, t - 2 * t2 + t3, 3 * t2 - 2 * t3, t3 - t2]
        d = [6 * t2 - 6 * t, 1 - 4 * t + 3 * t2, 6 * t - 6 * t2, 3 * t2 - 2 * t]
        return torch.stack(w), torch.stack(d), None
    node = [j - N // 2 + 1 for j in range(N)]
    w, d = [], []
    for j in range(N):
        rest = [node[k] for k in range(N) if k != j]
        scale = 1.0 / math.prod(node[j] - m for m in rest)
        w.append(math.prod(t - m for m in rest) * scale)
        total = torch.zeros_like(t)
        for skip in rest:
            total = total + math.prod([t - m for m in rest if m != skip], start=torch.ones_like(t))
        d.append(total * scale)
    return torch.stack(w), torch.stack(d), None


def _exact_eval(grid, pos, n, N, basis, hess=False, chunk=1 << 19):
    cs, lo = (2, 0) if basis == "hermite" else (1, N // 2 - 1)
    C = grid.shape[0]
    m = grid.shape[1:]
    P = pos.shape[0]
    u = torch.empty((P, C), dtype=torch.float64, device="cuda")
    g = torch.empty((P, C, 3), dtype=torch.float64, device="cuda")
    h = torch.empty((P, C, 6), dtype=torch.float64, device="cuda") if hess else None
    flat = grid.reshape(C, -1)
    for b in range(0, P, chunk):
        x = pos[b:b + chunk]
        at, w = [], []
        for d in range(3):
            s = x[:, d] * (n[d] / TWO_PI)
            f = torch.floor(s)
            f_ = f.to(torch.int64) * cs - lo
            at.append([torch.remainder(f_ + j, m[d]) for j in range(N)])
            scale = n[d] / TWO_PI
            ws = _weights(s - f, N, basis)
            w.append([ws[0], ws[1] * scale, None if ws[2] is None else ws[2] * (scale * scale)])
        ks = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
        if hess:
            ks += [(2, 0, 0), (1, 1, 0), (1, 0, 1), (0, 2, 0), (0, 1, 1), (0, 0, 2)]
        acc = [torch.zeros((C, x.shape[0]), dtype=torch.float64, device="cuda") for _ in ks]
        for ia in range(N):
            for ib in range(N):
                row = (at[0][ia] * m[1] + at[1][ib]) * m[2]
                t = [torch.zeros((C, x.shape[0]), dtype=torch.float64, device="cuda") for _ in range(3)]
                for ic in range(N):
                    v = flat[:, row + at[2][ic]]
                    for l in range(3 if hess else 2):
                        t[l].addcmul_(v, w[2][l][ic])
                for q, (a, bb, cc) in enumerate(ks):
                    acc[q].addcmul_(t[cc], w[0][a][ia] * w[1][bb][ib])
        u[b:b + chunk] = acc[0].t()
        for d in range(3):
            g[b:b + chunk, :, d] = acc[1 + d].t()
        for q in range(6 if hess else 0):
            h[b:b + chunk, :, q] = acc[4 + q].t()
    return u, g, h


def exact(case, seed):
    if case["kind"] in ("batch", "serve"):
        grids, out = {}, []
        for i, (f, P, key) in enumerate(_members(case)):
            if key not in grids:
                if case["kind"] == "batch":
                    grids.clear()
                uhat = _spectrum(f["n"], f["ncomp"], _field_seed(seed, key), "c128")
                grids[key] = _exact_grid(uhat, f["n"], f["order"], "l2opt", "bspline")
            cloud = "clustered" if case["kind"] == "serve" and i % 2 else "uniform"
            u, g, _ = _exact_eval(grids[key], _positions(P, cloud, _positions_seed(seed, i)), f["n"], f["order"],
                                  "bspline")
            out.append((u, g) if case["kind"] == "batch" else (u.cpu(), g.cpu()))
        return out
    n = _n(case)
    hess = case["kind"] == "hessian"
    grid = _exact_grid(_spectrum(n, case["ncomp"], seed, case["spectrum"]), n, case["order"], case["prefilter"],
                       case["basis"])
    u, g, h = _exact_eval(grid, _positions(case["P"], case["cloud"], seed), n, case["order"], case["basis"], hess)
    if hess:
        return u, g, h
    return (u, g) if case["grad"] else (u,)
