"""Performance cases: what a user of the library has it do, from one thin Rayleigh layer to a single
layer at the largest quadrature.

A case is a dict of plain values:
  kind       "layers" (plan of independent layers), "spectral" (SpectralBRDF), "adjoint" (forward and
             backward through DifferentiableBRDF), "stack" (layers on top of one another over a base),
             "beams" (off-node incident and outgoing cosines), "noalloc" (allocation-free entry point)
  layers     number of layers
  N          nodes per hemisphere; a comma-separated text is dealt to the layers in turn
  L, M, P    coefficients, Fourier orders, azimuth samples; 0 stands for 2 N
  phase      "hg" (Henyey-Greenstein-like set, redrawn until it is a valid scattering matrix) or
             "rayleigh"
  tau0, tau1, omega0, omega1   ranges of the optical thickness (logarithmic) and of the albedo
  and, by kind: precision, graph, base, n_mu0, n_mu_out.
"""

import functools
import math

import numpy as np
import torch

from paper_1707_05882_amd import api, binding

OMEGA_MAX = 1.0 - 1e-12
# largest sum over layers and orders of M (8N)^3 for which exact() is quick enough
EXACT_LIMIT = 3e9
# largest sum over layers and orders of (4N)^3 of a drawn case (the largest listed one has 3.7e10)
DRAW_LIMIT = 1.5e10


def _case(name, kind, layers, N, L=0, M=0, P=0, phase="hg", tau=(0.1, 100.0), omega=(0.5, 0.999), **more):
    c = dict(kind=kind, layers=layers, N=str(N), L=L, M=M, P=P, phase=phase, tau0=tau[0], tau1=tau[1],
             omega0=omega[0], omega1=omega[1], **more)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one molecular layer, three orders (the smoke workload); launches dominate
        _case("rayleigh_N8", "layers", 1, 8, 3, 3, 16, "rayleigh", (0.3, 3.0), (0.8, 0.95)),
        # small odd layers replayed as one graph, as a serving loop does
        _case("graph_4xN13", "layers", 4, 13, 29, 21, 17, graph=True),
        # one layer through the allocation-free entry point (code that cannot call hipMalloc)
        _case("noalloc_N16", "noalloc", 1, 16),
        # the ordinary single material (the particulate workload)
        _case("particulate_N32", "layers", 1, 32, tau=(3.0, 30.0), omega=(0.9, 0.999)),
        # a rendering's materials: 8 materials at 9 wavelengths in one plan (the spectral workload)
        _case("spectral_8x9_N32", "spectral", 72, 32, 64, 64, 32, tau=(0.3, 30.0), omega=(0.8, 0.999)),
        # a library of layers of mixed resolution (the batched workload, a quarter of it)
        _case("uneven_64", "layers", 64, "16,24,32,48,64"),
        # one thick layer at the largest quadrature (the large workload)
        _case("large_N128", "layers", 1, 128, tau=(30.0, 100.0), omega=(0.99, 0.999)),
        # the FP32-refined boundary solve on a few layers
        _case("refined_4xN24", "layers", 4, 24, precision="fp32_refined"),
        # a paint: four layers over a Lambertian base
        _case("stack4_lambertian_N24", "stack", 4, 24, P=32, tau=(0.2, 10.0), base="lambertian"),
        # a coating over a measured (general Mueller) base; 4N = 160 is not a power of two
        _case("stack2_mueller_N40", "stack", 2, 40, 80, 24, 36, tau=(0.2, 10.0), base="mueller"),
        # light sources and viewers off the quadrature nodes
        _case("beams_N32", "beams", 1, 32, tau=(0.3, 10.0), omega=(0.8, 0.99), n_mu0=8, n_mu_out=8),
        # inverse rendering step: loss and gradients of 64 layers (the differentiation workload)
        _case("adjoint_64xN32", "adjoint", 64, 32, 64, 32, 32),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.choice(["layers", "layers", "layers", "layers", "noalloc", "stack", "beams", "adjoint", "spectral"])
    N = _log_int(rng, 6, 128 if kind == "layers" else 48)
    L = min(256, max(4, int(N * rng.uniform(1.0, 2.5))))
    M = max(1, int(L * rng.uniform(0.4, 1.0)))
    P = _log_int(rng, 7, 2 * N)
    limit = DRAW_LIMIT / (8.0 if kind in ("adjoint", "stack", "beams") else 1.0)
    if kind == "noalloc":  # its static scratch array holds about 8 M (4N)^2 doubles
        M = max(1, min(M, int((70 << 20) / (8.0 * (8 * 16 * N * N + 3 * L * N)))))
    while M * (4 * N) ** 3 > limit:
        M = max(1, M // 2)
    most = max(1, min(72, int(limit / (M * (4.0 * N) ** 3))))
    if kind in ("noalloc", "beams"):
        n = 1
    elif kind == "stack":
        n = rng.randint(1, max(1, min(5, most)))
    elif kind == "spectral":
        n = 3 * max(1, _log_int(rng, 1, max(1, most // 3)))
    else:
        n = _log_int(rng, 1, most)
    more = {}
    if kind == "layers":
        more = rng.choice([{}, {}, {"graph": True}, {"precision": "fp32_refined"}])
    elif kind == "stack":
        more = {"base": rng.choice(["black", "lambertian", "mueller"])}
    elif kind == "beams":
        more = {"n_mu0": rng.randint(1, min(N, 16)), "n_mu_out": rng.randint(0, min(N, 16))}
    tau0 = 10.0 ** rng.uniform(-1.0, 1.0)
    omega0 = rng.uniform(0.5, 0.95)
    return _case("", kind, n, N, L, M, P, tau=(tau0, 10.0 * tau0), omega=(omega0, rng.uniform(omega0, 0.999)), **more)


# ---------------------------------------------------------------------------------------- inputs


def _shapes(case):
    Ns = [int(x) for x in case["N"].split(",")]
    N = [Ns[l % len(Ns)] for l in range(case["layers"])]
    of = lambda k: [case[k] or 2 * n for n in N]
    return N, of("L"), of("M"), of("P")


def _wigner(L, m, n, x):
    """d^l_{mn}, l = 0..L-1, at the cosines x, by the three-term recurrence in l."""
    out = np.zeros((L,) + x.shape)
    l0 = max(abs(m), abs(n))
    if l0 >= L:
        return out
    log_c = 0.5 * (math.lgamma(2 * l0 + 1) - math.lgamma(abs(m - n) + 1) - math.lgamma(abs(m + n) + 1))
    sign = 1.0 if n >= m else (-1.0) ** (m - n)
    out[l0] = sign * math.exp(log_c - l0 * math.log(2.0)) * (1 - x) ** (abs(m - n) / 2) * (1 + x) ** (abs(m + n) / 2)
    for l in range(l0, L - 1):
        if l == 0:
            out[1] = x * out[0]
            continue
        a = (2 * l + 1) * (l * (l + 1) * x - m * n)
        b = (l + 1) * math.sqrt((l * l - m * m) * (l * l - n * n))
        c = l * math.sqrt(((l + 1) ** 2 - m * m) * ((l + 1) ** 2 - n * n))
        out[l + 1] = (a * out[l] - b * out[l - 1]) / c
    return out


@functools.lru_cache(maxsize=8)
def _check_tables(L):
    x = np.polynomial.legendre.leggauss(1024)[0]
    return tuple(_wigner(L, m, n, x) for m, n in ((0, 0), (2, 2), (2, -2), (0, 2)))


def _valid(coef):
    """The inequalities that a single-scattering matrix fulfils, on a Gauss grid."""
    d00, d22, d2m, d02 = _check_tables(coef.shape[1])
    a1, a4, s, d = coef[0] @ d00, coef[3] @ d00, (coef[1] + coef[2]) @ d22, (coef[1] - coef[2]) @ d2m
    a2, a3, b1, b2 = (s + d) / 2, (s - d) / 2, -(coef[4] @ d02), -(coef[5] @ d02)
    t = 1e-12 * max(1.0, np.abs(a1).max())
    return (all((np.abs(e) <= a1 + t).all() for e in (a2, a3, a4, b1, b2))
            and ((a3 + a4) ** 2 + 4 * b2 ** 2 <= (a1 + a2) ** 2 - 4 * b1 ** 2 + t).all()
            and (np.abs(a3 - a4) <= a1 - a2 + t).all())


def _hg(rng, L):
    """Henyey-Greenstein-like set: decay g, polarised and circular shares drawn with it."""
    l = np.arange(L)
    while True:
        # a truncated expansion rings when g^L is not small, so few coefficients take a smaller g
        g = rng.uniform(0.5, 0.9) if L > 24 else rng.uniform(0.2, 0.6)
        rho, rho4, eta, zeta = rng.uniform(0.5, 0.95), rng.uniform(0.5, 0.95), rng.uniform(0, 0.3), rng.uniform(0, 0.1)
        base = (2 * l + 1) * g ** l
        hi = base * (l >= 2)
        coef = np.stack([base, rho * hi, rho * hi, rho4 * base, -eta * hi, zeta * hi])
        coef[:, np.arange(L) > 0] *= 1.0 if L > 24 else 0.7  # the short sets are mixed with isotropic scattering
        if _valid(coef):
            return coef


def _rayleigh():
    c = np.zeros((6, 3))
    c[0] = 1.0, 0.0, 0.5
    c[1, 2], c[3, 1], c[4, 2] = 3.0, 1.5, math.sqrt(6.0) / 2
    return c


def _inputs(case, seed):
    rng = np.random.default_rng([1707, int(seed)])
    N, L, M, P = _shapes(case)
    n = len(N)
    x = {"tau": np.exp(rng.uniform(math.log(case["tau0"]), math.log(case["tau1"]), n)),
         "omega": rng.uniform(case["omega0"], case["omega1"], n),
         "coef": [_rayleigh() if case["phase"] == "rayleigh" else _hg(rng, l) for l in L]}
    if case["kind"] == "stack" and case["base"] == "lambertian":
        x["base"] = np.full(n, rng.uniform(0.2, 0.8))
    elif case["kind"] == "stack" and case["base"] == "mueller":
        Rb = np.stack([rng.standard_normal((N[0], 4, N[0], 4)) * (0.05 / (1 + m) / N[0]) for m in range(M[0])])
        Rb[0, :, 0, :, 0] += 0.8
        x["base"] = Rb.reshape(M[0], 4 * N[0], 4 * N[0])
    if case["kind"] == "beams":
        spread = lambda k: (np.arange(k) + rng.uniform(0.1, 0.9, k)) / k
        x["mu0"], x["mu_out"] = spread(case["n_mu0"]), spread(case["n_mu_out"])
    if case["kind"] == "adjoint":  # the target material: everything a few per cent off
        x["target"] = (x["tau"] * (1 + 0.05 * rng.standard_normal(n)),
                       np.minimum(x["omega"] + 0.01 * rng.standard_normal(n), 0.999),
                       [c * np.where(np.arange(c.shape[1]) > 0, 0.98, 1.0) for c in x["coef"]])
    return x


# ---------------------------------------------------------------------------------------- running


def prepare(case, seed):
    x = _inputs(case, seed)
    N, L, M, P = _shapes(case)
    kind = case["kind"]
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")
    st = {"kind": kind}
    if kind == "spectral":  # host arrays in, as a renderer holds its materials
        A = 3 if case["layers"] % 9 else case["layers"] // 9
        W = case["layers"] // A
        st["solver"] = api.SpectralBRDF(A, W, N[0], L[0], M[0], P[0])
        st["args"] = (x["tau"].reshape(A, W), x["omega"].reshape(A, W),
                      np.stack(x["coef"]).reshape(A, W, 6, L[0]))
        return st
    st["tau"], st["omega"], st["coef"] = dev(x["tau"]), dev(x["omega"]), dev(api.pack_coefficients(x["coef"]))
    if kind == "noalloc":
        st["shape"] = (N[0], L[0], M[0], P[0])
        st["F"] = torch.empty(N[0], N[0], P[0], 4, 4, dtype=torch.float64, device="cuda")
        st["status"] = torch.empty(1, dtype=torch.int32, device="cuda")
        return st
    if kind == "adjoint":
        st["model"] = api.DifferentiableBRDF(N, L, M, P)
        t, w, c = x["target"]
        with torch.no_grad():
            st["target"] = st["model"](dev(t), dev(w), dev(api.pack_coefficients(c)))
        for k in ("tau", "omega", "coef"):
            st[k].requires_grad_()
        return st
    kw = {}
    if case.get("precision") == "fp32_refined":
        kw["precision"] = binding.PRECISION_FP32_REFINED
    if case.get("graph"):
        kw["flags"] = binding.FLAG_GRAPH
        st["stream"] = torch.cuda.Stream()
    if kind == "stack":
        kw["below"] = list(range(1, len(N))) + [-1]
        kw["base"] = {"black": binding.BASE_BLACK, "lambertian": binding.BASE_LAMBERTIAN,
                      "mueller": binding.BASE_MUELLER}[case["base"]]
        st["base"] = dev(x["base"].ravel()) if "base" in x else None
    if kind == "beams":
        kw["mu0"] = x["mu0"]
        kw["mu_out"] = x["mu_out"] if len(x["mu_out"]) else None
    st["solver"] = api.BRDFSolver(N, L, M, P, **kw)
    return st


def run(st):
    kind = st["kind"]
    if kind == "spectral":
        st["solver"](*st["args"])
        return {"F": st["solver"].solver.F}
    if kind == "noalloc":
        binding.solve_noalloc(*st["shape"], st["tau"], st["omega"], st["coef"], st["F"], st["status"],
                              torch.cuda.current_stream().cuda_stream)
        return {"F": st["F"], "status": st["status"]}
    if kind == "adjoint":
        F = st["model"](st["tau"], st["omega"], st["coef"])
        loss = 0.5 * (F - st["target"]).square().sum()
        g = torch.autograd.grad(loss, [st["tau"], st["omega"], st["coef"]])
        return {"F": F, "loss": loss, "dtau": g[0], "domega": g[1], "dcoef": g[2]}
    s = st["solver"]
    s.solve_device(st["tau"], st["omega"], st["coef"], stream=st.get("stream"), base_d=st.get("base"))
    out = {"F": s.F, "status": s.status}
    if s.F_beam is not None:
        out["F_beam"] = s.F_beam
    return out


def work(case):
    """Bytes: inputs read once, outputs written once. Flops per order, n = 4N: the assembly, the product
    FE, the mode vectors and their boundary factorisations and right divisions (2 (2/3 + 2) n^3); not
    the steps of the eigen-decomposition, whose number depends on the method. A stack adds its adding
    step, the adjoint the products of its reverse pass."""
    N, L, M, P = _shapes(case)
    by = fl = 0.0
    kind = case["kind"]
    for n, l, m, p in zip(N, L, M, P):
        d = (4.0 * n) ** 3
        fl += m * (4.0 + 16.0 / 3.0) * d + sum(72.0 * n * n * (l - k) for k in range(m)) + 2.0 * m * 16 * n * n * p
        by += 8.0 * (6 * l + 2 + 16 * n * n * p)
        if kind == "stack":
            fl += m * (6.0 + 8.0 / 3.0) * d
        if kind == "adjoint":
            fl += m * 20.0 * d
            by += 8.0 * (6 * l + 2 + 2 * 16 * n * n * p)
        if kind == "beams":
            by += 8.0 * 16 * (n + case["n_mu_out"]) * case["n_mu0"] * p
    if kind == "stack" and case["base"] == "mueller":
        by += 8.0 * M[0] * (4 * N[0]) ** 2
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------------------------------- 64-bit values


def _legendre_matrices(L, m, mu):
    pb, dp, dm = (_wigner(L, m, k, mu) for k in (0, 2, -2))
    r, t = -0.5 * (dp + dm), -0.5 * (dp - dm)
    Z = np.zeros((L, len(mu), 4, 4))
    Z[..., 0, 0] = Z[..., 3, 3] = pb
    Z[..., 1, 1] = Z[..., 2, 2] = r
    Z[..., 1, 2] = Z[..., 2, 1] = -t
    return Z


def _order(coef, omega, tau, m, mu, alpha, mu0=(), mu_out=()):
    """Upward radiance at the top and downward radiance at the base for unit radiance entering at the top
    on each downward node (and, in the last columns, for beams of unit flux at mu0; in the last rows of
    the upward field towards mu_out), from the full eigen-decomposition of the order's transfer system
    on all directions. Beams and extra outgoing directions are streams of zero weight."""
    N, nb, no = len(mu), len(mu0), len(mu_out)
    down, up = np.concatenate([mu, mu0]), np.concatenate([mu, mu_out])
    mus = np.concatenate([down, -up])
    L = coef.shape[1]
    B = np.zeros((L, 4, 4))
    B[:, 0, 0], B[:, 1, 1], B[:, 2, 2], B[:, 3, 3] = coef[0], coef[1], coef[2], coef[3]
    B[:, 0, 1] = B[:, 1, 0] = coef[4]
    B[:, 2, 3], B[:, 3, 2] = coef[5], -coef[5]
    Z = _legendre_matrices(L, m, mus)[m:]  # (l, direction, 4, 4)
    left = Z.transpose(1, 2, 0, 3).reshape(4 * len(mus), -1)
    A = left @ (B[m:, None] @ Z).transpose(0, 2, 1, 3).reshape(left.shape[1], -1)
    w = np.concatenate([alpha, np.full(nb, 1 / math.pi), alpha, np.zeros(no)])
    K = 0.5 * omega * A * np.repeat(w, 4)[None, :]
    K[4 * N:4 * (N + nb), :] = 0.0  # nothing scatters into a beam
    K = (K - np.eye(len(K))) / np.repeat(mus, 4)[:, None]
    kappa, V = np.linalg.eig(K)
    nd = 4 * (N + nb)
    dec = kappa.real < 0
    if dec.sum() != nd:
        raise FloatingPointError("the modes do not split into decaying and growing ones")
    H0 = V * np.exp(np.where(dec, 0.0, -kappa * tau))
    H1 = V * np.exp(np.where(dec, kappa * tau, 0.0))
    rhs = np.zeros((len(K), nd))
    rhs[:nd] = np.eye(nd)
    c = np.linalg.solve(np.vstack([H0[:nd], H1[nd:]]), rhs)
    return (H0[nd:] @ c).real, (H1[:nd] @ c).real


def _synthesis(R, mu_in, P):
    """F[i, q, k, r, p] = 1 / (2 mu_q) sum_m c_m t_rp(m phi_k) R^m[(i, r), (q, p)]."""
    M, ni, nq = len(R), R[0].shape[0] // 4, R[0].shape[1] // 4
    ang = (np.outer(np.arange(P), np.arange(M)) % P) * (2 * math.pi / P)
    cm = np.where(np.arange(M) == 0, 1.0, 2.0)
    c, s = np.cos(ang) * cm, np.sin(ang) * cm
    Rs = np.stack(R).reshape(M, ni, 4, nq, 4)
    F = np.empty((ni, nq, P, 4, 4))
    for r in range(4):
        for p in range(4):
            t = c if (r < 2) == (p < 2) else s if p < 2 else -s
            F[:, :, :, r, p] = np.tensordot(t, Rs[:, :, r, :, p], 1).transpose(1, 2, 0)
    return F / (2 * np.asarray(mu_in)[None, :, None, None, None])


def exact(case, seed):
    N, L, M, P = _shapes(case)
    kind = case["kind"]
    if sum(m * (8.0 * n) ** 3 for m, n in zip(M, N)) > EXACT_LIMIT or kind == "adjoint":
        return None  # above the limit it takes too long; the gradients have no plain 64-bit reference
    x = _inputs(case, seed)
    flat, beam = [], []
    level = {}  # stacks: the reflection of what lies beneath, per order
    for l in reversed(range(len(N))):
        g, wg = np.polynomial.legendre.leggauss(N[l])
        mu, alpha = (1 + g) / 2, wg / 2
        mirror = np.tile([1.0, 1.0, -1.0, -1.0], N[l])
        R, Rb = [], []
        for m in range(M[l]):
            mu0, mu_out = x.get("mu0", ()), x.get("mu_out", ())
            up, down = _order(x["coef"][l], min(x["omega"][l], OMEGA_MAX), x["tau"][l], m, mu, alpha, mu0, mu_out)
            n4 = 4 * N[l]
            r, t = up[:n4, :n4], down[:n4, :n4]
            if kind == "stack":
                rt = mirror[:, None] * r  # upward fields stored mirrored: alike from above and below
                X = level.get(m)
                if l == len(N) - 1 and case["base"] != "black":
                    base = np.zeros((n4, n4))
                    if case["base"] == "mueller":
                        base = x["base"][m]
                    elif m == 0:
                        base[::4, ::4] = 2 * x["base"][l]
                    X = mirror[:, None] * base * np.repeat(alpha * mu, 4)[None, :]
                if X is not None:
                    rt = rt + t @ np.linalg.solve(np.eye(n4) - X @ rt, X @ t)
                level[m] = rt
                r = mirror[:, None] * rt
            R.append(r / np.repeat(math.pi * alpha, 4)[None, :])
            Rb.append(up[:, n4:])
        flat.append(_synthesis(R, mu, P[l]).ravel())
        if len(x.get("mu0", ())):
            beam.append(_synthesis(Rb, x["mu0"], P[l]).ravel())
    F = np.concatenate(flat[::-1])
    if kind == "noalloc":
        F = F.reshape(N[0], N[0], P[0], 4, 4)
    if kind == "spectral":
        return {"F": F}
    out = {"F": F, "status": None}
    if beam:
        out["F_beam"] = np.concatenate(beam)
    return out
