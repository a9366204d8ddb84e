"""The work a user of the library has it do, as timed cases through its public
entry points, over the sizes the path is used at.

A case is one call (or the few calls that always go together) with everything
a program holds beforehand -- packed links, sources, momenta, workspaces,
rational approximations -- prepared on the GPU:

  hop         D_oe on a batch of packed spinors
  apply_A     the even-site operator m^2 + sigma - D_eo D_oe
  cg          conjugate gradient on one shift, FP64
  multishift  the mixed-precision multi-shift solve of all shifts
  force       the fermion force from the solutions of a multi-shift solve
  gauge       the Symanzik (or Wilson) gauge force
  energy      kinetic energy and gauge action, the pure-gauge part of H
  md          one momentum step and one link step of the integrator
  stout       stout smearing and the force carried back through the levels
  trajectory  a whole RHMC trajectory: heatbath, MD, energies, accept/reject
  layout      packing links and sources, the inner-precision copy, unpacking

Sizes run from 4^4 and 8^4 (tests, tuning runs) over the 16^4 - 32^3 x 48
lattices of everyday runs to 48^4 (one GPU's share of 96^4); extents are even
but otherwise arbitrary, right-hand sides 1 to 8, shifts 1 to 12.
"""
from __future__ import annotations

import functools
import math

import torch

import paper_1801_01473_amd as lq

DEV = "cuda"
C1 = lq.SYMANZIK_C1
RHO = 0.1


def listed():
    return [
        # one hopping term on a test-sized lattice: launch latency only
        case("hop", "8 8 8 8", name="hop_8_f64", prec=64, fmt=18, n=1),
        # the operator on a lattice with no round extents, a few vectors
        case("apply_A", "18 22 20 26", name="apply_A_ragged_f64", prec=64, fmt=18, n=3),
        # the solver's inner operator on one GPU's share of a 96^4 lattice
        case("hop", "48 48 48 48", name="hop_48_f32_8rhs", prec=32, fmt=12, n=8),
        # a single FP64 inversion (a measurement, a test solve) on a small lattice
        case("cg", "16 16 16 16", name="cg_16_f64", n=1, mass=0.05),
        # the solve that RHMC spends its time in: 8 pseudofermions, 12 shifts
        case("multishift", "32 32 32 32", name="multishift_32_8rhs", n=8, shifts=12, mass=0.05),
        # fermion force of one MD step on the paper's lattice
        case("force", "32 32 32 48", name="force_32x48_4pf", n=4, shifts=12),
        # gauge force of one MD substep
        case("gauge", "48 48 48 48", name="gauge_force_48", symanzik=True),
        # gauge and kinetic energy at both ends of a trajectory
        case("energy", "24 24 24 48", name="energy_24x48", symanzik=True),
        # kick and drift of one MD substep
        case("md", "32 32 32 48", name="md_step_32x48"),
        # two smearing levels and the way back, each fermion-force evaluation
        case("stout", "24 24 24 32", name="stout_2_levels_24x32", levels=2),
        # a short trajectory on a lattice small enough to be launch-bound
        case("trajectory", "16 16 16 16", name="trajectory_16", n=1, steps=2, substeps=2, levels=0),
        # bringing a configuration and sources in, and fields out
        case("layout", "32 32 32 32", name="layout_32", n=4),
    ]


def case(kind, extents, **kw):
    return dict(kw, kind=kind, L=extents)


def draw(rng):
    kinds = ["hop", "apply_A", "cg", "multishift", "force", "gauge", "energy", "md", "stout",
             "trajectory", "layout"]
    kind = rng.choice(kinds)
    prec, fmt = rng.choice([(64, 18), (64, 12), (32, 18), (32, 12)])
    n = rng.choice([1, 1, 2, 3, 4, 5, 6, 8])
    shifts = rng.randint(2, 12)
    if kind in ("hop", "apply_A"):
        return case(kind, lattice(rng, 4, 48 if n <= 4 else 40), prec=prec, fmt=fmt, n=n)
    if kind == "cg":
        return case(kind, lattice(rng, 4, 28), n=min(n, 4), mass=rng.choice([0.05, 0.1, 0.3]))
    if kind == "multishift":
        return case(kind, lattice(rng, 6, 28), n=n, shifts=shifts, mass=rng.choice([0.05, 0.1]))
    if kind == "force":
        return case(kind, lattice(rng, 4, 32), n=min(n, 4), shifts=shifts)
    if kind == "gauge":
        return case(kind, lattice(rng, 4, 44), symanzik=rng.random() < 0.8)
    if kind == "energy":
        return case(kind, lattice(rng, 4, 40), symanzik=rng.random() < 0.8)
    if kind == "md":
        return case(kind, lattice(rng, 4, 40))
    if kind == "stout":
        return case(kind, lattice(rng, 4, 26), levels=rng.randint(1, 3))
    if kind == "trajectory":
        return case(kind, lattice(rng, 4, 14), n=rng.choice([1, 2]), steps=rng.randint(1, 3),
                    substeps=rng.randint(1, 3), levels=rng.randint(0, 1))
    return case("layout", lattice(rng, 4, 36), n=n)


def lattice(rng, lo, hi):
    """Even extents whose geometric mean is spread over [lo, hi] on a log scale."""
    mean = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    ext = [min(max(mean * math.exp(rng.uniform(-0.25, 0.25)), 4), 48) for _ in range(4)]
    scale = min(1.0, (hi ** 4 / math.prod(ext)) ** 0.25)
    return " ".join(str(max(4, 2 * int(e * scale / 2))) for e in ext)


# ------------------------------------------------------------------ inputs
# Everything is drawn on the GPU from the seed.  Matrix fields are kept as
# [3][3][T][Z][Y][X], vector fields as [3][T][Z][Y][X], and brought to the
# layouts the library takes at the end.

def extents(c):
    return tuple(int(v) for v in c["L"].split())


def generator(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 64 + stream)
    return g


def hermitian(L, g):
    """Traceless Hermitian sum_a c_a lambda_a / 2 with Gaussian c_a."""
    shape = (L[3], L[2], L[1], L[0])
    c = torch.randn((8,) + shape, generator=g, device=DEV, dtype=torch.float64) * 0.5
    h = torch.zeros((3, 3) + shape, dtype=torch.complex128, device=DEV)
    for (i, j), (a, b) in {(0, 1): (0, 1), (0, 2): (3, 4), (1, 2): (5, 6)}.items():
        h[i, j] = torch.complex(c[a], -c[b])
        h[j, i] = h[i, j].conj()
    h[0, 0] = c[2] + c[7] / math.sqrt(3)
    h[1, 1] = -c[2] + c[7] / math.sqrt(3)
    h[2, 2] = -2 * c[7] / math.sqrt(3)
    return h


def links(L, seed):
    """SU(3) links of a moderately rough configuration: the rows of
    1 + i s H - (s H)^2 / 2, s = 0.5, orthonormalised; [4][3][3][T][Z][Y][X]."""
    out = []
    for mu in range(4):
        h = hermitian(L, generator(seed, mu)) * 0.5j
        e = h + 0.5 * mul(h, h)
        for i in range(3):
            e[i, i] += 1
        r0 = e[0] / e[0].abs().square().sum(0).sqrt()
        r1 = e[1] - (r0.conj() * e[1]).sum(0) * r0
        r1 = r1 / r1.abs().square().sum(0).sqrt()
        r2 = torch.stack([(r0[(j + 1) % 3] * r1[(j + 2) % 3] - r0[(j + 2) % 3] * r1[(j + 1) % 3])
                          for j in range(3)]).conj()
        out.append(torch.stack([r0, r1, r2]))
    return torch.stack(out)


def even_vectors(L, n, seed):
    """[n][3][T][Z][Y][X] complex Gaussian on the even sites, zero on the odd ones."""
    g = generator(seed, 8)
    shape = (n, 3, L[3], L[2], L[1], L[0], 2)
    v = torch.randn(shape, generator=g, device=DEV, dtype=torch.float64) * math.sqrt(0.5)
    return torch.view_as_complex(v) * (parity(L) == 0)


def momenta(L, seed):
    return torch.stack([hermitian(L, generator(seed, 16 + mu)) * math.sqrt(2) for mu in range(4)])


def parity(L):
    ax = [torch.arange(n, device=DEV) for n in (L[3], L[2], L[1], L[0])]
    return (ax[0][:, None, None, None] + ax[1][:, None, None] + ax[2][:, None] + ax[3]) & 1


def natural_links(u):
    """[4][3][3][T][Z][Y][X] -> natural [4][V][3][3]."""
    return u.reshape(4, 3, 3, -1).permute(0, 3, 1, 2).contiguous()


def natural_vectors(v):
    return v.reshape(v.shape[0], 3, -1).permute(0, 2, 1).contiguous()


def packed(L, f, par):
    """Sites of one parity of f [...][T][Z][Y][X] as [...][Vh], in the packed order."""
    t, z, y, x = torch.meshgrid(*[torch.arange(n, device=DEV) for n in (L[3], L[2], L[1], L[0] // 2)],
                                indexing="ij")
    lex = (2 * x + ((y + z + t + par) & 1)) + L[0] * (y + L[1] * (z + L[2] * t))
    return f.reshape(f.shape[:-4] + (-1,))[..., lex.reshape(-1)]


def packed_links(L, u):
    return torch.stack([packed(L, u.reshape((4, 9) + u.shape[3:]), p) for p in (0, 1)])


def rational(n):
    """Shifts log-spaced on [1e-4, 10] and positive residues."""
    s = [10 ** (-4 + 5 * i / max(n - 1, 1)) for i in range(n)]
    return s, [0.225 * v ** 0.75 * (math.log(1e5) / max(n - 1, 1)) for v in s]


@functools.lru_cache(maxsize=None)
def approximation(power, mass, degree):
    return lq.minimax(power, *lq.spectral_bounds(mass), degree)


PREC = {64: lq.F64, 32: lq.F32}
FMT = {18: lq.LINKS18, 12: lq.LINKS12}
TRAJ_MASS = 0.1


def prepare(c, seed):
    L = extents(c)
    g = lq.Geometry(L)
    k = c["kind"]
    s = dict(c, g=g)
    nat = natural_links(links(L, seed))
    if k == "layout":
        s["nat"], s["src"] = nat, natural_vectors(even_vectors(L, c["n"], seed))
        return s
    if k in ("hop", "apply_A"):
        p = PREC[c["prec"]]
        s["U"] = lq.pack_links(g, nat, p, FMT[c["fmt"]])
        s["x"] = lq.pack_spinor(g, natural_vectors(even_vectors(L, c["n"], seed)), 0, p)
        s["out"], s["tmp"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
        return s
    s["U"] = lq.pack_links(g, nat)
    if k in ("cg", "multishift"):
        s["b"] = lq.pack_spinor(g, natural_vectors(even_vectors(L, c["n"], seed)), 0)
        if k == "cg":
            s["params"] = lq.solver_params(mass=c["mass"], tol=1e-10)
        else:
            s["params"] = lq.solver_params(mass=c["mass"], tol=1e-10, inner_prec=lq.F32,
                                           inner_fmt=lq.LINKS12)
            s["sigma"], _ = rational(c["shifts"])
    elif k == "force":
        v = lq.pack_spinor(g, natural_vectors(even_vectors(L, c["n"], seed)), 0)
        sig, s["alpha"] = rational(c["shifts"])
        s["X"] = torch.stack([v / (q + 1.0) for q in sig], 1).contiguous()
        s["F"] = lq.empty_links(g)
    elif k == "gauge":
        s["F"] = lq.empty_links(g)
    elif k == "energy":
        s["H"] = lq.pack_links(g, natural_links(momenta(L, seed)))
    elif k == "md":
        s["H"] = lq.pack_links(g, natural_links(momenta(L, seed)))
        s["F"] = lq.pack_links(g, natural_links(1j * momenta(L, seed + 1)))
        s["eps"] = 0.05
    elif k == "stout":
        s["G"] = lq.pack_links(g, natural_links(raw_gradient(L, seed)))
    elif k == "trajectory":
        s["params"] = lq.solver_params(mass=TRAJ_MASS, tol=1e-10, inner_prec=lq.F32,
                                       inner_fmt=lq.LINKS12)
        s["eighth"] = approximation(0.125, TRAJ_MASS, 8)
        s["quarter"] = approximation(-0.25, TRAJ_MASS, 8)
        s["xi"] = lq.pack_spinor(g, natural_vectors(even_vectors(L, c["n"], seed)), 0)
        s["H"] = lq.pack_links(g, natural_links(momenta(L, seed)))
    return s


def raw_gradient(L, seed):
    g = generator(seed, 24)
    shape = (4, 3, 3, L[3], L[2], L[1], L[0], 2)
    return torch.view_as_complex(torch.randn(shape, generator=g, device=DEV, dtype=torch.float64))


def run(s):
    g, k = s["g"], s["kind"]
    if k == "hop":
        return lq.doe(g, s["U"], s["x"], out=s["out"])
    if k == "apply_A":
        return lq.apply_A(g, s["U"], 0.05, 0.01, s["x"], out=s["out"], tmp=s["tmp"])
    if k == "cg":
        return lq.cg(g, s["params"], s["U"], s["b"])[0]
    if k == "multishift":
        return lq.cg_multishift(g, s["params"], s["U"], s["sigma"], s["b"])[0]
    if k == "force":
        return lq.fermion_force(g, s["U"], s["alpha"], s["X"], out=s["F"])
    if k == "gauge":
        return lq.gauge_force(g, s["U"], 4.0, C1 if s["symanzik"] else 0.0, out=s["F"])
    if k == "energy":
        return {"kinetic": lq.kinetic_energy(g, s["H"]),
                "gauge": lq.gauge_action(g, s["U"], 4.0, C1 if s["symanzik"] else 0.0)}
    if k == "md":
        # repeated passes go forth and back along the same step, so that the
        # momenta stay those of a trajectory
        lq.md_update_momenta(g, s["H"], s["F"], s["eps"])
        lq.md_update_links(g, s["U"], s["H"], s["eps"])
        s["eps"] = -s["eps"]
        return {"H": s["H"], "U": s["U"]}
    if k == "stout":
        chain = lq.stout_smear(g, s["U"], RHO, s["levels"])
        return {"top": chain[-1], "F": lq.stout_force(g, chain, RHO, s["G"])}
    if k == "trajectory":
        U, H = s["U"].clone(), s["H"].clone()
        r = lq.rhmc_trajectory(g, s["params"], U, 5.0, s["eighth"], s["quarter"], s["xi"], H,
                               u=0.0, tau=0.2, nsteps=s["steps"], gauge_substeps=s["substeps"],
                               stout_rho=RHO, stout_levels=s["levels"])
        return {"U": U, "H": H, "H0": r["H0"], "H1": r["H1"]}
    U = lq.pack_links(g, s["nat"])
    V = lq.convert_links(g, U, lq.F64, lq.LINKS18, lq.F32, lq.LINKS12)
    b = lq.pack_spinor(g, s["src"], 0)
    return {"U": U, "U12": V, "b": b, "back": lq.unpack_links(g, U), "src": lq.unpack_spinor(g, b, 0)}


# ------------------------------------------------------------------ least work

MM = 198.0  # real operations of one 3 x 3 complex product


def iterations(mass, sigma):
    """Conjugate-gradient iterations to 1e-10 on a spectrum that fills
    [mass^2 + sigma, mass^2 + sigma + 16] (rough links reach most of it)."""
    lo = mass * mass + sigma
    return 0.5 * math.sqrt((lo + 16) / lo) * math.log(2e10) * 0.5


def work(c):
    L = extents(c)
    V = math.prod(L)
    k = c["kind"]
    M = 576.0 * V  # one FP64 18-real link field
    if k in ("hop", "apply_A"):
        real = c["prec"] / 8
        vec = 6 * real * (V // 2) * c["n"]
        return {"bytes": 4 * V * c["fmt"] * real + 2 * vec,
                "flops": 570.0 * (V // 2) * c["n"] * (1 if k == "hop" else 2)}
    vec = 48.0 * (V // 2)
    if k == "cg":
        it = iterations(c["mass"], 0.0)
        return {"bytes": M + 2 * vec * c["n"], "flops": it * (1140.0 + 100) * (V // 2) * c["n"]}
    if k == "multishift":
        it = iterations(c["mass"], 1e-4)
        return {"bytes": M + vec * c["n"] * (1 + c["shifts"]),
                "flops": it * (1140.0 + 100) * (V // 2) * c["n"]}
    if k == "force":
        pairs = c["n"] * c["shifts"]
        return {"bytes": 2 * M + vec * pairs, "flops": (570.0 + 8 * 72) * (V // 2) * pairs}
    if k == "gauge":  # per plane and site: 3 quadrants of one or three loops, 3 products a loop
        return {"bytes": 2 * M, "flops": MM * 6 * V * (40 if c["symanzik"] else 9)}
    if k == "energy":
        return {"bytes": 2 * M, "flops": MM * 6 * V * (9 if c["symanzik"] else 2.3)}
    if k == "md":
        return {"bytes": 5 * M, "flops": MM * 4 * V * 5}
    if k == "stout":
        return {"bytes": M * c["levels"] * 2 + M * c["levels"] * 3,
                "flops": MM * 4 * V * c["levels"] * (17 + 13 + 15 + 37)}
    if k == "trajectory":
        solves = 3 + 2 * c["steps"] + 1
        it = iterations(TRAJ_MASS, 0.0)
        return {"bytes": 2 * M + 2 * M, "flops": solves * it * 1240.0 * (V // 2) * c["n"]}
    return {"bytes": M + M + M + M / 3 + M + M + c["n"] * (4 * vec + vec), "flops": 0}


# ------------------------------------------------------------------ 64-bit values

def mul(a, b):
    return torch.stack([torch.stack([a[i, 0] * b[0, j] + a[i, 1] * b[1, j] + a[i, 2] * b[2, j]
                                     for j in range(3)]) for i in range(3)])


def dag(a):
    return a.transpose(0, 1).conj()


def mat_vec(u, v):  # u [3][3]..., v [n][3]...
    return torch.stack([u[i, 0] * v[:, 0] + u[i, 1] * v[:, 1] + u[i, 2] * v[:, 2]
                        for i in range(3)], 1)


def at(f, mu, d):
    """f at x + d mu (the last four axes are t, z, y, x)."""
    return torch.roll(f, -d, -1 - mu)


def phases(L):
    """eta_mu(x) times the sign of the antiperiodic time links, [4][T][Z][Y][X]."""
    ax = [torch.arange(n, device=DEV) for n in (L[3], L[2], L[1], L[0])]
    t, z, y, x = torch.meshgrid(*ax, indexing="ij")
    eta = torch.stack([torch.zeros_like(x), x, x + y, x + y + z])
    sign = 1.0 - 2.0 * (eta & 1).double()
    sign[3] = torch.where(t == L[3] - 1, -sign[3], sign[3])
    return sign


def hop(ph, u, v):
    """D v on the whole lattice."""
    out = torch.zeros_like(v)
    for mu in range(4):
        w = 0.5 * ph[mu] * u[mu]
        out += mat_vec(w, at(v, mu, 1)) - at(mat_vec(dag(w), v), mu, -1)
    return out


def solve(ph, u, diag, b):
    """(diag - D D) x = b on the even sites by conjugate gradient to rounding."""
    dot = lambda p, q: (p.conj() * q).real.flatten(1).sum(1)[:, None, None, None, None, None]  # noqa: E731
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rr = dot(r, r)
    stop = rr.max() * 1e-29
    for it in range(5000):
        w = diag * p - hop(ph, u, hop(ph, u, p))
        a = rr / dot(p, w)
        x += a * p
        r -= a * w
        new = dot(r, r)
        p = r + (new / rr) * p
        rr = new
        if it % 20 == 0 and bool(rr.max() < stop):
            break
    return x


def traceless(w):
    r = 0.5 * (w - dag(w))
    tr = (r[0, 0] + r[1, 1] + r[2, 2]) / 3
    return torch.stack([torch.stack([r[i, j] - tr if i == j else r[i, j] for j in range(3)])
                        for i in range(3)])


def re_tr(a, b):
    """Re Tr[a b^dag] summed over the lattice."""
    return (a.real * b.real + a.imag * b.imag).sum()


def plane_action(ua, ub, a, b, c1):
    """sum of c0 (1 - Re Tr P / 3) + c1 (1 - Re Tr R / 3) over one plane."""
    n = ua[0, 0].numel()
    c = mul(ua, at(ub, a, 1))
    d = mul(ub, at(ua, b, 1))
    s = (1 - 8 * c1) * (n - re_tr(c, d) / 3)
    if c1:
        s = s + c1 * (n - re_tr(mul(ua, at(c, a, 1)), mul(d, at(at(ua, a, 1), b, 1))) / 3)
        s = s + c1 * (n - re_tr(mul(c, at(at(ub, a, 1), b, 1)), mul(ub, at(d, b, 1))) / 3)
    return s


PLANES = [(a, b) for a in range(4) for b in range(a + 1, 4)]


def gauge_force(u, beta, c1):
    """TA(U M) of S_g, the derivative taken by autograd plane by plane."""
    m = torch.zeros_like(u)
    for a, b in PLANES:
        ua, ub = u[a].clone().requires_grad_(), u[b].clone().requires_grad_()
        plane_action(ua, ub, a, b, c1).backward()
        m[a] += ua.grad
        m[b] += ub.grad
    return torch.stack([traceless(mul(u[mu], dag(beta * m[mu]))) for mu in range(4)])


def expm(x):
    """exp of matrices of norm below about one, 24 terms."""
    one = torch.zeros_like(x)
    for i in range(3):
        one[i, i] = 1
    e = one
    for k in range(24, 0, -1):
        e = one + mul(x, e) / k
    return e


def smear(u):
    out = []
    for a in range(4):
        w = 0
        for b in range(4):
            if b != a:
                up = mul(u[b], mul(at(u[a], b, 1), dag(at(u[b], a, 1))))
                dn = mul(dag(u[b]), mul(u[a], at(u[b], a, 1)))
                w = w + up + at(dn, b, -1)
        x = traceless(RHO * mul(w, dag(u[a])))
        out.append(mul(expm(x), u[a]))
    return torch.stack(out)


def exact(c, seed):
    L = extents(c)
    V = math.prod(L)
    k = c["kind"]
    u = links(L, seed)
    if k in ("hop", "apply_A"):
        v = even_vectors(L, c["n"], seed)
        v = v.to(torch.complex64).to(torch.complex128) if c["prec"] == 32 else v
        ph = phases(L)
        if k == "hop":
            return torch.cat([packed(L, hop(ph, u, v[j:j + 1]), 1) for j in range(c["n"])])
        return torch.cat([packed(L, (0.05 ** 2 + 0.01) * w - hop(ph, u, hop(ph, u, w)), 0)
                          for w in v.split(1)])
    if k == "cg":
        if V * c["n"] > 300_000:
            return None
        return packed(L, solve(phases(L), u, c["mass"] ** 2, even_vectors(L, c["n"], seed)), 0)
    if k == "multishift":
        if V * c["n"] > 30_000:
            return None
        b = even_vectors(L, c["n"], seed)
        return torch.stack([packed(L, solve(phases(L), u, c["mass"] ** 2 + q, b), 0)
                            for q in rational(c["shifts"])[0]], 1)
    if k == "force":
        v = even_vectors(L, c["n"], seed)
        sig, al = rational(c["shifts"])
        ph = phases(L)
        # X_ji = phi_j / (sigma_i + 1), so the sum over i factors out
        weight = sum(a / (q + 1.0) ** 2 for q, a in zip(sig, al))
        sgn = 1.0 - 2.0 * parity(L).double()
        out = []
        chi = [hop(ph, u, w) for w in v.split(1)]
        for mu in range(4):
            m = torch.zeros_like(u[mu])
            for x, y in zip(v, chi):
                w = x + y[0]  # even sites hold X, odd sites chi
                m += torch.stack([torch.stack([at(w[i], mu, 1) * w[j].conj() for j in range(3)])
                                  for i in range(3)])
            out.append(traceless(mul(u[mu], weight * ph[mu] * sgn * m)))
        return packed_links(L, torch.stack(out))
    if k == "gauge":
        return packed_links(L, gauge_force(u, 4.0, C1 if c["symanzik"] else 0.0))
    if k == "energy":
        s = sum(plane_action(u[a], u[b], a, b, C1 if c["symanzik"] else 0.0) for a, b in PLANES)
        return {"kinetic": 0.5 * float(momenta(L, seed).abs().square().sum()),
                "gauge": 4.0 * float(s)}
    if k == "md":
        h = momenta(L, seed) + 0.05 * momenta(L, seed + 1)
        new = torch.stack([mul(expm(0.05j * h[mu]), u[mu]) for mu in range(4)])
        return {"H": packed_links(L, h), "U": packed_links(L, new)}
    if k == "stout":
        if V > 500_000:
            return None
        chain = [u]
        for _ in range(c["levels"]):
            chain.append(smear(chain[-1]))
        grad = raw_gradient(L, seed)
        for low in reversed(chain[:-1]):
            w = low.clone().requires_grad_()
            top = smear(w)
            (top.real * grad.real + top.imag * grad.imag).sum().backward()
            grad = w.grad
        f = torch.stack([traceless(mul(u[mu], dag(grad[mu]))) for mu in range(4)])
        return {"top": packed_links(L, chain[-1]), "F": packed_links(L, f)}
    if k == "trajectory":
        return None
    nat = natural_links(u)
    src = natural_vectors(even_vectors(L, c["n"], seed))
    p = packed_links(L, u)
    return {"U": p, "U12": p[:, :, :6], "b": packed(L, even_vectors(L, c["n"], seed), 0),
            "back": nat, "src": src}
