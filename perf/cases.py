"""The workloads of this library whose speed is tracked, through its Python entry points.

Each case is one thing that a program using the library does between two
points at which it looks at the result: hand over a configuration, run a
number of overrelaxation (or heat-bath) sweeps, look at theta and F, take the
links back.  The sizes and options are those of the repository's benchmark,
tests and README: 8^4 to 48^3x96, float64, float32 and mixed precision, links
in 12 or 8 reals, Landau and Coulomb gauge, SU(3) and SU(2), one lattice or a
pool of them.

`exact` repeats the iteration of a case in complex128 with plain torch on
whole-lattice arrays.
"""

import math

import numpy as np
import torch

from paper_1412_3655_amd import gf

PREC = {"f64": gf.GF_FP64, "f32": gf.GF_FP32, "mixed": gf.GF_MIXED}
SUBGROUPS = {3: ((0, 1), (0, 2), (1, 2)), 2: ((0, 1),)}


# ------------------------------------------------------------------- cases --


# start: "hot" links have a Haar-random gauge, as a fresh configuration has; "near" ones a small random
# rotation at every site, as after the first sweeps, which is where most sweeps of a run to theta < 1e-12
# are done.  Single precision starts near: from a hot start a rounding can decide which maximum a site
# takes, and two equally good results then differ.


def _case(kind, dims, prec="f64", reals=12, group=3, gauge="landau", mode="exact", omega=1.7, eps=0.8, sweeps=10,
          tune=False, **more):
    return dict(kind=kind, dims=dims, prec=prec, reals=reals, group=group, gauge=gauge, mode=mode, omega=omega,
                eps=eps, start="hot" if prec == "f64" else "near", sweeps=sweeps, tune=tune, **more)


def listed():
    return [
        # one check interval on the smallest lattice of the benchmark: launches and latency
        dict(_case("sweeps", "8x8x8x8", eps=0.6), name="or_8x4_f64"),
        # the benchmark's smallest run to theta < 1e-12, as one call
        dict(_case("fix", "8x8x8x8", eps=0.6, sweeps=400), name="fix_8x4_f64"),
        # uneven extents, half extents that are no multiple of a wavefront, the binomial power, no tuning
        dict(_case("sweeps", "14x18x10x22", prec="f32", mode="binomial", omega=1.9), name="or_ragged_f32"),
        # the headline lattice in float64, tuned as the README does
        dict(_case("sweeps", "32x32x32x32", tune=True, sweeps=20), name="or_32x4_f64"),
        # the bulk phase of mixed precision on it (float32 links in 8 reals, g tracked), then the float64 rebuild
        dict(_case("sweeps", "32x32x32x32", prec="mixed", reals=8, tune=True, sweeps=20), name="or_32x4_mixed8"),
        # the full-size lattice: links far beyond the Infinity Cache
        dict(_case("sweeps", "48x48x48x96", eps=1.0, tune=True), name="or_48x96_f64"),
        dict(_case("sweeps", "48x48x48x96", prec="f32", reals=8, eps=1.0, tune=True), name="or_48x96_f32_8"),
        # Coulomb gauge with the smallest float64 storage
        dict(_case("sweeps", "24x24x24x48", reals=8, gauge="coulomb", tune=True), name="coulomb_24x48_f64_8"),
        # gauge group SU(2)
        dict(_case("sweeps", "32x32x32x64", group=2, sweeps=20), name="su2_32x64_f64"),
        # the simulated-annealing prelude in single precision
        dict(_case("anneal", "32x32x32x32", prec="f32", reals=8, sweeps=10), name="anneal_32x4_f32_8"),
        # theta, F and the plaquette of a configuration that was loaded
        dict(_case("observe", "32x32x32x32"), name="observe_32x4_f64"),
        # jobs of uneven volume through the pool, from host memory and back to it
        dict(_case("pool", "mix", prec="mixed", reals=8, eps=0.6, sweeps=500, jobs=8), name="pool_8_mixed8"),
    ]


def _even(x, least=4):
    return max(least, 2 * int(round(x / 2)))


def draw(rng):
    kind = rng.choices(("sweeps", "fix", "anneal", "observe", "pool"), (12, 2, 2, 2, 2))[0]
    omega = round(rng.uniform(1.0, 1.95), 3)
    eps = round(rng.uniform(0.4, 1.0), 3)
    if kind == "pool":
        return _case("pool", "mix", prec=rng.choice(("mixed", "f64")), reals=8, omega=1.7, eps=round(rng.uniform(0.4, 0.7), 3),
                     sweeps=10 * rng.randint(10, 40), jobs=rng.randint(2, 8))
    if kind == "fix":
        dims = "x".join(str(_even(rng.uniform(6, 13))) for _ in range(4))
        return _case("fix", dims, omega=round(rng.uniform(1.6, 1.8), 3), eps=round(rng.uniform(0.4, 0.6), 3),
                     sweeps=rng.randint(100, 300), mode=rng.choice(("exact", "binomial")))
    side = math.exp(rng.uniform(math.log(4096), math.log(3e6))) ** 0.25
    extents = [_even(side * rng.uniform(0.7, 1.3)) for _ in range(4)]
    dims = "x".join(map(str, extents))
    most = int(4e7 / math.prod(extents))  # sweeps that cost less than the full-size cases
    if kind == "observe":
        return _case("observe", dims, prec=rng.choice(("f64", "f32")), reals=rng.choice((12, 8)), eps=eps,
                     gauge=rng.choice(("landau", "landau", "coulomb")))
    prec = rng.choice(("f64", "f32", "mixed"))
    case = _case(kind, dims, prec=prec, reals=rng.choice((12, 8)), omega=omega, eps=eps, sweeps=max(1, min(rng.randint(1, 20), most)),
                 gauge=rng.choice(("landau", "landau", "landau", "coulomb")), tune=rng.random() < 0.5,
                 mode=rng.choice(("exact", "exact", "exact", "binomial")))
    if kind == "sweeps" and prec != "mixed" and rng.random() < 0.2:
        case.update(group=2, reals=12)
    if kind == "anneal":
        case.update(mode="exact", omega=1.7, sweeps=min(case["sweeps"], 10))
    return case


def _dims(case):
    return tuple(int(d) for d in case["dims"].split("x"))


POOL_SHAPES = ((12, 12, 12, 12), (16, 16, 16, 16), (12, 12, 12, 12), (16, 16, 16, 32))


def _pool_dims(case):
    return [POOL_SHAPES[k % len(POOL_SHAPES)] for k in range(case["jobs"])]


# ------------------------------------------------------------------ inputs --
#
# A matrix field is a complex128 tensor (n, n, sites...): the matrix indices
# come first, so products are elementwise over the sites.


def _mul(a, b):
    out = a[:, 0].unsqueeze(1) * b[0].unsqueeze(0)
    for k in range(1, a.shape[0]):
        out.addcmul_(a[:, k].unsqueeze(1), b[k].unsqueeze(0))
    return out


def _dag(a):
    return a.transpose(0, 1).conj()


def _unit(n, like):
    e = torch.zeros_like(like)
    for i in range(n):
        e[i, i] = 1.0
    return e


def _normal(shape, gen):
    return torch.randn(shape, generator=gen, dtype=torch.float64, device="cuda")


def _rotation(n, shape, gen):
    """Haar-random SU(n) matrices."""
    if n == 2:
        q = _normal((4, *shape), gen)
        q = q / q.square().sum(0, keepdim=True).sqrt()
        a, b = torch.complex(q[0], q[3]), torch.complex(q[2], q[1])
        return torch.stack([torch.stack([a, b]), torch.stack([-b.conj(), a.conj()])])
    r = torch.complex(_normal((2, 3, *shape), gen), _normal((2, 3, *shape), gen))
    r0 = r[0] / r[0].abs().square().sum(0, keepdim=True).sqrt()
    r1 = r[1] - (r0.conj() * r[1]).sum(0, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(0, keepdim=True).sqrt()
    r2 = torch.stack([(r0[(j + 1) % 3] * r1[(j + 2) % 3] - r0[(j + 2) % 3] * r1[(j + 1) % 3]).conj() for j in range(3)])
    return torch.stack([r0, r1, r2])


def _rough(n, shape, eps, gen):
    """exp(i eps H), H random traceless Hermitian with N(0, 1) entries: 12th-order series of eps H / 8, squared thrice."""
    h = torch.zeros((n, n, *shape), dtype=torch.complex128, device="cuda")
    d = _normal((n, *shape), gen)
    d -= d.mean(0, keepdim=True)
    for i in range(n):
        h[i, i] = d[i]
        for j in range(i + 1, n):
            z = torch.complex(_normal(shape, gen), _normal(shape, gen)) / math.sqrt(2.0)
            h[i, j] = z
            h[j, i] = z.conj()
    h *= 1j * eps / 8
    one = _unit(n, h)
    e = one + h / 12
    for k in range(11, 0, -1):
        e = one + _mul(h, e) / k
    for _ in range(3):
        e = _mul(e, e)
    return e


def _field(case, dims, seed):
    """The four link fields U_mu, (n, n, Nt, Nz, Ny, Nx): exp(i eps H) after a random gauge transformation (see start)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, shape = case["group"], tuple(reversed(dims))
    g = _rotation(n, shape, gen) if case["start"] == "hot" else _rough(n, shape, 0.2, gen)
    return [_mul(_mul(g, _rough(n, shape, case["eps"], gen)), _dag(torch.roll(g, -1, -1 - mu))) for mu in range(4)]


def _canonical(U):
    """Canonical float64 links (V, 4, n, n, 2)."""
    n = U[0].shape[0]
    out = torch.empty((U[0][0, 0].numel(), 4, n, n, 2), dtype=torch.float64, device="cuda")
    for mu in range(4):
        out[:, mu] = torch.view_as_real(U[mu].reshape(n, n, -1).permute(2, 0, 1).contiguous())
    return out


def _single(case):
    """Whether the links that come back carry single precision (float32 sweeps, or float64 links rebuilt from float32 g)."""
    return case["prec"] != "f64"


# ------------------------------------------------------------ library side --


def prepare(case, seed):
    mode = gf.GF_OR_EXACT if case["mode"] == "exact" else gf.GF_OR_BINOMIAL1
    if case["kind"] == "pool":
        jobs = []
        for k, dims in enumerate(_pool_dims(case)):
            links = _canonical(_field(case, dims, 1000 * seed + k)).cpu().numpy()
            jobs.append((dims, links))
        pool = gf.Pool(2 << 30, 16, PREC[case["prec"]], check_every=10, mode=mode,
                       reals32=case["reals"] if case["prec"] == "mixed" else 12)
        return dict(case=case, pool=pool, jobs=jobs)
    dims = _dims(case)
    links = _canonical(_field(case, dims, seed))
    torch.cuda.empty_cache()
    lat = gf.Lattice(dims, PREC[case["prec"]], stream=torch.cuda.Stream(),
                     gauge=gf.GF_COULOMB if case["gauge"] == "coulomb" else gf.GF_LANDAU, group=case["group"],
                     storage=case["reals"])
    lat.set_links(links)
    if case["tune"] and case["kind"] == "anneal":
        lat.autotune_anneal(None, n_sweeps=2)
    elif case["tune"]:
        lat.autotune(None, n_sweeps=2)
    return dict(case=case, lat=lat, links=links, out=torch.empty_like(links), mode=mode)


def _scalars(case, theta, F):
    kind = np.float32 if _single(case) else np.float64
    return dict(theta=kind(theta), F=kind(F))


def _taken(case, state):
    """The links back, in the precision that they carry."""
    state["lat"].get_links(state["out"])
    return state["out"].float() if _single(case) else state["out"]


def run(state):
    case = state["case"]
    if case["kind"] == "pool":
        pool, jobs = state["pool"], state["jobs"]
        for k, (dims, links) in enumerate(jobs):
            if not pool.admit(k, dims, links, omega=case["omega"], max_sweeps=case["sweeps"]):
                raise RuntimeError("the pool has no room for job %d" % k)
        got = {}
        while len(got) < len(jobs):
            pool.step()
            for d in pool.poll():
                got[d["job_id"]] = d["result"]
        links = [pool.fetch_links(k) for k in range(len(jobs))]
        if _single(case):
            links = [u.astype(np.float32) for u in links]
        out = [dict(links=u, **_scalars(case, got[k].theta, got[k].F)) for k, u in enumerate(links)]
        if _single(case):
            # hundreds of float32 sweeps end near the rounding floor of theta, where its value is noise
            for o in out:
                del o["theta"]
        return out
    lat = state["lat"]
    lat.set_links(state["links"])
    if case["kind"] == "fix":
        r = lat.fix_until(omega=case["omega"], mode=state["mode"], theta_target=1e-12, max_sweeps=case["sweeps"])
        return dict(links=_taken(case, state), sweeps=r.sweeps, **_scalars(case, r.theta, r.F))
    if case["kind"] == "observe":
        theta, F = lat.measure()
        P = lat.plaquette()
        kind = np.float32 if _single(case) else np.float64
        return dict(P=kind(P), **_scalars(case, theta, F))
    if case["kind"] == "anneal":
        lat.anneal(case["sweeps"], 1.25, 0.5, 7)
    else:
        lat.sweep(case["sweeps"], case["omega"], state["mode"])
    if case["prec"] == "mixed":
        lat.promote_fp64()
    theta, F = lat.measure()
    return dict(links=_taken(case, state), **_scalars(case, theta, F))


# ---------------------------------------------------------- 64-bit results --


def _K(U, directions):
    K = torch.zeros_like(U[0])
    for mu in range(directions):
        K += U[mu]
        K += _dag(torch.roll(U[mu], 1, -1 - mu))
    return K


def _half_sweep(U, colour, even, omega, mode, directions):
    n = U[0].shape[0]
    K = _K(U, directions)
    G = _unit(n, K)
    for i, j in SUBGROUPS[n]:
        a0 = K[i, i].real + K[j, j].real
        a1 = K[i, j].imag + K[j, i].imag
        a2 = K[i, j].real - K[j, i].real
        a3 = K[i, i].imag - K[j, j].imag
        v = (a1 * a1 + a2 * a2 + a3 * a3).sqrt()
        if mode == "exact":
            phi = omega * torch.atan2(v, a0)
            b0, f = torch.cos(phi), -torch.sin(phi) / v
        else:
            m = (a0 * a0 + v * v).sqrt()
            b0, f = 1 - omega + omega * a0 / m, -omega / m
            m = (b0 * b0 + f * f * v * v).sqrt()
            b0, f = b0 / m, f / m
        p, q = torch.complex(b0, f * a3), torch.complex(f * a2, f * a1)
        for M in (G, K):
            x, y = M[i].clone(), M[j].clone()
            M[i] = p * x + q * y
            M[j] = -q.conj() * x + p.conj() * y
    G = torch.where(even if colour == 0 else ~even, G, _unit(n, G))
    for mu in range(4):
        U[mu] = _mul(_mul(G, U[mu]), _dag(torch.roll(G, -1, -1 - mu)))


def _even_sites(U):
    nt, nz, ny, nx = U[0].shape[2:]
    r = [torch.arange(k, device=U[0].device) for k in (nt, nz, ny, nx)]
    s = r[0].view(-1, 1, 1, 1) + r[1].view(-1, 1, 1) + r[2].view(-1, 1) + r[3]
    return s % 2 == 0


def _theta_F(U, gauge):
    n, directions = U[0].shape[0], 3 if gauge == "coulomb" else 4
    K = _K(U, directions)
    D = (K - _dag(K)) / 2j
    tr = sum(D[i, i] for i in range(n)) / n
    for i in range(n):
        D[i, i] -= tr
    th = D.abs().square().sum((0, 1)).sum((1, 2, 3)) / n
    F = sum(U[mu][i, i].real for mu in range(directions) for i in range(n)).sum((1, 2, 3)) / (n * directions)
    per = K[0, 0, 0].numel()
    if gauge == "coulomb":
        return float((th / per).max()), float((F / per).mean())
    return float(th.sum()) / (per * K.shape[2]), float(F.sum()) / (per * K.shape[2])


def _plaquette(U):
    n, total = U[0].shape[0], 0.0
    for mu in range(4):
        for nu in range(mu + 1, 4):
            p = _mul(U[mu], torch.roll(U[nu], -1, -1 - mu))
            q = _mul(U[nu], torch.roll(U[mu], -1, -1 - nu))
            total += float((p * q.conj()).real.sum())
    return total / (6 * n * U[0][0, 0].numel())


def exact(case, seed):
    # a heat bath accepts and rejects by its own rounding; a pool's jobs would take minutes
    if case["kind"] in ("anneal", "pool"):
        return None
    U = _field(case, _dims(case), seed)
    directions = 3 if case["gauge"] == "coulomb" else 4
    even = _even_sites(U)
    if case["kind"] == "observe":
        theta, F = _theta_F(U, case["gauge"])
        return dict(P=_plaquette(U), theta=theta, F=F)
    done = 0
    theta, F = _theta_F(U, case["gauge"])
    while done < case["sweeps"]:
        _half_sweep(U, 0, even, case["omega"], case["mode"], directions)
        _half_sweep(U, 1, even, case["omega"], case["mode"], directions)
        done += 1
        if case["kind"] == "fix" and (done % 10 == 0 or done == case["sweeps"]):
            theta, F = _theta_F(U, case["gauge"])
            if theta < 1e-12:
                break
    if case["kind"] == "sweeps":
        theta, F = _theta_F(U, case["gauge"])
        return dict(links=_canonical(U), theta=theta, F=F)
    return dict(links=_canonical(U), sweeps=done, theta=theta, F=F)


# ------------------------------------------------------------ bytes, flops --

LINK_BYTES = {("f64", 12): 96, ("f64", 8): 64, ("f32", 12): 48, ("f32", 8): 32, ("mixed", 12): 48, ("mixed", 8): 32}


def work(case):
    # 2350 operations per site update is the convention of the method's paper for SU(3); SU(2) by count
    update = 2350 if case["group"] == 3 else 330
    if case["kind"] == "pool":
        sites = sum(math.prod(d) for d in _pool_dims(case))
    else:
        sites = math.prod(_dims(case))
    link = LINK_BYTES[case["prec"], case["reals"]] if case["group"] == 3 else (32 if case["prec"] == "f64" else 16)
    canon = 4 * 2 * case["group"] ** 2 * 8
    out = canon // 2 if _single(case) else canon
    if case["kind"] == "observe":
        # the configuration in, then every link once for theta and F and once for the plaquette
        return dict(bytes=sites * (canon + 2 * 4 * link), flops=sites * (6 * 432 + 8 * 60))
    sweeps = case["sweeps"]
    # a sweep reads and writes every link once (mixed: and g(x)); the configuration comes in and goes out once
    per_sweep = 2 * 4 * link + (2 * 48 if case["prec"] == "mixed" else 0)
    return dict(bytes=sites * (canon + out + sweeps * per_sweep), flops=sites * sweeps * update)
