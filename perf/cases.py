"""Performance cases of the library's public entry points.

Each case is one pass of work that a lattice program has the library do on one
GPU: smear gauge links, take plaquettes, evaluate the shift expression, run
the chain or the Jacobi smearing, smear a batch of lattices, push and pop
fields, evaluate a run-time compiled expression.  ``listed()`` names twelve of
them, ``draw(rng)`` gives others of the same ranges, ``prepare`` makes what a
program has in hand before the call, ``run`` makes the calls, ``work`` says
what a pass cannot do without and ``exact`` computes its results in 64 bits
with torch alone.

The context is the package's own: the stored launch table for the shapes it
holds, the library's default launch geometry for every other shape.
"""

from __future__ import annotations

import math
import random

import torch

import paper_1105_2279_amd as q
from paper_1105_2279_amd import tuning

ALPHA = 0.5           # APE weight
A_PHI, C_CHAIN = 0.3, 0.1  # axpy and chain coefficients
KAPPA = 0.21          # Jacobi hopping parameter
BATCH_CHOICES = ("8x8x8x8", "12x12x12x24", "16x16x16x32", "24x24x24x48")
# one iteration of the smearing listing as an expression
EXPR = "(add f1 (scale s0 (sum 0xF (add (umul m (shift f0 + m)) (shift (uadj m f0) - m)))))"


# ----------------------------------------------------------------- the cases
def _ape(name, L, prec, reals, steps, mask=15, proj="rows", plaq="last", links="haar"):
    """plaq: "none", "last" (qdpx_plaquette on the result) or "every" (of the
    input and of every step, from the smearing call)."""
    return {"name": name, "kind": "ape", "L": L, "prec": prec, "reals": reals, "steps": steps, "mask": mask,
            "proj": proj, "plaq": plaq, "links": links}


def listed():
    return [
        # one step on the smallest lattice: a regression check or a toy study, where
        # launches and host time are everything
        _ape("ape 4^4 f64", "4x4x4x4", "f64", 18, 1, plaq="every"),
        # the shift expression with its norm at the size of one propagator source
        {"name": "shift 16^3x32 f64", "kind": "shift", "L": "16x16x16x32", "prec": "f64", "reals": 18, "mask": 15,
         "sign": 1, "links": "haar"},
        # production smearing before a measurement: ten single-precision steps and the
        # plaquette of the result
        _ape("ape 32^3x64 f32-12", "32x32x32x64", "f32", 12, 10),
        # the same in double with the plaquette history that a smearing study records
        _ape("ape 24^3x48 f64 plaq", "24x24x24x48", "f64", 18, 5, plaq="every"),
        # uneven extents, 18-real single precision links, no plaquette
        _ape("ape 14x18x22x30 f32-18", "14x18x22x30", "f32", 18, 4, plaq="none", links="near"),
        # spatial smearing with the gauge-covariant projection, as for source smearing
        _ape("ape spatial polar f64", "24x24x24x48", "f64", 18, 3, mask=7, proj="polar", plaq="last"),
        # Jacobi smearing of a source, all four directions, the largest lattice of the
        # routine's own benchmark
        {"name": "jacobi 32^3x64 f32-12", "kind": "jacobi", "L": "32x32x32x64", "prec": "f32", "reals": 12,
         "iters": 20, "mask": 15, "links": "haar"},
        # ... in double, in the spatial directions, on extents that no brick divides
        {"name": "jacobi 20^3x40 f64 spatial", "kind": "jacobi", "L": "20x20x20x40", "prec": "f64", "reals": 18,
         "iters": 20, "mask": 7, "links": "near"},
        # the iterated expression with a norm per iteration on the largest lattice
        {"name": "chain 48^3x96 f64", "kind": "chain", "L": "48x48x48x96", "prec": "f64", "reals": 18, "iters": 8,
         "links": "haar"},
        # an ensemble of 64 lattices of four sizes smeared as one job
        {"name": "batch 64 f32-12", "kind": "batch", "lattices": 64, "extents_seed": 1400, "uneven": False,
         "prec": "f32", "reals": 12, "steps": 5},
        # push a configuration and a source into the library's layout and pop them back
        {"name": "push pop 32^3x64 f32-12", "kind": "fields", "L": "32x32x32x64", "prec": "f32", "reals": 12,
         "links": "haar"},
        # an expression the library has no kernel for, compiled at run time
        {"name": "expression 24^3x48 f64", "kind": "jit", "L": "24x24x24x48", "prec": "f64", "reals": 18,
         "links": "haar"},
    ]


def _extents(rng, lo, hi):
    """Extents of a lattice of about lo..hi sites (log-uniform): cubic with
    t twice as long, even, or anything."""
    target = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    style = rng.choice(("cubic", "cubic", "even", "odd"))
    if style == "cubic":
        step = rng.choice((2, 4, 8))
        n = max(step, int(round((target / 2) ** 0.25 / step)) * step)
        L = [n, n, n, 2 * n]
    else:
        b = target ** 0.25
        L = [max(3, int(round(b * rng.uniform(0.65, 1.5)))) for _ in range(4)]
        if style == "even":
            L = [n + n % 2 for n in L]
    while L[0] * L[1] * L[2] * L[3] > hi:
        k = max(range(4), key=lambda d: L[d])
        L[k] -= 2
    return "x".join(str(n) for n in L)


def draw(rng):
    kind = rng.choice(("ape", "ape", "ape", "shift", "chain", "jacobi", "jacobi", "batch", "fields", "jit"))
    prec, reals = rng.choice((("f64", 18), ("f32", 12), ("f32", 18)))
    links = rng.choice(("haar", "near"))
    if kind == "batch":
        return {"kind": kind, "lattices": rng.randint(3, 40), "extents_seed": rng.randrange(10 ** 6),
                "uneven": rng.random() < 0.5, "prec": prec, "reals": reals, "steps": rng.randint(1, 5)}
    L = _extents(rng, 256, 1 << 20)
    base = {"kind": kind, "L": L, "prec": prec, "reals": reals, "links": links}
    if kind == "ape":
        polar = rng.random() < 0.25
        return dict(base, steps=rng.randint(1, 3 if polar else 10), mask=rng.choice((15, 15, 7)),
                    proj="polar" if polar else "rows", plaq=rng.choice(("none", "last", "last", "every")))
    if kind == "shift":
        return dict(base, mask=rng.choice((15, 15, 7)), sign=rng.choice((1, -1)))
    if kind == "chain":
        return dict(base, iters=rng.randint(1, 16))
    if kind == "jacobi":
        return dict(base, iters=rng.randint(5, 40), mask=rng.choice((15, 7)))
    return base


# -------------------------------------------------------------------- helpers
_PROGRAM = {}  # what a program makes once: its context and its compiled expressions


def _context():
    if "ctx" not in _PROGRAM:
        _PROGRAM["ctx"] = tuning.context(0)
    return _PROGRAM["ctx"]


def _kernel(prec, fmt):
    key = (prec, fmt)
    if key not in _PROGRAM:
        _PROGRAM[key] = q.qdpx_jit_compile(_context(), EXPR, prec, fmt, 2, 1)
    return _PROGRAM[key]


def _dims(text):
    return tuple(int(n) for n in text.split("x"))


def _volume(L):
    return L[0] * L[1] * L[2] * L[3]


def _batch_extents(case):
    rng = random.Random(case["extents_seed"])
    out = []
    for _ in range(case["lattices"]):
        L = list(_dims(rng.choice(BATCH_CHOICES)))
        if case["uneven"]:
            L = [max(3, n - rng.choice((0, 1, 2))) for n in L]
        out.append(tuple(L))
    return out


def _types(case):
    prec = q.F64 if case["prec"] == "f64" else q.F32
    return prec, q.LINK12 if case["reals"] == 12 else q.LINK18


def _dtype(case):
    return torch.float64 if case["prec"] == "f64" else torch.float32


def _links(gen, L, kind):
    """Canonical FP64 SU(3) links complex128[V, 4, 3, 3]: rows by Gram-Schmidt,
    the third the conjugate cross product.  Haar (Gaussian rows), or near unit."""
    V = _volume(L)
    z = torch.view_as_complex(torch.randn((V, 4, 2, 3, 2), generator=gen, device="cuda", dtype=torch.float64))
    if kind == "near":
        z = 0.1 * z
        z[:, :, 0, 0] += 1.0
        z[:, :, 1, 1] += 1.0
    u = torch.empty((V, 4, 3, 3), device="cuda", dtype=torch.complex128)
    a = z[:, :, 0] / z[:, :, 0].abs().square().sum(-1, keepdim=True).sqrt()
    b = z[:, :, 1] - (a.conj() * z[:, :, 1]).sum(-1, keepdim=True) * a
    b = b - (a.conj() * b).sum(-1, keepdim=True) * a
    b = b / b.abs().square().sum(-1, keepdim=True).sqrt()
    u[:, :, 0] = a
    u[:, :, 1] = b
    for k in range(3):
        i, j = (k + 1) % 3, (k + 2) % 3
        u[:, :, 2, k] = (a[..., i] * b[..., j] - a[..., j] * b[..., i]).conj()
    return u


def _field(gen, L):
    """Canonical FP64 Dirac field complex128[V, 4, 3], parts N(0, 1)."""
    return torch.view_as_complex(torch.randn((_volume(L), 4, 3, 2), generator=gen, device="cuda",
                                             dtype=torch.float64))


def _inputs(case, seed, n_fields):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000_003 * int(seed) + 17)
    L = _dims(case["L"])
    return L, _links(gen, L, case["links"]), [_field(gen, L) for _ in range(n_fields)]


def _zeros(nbytes):
    # zeroed once, so that the padding of an output is the same in every run
    return torch.zeros(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")


def _pack_links(ctx, L, u, prec, fmt):
    soa = _zeros(q.qdpx_links_bytes(L, prec, fmt))
    q.qdpx_pack_links(ctx, L, torch.view_as_real(u), prec, fmt, soa)
    return soa


def _pack_field(ctx, L, f, prec):
    soa = _zeros(q.qdpx_fermion_bytes(L, prec))
    q.qdpx_pack_fermion(ctx, L, torch.view_as_real(f), prec, soa)
    return soa


def _doubles(n):
    return torch.zeros(n, dtype=torch.float64, device="cuda")


# -------------------------------------------------------------------- prepare
def prepare(case, seed):
    ctx = _context()
    prec, fmt = _types(case)
    s = {"case": dict(case), "ctx": ctx, "prec": prec, "fmt": fmt, "dtype": _dtype(case)}
    kind = case["kind"]
    if kind == "batch":
        Ls = _batch_extents(case)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(1_000_003 * int(seed) + 17)
        sizes = [q.qdpx_links_bytes(L, prec, fmt) for L in Ls]
        arena = _zeros(sum(sizes))
        outs, at = [], 0
        for n in sizes:
            outs.append(arena[at:at + n])
            at += n
        s.update(Ls=Ls, U=[_pack_links(ctx, L, _links(gen, L, "haar"), prec, fmt) for L in Ls], outs=outs,
                 out=arena.view(s["dtype"]), plaq=_doubles(3 * len(Ls)),
                 work=q.alloc_workspace(q.OP_BATCHED, Ls, prec, fmt))
        return s
    n_fields = {"ape": 0, "shift": 2, "chain": 2, "jacobi": 1, "fields": 1, "jit": 2}[kind]
    L, u, fields = _inputs(case, seed, n_fields)
    s["L"] = L
    if kind == "fields":
        s.update(u=torch.view_as_real(u), f=torch.view_as_real(fields[0]), U=_zeros(q.qdpx_links_bytes(L, prec, fmt)),
                 F=_zeros(q.qdpx_fermion_bytes(L, prec)))
        s.update(u2=torch.zeros_like(s["u"]), f2=torch.zeros_like(s["f"]))
        return s
    s["U"] = _pack_links(ctx, L, u, prec, fmt)
    s["F"] = [_pack_field(ctx, L, f, prec) for f in fields]
    if kind == "ape":
        n = case["steps"]
        s.update(out=torch.zeros_like(s["U"]), work=q.alloc_workspace(q.OP_APE, L, prec, fmt, n),
                 plaq=_doubles(3 * (n + 1) if case["plaq"] == "every" else 3),
                 plaq_work=q.alloc_workspace(q.OP_PLAQ, L, prec, fmt))
    elif kind in ("shift", "jit"):
        s.update(out=torch.zeros_like(s["F"][0]), norm=_doubles(1), work=q.alloc_workspace(q.OP_SHIFT, L, prec, fmt))
        if kind == "jit":
            s["kernel"] = _kernel(prec, fmt)
    elif kind == "chain":
        s.update(out=torch.zeros_like(s["F"][0]), norm=_doubles(case["iters"]),
                 work=q.alloc_workspace(q.OP_CHAIN, L, prec, fmt, case["iters"]))
    else:
        s.update(out=torch.zeros_like(s["F"][0]), work=q.alloc_workspace(q.OP_JACOBI, L, prec, fmt))
    return s


# ------------------------------------------------------------------------ run
def run(s):
    c, ctx, prec, fmt = s["case"], s["ctx"], s["prec"], s["fmt"]
    kind, dt = c["kind"], s["dtype"]
    if kind == "batch":
        q.qdpx_ape_smear_batched(ctx, s["Ls"], prec, fmt, s["U"], s["outs"], ALPHA, c["steps"], s["plaq"], s["work"])
        return {"links": s["out"], "plaq": s["plaq"]}
    L = s["L"]
    if kind == "ape":
        every = c["plaq"] == "every"
        q.qdpx_ape_smear(ctx, L, prec, fmt, s["U"], s["out"], ALPHA, c["steps"], plaq=s["plaq"] if every else None,
                         work=s["work"], smear_mask=c["mask"],
                         projection=q.PROJ_POLAR if c["proj"] == "polar" else q.PROJ_GRAM_SCHMIDT)
        if c["plaq"] == "last":
            q.qdpx_plaquette(ctx, L, prec, fmt, s["out"], s["plaq"], s["plaq_work"])
        out = {"links": s["out"].view(dt)}
        if c["plaq"] != "none":
            out["plaq"] = s["plaq"]
        return out
    if kind == "shift":
        q.qdpx_eval_shift_mul_axpy(ctx, L, prec, fmt, s["U"], s["F"][0], s["F"][1], A_PHI, s["out"], s["norm"],
                                   s["work"], dir_mask=c["mask"], sign=c["sign"])
        return {"chi": s["out"].view(dt), "norm": s["norm"]}
    if kind == "jit":
        q.qdpx_jit_eval(ctx, s["kernel"], L, s["U"], s["F"], [KAPPA], s["out"], s["norm"], s["work"])
        return {"out": s["out"].view(dt), "norm": s["norm"]}
    if kind == "chain":
        s["out"].copy_(s["F"][0])  # updated in place; the program keeps its source
        q.qdpx_shift_chain(ctx, L, prec, fmt, s["U"], s["out"], s["F"][1], A_PHI, C_CHAIN, c["iters"], s["norm"],
                           s["work"])
        return {"psi": s["out"].view(dt), "norms": s["norm"]}
    if kind == "jacobi":
        s["out"].copy_(s["F"][0])  # smeared in place; the program keeps its source
        q.qdpx_jacobi_smear(ctx, L, prec, fmt, s["U"], s["out"], KAPPA, c["iters"], 1.0, c["mask"], s["work"])
        return {"chi": s["out"].view(dt)}
    q.qdpx_pack_links(ctx, L, s["u"], prec, fmt, s["U"])
    q.qdpx_pack_fermion(ctx, L, s["f"], prec, s["F"])
    q.qdpx_unpack_links(ctx, L, s["U"], prec, fmt, s["u2"])
    q.qdpx_unpack_fermion(ctx, L, s["F"], prec, s["f2"])
    return {"U": s["U"].view(dt), "F": s["F"].view(dt), "u": s["u2"], "f": s["f2"]}


# ----------------------------------------------------------------------- work
def _site_bytes(case):
    """Bytes of one site's links as read (rows 0 and 1 suffice in double) and
    as written, and of one site's Dirac field."""
    r = 8 if case["prec"] == "f64" else 4
    read = 4 * r * (12 if case["prec"] == "f64" else case["reals"])
    return read, 4 * r * case["reals"], 24 * r


def work(case):
    """Every field once per step or iteration (each needs the whole result of
    the one before), and the arithmetic of the expressions as the method has
    it: rows 0 and 1 of every staple with a plane's upper product formed once
    (1512 flop a link), 72 for the combination, 126 for the row projection; a
    Dirac-field hop 288 flop a site and direction."""
    rd, wr, fb = _site_bytes(case)
    kind = case["kind"]
    ndir = bin(case.get("mask", 15)).count("1")
    if kind == "batch":
        V, n = sum(_volume(L) for L in _batch_extents(case)), case["steps"]
        return {"bytes": V * (n * (rd + wr) + rd), "flops": V * (n * 4 * 1710 + 2808)}
    V = _volume(_dims(case["L"]))
    if kind == "ape":
        n = case["steps"]
        plaqs = {"none": 0, "last": 1, "every": 1 if case["prec"] == "f64" else n + 1}[case["plaq"]]
        link = 1710 * (ndir - 1) / 3 if case["proj"] == "rows" else 2268 * (ndir - 1) / 3 + 3000
        return {"bytes": V * (n * (rd + wr) + plaqs * rd), "flops": V * (n * ndir * link + plaqs * 2808)}
    if kind == "shift":
        return {"bytes": V * (rd * ndir / 4 + 3 * fb), "flops": V * (ndir * 288 + 96)}
    if kind == "chain":
        n = case["iters"]
        return {"bytes": V * n * (rd + 3 * fb), "flops": V * n * (4 * 288 + 144)}
    if kind == "jacobi":
        n = case["iters"]
        return {"bytes": V * n * (rd * ndir / 4 + 3 * fb), "flops": V * n * (2 * ndir * 288 + 48)}
    if kind == "jit":
        return {"bytes": V * (rd + 3 * fb), "flops": V * (8 * 288 + 96)}
    return {"bytes": V * (2 * (4 * 144 + 192) + 2 * (wr + fb)), "flops": 0}


# ---------------------------------------------------------------------- exact
# Links as a list of four complex128[3, 3, Lt, Lz, Ly, Lx], fields as
# complex128[4, 3, Lt, Lz, Ly, Lx]; torch arithmetic in 64 bits.
def _at(f, mu, sign):
    """f at x + mu (sign 1) or x - mu (sign -1)."""
    return torch.roll(f, -sign, -1 - mu)


def _mm(a, b):
    return (a[:, :, None] * b[None]).sum(1)


def _dag(a):
    return a.transpose(0, 1).conj()


def _row2(u):
    a, b = u[0], u[1]
    return torch.stack([(a[(k + 1) % 3] * b[(k + 2) % 3] - a[(k + 2) % 3] * b[(k + 1) % 3]).conj() for k in range(3)])


def _stored_links(case, L, u):
    """The links that the library holds, in 64 bits: as rounded by the link format."""
    out = []
    for mu in range(4):
        m = u[:, mu].permute(1, 2, 0)
        if case["prec"] == "f32":
            m = m.to(torch.complex64).to(torch.complex128)
            if case["reals"] == 12:
                m = torch.cat([m[:2], _row2(m)[None]])
        out.append(m.reshape(3, 3, L[3], L[2], L[1], L[0]).contiguous())
    return out


def _stored_field(case, L, f):
    m = f.permute(1, 2, 0)
    if case["prec"] == "f32":
        m = m.to(torch.complex64).to(torch.complex128)
    return m.reshape(4, 3, L[3], L[2], L[1], L[0]).contiguous()


def _padded(x, V):
    """x[..., V] with its last axis padded with zeros to a multiple of 256."""
    out = torch.zeros(x.shape[:-1] + ((V + 255) // 256 * 256,), device=x.device, dtype=x.dtype)
    out[..., :V] = x
    return out


def _links_out(case, u):
    """Links in the library's layout, as float64."""
    rows = 2 if case["reals"] == 12 else 3
    got = []
    for m in u:
        V = m[0, 0].numel()
        e = _padded(m[:rows].reshape(3 * rows, V), V)
        if case["prec"] == "f32":
            pairs = e[:3 * rows // 2 * 2].reshape(3 * rows // 2, 2, -1).transpose(1, 2)
            got.append(torch.view_as_real(pairs.resolve_conj().contiguous()).reshape(-1))
            e = e[3 * rows // 2 * 2:]
        got.append(torch.view_as_real(e.resolve_conj().contiguous()).reshape(-1))
    return torch.cat(got)


def _field_out(case, f):
    V = f[0, 0].numel()
    e = _padded(f.reshape(12, V), V)
    if case["prec"] == "f32":
        e = e.reshape(6, 2, -1).transpose(1, 2)
    return torch.view_as_real(e.contiguous()).reshape(-1)


def _project_rows(w):
    a = w[0] / w[0].abs().square().sum(0).sqrt()
    b = w[1] - (a.conj() * w[1]).sum(0) * a
    b = b / b.abs().square().sum(0).sqrt()
    u = torch.stack([a, b])
    return torch.cat([u, _row2(u)[None]])


def _project_polar(w):
    def cof(x):
        return torch.stack([torch.stack([x[(i + 1) % 3][(j + 1) % 3] * x[(i + 2) % 3][(j + 2) % 3]
                                         - x[(i + 1) % 3][(j + 2) % 3] * x[(i + 2) % 3][(j + 1) % 3]
                                         for j in range(3)]) for i in range(3)])
    x = w
    for _ in range(12):  # scaled Newton iteration for the unitary factor
        c = cof(x)
        d = (x[0] * c[0]).sum(0)
        y = (c / d).conj()  # inverse, conjugate transposed
        g = (y.abs().square().sum((0, 1)) / x.abs().square().sum((0, 1))) ** 0.25
        x = 0.5 * (g * x + y / g)
    d = (x[0] * cof(x)[0]).sum(0)
    return x * torch.polar(torch.ones_like(d.real), -d.angle() / 3)


def _ape_step(u, mask, polar):
    dirs = [mu for mu in range(4) if mask >> mu & 1]
    out = []
    for mu in range(4):
        if mu not in dirs:
            out.append(u[mu])
            continue
        w = (1 - ALPHA) * u[mu]
        c = ALPHA / (2 * (len(dirs) - 1))
        for nu in dirs:
            if nu == mu:
                continue
            w = w + c * _mm(_mm(u[nu], _at(u[mu], nu, 1)), _dag(_at(u[nu], mu, 1)))
            low = _mm(_mm(_dag(u[nu]), u[mu]), _at(u[nu], mu, 1))
            w = w + c * _at(low, nu, -1)
        out.append(_project_polar(w) if polar else _project_rows(w))
    return out


def _plaquette(u):
    part = [0.0, 0.0]
    for nu in range(4):
        for mu in range(nu):
            a, b = _mm(u[mu], _at(u[nu], mu, 1)), _mm(u[nu], _at(u[mu], nu, 1))
            part[nu == 3] = part[nu == 3] + (a * b.conj()).real.sum()
    V = u[0][0, 0].numel()
    return torch.stack([(part[0] + part[1]) / (18.0 * V), part[0] / (9.0 * V), part[1] / (9.0 * V)])


def _hop(u, psi, mask, fwd=True, bwd=True):
    out = torch.zeros_like(psi)
    for mu in range(4):
        if not mask >> mu & 1:
            continue
        if fwd:
            p = _at(psi, mu, 1)
            out += torch.stack([sum(u[mu][a, b] * p[:, b] for b in range(3)) for a in range(3)], 1)
        if bwd:
            h = torch.stack([sum(u[mu][b, a].conj() * psi[:, b] for b in range(3)) for a in range(3)], 1)
            out += _at(h, mu, -1)
    return out


def _norm2(f):
    return f.abs().square().sum().reshape(1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(1_000_003 * int(seed) + 17)
        links, plaqs = [], []
        for L in _batch_extents(case):
            u = _stored_links(case, L, _links(gen, L, "haar"))
            for _ in range(case["steps"]):
                u = _ape_step(u, 15, False)
            links.append(_links_out(case, u))
            plaqs.append(_plaquette(u))
        return {"links": torch.cat(links), "plaq": torch.cat(plaqs)}
    n_fields = {"ape": 0, "shift": 2, "chain": 2, "jacobi": 1, "fields": 1, "jit": 2}[kind]
    L, aos, fields = _inputs(case, seed, n_fields)
    u = _stored_links(case, L, aos)
    f = [_stored_field(case, L, x) for x in fields]
    if kind == "ape":
        every = case["plaq"] == "every"
        plaqs = [_plaquette(u)] if every else []
        for k in range(case["steps"]):
            u = _ape_step(u, case["mask"], case["proj"] == "polar")
            if every or (case["plaq"] == "last" and k == case["steps"] - 1):
                plaqs.append(_plaquette(u))
        out = {"links": _links_out(case, u)}
        if plaqs:
            out["plaq"] = torch.cat(plaqs)
        return out
    if kind == "shift":
        chi = A_PHI * f[1] + _hop(u, f[0], case["mask"], case["sign"] > 0, case["sign"] < 0)
        return {"chi": _field_out(case, chi), "norm": _norm2(chi)}
    if kind == "jit":
        out = f[1] + KAPPA * _hop(u, f[0], 15)
        return {"out": _field_out(case, out), "norm": _norm2(out)}
    if kind == "chain":
        psi, norms = f[0], []
        for _ in range(case["iters"]):
            chi = A_PHI * f[1] + _hop(u, psi, 15, True, False)
            norms.append(_norm2(chi))
            psi = psi - C_CHAIN * chi
        return {"psi": _field_out(case, psi), "norms": torch.cat(norms)}
    if kind == "jacobi":
        chi = f[0]
        for _ in range(case["iters"]):
            chi = f[0] + KAPPA * _hop(u, chi, case["mask"])
        return {"chi": _field_out(case, chi)}
    back = torch.stack([m.reshape(3, 3, -1) for m in u]).permute(3, 0, 1, 2)
    field = f[0].reshape(4, 3, -1).permute(2, 0, 1)
    return {"U": _links_out(case, u), "F": _field_out(case, f[0]),
            "u": torch.view_as_real(back.resolve_conj().contiguous()), "f": torch.view_as_real(field.contiguous())}
