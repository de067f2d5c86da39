"""The work that a user of this framework has it do, as cases that can be timed.

A case is one call, or the few calls that a program makes one after the other, through the public
entry points in paper_0807_0264_amd.api and paper_0807_0264_amd.autograd:

  smear     api.smear: n stout or over-improved stout steps of one field
  grad      autograd.stout_mcg_loss, its value and its gradients (forward and backward)
  fix       api.fix on one field, or api.fix_batch on several fields or on copies of one field
  pipeline  api.precondition_batch: smear, fix, carry back and fix, project, count
  analyse   api.center_project, api.count_vortices and api.vortex_field of a fixed field
  wilson    api.wilson_loops
  convert   api.to_links / from_links and api.to_gauge / from_gauge
  monitor   api.plaquette, api.functional and the check of api.unitarity on one field

Fixes run a set number of sweeps (a tolerance that is never met), so that every run of a case does
the same work.  Fields are thermalised by the seeded heatbath of the package's input generator.
Loops and losses measured with FP32 links are kept as FP32 numbers, those measured with FP64 links as
FP64; fields and transforms are returned as the library holds them.
`exact` repeats the mathematics of each case in 64 bits with plain torch.
"""
import itertools
import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_0807_0264_amd import api, autograd, synth
from paper_0807_0264_amd import _abi

HEATBATH_SWEEPS = 15  # the plaquette is within a few percent of its equilibrium value by then
BETA = 5.7
OMEGA = 1.7
RE_UNIT = 50
# spatial directions of Wilson loops, in the order in which a case takes them
DIRECTIONS = [(1, 0, 0), (1, 1, 0), (2, 1, 0), (1, 1, 1), (2, 1, 1), (2, 2, 1)]


# ---- the cases ------------------------------------------------------------------------
def listed():
    return [
        # smearing before the fix: ten stout steps of the largest field of the benchmark's batch
        dict(name="smear_stout_f32_32x64", kind="smear", lat="32x32x32x64", prec="f32", n=10, rho=0.1, eps=1.0),
        # the paper's over-improved smearing at the paper's volume: a quarter of its 80 steps
        dict(name="smear_oi_f32_20x40", kind="smear", lat="20x20x20x40", prec="f32", n=20, rho=0.06, eps=-0.25),
        # one training step on the smearing parameters and the links, as the benchmark's backward
        dict(name="grad_oi_f32_16", kind="grad", lat="16x16x16x16", prec="f32", n=20, rho=0.06, eps=-0.25,
             ckpt=5),
        # the same in double precision on a lattice whose slices do not fill whole tiles
        dict(name="grad_stout_f64_ragged", kind="grad", lat="12x12x10x6", prec="f64", n=6, rho=0.1, eps=1.0,
             ckpt=4),
        # the fixing loop over the benchmark's four lattices together, three blocks of fifty sweeps
        dict(name="fix_batch_f32", kind="fix", lat="32x32x32x64+24x24x24x48+20x20x20x40+16x16x16x16",
             prec="f32", copies=1, sweeps=150),
        # Gribov copies of one small field, fixed together
        dict(name="copies_f32_16", kind="fix", lat="16x16x16x16", prec="f32", copies=16, sweeps=100),
        # one small field fixed alone, where launches and latency count
        dict(name="fix_f32_8", kind="fix", lat="8x8x8x8", prec="f32", copies=1, sweeps=200),
        # the whole path in double precision (the reference run of a precision comparison)
        dict(name="pipeline_f64_20x40", kind="pipeline", lat="20x20x20x40+16x16x16x16", prec="f64", n=10,
             rho=0.1, eps=1.0, sweeps=12),
        # centre projection, vortex count and vortex removal of the largest fixed field
        dict(name="analyse_f32_32x64", kind="analyse", lat="32x32x32x64", prec="f32"),
        # on- and off-axis Wilson loops of one field of the paper's volume
        dict(name="wilson_f32_20x40", kind="wilson", lat="20x20x20x40", prec="f32", dirs=6, rmax=5, tmax=10),
        # a field and its transform taken in from, and given out to, the interchange layout
        dict(name="convert_f32_24x48", kind="convert", lat="24x24x24x48", prec="f32"),
        # the numbers a program logs for every field it reads, on the smallest lattice in use
        dict(name="monitor_f64_6", kind="monitor", lat="6x4x4x8", prec="f64"),
    ]


def _draw_lattice(rng, vmin, vmax):
    """Even extents, not all equal as a rule, with about as many sites as a draw between the two."""
    while True:
        v = math.exp(rng.uniform(math.log(vmin), math.log(vmax)))
        t_ratio = rng.choice([1.0, 1.0, 2.0, 2.0, 1.5])
        s = (v / t_ratio) ** 0.25
        e = [max(4, 2 * round(s * rng.uniform(0.8, 1.25) / 2)) for _ in range(3)]
        t = max(4, 2 * round(v / (e[0] * e[1] * e[2]) / 2))
        vol = e[0] * e[1] * e[2] * t
        if vmin <= vol <= vmax and t <= 6 * max(e):
            return "x".join(str(k) for k in e + [t])


def draw(rng):
    kind = rng.choice(["smear", "smear", "grad", "fix", "fix", "copies", "pipeline", "analyse", "wilson", "convert",
                       "monitor"])
    prec = rng.choice(["f32", "f32", "f64"])
    stout = rng.random() < 0.5
    rho = round(rng.uniform(0.05, 0.12) if stout else rng.uniform(0.03, 0.06), 3)
    eps = 1.0 if stout else round(rng.uniform(-0.5, 0.5), 2)
    if kind == "smear":
        lat = _draw_lattice(rng, 256, 1 << 21 if prec == "f32" else 1 << 20)
        return dict(kind="smear", lat=lat, prec=prec, n=rng.randint(1, 10 if stout else 4), rho=rho, eps=eps)
    if kind == "grad":
        n = rng.randint(1, 12)
        return dict(kind="grad", lat=_draw_lattice(rng, 256, 1 << 17), prec=prec, n=n, rho=rho, eps=eps,
                    ckpt=rng.randint(1, n))
    if kind == "fix":
        lats = [_draw_lattice(rng, 256, 600000) for _ in range(rng.randint(1, 3))]
        return dict(kind="fix", lat="+".join(lats), prec=prec, copies=1, sweeps=rng.randint(10, 100))
    if kind == "copies":
        return dict(kind="fix", lat=_draw_lattice(rng, 256, 100000), prec=prec, copies=rng.randint(2, 16),
                    sweeps=rng.randint(10, 60))
    if kind == "pipeline":  # in double precision: with FP32 links rounding decides where a fix after smearing ends
        lats = [_draw_lattice(rng, 1000, 200000) for _ in range(rng.randint(1, 3))]
        return dict(kind="pipeline", lat="+".join(lats), prec="f64", n=rng.randint(1, 10), rho=rho, eps=eps,
                    sweeps=rng.randint(4, 12))
    if kind == "wilson":  # averages over sites: lattices large enough for them to mean something
        d = rng.randint(1, 6)
        return dict(kind="wilson", lat=_draw_lattice(rng, 20000, 400000), prec=prec, dirs=d, rmax=rng.randint(2, 4),
                    tmax=rng.randint(3, 10))
    if kind == "monitor":
        return dict(kind="monitor", lat=_draw_lattice(rng, 256, 1 << 20), prec=prec)
    return dict(kind=kind, lat=_draw_lattice(rng, 256, 1 << 21 if prec == "f32" else 1 << 20), prec=prec)


def _lats(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["lat"].split("+")]


def _vol(L):
    return L[0] * L[1] * L[2] * L[3]


def _rmax(case, v):
    lmin = min(_lats(case)[0][:3])
    return min(case["rmax"], lmin // max(v))


# ---- inputs -----------------------------------------------------------------------------
def _field64(L, seed, k=0):
    """A thermalised field in the interchange layout, complex128 on the GPU."""
    return synth.heatbath_field_gpu(L, synth.sub_seed(11, seed, k), BETA, HEATBATH_SWEEPS)


def _inputs64(case, seed):
    """The fields of a case as the library sees them (rounded to its link precision), complex128."""
    out = [_field64(L, seed, k) for k, L in enumerate(_lats(case))]
    return [U.to(torch.complex64).to(torch.complex128) if case["prec"] == "f32" else U for U in out]


def _start64(case, seed, c):
    return synth.haar_gauge_gpu(_lats(case)[0], synth.sub_seed(12, seed), c)


def _fixing64(U, sweeps):
    """A transform that takes U most of the way to the gauge: a few sweeps in plain torch."""
    return _t_fix(U, None, sweeps)[0]


def prepare(case, seed):
    kind, prec = case["kind"], (0 if case["prec"] == "f64" else 1)
    s = dict(case=case)
    U64 = _inputs64(case, seed)
    if kind == "grad":
        ctype, rtype = (torch.complex128, torch.float64) if prec == 0 else (torch.complex64, torch.float32)
        s["U"] = U64[0].to(ctype).requires_grad_(True)
        s["rho"] = torch.tensor(case["rho"], dtype=rtype, requires_grad=True)
        s["eps"] = torch.tensor(case["eps"], dtype=rtype, requires_grad=True)
        s["G"] = api.to_gauge(_fixing64(U64[0], 4))
    elif kind == "convert":
        s["U"] = U64[0].to(torch.complex128 if prec == 0 else torch.complex64)
        s["G"] = _start64(case, seed, 0)
    else:
        s["U"] = [api.to_links(U, prec) for U in U64]
        if kind == "fix" and case["copies"] > 1:
            s["G"] = [api.to_gauge(_start64(case, seed, c)) for c in range(case["copies"])]
        if kind == "analyse":
            s["G"] = api.to_gauge(_fixing64(U64[0], 4))
    return s


# ---- one pass ---------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "smear":
        return api.smear(s["U"][0], case["rho"], case["eps"], case["n"]).data
    if kind == "grad":
        U, rho, eps = s["U"], s["rho"], s["eps"]
        loss = autograd.stout_mcg_loss(U, rho, eps, case["n"], s["G"], case["ckpt"])
        gU, gr, ge = torch.autograd.grad(loss, (U, rho, eps))
        return dict(loss=loss.detach().to(rho.dtype), gU=gU, rho=gr, eps=ge)
    if kind == "fix":
        kw = dict(tol=-1.0, max_sweeps=case["sweeps"], omega=OMEGA, reunit_every=RE_UNIT)
        if case["copies"] > 1:
            Gs, res = api.fix_batch([s["U"][0]] * case["copies"], [G.clone() for G in s["G"]], **kw)
        elif len(s["U"]) > 1:
            Gs, res = api.fix_batch(s["U"], None, **kw)
        else:
            G, r = api.fix(s["U"][0], None, **kw)
            Gs, res = [G], [r]
        return dict(G=[G.data for G in Gs], R=[r["R"] for r in res], theta=[r["theta"] for r in res])
    if kind == "pipeline":
        Gs, Zs, res = api.precondition_batch(s["U"], case["rho"], case["eps"], case["n"], tol=-1.0,
                                             max_sweeps=case["sweeps"], omega=OMEGA, reunit_every=RE_UNIT)
        return dict(G=[G.data for G in Gs], Z=Zs, Rs=[r["smeared"]["R"] for r in res],
                    R=[r["fixed"]["R"] for r in res], vortices=[r["vortices"]["per_plane"] for r in res])
    if kind == "analyse":
        U, G = s["U"][0], s["G"]
        Z, margin = api.center_project(U, G)
        v = api.count_vortices(Z, U.L)
        rem = api.vortex_field(U, G, Z, _abi.MCG_VORTEX_REMOVED)
        return dict(Z=Z, margin=margin, counts=[v["total"]] + v["per_plane"] + v["per_charge"], removed=rem.data)
    if kind == "wilson":
        U = s["U"][0]
        W = [api.wilson_loops(U, [v], _rmax(case, v), min(case["tmax"], U.L[3])) for v in DIRECTIONS[: case["dirs"]]]
        return W if case["prec"] == "f64" else [w.astype(np.float32) for w in W]
    if kind == "convert":
        U, G = api.to_links(s["U"]), api.to_gauge(s["G"])
        return dict(U=U.data, G=G.data, u=api.from_links(U), g=api.from_gauge(G))
    U = s["U"][0]
    return [api.plaquette(U), api.functional(U), api.unitarity(U)[0] < 1e-5]


# ---- what a pass cannot do without --------------------------------------------------------
def work(case):
    kind, sz = case["kind"], (8 if case["prec"] == "f64" else 4)
    Ls = _lats(case)
    V = sum(_vol(L) for L in Ls) * case.get("copies", 1)
    field, gauge = V * 72 * sz, V * 144
    stout = case.get("eps") == 1.0
    step = 4 * V * (3270 if stout else 16338)  # flop of one smearing step
    if kind == "smear":
        return dict(bytes=2 * field * case["n"], flops=step * case["n"])
    if kind == "grad":
        # the forward step reads and writes a field; its adjoint reads U and a gradient and writes one
        return dict(bytes=5 * field * case["n"], flops=4 * step * case["n"])
    if kind == "fix":
        # a sweep reads and writes the links once as two rows each and passes on one g per site
        return dict(bytes=case["sweeps"] * V * (2 * 48 * sz + 12 * sz), flops=case["sweeps"] * V * 2700)
    if kind == "pipeline":
        sw = 2 * case["sweeps"]
        return dict(bytes=2 * field * case["n"] + sw * V * 108 * sz + field + gauge + 4 * V,
                    flops=step * case["n"] + sw * V * 2700)
    if kind == "analyse":
        return dict(bytes=3 * field + 2 * gauge + 3 * 4 * V, flops=V * 4 * (216 + 72 + 432 + 54))
    if kind == "wilson":
        T, b, f = min(case["tmax"], Ls[0][3]), 0, 0
        for v in DIRECTIONS[: case["dirs"]]:
            n = len(_images(v)) * _rmax(case, v)
            b += n * V * 18 * sz * 2
            f += n * V * (216 * sum(v) + 36 * T)
        return dict(bytes=field + b, flops=f)
    if kind == "convert":
        return dict(bytes=4 * field + 4 * gauge, flops=0)
    return dict(bytes=3 * field, flops=V * (6 * 252 + 4 * 8 + 4 * 216))


# ---- the mathematics in 64 bits, with plain torch --------------------------------------------
def _mm(a, b):
    return a[..., :, 0:1] * b[..., 0:1, :] + a[..., :, 1:2] * b[..., 1:2, :] + a[..., :, 2:3] * b[..., 2:3, :]


def _dg(a):
    return a.conj().transpose(-1, -2)


def _tr(a):
    return a[..., 0, 0] + a[..., 1, 1] + a[..., 2, 2]


def _at(F, mu, n):
    """F at x + n mu."""
    return torch.roll(F, -n, 3 - mu)


def _eye(F):
    return torch.eye(3, dtype=F.dtype, device=F.device)


def _soa(U):
    """Interchange links [.., 4, 3, 3] or transforms [.., 3, 3] as the flat even/odd arrays of the library."""
    nmu = 4 if U.dim() == 7 else 1
    Lt, Lz, Ly, Lx = U.shape[:4]
    t, z, y = torch.meshgrid(*(torch.arange(n, device=U.device) for n in (Lt, Lz, Ly)), indexing="ij")
    p0 = ((t + z + y) % 2)[..., None].expand(Lt, Lz, Ly, Lx // 2).reshape(-1)  # parity of the pair's first site
    P = U.reshape(-1, 2, nmu, 9)
    odd = (p0 == 1)[:, None, None]
    even_odd = torch.stack([torch.where(odd, P[:, 1], P[:, 0]), torch.where(odd, P[:, 0], P[:, 1])])  # [par, h, mu, k]
    return torch.view_as_real(even_odd.permute(2, 0, 3, 1).contiguous()).reshape(-1)


def _exp(A):
    B, E = A / 16, _eye(A)
    for k in range(14, 0, -1):
        E = _eye(A) + _mm(B, E.expand_as(B)) / k
    for _ in range(4):
        E = _mm(E, E)
    return E


def _t_smear_step(U, rho, eps):
    links = [U[..., mu, :, :] for mu in range(4)]
    wp, wr = (5.0 - 2.0 * eps) / 3.0, -(1.0 - eps) / 12.0
    rect = not (isinstance(eps, float) and eps == 1.0)
    out = []
    for mu in range(4):
        Um = links[mu]
        Cp = Cr = 0.0
        for nu in range(4):
            if nu == mu:
                continue
            Un = links[nu]
            Unm = _at(Un, mu, 1)
            up = _mm(Un, _at(Um, nu, 1))  # U_nu(x) U_mu(x+nu)
            dn = _mm(_dg(Un), Um)         # at x: U_nu(x)^dag U_mu(x), used at x-nu
            Cp = Cp + _mm(up, _dg(Unm)) + _at(_mm(dn, Unm), nu, -1)
            if rect:
                Umd = _dg(_at(Um, mu, 1))
                Um2, Un2 = _at(Um, mu, 1), _at(Un, mu, 2)
                # ahead: around x+mu .. x+2mu, closed by U_mu(x+mu)^dag
                a_up = _mm(_mm(up, _at(Um2, nu, 1)), _dg(Un2))
                a_dn = _at(_mm(_mm(dn, Um2), Un2), nu, -1)
                Cr = Cr + _mm(a_up + a_dn, Umd)
                # behind: opened by U_mu(x-mu)^dag
                Umb, Unb = _at(Um, mu, -1), _at(Un, mu, -1)
                b_up = _mm(_mm(_mm(Unb, _at(Umb, nu, 1)), _at(Um, nu, 1)), _dg(Unm))
                b_dn = _at(_mm(_mm(_mm(_dg(Unb), Umb), Um), Unm), nu, -1)
                Cr = Cr + _mm(_dg(Umb), b_up + b_dn)
                # two steps along nu
                Unn = _mm(Un, _at(Un, nu, 1))
                Unnm = _at(Unn, mu, 1)
                Cr = Cr + _mm(_mm(Unn, _at(Um, nu, 2)), _dg(Unnm))
                Cr = Cr + _at(_mm(_mm(_dg(Unn), Um), Unnm), nu, -2)
        O = rho * _mm(wp * Cp + (wr * Cr if rect else 0.0), _dg(Um))
        A = 0.5 * (O - _dg(O))
        A = A - (_tr(A) / 3.0)[..., None, None] * _eye(A)
        out.append(_mm(_exp(A), Um))
    return torch.stack(out, dim=4)


def _t_smear(U, rho, eps, n):
    for _ in range(n):
        U = _t_smear_step(U, rho, eps)
    return U


def _t_gauge(U, G):
    return torch.stack([_mm(_mm(G, U[..., mu, :, :]), _dg(_at(G, mu, 1))) for mu in range(4)], dim=4)


def _t_R(W):
    t = _tr(W)
    return (t.real ** 2 + t.imag ** 2).sum() / (9.0 * t.numel())


def _t_X(W):
    X = 0.0
    for mu in range(4):
        F = W[..., mu, :, :]
        B = _at(F, mu, -1)
        X = X + _tr(F).conj()[..., None, None] * F + _tr(B)[..., None, None] * _dg(B)
    return X


def _su2(Y, g, i, j, update):
    a, b, c, d = Y[..., i, i], Y[..., i, j], Y[..., j, i], Y[..., j, j]
    v = torch.stack([a.real + d.real, -(b.imag + c.imag), c.real - b.real, -(a.imag - d.imag)])
    v = v / v.norm(dim=0).clamp_min(1e-300)
    q = OMEGA * v
    q[0] += 1.0 - OMEGA
    q = q / q.norm(dim=0).clamp_min(1e-300)
    s = [torch.complex(q[0], q[3]), torch.complex(q[2], q[1]), torch.complex(-q[2], q[1]), torch.complex(q[0], -q[3])]

    def left(M):
        M = M.clone()
        ri, rj = M[..., i, :].clone(), M[..., j, :].clone()
        M[..., i, :] = s[0][..., None] * ri + s[1][..., None] * rj
        M[..., j, :] = s[2][..., None] * ri + s[3][..., None] * rj
        return M

    return (left(Y) if update else Y), left(g)


def _t_fix(U, G, sweeps):
    """The fixing sweeps from G (identity if None): the transform and the fixed field."""
    W = U if G is None else _t_gauge(U, G)
    I = _eye(U).expand(U.shape[:4] + (3, 3))
    G = I.clone() if G is None else G
    ax = [torch.arange(n, device=U.device) for n in U.shape[:4]]
    par = (ax[0][:, None, None, None] + ax[1][:, None, None] + ax[2][:, None] + ax[3]) % 2
    for _ in range(sweeps):
        for p in (0, 1):
            Y, g = _t_X(W), I
            Y, g = _su2(Y, g, 0, 1, True)
            Y, g = _su2(Y, g, 1, 2, True)
            Y, g = _su2(Y, g, 0, 2, False)
            g = torch.where((par == p)[..., None, None], g, I)
            W = _t_gauge(W, g)
            G = _mm(g, G)
    return G, W


def _t_theta(W):
    X = _t_X(W)
    A = 0.5 * (X - _dg(X))
    A = A - (_tr(A) / 3.0)[..., None, None] * _eye(A)
    return float((A.abs() ** 2).sum() / (A.numel() // 9))


def _steps(v):
    """Unit steps of the staircase from 0 to v: along the axis with steps left whose
    (taken + 1/2) / |v_axis| is smallest, the lower axis on a tie."""
    taken, out = [0, 0, 0], []
    for _ in range(sum(v)):
        a = min((k for k in range(3) if taken[k] < v[k]), key=lambda k: ((2 * taken[k] + 1) / v[k], k))
        taken[a] += 1
        out.append(a + 1)
    return out


def _images(v):
    """Distinct images of the staircase under the 48 axis permutations and reflections, each with the
    images (itself and its reversal, the same averaged loop) it stands for."""
    every = set()
    for p in itertools.permutations(range(3)):
        for sg in itertools.product((1, -1), repeat=3):
            every.add(tuple(sg[a - 1] * (p[a - 1] + 1) for a in _steps(v)))
    out = {}
    for im in sorted(every):
        back = tuple(-q for q in reversed(im))
        out[back if back in out else im] = out.get(back if back in out else im, 0) + 1
    return out


def _t_wilson(U, v, rmax, tmax):
    L = [U[..., mu, :, :].contiguous() for mu in range(4)]
    A = [L[3]]
    for t in range(1, tmax):
        A.append(_mm(A[-1], _at(L[3], 3, t)))
    imgs, W = _images(v), np.zeros((1, rmax, tmax))
    for im, weight in imgs.items():
        d, S, y = [0, 0, 0], None, [0, 0, 0]

        def moved(F, o):
            return torch.roll(F, (-o[0], -o[1], -o[2]), (3, 2, 1))

        for q in im:
            d[abs(q) - 1] += 1 if q > 0 else -1
        for k in range(1, rmax + 1):
            for q in im:
                a = abs(q) - 1
                if q > 0:
                    f = moved(L[a], y)
                    y[a] += 1
                else:
                    y[a] -= 1
                    f = _dg(moved(L[a], y))
                S = f if S is None else _mm(S, f)
            D = [k * e for e in d]
            for t in range(1, tmax + 1):
                P = _mm(S, moved(A[t - 1], D))
                Q = _mm(A[t - 1], _at(S, 3, t))
                W[0, k - 1, t - 1] += weight * float((P.real * Q.real + P.imag * Q.imag).sum())
    return W / (3.0 * sum(imgs.values()) * L[3].numel() / 9)


def exact(case, seed):
    kind = case["kind"]
    V = sum(_vol(L) for L in _lats(case)) * case.get("copies", 1)
    U64 = _inputs64(case, seed)
    if kind == "smear":
        return _soa(_t_smear(U64[0], case["rho"], case["eps"], case["n"]))
    if kind == "grad":
        def rounded(x):
            return float(np.float32(x)) if case["prec"] == "f32" else x

        G = _fixing64(U64[0], 4)
        U = U64[0].clone().requires_grad_(True)
        rho, eps = (torch.tensor(rounded(case[k]), dtype=torch.float64, device=U.device, requires_grad=True)
                    for k in ("rho", "eps"))
        S = U
        for _ in range(case["n"]):
            S = checkpoint(_t_smear_step, S, rho, eps, use_reentrant=False)
        loss = _t_R(_t_gauge(S, G))
        gU, gr, ge = torch.autograd.grad(loss, (U, rho, eps))
        return dict(loss=loss.detach(), gU=gU, rho=gr, eps=ge)
    if kind == "fix":
        if V * case["sweeps"] > 20_000_000 or case["sweeps"] > 20 and case["prec"] == "f32":
            return None  # takes too long, or rounding has grown to the size of the result
        starts = [_start64(case, seed, c) for c in range(case["copies"])] if case["copies"] > 1 else [None] * len(U64)
        done = [_t_fix(U64[min(c, len(U64) - 1)], G, case["sweeps"]) for c, G in enumerate(starts)]
        return dict(G=[_soa(G) for G, _ in done], R=[float(_t_R(W)) for _, W in done],
                    theta=[_t_theta(W) for _, W in done])
    if kind == "pipeline":
        G, Rs, R = [], [], []
        for U in U64:
            g, W = _t_fix(_t_smear(U, case["rho"], case["eps"], case["n"]), None, case["sweeps"])
            Rs.append(float(_t_R(W)))
            g, W = _t_fix(U, g, case["sweeps"])
            R.append(float(_t_R(W)))
            G.append(_soa(g))
        return dict(G=G, Z=None, Rs=Rs, R=R, vortices=None)
    if kind == "analyse":
        W = _t_gauge(U64[0], _fixing64(U64[0], 4))
        t = _tr(W)
        m = torch.round(t.angle() * 1.5 / math.pi)  # the nearest centre phase
        margin = float((math.pi / 3 - (t.angle() - m * (2 * math.pi / 3)).abs()).min())
        z = torch.polar(torch.ones_like(m), m * (2 * math.pi / 3))
        return dict(Z=None, margin=margin, counts=None, removed=_soa(z.conj()[..., None, None] * W))
    if kind == "wilson":
        tmax = min(case["tmax"], _lats(case)[0][3])
        return [_t_wilson(U64[0], v, _rmax(case, v), tmax) for v in DIRECTIONS[: case["dirs"]]]
    if kind == "convert":
        G = _start64(case, seed, 0)
        return dict(U=_soa(U64[0]), G=_soa(G), u=U64[0], g=G)
    U, plaq = U64[0], 0.0
    for mu in range(4):
        for nu in range(mu + 1, 4):
            A, B = U[..., mu, :, :], U[..., nu, :, :]
            plaq += float(_tr(_mm(_mm(A, _at(B, mu, 1)), _dg(_mm(B, _at(A, nu, 1))))).real.sum())
    return [plaq / (18 * V), float(_t_R(U)), None]
