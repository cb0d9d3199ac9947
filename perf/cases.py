"""The workloads whose speed this framework is judged by, with their inputs, their exact
results in plain torch (64 bits) and the work they cannot do without.

A case is a dict of plain values.  `kind` says which public entry points a pass calls:

  apply       Lattice.dslash on packed fields (a solver or a measurement program that keeps
              its fields packed)
  operator    Lattice.pack, dslash, unpack: the operator on canonical fields
  cg          Lattice.cg: one linear solve for all right-hand sides
  multishift  Lattice.cg_multishift: the shifted solves of rational HMC
  action      PseudofermionAction forward and backward through torch autograd
  hmc         Lattice.hmc_trajectory with an even-odd pseudofermion
  quenched    Lattice.hmc_trajectory of the pure gauge theory
  configure   a new gauge configuration for FLIC measurements: ape_smear, set_gauge,
              set_fat_gauge (with the clover blocks) and the first operator application

Inputs are the synthetic fields of the package's own benchmark and tests: SU(3) links mixed
0.3 toward the identity, complex Gaussian or point sources, antiperiodic time.
"""
import math

import numpy as np
import torch

from paper_2302_00850_amd import cola
from paper_2302_00850_amd.synth import Synth, point_sources, unit_gauge

C128 = torch.complex128
OPS = {"hop": cola.COLA_OP_HOP, "hop_dag": cola.COLA_OP_HOP_DAG, "m": cola.COLA_OP_M,
       "mdag": cola.COLA_OP_MDAG, "mdagm": cola.COLA_OP_MDAGM, "schur": cola.COLA_OP_SCHUR,
       "schur_dag": cola.COLA_OP_SCHUR_DAG, "schur_normal": cola.COLA_OP_SCHUR_DAGSCHUR}
FULL_OPS = ("m", "mdag", "mdagm")
PREC = {"fp64": cola.COLA_FP64, "fp64_12": cola.COLA_FP64_12, "fp32": cola.COLA_FP32,
        "fp16": cola.COLA_FP16}
SYSTEMS = {"mdagm": cola.COLA_SYS_MDAGM, "schur": cola.COLA_SYS_SCHUR,
           "propagator": cola.COLA_SYS_PROPAGATOR}
SCHEMES = {"fp64": cola.COLA_CG_FP64, "fp32_reliable": cola.COLA_CG_FP32_RELIABLE,
           "fp16_defect": cola.COLA_CG_FP16_DEFECT, "fp32_defect": cola.COLA_CG_FP32_DEFECT}
BC = np.array([[1.0, 0.0], [1.0, 0.0], [1.0, 0.0], [-1.0, 0.0]])
PHASE = (1.0, 1.0, 1.0, -1.0)


def _case(kind, lattice, **more):
    lx, ly, lz, lt = lattice
    return {"kind": kind, "lx": lx, "ly": ly, "lz": lz, "lt": lt, **more}


def listed():
    return [
        # the smallest call: M on a 4^4 test lattice, where launches and host work are all
        dict(_case("apply", (4, 4, 4, 4), op="m", prec="fp64", nrhs=1, kappa=0.12, csw=0.0),
             name="m_fp64_4x4x4x4"),
        # the operator on canonical fields, on a ragged lattice no tile divides, with a
        # number of sources that is neither 1 nor 12
        dict(_case("operator", (20, 18, 14, 30), op="m", prec="fp32", nrhs=5, kappa=0.118,
                   csw=1.0), name="m_clover_fp32_5rhs_ragged"),
        # one application of M^H M to a packed field: the full-lattice operator of an HMC or
        # an eigensolver in plain FP64
        dict(_case("apply", (32, 32, 32, 64), op="mdagm", prec="fp64", nrhs=1, kappa=0.12,
                   csw=0.0), name="mdagm_fp64_32x64"),
        # the even-odd normal operator in FP16 storage on the 12 sources of a propagator
        dict(_case("apply", (32, 32, 32, 64), op="schur_normal", prec="fp16", nrhs=12,
                   kappa=0.12, csw=0.0), name="schur_normal_fp16_12rhs_32x64"),
        # the largest: the clover Schur operator on the benchmark's 48^3 x 96, 12 sources
        dict(_case("apply", (48, 48, 48, 96), op="schur", prec="fp32", nrhs=12, kappa=0.118,
                   csw=1.0), name="schur_clover_fp32_12rhs_48x96"),
        # a small mixed-precision solve (one source), bound by launches and host checks
        dict(_case("cg", (16, 16, 16, 32), system="schur", scheme="fp32_reliable", block=0,
                   nrhs=1, point=False, kappa=0.12, csw=0.0, tol=1e-12),
             name="cg_fp32_reliable_16x32"),
        # the 12 propagators of a configuration: clover, FP32 inner solves, FP64 outer
        dict(_case("cg", (24, 24, 24, 48), system="propagator", scheme="fp32_defect", block=0,
                   nrhs=12, point=True, kappa=0.118, csw=1.0, tol=1e-12),
             name="propagators_clover_24x48"),
        # the 12 shifted systems of a rational approximation
        dict(_case("multishift", (24, 24, 24, 48), nshift=12, system="schur", kappa=0.12,
                   csw=0.0, tol=1e-10), name="multishift_12_24x48"),
        # the pseudofermion action and its gradient with respect to the links
        dict(_case("action", (16, 16, 16, 32), kappa=0.12, csw=0.0, tol=1e-12),
             name="action_gradient_16x32"),
        # an HMC trajectory with fermions: two time scales, mixed-precision solves
        dict(_case("hmc", (24, 24, 24, 48), beta=5.6, kappa=0.12, eps=0.04, nsteps=5, n_gauge=4,
                   integrator="leapfrog_mts", scheme="fp32_reliable", tol=1e-12),
             name="hmc_two_scales_24x48"),
        # the quenched sampler's small lattice: hundreds of short launches
        dict(_case("quenched", (8, 8, 8, 8), beta=6.0, eps=0.05, nsteps=20, n_gauge=1,
                   integrator="omelyan", cold=True), name="quenched_8x8"),
        # a new configuration for FLIC measurements: smearing, packing, clover blocks, M
        dict(_case("configure", (24, 24, 24, 48), alpha=0.7, nsweeps=4, prec="fp32", nrhs=1,
                   kappa=0.118, csw=1.0), name="flic_configure_24x48"),
    ]


def _draw_lattice(rng, vmin, vmax):
    """Even extents of a volume spread over its logarithm; ragged as often as not."""
    v = math.exp(rng.uniform(math.log(vmin), math.log(vmax)))
    base = (v / 2.0) ** 0.25
    step = rng.choice((2, 2, 4, 8)) if base >= 8 else 2
    ext = [max(step, step * round(base * rng.uniform(0.8, 1.25) / step)) for _ in range(3)]
    lt = max(4, 2 * round(v / (ext[0] * ext[1] * ext[2]) / 2.0))
    return ext[0], ext[1], ext[2], min(lt, 96)


def draw(rng):
    kind = rng.choice(("apply", "apply", "apply", "operator", "cg", "cg", "multishift",
                       "action", "hmc", "quenched", "configure"))
    csw = float(rng.choice((0, 1)))
    kappa = 0.118 if csw else 0.12
    if kind in ("apply", "operator"):
        nrhs = rng.choice((1, 1, 2, 3, 4, 5, 6, 8, 11, 12, 12, 12, 16))
        vmax = 2.0 ** 21 if kind == "apply" else 2.0 ** 20 / max(1, nrhs / 4)
        ops = sorted(OPS) if kind == "apply" else ["m", "mdag", "mdagm"]
        return _case(kind, _draw_lattice(rng, 256, vmax), op=rng.choice(ops),
                     prec=rng.choice(("fp64", "fp64_12", "fp32", "fp32", "fp16")), nrhs=nrhs,
                     kappa=kappa, csw=csw)
    if kind == "cg":
        nrhs = rng.choice((1, 1, 2, 4, 12, 12))
        system = rng.choice(("mdagm", "schur", "schur", "propagator", "propagator"))
        scheme = rng.choice(sorted(SCHEMES))
        vmax = 131072 if system == "mdagm" or scheme == "fp64" else 331776
        block = 1 if nrhs == 12 and scheme.endswith("defect") and system != "mdagm" \
            and rng.random() < 0.3 else 0
        return _case("cg", _draw_lattice(rng, 4096, vmax), system=system, scheme=scheme,
                     block=block, nrhs=nrhs, point=nrhs == 12, kappa=kappa, csw=csw, tol=1e-12)
    if kind == "multishift":
        return _case("multishift", _draw_lattice(rng, 4096, 331776), nshift=rng.randint(2, 16),
                     system=rng.choice(("schur", "mdagm")), kappa=kappa, csw=csw, tol=1e-10)
    if kind == "action":
        return _case("action", _draw_lattice(rng, 4096, 262144), kappa=0.12, csw=0.0, tol=1e-12)
    if kind == "hmc":
        integrator = rng.choice(("leapfrog", "omelyan", "leapfrog_mts"))
        return _case("hmc", _draw_lattice(rng, 4096, 262144), beta=5.6, kappa=0.12, eps=0.02,
                     nsteps=rng.randint(2, 3), n_gauge=rng.randint(2, 4), integrator=integrator,
                     scheme=rng.choice(("fp64", "fp32_reliable")), tol=1e-12)
    if kind == "quenched":
        integrator = rng.choice(("leapfrog", "omelyan", "leapfrog_mts"))
        return _case("quenched", _draw_lattice(rng, 2048, 2.0 ** 20), beta=6.0, eps=0.05,
                     nsteps=rng.randint(2, 8), n_gauge=rng.randint(1, 4), integrator=integrator,
                     cold=False)
    return _case("configure", _draw_lattice(rng, 4096, 2.0 ** 19), alpha=0.7,
                 nsweeps=rng.randint(1, 6), prec=rng.choice(("fp64", "fp32")),
                 nrhs=rng.choice((1, 4)), kappa=kappa, csw=csw)


# ------------------------------------------------------------------ inputs

def _dims(c):
    return c["lx"], c["ly"], c["lz"], c["lt"]


def _site_shape(c):
    return c["lt"], c["lz"], c["ly"], c["lx"]


def _volume(c):
    return c["lx"] * c["ly"] * c["lz"] * c["lt"]


def _gaussian(gen, shape):
    z = torch.empty(shape, dtype=C128, device="cuda")
    torch.view_as_real(z).normal_(0.0, math.sqrt(0.5), generator=gen)
    return z


def _inputs(c, seed):
    """The fields of a case, from the seed alone: links U, spinors psi, momenta P."""
    s = Synth(seed, device="cuda", rng="torch")
    if c["kind"] == "quenched" and c["cold"]:
        f = {"U": unit_gauge(_dims(c), device="cuda")}
    else:
        f = {"U": s.gauge(_dims(c))}
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 1)
    nrhs = c.get("nrhs", 1)
    if c["kind"] == "cg" and c["point"]:
        # the 12 spin-colour point sources at a site of the seed's choice
        at = [int(v) for v in np.random.RandomState(seed % 2**31).randint(0, _dims(c))]
        b = point_sources(_dims(c), device="cuda")[:nrhs]
        f["psi"] = torch.roll(b, (at[3], at[2], at[1], at[0]), (1, 2, 3, 4)).contiguous()
    elif c["kind"] != "quenched":
        f["psi"] = _gaussian(gen, (nrhs,) + _site_shape(c) + (4, 3))
    if c["kind"] in ("hmc", "quenched"):
        f["P"] = s.momenta(_dims(c))
    if c["kind"] == "action":  # the heat bath phi = M^H eta
        f["psi"] = _Plain(f["U"], c["kappa"]).m(f["psi"], dag=True)
    if c["kind"] == "hmc":  # phi_e = S^H eta_e
        plain = _Plain(f["U"], c["kappa"])
        f["psi"] = plain.schur(plain.even(f["psi"]), dag=True)
    return f


def prepare(c, seed):
    f = _inputs(c, seed)
    kind = c["kind"]
    lat = cola.Lattice(_dims(c), c.get("kappa", 0.12), BC, c.get("csw", 0.0))
    st = {"case": c, "lat": lat}
    if kind in ("apply", "operator", "cg", "multishift"):
        lat.set_gauge(f["U"])
    if kind == "apply":
        full = c["op"] in FULL_OPS
        parity = -1 if full else (1 if c["op"] in ("hop", "hop_dag") else 0)
        prec = PREC[c["prec"]]
        st["in"] = lat.pack(f["psi"], prec, parity)
        st["out"] = lat.empty_packed(prec, c["nrhs"], -1 if full else 0)
    elif kind in ("operator", "cg"):
        st["psi"] = f["psi"]
    elif kind == "multishift":
        st["psi"] = f["psi"][0]
        st["shifts"] = _shifts(c)
    elif kind == "action":
        st["U"], st["psi"] = f["U"].requires_grad_(True), f["psi"][0]
    elif kind in ("hmc", "quenched"):
        st["U"], st["P"] = f["U"], f["P"]
        st["phi"] = f["psi"][0].contiguous() if kind == "hmc" else None
    else:
        st["U"], st["psi"] = f["U"], f["psi"]
    del f
    if _volume(c) > 4 * 2**20:
        torch.cuda.empty_cache()  # the generator's temporaries
    return st


def _shifts(c):
    return [0.0] + [float(v) for v in np.geomspace(1e-3, 3.0, c["nshift"] - 1)]


# ------------------------------------------------------------------ one pass

def _values(packed, prec, blocks):
    """A packed field as its numbers: one array, or for FP16 halves and site scales."""
    if prec in (cola.COLA_FP64, cola.COLA_FP64_12):
        return packed.view(torch.float64)
    if prec == cola.COLA_FP32:
        return packed.view(torch.float32)
    out = []
    for blk in packed.view(blocks, -1):
        n = blk.numel() // 13 * 12
        out += [blk[:n].view(torch.float16), blk[n:].view(torch.float32)]
    return out


def run(st):
    c, lat, kind = st["case"], st["lat"], st["case"]["kind"]
    if kind == "apply":
        prec, full = PREC[c["prec"]], c["op"] in FULL_OPS
        lat.dslash(st["out"], st["in"], OPS[c["op"]], -1 if full else 0, prec, c["nrhs"])
        return _values(st["out"], prec, 2 if full else 1)
    if kind == "operator":
        prec = PREC[c["prec"]]
        packed = lat.pack(st["psi"], prec)
        out = lat.empty_packed(prec, c["nrhs"])
        lat.dslash(out, packed, OPS[c["op"]], -1, prec, c["nrhs"])
        return lat.unpack(out, prec, c["nrhs"])
    if kind == "cg":
        return lat.cg(st["psi"], system=SYSTEMS[c["system"]], scheme=SCHEMES[c["scheme"]],
                      tol=c["tol"], block=c["block"])[0]
    if kind == "multishift":
        return lat.cg_multishift(st["psi"], st["shifts"], system=SYSTEMS[c["system"]],
                                 tol=c["tol"])[0]
    if kind == "action":
        st["U"].grad = None
        s = cola.PseudofermionAction.apply(st["U"], st["psi"], lat, c["tol"])
        s.backward()
        return {"S": s.detach(), "grad": st["U"].grad}
    if kind in ("hmc", "quenched"):
        # the Metropolis step keeps the old fields, so the trajectory moves copies
        U, P = st["U"].clone(), st["P"].clone()
        more = {} if kind == "quenched" else {"phi": st["phi"], "cg_tol": c["tol"], "eo": True,
                                              "cg_scheme": SCHEMES[c["scheme"]]}
        info = lat.hmc_trajectory(U, P, c["beta"], c["eps"], c["nsteps"],
                                  integrator=c["integrator"], n_gauge=c["n_gauge"], **more)
        return {"U": U, "P": P, "H0": info["H0"], "H1": info["H1"]}
    prec = PREC[c["prec"]]
    F = lat.ape_smear(st["U"], c["alpha"], c["nsweeps"])
    lat.set_gauge(st["U"])
    lat.set_fat_gauge(F)
    packed = lat.pack(st["psi"], prec)
    out = lat.empty_packed(prec, c["nrhs"])
    lat.dslash(out, packed, cola.COLA_OP_M, -1, prec, c["nrhs"])
    return {"F": F, "M": lat.unpack(out, prec, c["nrhs"])}


# ------------------------------------------------------------------ necessary work

def work(c):
    """Bytes and flops of one pass.  Every field of an operator application is read or
    written once; an iterative solve streams its operator and its vectors once per
    iteration (the iteration counts of the synthetic fields: 60 to 110 on even sites)."""
    V, kind = float(_volume(c)), c["kind"]
    nrhs = c.get("nrhs", 1)
    spin = {"fp64": 192.0, "fp64_12": 192.0, "fp32": 96.0, "fp16": 52.0}
    link = {"fp64": 144.0, "fp64_12": 96.0, "fp32": 48.0, "fp16": 24.0}
    clov = {"fp64": 576.0, "fp64_12": 576.0, "fp32": 288.0, "fp16": 288.0}

    def op_work(op, prec):
        # links once per use of the operator D on each parity: 4 V links per full hop
        hops = {"hop": 0.5, "hop_dag": 0.5, "m": 1, "mdag": 1, "mdagm": 2, "schur": 1,
                "schur_dag": 1, "schur_normal": 2}[op]
        ends = 2 * V if op in FULL_OPS else V
        cl = V * hops * clov[prec] if c.get("csw") and op not in ("hop", "hop_dag") else 0.0
        links = min(hops, 1.0) * 4 * V * link[prec]
        return links + ends * spin[prec] * nrhs + min(cl, V * clov[prec]), \
            hops * V * nrhs * (1320.0 + 48.0 + (552.0 if cl else 0.0))

    def cg_iteration(prec, system):
        # operator, and x, r, p read and written (one block on even sites, two in full)
        b, f = op_work("mdagm" if system == "mdagm" else "schur_normal", prec)
        n = V if system == "mdagm" else V / 2
        return b + 6 * n * spin[prec] * nrhs, f + 12 * 24 * n * nrhs

    canon = 192.0 * V * nrhs  # one canonical field
    if kind == "apply":
        b, f = op_work(c["op"], c["prec"])
        return {"bytes": b, "flops": f}
    if kind == "operator":
        b, f = op_work(c["op"], c["prec"])
        return {"bytes": 2 * canon + b - 2 * V * spin[c["prec"]] * nrhs, "flops": f}
    if kind in ("cg", "multishift"):
        n = 240 if c["system"] == "mdagm" else 90
        prec = "fp64" if kind == "multishift" or c["scheme"] == "fp64" else \
            "fp16" if c["scheme"] == "fp16_defect" else "fp32"
        b, f = cg_iteration(prec, c["system"])
        if kind == "multishift":
            block = V if c["system"] == "mdagm" else V / 2
            b += c["nshift"] * 4 * block * 192.0 / 2  # half of the shifts stop early
            f += c["nshift"] * 96 * block / 2
            canon *= (1 + c["nshift"]) / 2
        return {"bytes": n * b + 2 * canon, "flops": n * f}
    force = V * (4 * 144.0 + 4 * 144.0)  # links read, force written
    if kind == "action":
        b, f = cg_iteration("fp64", "mdagm")
        return {"bytes": 240 * b + 3 * canon + 4 * V * 144.0 * 2, "flops": 240 * f + V * 4e3}
    if kind in ("hmc", "quenched"):
        per = {"leapfrog": 1, "omelyan": 2, "leapfrog_mts": c["n_gauge"]}[c["integrator"]]
        steps = per * c["nsteps"]
        # per gauge step: force, link update (U, P read, U written), momentum (P, F, P)
        b = steps * (force + V * 4 * 144.0 * 6)
        f = steps * V * 4 * 7e3
        if kind == "hmc":
            n = {"omelyan": 2 * c["nsteps"]}.get(c["integrator"], c["nsteps"]) + 1
            ib, iflops = cg_iteration("fp64" if c["scheme"] == "fp64" else "fp32", "schur")
            b += n * (70 * ib + force + 4 * canon)
            f += n * (70 * iflops + V * 4e3)
        return {"bytes": b, "flops": f}
    b, f = op_work("m", c["prec"])
    pack = V * 4 * (144.0 + link[c["prec"]])
    return {"bytes": c["nsweeps"] * force + 2 * pack + b + 2 * canon +
            (V * (clov[c["prec"]] * 2 + 4 * 144.0) if c["csw"] else 0.0),
            "flops": c["nsweeps"] * V * 4 * 7e3 + 2 * f + (V * 3e4 if c["csw"] else 0.0)}


# ------------------------------------------------------------------ exact results

def _mul(a, b, da=False, db=False):
    """Products of 3 x 3 matrices, either factor as its Hermitian conjugate."""
    a = a.conj().transpose(-1, -2) if da else a
    b = b.conj().transpose(-1, -2) if db else b
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _shift(m, mu, d):
    """m(x + d mu) of a link-like field [t, z, y, x, ...]."""
    return torch.roll(m, -d, 3 - mu)


def _traceless_hermitian(w):
    """Traceless part of i (W - W^H) / 2."""
    x = 0.5j * (w - w.conj().transpose(-1, -2))
    tr = torch.diagonal(x, dim1=-2, dim2=-1).sum(-1)
    return x - (tr / 3.0)[..., None, None] * torch.eye(3, dtype=C128, device=x.device)


class _Plain:
    """The Wilson(-clover) and FLIC operators in plain torch on canonical fields."""

    # g_mu psi for the upper spins, (source spin, factor) of rows 0 and 1, and of the lower
    # spins from the upper ones (rows 2 and 3): chiral basis
    UP = (((3, 1j), (2, 1j)), ((3, -1), (2, 1)), ((2, 1j), (3, -1j)), ((2, 1), (3, 1)))
    LOW = (((1, -1j), (0, -1j)), ((1, 1), (0, -1)), ((0, -1j), (1, 1j)), ((0, 1), (1, 1)))

    def __init__(self, U, kappa, csw=0.0, F=None):
        self.U, self.F, self.kappa = U, F, kappa
        lt, lz, ly, lx = U.shape[:4]
        ar = [torch.arange(n, device=U.device) for n in (lt, lz, ly, lx)]
        par = (ar[0][:, None, None, None] + ar[1][:, None, None] + ar[2][:, None] + ar[3]) % 2
        self.is_even = (par == 0)[..., None, None]
        self.A = self._clover(U if F is None else F, kappa * csw) if csw else None
        self.Ainv = None

    def even(self, v):
        return torch.where(self.is_even, v, torch.zeros((), dtype=C128, device=v.device))

    def odd(self, v):
        return v - self.even(v)

    @staticmethod
    def _edge(v, mu, last, phase):
        if phase != 1.0:
            v.select(4 - mu, v.shape[4 - mu] - 1 if last else 0).mul_(phase)
        return v

    def _term(self, out, v, mu, sg, link, back):
        """out += (1 + sg g_mu) applied to link times v (forward) or, for back, to the
        backward neighbour's link^H v."""
        h = torch.stack([v[..., a, :] + (sg * f) * v[..., s, :]
                         for a, (s, f) in enumerate(self.UP[mu])], -2)
        if back:
            w = sum(link[..., None, b, :].conj() * h[..., b, None] for b in range(3))
            w = self._edge(torch.roll(w, 1, 4 - mu), mu, False, PHASE[mu])
        else:
            w = sum(link[..., None, :, b] * h[..., b, None] for b in range(3))
        out[..., :2, :] += w
        for a, (s, f) in enumerate(self.LOW[mu]):
            out[..., 2 + a, :] += (sg * f) * w[..., s, :]

    def hop(self, psi, dag=False):
        out = torch.zeros_like(psi)
        s = 1.0 if dag else -1.0
        for mu in range(4):
            u = self.U[..., mu, :, :]
            fwd = self._edge(torch.roll(psi, -1, 4 - mu), mu, True, PHASE[mu])
            if self.F is None:
                self._term(out, fwd, mu, s, u, False)
                self._term(out, psi, mu, -s, u, True)
            else:  # F + s g U = [(1 + s g)(F + U) + (1 - s g)(F - U)] / 2
                f = self.F[..., mu, :, :]
                for sg, l in ((s, 0.5 * (f + u)), (-s, 0.5 * (f - u))):
                    self._term(out, fwd, mu, sg, l, False)
                    self._term(out, psi, mu, -sg, l, True)
        return out

    def _clover(self, U, k):
        def strength(mu, nu):
            a, b = U[..., mu, :, :], U[..., nu, :, :]
            # one leaf (the plaquette at x), the others are its transports back to x
            bm, an = _shift(b, mu, 1), _shift(a, nu, 1)
            q = _mul(_mul(a, bm), _mul(b, an), db=True)
            am, bmm = _shift(a, mu, -1), _shift(b, mu, -1)
            q = q + _mul(_mul(b, _shift(an, mu, -1), db=True), _mul(bmm, am, da=True))
            bn = _shift(b, nu, -1)
            q = q + _mul(_mul(_shift(bmm, nu, -1), am), _mul(_shift(am, nu, -1), bn), da=True)
            q = q + _mul(_mul(bn, _shift(a, nu, -1), da=True),
                         _mul(a, _shift(bn, mu, 1), db=True).conj().transpose(-1, -2))
            return -0.25 * _traceless_hermitian(q)

        f = {(m, n): strength(m, n) for m in range(4) for n in range(m + 1, 4)}
        out = []
        for sg in (-1.0, 1.0):
            b3 = f[0, 1] + sg * f[2, 3]
            b2 = f[0, 2] - sg * f[1, 3]
            b1 = f[1, 2] + sg * f[0, 3]
            top = torch.cat([-k * b3, -k * (b1 - 1j * b2)], -1)
            low = torch.cat([-k * (b1 + 1j * b2), k * b3], -1)
            blk = torch.cat([top, low], -2)
            torch.diagonal(blk, dim1=-2, dim2=-1).add_(1.0)
            out.append(blk)
        return out

    def _blocks(self, blocks, v):
        h = v.reshape(v.shape[:-2] + (2, 6))
        y = torch.stack([sum(b[..., :, k] * h[..., i, k, None] for k in range(6))
                         for i, b in enumerate(blocks)], -2)
        return y.reshape(v.shape)

    def a(self, v):
        return v if self.A is None else self._blocks(self.A, v)

    def a_inv(self, v):
        if self.A is None:
            return v
        if self.Ainv is None:
            self.Ainv = []
            for blk in self.A:  # Gauss-Jordan without pivoting (positive definite blocks)
                m = blk.clone()
                for k in range(6):
                    p = 1.0 / m[..., k, k]
                    row = m[..., k, :] * p[..., None]
                    col = m[..., :, k].clone()
                    m -= col[..., :, None] * row[..., None, :]
                    m[..., k, :] = row
                    m[..., :, k] = -col * p[..., None]
                    m[..., k, k] = p
                self.Ainv.append(m)
        return self._blocks(self.Ainv, v)

    def m(self, v, dag=False):
        return self.a(v) - self.kappa * self.hop(v, dag)

    def schur(self, v, dag=False):
        """S on fields that vanish on the odd sites."""
        t = self.a_inv(self.odd(self.hop(v, dag)))
        return self.even(self.a(v) - self.kappa ** 2 * self.hop(t, dag))

    def normal(self, system):
        if system == "mdagm":
            return lambda v: self.m(self.m(v), dag=True)
        return lambda v: self.schur(self.schur(v), dag=True)


def _dot(a, b):
    """Re <a, b> per leading index, broadcastable against the fields."""
    d = (torch.view_as_real(a) * torch.view_as_real(b)).flatten(1).sum(1)
    return d.reshape(-1, 1, 1, 1, 1, 1, 1)


def _bicgstab(op, b, tol=1e-15, max_iter=1000):
    """op x = b by BiCGStab, restarted from the true residual until it stalls."""
    def cdot(u, v):
        return (u.conj() * v).flatten(1).sum(1).reshape(-1, 1, 1, 1, 1, 1, 1)

    x, r = torch.zeros_like(b), b
    norm = _dot(b, b).clamp_min(1e-300)
    for _ in range(3):
        r0, p = r, r
        rho, start = cdot(r0, r), _dot(r, r)
        for k in range(max_iter):
            v = op(p)
            alpha = rho / cdot(r0, v)
            s = r - alpha * v
            t = op(s)
            omega = cdot(t, s) / _dot(t, t)
            x = x + alpha * p + omega * s
            r = s - omega * t
            new = cdot(r0, r)
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            rho = new
            left = float((_dot(r, r) / norm).max())
            if left <= tol * tol or float((_dot(r, r) / start).max()) <= 1e-24:
                break
        r = b - op(x)
        if float((_dot(r, r) / norm).max()) <= tol * tol:
            break
    return x


def _solve(plain, system, b):
    """x of the system that the solver entry points solve, by solves of M or S and its
    adjoint (M^H M x = b: M^H y = b, M x = y)."""
    if system == "mdagm":
        y = _bicgstab(lambda v: plain.m(v, dag=True), b)
        return _bicgstab(plain.m, y)
    if system == "schur":
        y = _bicgstab(lambda v: plain.schur(v, dag=True), plain.even(b))
        return _bicgstab(plain.schur, y)
    bo = plain.odd(b)
    hat = plain.even(b) + plain.kappa * plain.even(plain.hop(plain.a_inv(bo)))
    xe = _bicgstab(plain.schur, hat)
    return xe + plain.a_inv(bo + plain.kappa * plain.odd(plain.hop(xe)))


def _multishift(op, b, shifts):
    """(op + sigma) x = b for every shift from one Krylov space."""
    x = [torch.zeros_like(b) for _ in shifts]
    p = [b.clone() for _ in shifts]
    z, zo = [1.0] * len(shifts), [1.0] * len(shifts)
    r, q, ao, bo = b, b, 1.0, 0.0
    rho = float(_dot(r, r))
    stop = 1e-29 * rho
    while rho > stop:
        aq = op(q)
        alpha = rho / float(_dot(q, aq))
        r = r - alpha * aq
        new = float(_dot(r, r))
        beta = new / rho
        for i, s in enumerate(shifts):
            if z[i] * z[i] * rho <= stop:
                continue
            zn = z[i] * zo[i] * ao / (alpha * bo * (zo[i] - z[i]) + zo[i] * ao * (1 + s * alpha))
            x[i] += (alpha * zn / z[i]) * p[i]
            p[i] = zn * r + (beta * (zn / z[i]) ** 2) * p[i]
            zo[i], z[i] = z[i], zn
        q, ao, bo, rho = r + beta * q, alpha, beta, new
    return torch.cat(x)


def _packed(lattice, field, blocks, out):
    """Canonical [V, 12] of one right-hand side into out[block][c][site] (complex)."""
    lx, ly, lz, lt = lattice
    y, z, t = torch.meshgrid(*(torch.arange(n, device=field.device) for n in (ly, lz, lt)),
                             indexing="ij")
    odd = ((y + z + t) % 2).permute(2, 1, 0)[..., None].expand(lt, lz, ly, lx // 2)
    pair = field.reshape(lt * lz * ly * lx // 2, 2, 12)
    for k, p in enumerate(blocks):
        sel = ((odd + p) % 2 == 1).reshape(-1, 1)
        out[k][:, :pair.shape[0]] = torch.where(sel, pair[:, 1], pair[:, 0]).T


def _staples(U, mu):
    u, total = U[..., mu, :, :], 0
    for nu in range(4):
        if nu != mu:
            v = U[..., nu, :, :]
            vf = _shift(v, mu, 1)
            total = total + _mul(_mul(vf, _shift(u, nu, 1), db=True), v, db=True)
            total = total + _shift(_mul(_mul(u, vf), v, da=True), nu, -1)
    return total


def _gauge_force(U, beta):
    return torch.stack([(-beta / 3.0) * _traceless_hermitian(_mul(U[..., mu, :, :],
                                                                  _staples(U, mu)))
                        for mu in range(4)], -3)


def _gauge_action(U, beta):
    total, n = 0.0, U[..., 0, 0, 0].numel()
    for mu in range(4):
        for nu in range(mu + 1, 4):
            a, b = U[..., mu, :, :], U[..., nu, :, :]
            p = _mul(_mul(a, _shift(b, mu, 1)), _mul(b, _shift(a, nu, 1)), db=True)
            total += float(torch.diagonal(p, dim1=-2, dim2=-1).real.sum())
    return beta * (6.0 * n - total / 3.0)


def _expi(P, eps):
    x = 1j * eps * P
    norm = float(torch.linalg.matrix_norm(x).max())
    n = max(0, math.ceil(math.log2(max(norm, 1e-30) / 0.25)))
    x = x / 2.0 ** n
    eye = torch.eye(3, dtype=C128, device=P.device)
    e = eye.expand_as(x)
    for k in range(18, 0, -1):
        e = eye + _mul(x, e) / k
    for _ in range(n):
        e = _mul(e, e)
    return e


def _fermion_gradient(U, X, Y, kappa):
    """dS/dRe U + i dS/dIm U from the full-lattice solve vectors X and Y."""
    out = []
    for mu in range(4):
        g = 0
        for sg, here, there in ((-1.0, Y, X), (1.0, X, Y)):
            far = torch.roll(there, -1, 4 - mu)
            ha, hb = (torch.stack([v[0][..., a, :] + (sg * f) * v[0][..., s, :]
                                   for a, (s, f) in enumerate(_Plain.UP[mu])], -2)
                      for v in (here, far))
            g = g + sum(ha[..., k, :, None] * hb[..., k, None, :].conj() for k in range(2))
        if PHASE[mu] != 1.0:
            g.select(3 - mu, g.shape[3 - mu] - 1).mul_(PHASE[mu])
        out.append(2.0 * kappa * g)
    return torch.stack(out, -3)


def _trajectory(c, f):
    U, P, beta, eps = f["U"], f["P"], c["beta"], c["eps"]
    phi = f.get("psi")

    def fermions(U):
        plain = _Plain(U, c["kappa"])
        xe = _solve(plain, "schur", phi)
        ye = plain.schur(xe)
        X, Y = xe + plain.odd(plain.hop(xe)), ye + plain.odd(plain.hop(ye, dag=True))
        G = _fermion_gradient(U, X, Y, c["kappa"] ** 2)
        return _traceless_hermitian(_mul(U, G, db=True)), float(_dot(phi, xe))

    def both(U):
        if phi is None:
            return _gauge_force(U, beta), 0.0
        ff, sf = fermions(U)
        return _gauge_force(U, beta) + ff, sf

    def energy(U, P, sf):
        return 0.5 * float(P.abs().square().sum()) + _gauge_action(U, beta) + sf

    h0 = None
    if c["integrator"] == "leapfrog_mts":
        n = c["n_gauge"]
        ff, sf = fermions(U) if phi is not None else (0.0, 0.0)
        h0 = energy(U, P, sf)
        P = P - 0.5 * eps * ff
        for k in range(c["nsteps"]):
            P = P - 0.5 * (eps / n) * _gauge_force(U, beta)
            for j in range(n):
                U = _mul(_expi(P, eps / n), U)
                P = P - (eps / n) * (1.0 if j < n - 1 else 0.5) * _gauge_force(U, beta)
            ff, sf = fermions(U) if phi is not None else (0.0, 0.0)
            P = P - eps * (1.0 if k < c["nsteps"] - 1 else 0.5) * ff
    else:
        lam = 0.1931833275037836 if c["integrator"] == "omelyan" else 0.5
        F, sf = both(U)
        h0 = energy(U, P, sf)
        P = P - lam * eps * F
        for k in range(c["nsteps"]):
            if c["integrator"] == "omelyan":
                U = _mul(_expi(P, 0.5 * eps), U)
                P = P - (1.0 - 2.0 * lam) * eps * both(U)[0]
                U = _mul(_expi(P, 0.5 * eps), U)
            else:
                U = _mul(_expi(P, eps), U)
            F, sf = both(U)
            P = P - lam * eps * (2.0 if k < c["nsteps"] - 1 else 1.0) * F
    return {"U": U, "P": P, "H0": h0, "H1": energy(U, P, sf)}


def _smear(U, alpha, nsweeps):
    def det_inv_dag(x):
        r = [x[..., i, :] for i in range(3)]
        cof = torch.stack([torch.cross(r[1], r[2], dim=-1), torch.cross(r[2], r[0], dim=-1),
                           torch.cross(r[0], r[1], dim=-1)], -2)
        det = (r[0] * cof[..., 0, :]).sum(-1)
        return det, (cof / det[..., None, None]).conj()

    for _ in range(nsweeps):
        v = []
        for mu in range(4):
            total = _staples(U, mu).conj().transpose(-1, -2)
            v.append((1.0 - alpha) * U[..., mu, :, :] + (alpha / 6.0) * total)
        x = torch.stack(v, -3)
        for _ in range(14):  # Newton's iteration for the polar factor
            x = 0.5 * (x + det_inv_dag(x)[1])
        det = det_inv_dag(x)[0]
        U = x * torch.exp(-1j * torch.angle(det) / 3.0)[..., None, None]
    return U


def exact(c, seed):
    kind, V = c["kind"], _volume(c)
    # solves whose plain form takes too long
    if kind == "cg" and V * c["nrhs"] > 9 * 2**20:
        return None
    if kind in ("multishift", "action", "hmc") and V > 9 * 2**17:
        return None
    f = _inputs(c, seed)
    U, psi = f["U"], f.get("psi")
    with torch.no_grad():
        if kind in ("hmc", "quenched"):
            return _trajectory(c, f)
        if kind == "configure":
            F = _smear(U, c["alpha"], c["nsweeps"])
            return {"F": F, "M": _Plain(U, c["kappa"], c["csw"], F).m(psi)}
        plain = _Plain(U, c["kappa"], c.get("csw", 0.0))
        if kind == "cg":
            return _solve(plain, c["system"], psi)
        if kind == "multishift":
            b = plain.even(psi) if c["system"] == "schur" else psi
            return _multishift(plain.normal(c["system"]), b, _shifts(c))
        if kind == "action":
            x = _solve(plain, "mdagm", psi)
            return {"S": _dot(psi, x).reshape(()),
                    "grad": _fermion_gradient(U, x, plain.m(x), c["kappa"])}
        op = {"hop": lambda v: plain.hop(plain.odd(v)),
              "hop_dag": lambda v: plain.hop(plain.odd(v), dag=True),
              "m": plain.m, "mdag": lambda v: plain.m(v, dag=True),
              "mdagm": plain.normal("mdagm"), "schur": lambda v: plain.schur(plain.even(v)),
              "schur_dag": lambda v: plain.schur(plain.even(v), dag=True),
              "schur_normal": lambda v: plain.normal("schur")(plain.even(v))}[c["op"]]
        if kind == "operator":
            return op(psi)
        # packed: per block 12 component arrays of the padded parity volume, sources inside
        blocks = (0, 1) if c["op"] in FULL_OPS else (0,)
        S = (V // 2 + 63) // 64
        S = 64 * (S + 1 if S % 2 == 0 else S)
        out = torch.zeros((len(blocks), 12, S, c["nrhs"]), dtype=C128, device="cuda")
        for q in range(c["nrhs"]):
            _packed(_dims(c), op(psi[q:q + 1])[0].reshape(V, 12), blocks, out[..., q])
        if c["prec"] != "fp16":
            return torch.view_as_real(out).reshape(-1)
        res = []
        for blk in out:  # halves scaled by the site's largest real or imaginary part
            parts = torch.view_as_real(blk)
            top = parts.abs().amax((0, -1))
            scaled = parts / torch.where(top > 0, top, torch.ones_like(top))[..., None]
            res += [scaled.reshape(-1), top.reshape(-1)]
        return res
