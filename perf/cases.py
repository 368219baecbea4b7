"""What the speed of this framework is measured on: calls through its public
entry points (`paper_2010_01628_amd.lbm`), from a 32^3 validation box to
57 million nodes, over the collisions, storage types, streaming patterns,
boundaries and coupled lattices that it offers.

A case is a dict of plain values; `prepare` makes what a program holds before
the call (input fields on the GPU, the lattice, network or ensemble), `run` is
one pass, `work` what a pass cannot do without, `exact` the same outputs from
plain torch in 64 bits.

`work` counts the state once in and once out of a whole pass and the fields it
returns; the floating-point operations are those of every step.
"""
import math

import numpy as np
import torch

from paper_2010_01628_amd import lbm as L

DEV = "cuda"
F64 = torch.float64


# -- the cases ---------------------------------------------------------------

def listed():
    return [
        # the paper's smallest validation: a shear wave in a 32^3 FP64 box, its fields read every few steps
        dict(name="shear_32_fp64", kind="flow", nx=32, ny=32, nz=32, q=19, precision="fp64", streaming="ab",
             flow="shear", force="none", walls=False, nu=0.05, steps=10, io="moments"),
        # the headline workload: forced Taylor-Green 256^3, single precision, two buffers
        dict(name="taylor_green_256_fp32", kind="flow", nx=256, ny=256, nz=256, q=19, precision="fp32",
             streaming="ab", flow="vortex", force="kolmogorov", walls=False, nu=1e-3, steps=20, io="moments"),
        # a large box in the memory-saving form: half-precision storage, one buffer
        dict(name="taylor_green_384_fp16_aa", kind="flow", nx=384, ny=384, nz=384, q=19, precision="fp16",
             streaming="aa", flow="vortex", force="none", walls=False, nu=1e-3, steps=20, io="moments"),
        # a channel between walls, sides that divide nothing, an odd number of steps
        dict(name="channel_200x101x75_fp32", kind="flow", nx=200, ny=101, nz=75, q=19, precision="fp32",
             streaming="ab", flow="noise", force="uniform", walls=True, nu=0.01, steps=21, io="moments"),
        # the D3Q27 comparison lattice of the Taylor-Green study
        dict(name="taylor_green_128_q27", kind="flow", nx=128, ny=128, nz=128, q=27, precision="fp32",
             streaming="ab", flow="vortex", force="none", walls=False, nu=2e-3, steps=12, io="moments"),
        # learned rates with half-precision storage, resumed from a checkpoint and checkpointed again
        dict(name="learned_192_fp16", kind="learned", nx=192, ny=192, nz=192, q=19, precision="fp16",
             streaming="ab", flow="vortex", force="kolmogorov", walls=False, nu=1e-3, steps=12, io="populations"),
        # the two-phase droplet, from its initial interface
        dict(name="droplet_192", kind="droplet", nx=192, ny=192, nz=192, precision="fp32", steps=16),
        # the Hartmann channel of the magnetic validation
        dict(name="hartmann_32x128x32", kind="hartmann", nx=32, ny=128, nz=32, precision="fp32", steps=50),
        # the Shan-Chen static bubble
        dict(name="bubble_100", kind="bubble", nx=100, ny=100, nz=100, precision="fp32", steps=30),
        # the colour-gradient Rayleigh-Taylor column, from rest
        dict(name="rayleigh_taylor_64", kind="rayleigh_taylor", nx=64, ny=256, nz=64, precision="fp32", steps=24),
        # decaying turbulence in many uneven boxes at once: energies read after a block of steps, and the whole state
        # of one small box to the host
        dict(name="ensemble_32_boxes", kind="ensemble", boxes=32, q=19, learned=False, steps=48),
        # one training iteration's gradient: two samples, rollouts of 16 back-propagated steps
        dict(name="train_rollout_32", kind="train", n=32, nu=3e-4, samples=2, steps=16, energy=1e4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["flow"] * 5 + ["learned", "droplet", "hartmann", "bubble", "rayleigh_taylor", "ensemble",
                                      "train"])
    steps = _log_int(rng, 4, 40)
    if kind in ("flow", "learned"):
        size = [_log_int(rng, 24, 330) for _ in range(3)]
        if rng.random() < 0.4:  # sides that the lattice's users like
            size = [rng.choice([32, 48, 64, 96, 128, 160, 192, 256]) for _ in range(3)]
        while size[0] * size[1] * size[2] > 17_000_000:
            size[rng.randrange(3)] //= 2
        q = 27 if kind == "flow" and rng.random() < 0.2 else 19
        precision = rng.choice(["fp32", "fp64"] if q == 27 else
                               ["fp32", "fp16", "bf16"] if kind == "learned" else
                               ["fp32", "fp32", "fp64", "fp16", "fp16", "bf16"])
        c = dict(kind=kind, nx=size[0], ny=size[1], nz=size[2], q=q, precision=precision,
                 streaming=rng.choice(["ab", "ab", "aa"]), flow=rng.choice(["vortex", "noise", "shear"]),
                 force=rng.choice(["none", "uniform", "kolmogorov", "field"]), walls=rng.random() < 0.25,
                 nu=round(math.exp(rng.uniform(math.log(1e-3), math.log(0.05))), 6),
                 steps=min(steps, 20), io=rng.choice(["moments", "moments", "populations"]))
        if kind == "flow":
            c["moments"] = rng.choice(["central", "central", "raw"])
            if q == 19 and rng.random() < 0.2:
                c["omega_bulk"], c["omega_hi"] = round(rng.uniform(0.8, 1.4), 3), round(rng.uniform(0.8, 1.3), 3)
        return c
    if kind == "droplet":
        n = _log_int(rng, 64, 200)
        return dict(kind=kind, nx=n, ny=_log_int(rng, 64, 200), nz=_log_int(rng, 64, 200),
                    precision=rng.choice(["fp32", "fp32", "fp64"]), steps=min(steps, 16))
    if kind == "hartmann":
        return dict(kind=kind, nx=_log_int(rng, 16, 96), ny=_log_int(rng, 48, 160), nz=_log_int(rng, 16, 96),
                    precision=rng.choice(["fp32", "fp32", "fp64"]), steps=steps)
    if kind == "bubble":
        return dict(kind=kind, nx=_log_int(rng, 60, 160), ny=_log_int(rng, 60, 160), nz=_log_int(rng, 60, 160),
                    precision=rng.choice(["fp32", "fp32", "fp64"]), steps=min(steps, 30))
    if kind == "rayleigh_taylor":
        w = _log_int(rng, 24, 96)
        return dict(kind=kind, nx=w, ny=4 * w, nz=w, precision=rng.choice(["fp32", "fp32", "fp64"]),
                    steps=min(steps, 24))
    if kind == "ensemble":
        q = rng.choice([19, 19, 27])
        return dict(kind=kind, boxes=_log_int(rng, 4, 32), q=q, learned=q == 19 and rng.random() < 0.5, steps=steps)
    return dict(kind=kind, n=rng.choice([24, 32, 32, 48]), nu=round(math.exp(rng.uniform(math.log(1e-4), math.log(1e-3))), 6),
                samples=rng.choice([1, 2, 3]), steps=_log_int(rng, 1, 32), energy=rng.choice([0.0, 1e4]))


# -- inputs ------------------------------------------------------------------

def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + salt)
    return g


def _noise(shape, seed, salt=0):
    return torch.rand(shape, generator=_gen(seed, salt), dtype=F64, device=DEV) * 2 - 1


def _axes(nx, ny, nz):
    x = torch.arange(nx, dtype=F64, device=DEV)[None, None, :]
    y = torch.arange(ny, dtype=F64, device=DEV)[None, :, None]
    z = torch.arange(nz, dtype=F64, device=DEV)[:, None, None]
    return x, y, z


def _turbulence(n, seed, u_rms=0.04, k0=4.0):
    """Random-phase solenoidal field with E(k) ~ k^4 exp(-2 (k / k0)^2) on an n^3 box."""
    u = torch.fft.fftn(torch.randn((3, n, n, n), generator=_gen(seed, 7), dtype=F64, device=DEV), dim=(1, 2, 3))
    k = torch.fft.fftfreq(n, dtype=F64, device=DEV) * n
    kv = (k[None, None, :], k[None, :, None], k[:, None, None])
    k2 = kv[0] ** 2 + kv[1] ** 2 + kv[2] ** 2
    u = u * (k2.sqrt() * torch.exp(-k2 / k0 ** 2))
    div = (kv[0] * u[0] + kv[1] * u[1] + kv[2] * u[2]) / k2.clamp(min=1.0)
    u = torch.stack([u[d] - kv[d] * div for d in range(3)])
    u = torch.fft.ifftn(u, dim=(1, 2, 3)).real
    u = u - u.mean(dim=(1, 2, 3), keepdim=True)
    return (u * (u_rms / (u.square().sum(0).mean() / 3).sqrt())).contiguous()


def _flow_fields(c, seed):
    """(rho, u, force field or None) of a flow case."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    x, y, z = _axes(nx, ny, nz)
    shape = (nz, ny, nx)
    rho = torch.ones(shape, dtype=F64, device=DEV)
    u = torch.zeros((3,) + shape, dtype=F64, device=DEV)
    if c["flow"] == "shear":
        u[0] = 0.01 * torch.sin(2 * math.pi * (z / nz + 0.1 * seed))
        u += 1e-5 * _noise(u.shape, seed)
    else:
        a, b, d = (2 * math.pi * t / n for t, n in ((x, nx), (y, ny), (z, nz)))
        s, o = torch.sin, torch.cos
        u[0] = 0.05 * o(a) * s(b) * s(d)
        u[1] = -0.025 * s(a) * o(b) * s(d)
        u[2] = -0.025 * s(a) * s(b) * o(d)
        u += (1e-4 if c["flow"] == "vortex" else 5e-3) * _noise(u.shape, seed)
        if c["flow"] == "noise":
            rho += 5e-3 * _noise(shape, seed, 1)
    if c["walls"]:
        u *= torch.sin(math.pi * (y + 0.5) / ny)
    force = 1e-5 * _noise((3,) + shape, seed, 2) if c["force"] == "field" else None
    return rho, u, force


def _flow_params(c, force):
    kw = dict(precision=c["precision"], streaming=c["streaming"], omega=_omega(c["nu"]), q=c["q"],
              walls_y=c["walls"], moments=c.get("moments", "central"))
    if c["force"] == "uniform":
        kw.update(force_mode=L.LBM_FORCE_UNIFORM, force=(1e-6, 0.0, 2e-7))
    elif c["force"] == "kolmogorov":
        kw.update(force_mode=L.LBM_FORCE_KOLMOGOROV, kolmogorov_amp=1e-6)
    elif c["force"] == "field":
        kw.update(force_mode=L.LBM_FORCE_FIELD, force_field_ptr=force.data_ptr())
    if "omega_bulk" in c:
        kw.update(omega_bulk=c["omega_bulk"], omega_hi=[c["omega_hi"]] * 9)
    return L.make_params(c["nx"], c["ny"], c["nz"], **kw)


def _omega(nu):
    return 1.0 / (3.0 * nu + 0.5)


SCALES = [0.05, 0.02] + [5e-3] * 9


def _network(seed, out=0.02):
    """Random hidden layers and a small output layer: rates spread around 1."""
    r = np.random.default_rng(int(seed) + 17)
    p = np.zeros(1737)
    p[0:352] = r.normal(size=352) / math.sqrt(11)
    p[384:1408] = r.normal(size=1024) / math.sqrt(32)
    p[1440:1728] = r.normal(size=288) * out
    return p.astype(np.float32)


def _droplet_fields(c, seed):
    x, y, z = _axes(c["nx"], c["ny"], c["nz"])
    r = torch.sqrt((x - c["nx"] / 2) ** 2 + (y - c["ny"] / 2) ** 2 + (z - c["nz"] / 2) ** 2)
    phi = 0.5 + 0.5 * torch.tanh(2.0 * (min(c["nx"], c["ny"], c["nz"]) / 6 - r) / 4.0)
    phi = phi + 1e-3 * _noise(phi.shape, seed)
    return phi, torch.full_like(phi, 1.0 / 3.0), torch.zeros((3,) + phi.shape, dtype=F64, device=DEV)


PHASE = dict(rho_light=1.0, rho_heavy=10.0, sigma=1e-3, width=4.0, mobility=0.1)


def _hartmann(c, seed):
    """(b0, body force, rho, u, b): the channel at Hartmann number 10, with a little noise on the field."""
    ny = c["ny"]
    b0 = 2.0 / ny
    f = 0.02 * b0 ** 2 * math.tanh(10.0) / (0.1 * 10.0 * (1 - 1 / math.cosh(10.0)))
    shape = (c["nz"], ny, c["nx"])
    u = 1e-3 * _noise((3,) + shape, seed)
    b = 1e-2 * b0 * _noise((3,) + shape, seed, 1)
    b[1] += b0
    return b0, f, torch.ones(shape, dtype=F64, device=DEV), u, b


def _bubble_fields(c, seed):
    x, y, z = _axes(c["nx"], c["ny"], c["nz"])
    r = torch.sqrt((x - c["nx"] / 2) ** 2 + (y - c["ny"] / 2) ** 2 + (z - c["nz"] / 2) ** 2)
    rho = 0.15 + 0.9 * (1 - torch.tanh((r - 0.2 * min(c["nx"], c["ny"], c["nz"])) / 2.0))
    return rho * (1 + 1e-3 * _noise(rho.shape, seed)), torch.zeros((3,) + rho.shape, dtype=F64, device=DEV)


def _rayleigh_taylor(c, seed):
    """(parameters of the colour lattice, omega, rho_red, rho_blue, u)."""
    w = c["nx"]
    x, y, z = _axes(c["nx"], c["ny"], c["nz"])
    top = y > 2 * w + 0.05 * w * (torch.cos(2 * math.pi * x / w) + torch.cos(2 * math.pi * z / w))
    rr = torch.where(top, 3.0, 0.0).to(F64)
    rb = torch.where(top, 0.0, 1.0).to(F64)
    prm = dict(alpha_red=1.0 - (2.0 / 3.0) / 3.0, alpha_blue=1.0 / 3.0, A=1e-3, beta=0.7,
               gravity=(0.0, -0.04 ** 2 / w, 0.0), rho_ref=2.0)
    return prm, _omega(w * 0.04 / 512.0), rr, rb, 1e-4 * _noise((3,) + rr.shape, seed)


def _box_list(c, seed):
    """[(side, nu)]: the first box is small, its whole state is written out after each block of steps."""
    r = np.random.default_rng(int(seed) + 2010)
    sides = [32] + [int(r.choice([48, 64, 96])) for _ in range(c["boxes"] - 1)]
    return [(n, float(np.exp(r.uniform(math.log(1e-4), math.log(1e-3))))) for n in sides]


def _train_inputs(c, seed):
    """Per sample (f19, targets, sigma, step weights): D3Q27 states projected on the D3Q19 populations, the ten
    low moments of the D3Q27 steps that follow, and the scales that make the paper's rates score one per step."""
    n, steps, om = c["n"], c["steps"], _omega(c["nu"])
    out = []
    with torch.no_grad():
        for s in range(c["samples"]):
            rho = torch.ones((n, n, n), dtype=F64, device=DEV)
            f27 = _mix(Q27.minv, _pack(Q27, _eq_moments(Q27, rho, _turbulence(n, seed + 31 * s))))
            for _ in range(10):
                f27 = _stream(Q27, _plain_collide(Q27, f27, om))
            f19 = _mix(Q19.minv, _mix(Q19.basis(Q27.c), f27))
            tg = []
            for _ in range(steps):
                f27 = _stream(Q27, _plain_collide(Q27, f27, om))
                tg.append(_mix(LOW.basis(Q27.c), f27))
            err, f = [], f19
            for k in range(steps):
                f = _stream(Q19, _plain_collide(Q19, f, om))
                err.append((_mix(LOW.basis(Q19.c), f) - tg[k]).square().mean(dim=(1, 2, 3)))
            sigma = err[0].sqrt().clamp(min=1e-12)
            weight = [float(1.0 / (e / sigma ** 2).sum()) for e in err]
            out.append((f19.contiguous(), torch.stack(tg).float(), sigma.cpu().numpy(), np.array(weight)))
    return out


# -- states and passes -------------------------------------------------------

def prepare(case, seed):
    c, s = dict(case), {}
    kind = c["kind"]
    if kind in ("flow", "learned"):
        rho, u, force = _flow_fields(c, seed)
        lat = L.Lattice(_flow_params(c, force), force_field=force)
        lat.init(rho, u)
        if kind == "learned":
            s["mlp"] = L.Mlp(_network(seed), SCALES)
            lat.attach_mlp(s["mlp"])
        if c["io"] == "populations":
            s["f"] = lat.get_populations()
    elif kind == "droplet":
        s["fields"] = _droplet_fields(c, seed)
        lat = L.Lattice(L.make_params(c["nx"], c["ny"], c["nz"], precision=c["precision"], omega=1.25, phase=PHASE))
    elif kind == "hartmann":
        b0, f, rho, u, b = _hartmann(c, seed)
        lat = L.Lattice(L.make_params(c["nx"], c["ny"], c["nz"], precision=c["precision"], omega=1.25, walls_y=True,
                                      force_mode=L.LBM_FORCE_UNIFORM, force=(f, 0.0, 0.0),
                                      magnetic=dict(eta=0.1, b_wall=(0.0, b0, 0.0))))
        lat.init_magnetic(rho, u, b)
    elif kind == "bubble":
        rho, u = _bubble_fields(c, seed)
        lat = L.Lattice(L.make_params(c["nx"], c["ny"], c["nz"], precision=c["precision"], omega=_omega(0.0333),
                                      shan_chen=dict(G=-5.0)))
        lat.init(rho, u)
    elif kind == "rayleigh_taylor":
        prm, om, rr, rb, u = _rayleigh_taylor(c, seed)
        s["fields"] = (rr, rb, u)
        lat = L.Lattice(L.make_params(c["nx"], c["ny"], c["nz"], precision=c["precision"], omega=om, walls_y=True,
                                      colour=prm))
    elif kind == "ensemble":
        boxes = _box_list(c, seed)
        ens = L.Ensemble([(n, _omega(nu)) for n, nu in boxes], q=c["q"], precision="fp32")
        for b, (n, _) in enumerate(boxes):
            ens.init(b, np.ones((n, n, n)), _turbulence(n, seed + b).cpu().numpy())
        if c["learned"]:
            s["mlp"] = L.Mlp(_network(seed), SCALES)
            ens.set_mlp(s["mlp"])
        return dict(s, case=c, ens=ens)
    else:
        s["samples"] = _train_inputs(c, seed)
        s["mlp"] = L.Mlp(_network(seed), SCALES)
        s["mlp"].set_energy_weight(c["energy"])
        lat = L.Lattice(L.make_params(c["n"], c["n"], c["n"], precision="fp32", omega=_omega(c["nu"])))
        lat.attach_mlp(s["mlp"])
    return dict(s, case=c, lat=lat)


def run(state):
    c, kind = state["case"], state["case"]["kind"]
    if kind == "ensemble":
        ens = state["ens"]
        ens.step(c["steps"])
        ke, mass = ens.energy()
        return dict(ke=ke, mass=mass, box0=ens.get_populations(0))
    lat = state["lat"]
    if kind == "train":
        mlp, out = state["mlp"], []
        mlp.zero_grad()
        for f19, targets, sigma, weight in state["samples"]:
            lat.set_populations(f19)
            loss, per, dstate = lat.accumulate_rollout_grad(mlp, targets, sigma, step_weight=weight, want_dstate=True,
                                                            want_steps=True)
            out.append(dict(loss=loss, per_step=per.astype(np.float32), dstate=dstate))
        return dict(samples=out, grad=mlp.grad().astype(np.float32))
    if kind == "rayleigh_taylor":
        lat.init_colour(*state["fields"])
        lat.step(c["steps"])
        red, blue = lat.colour_fields()
        rho, u, diag = lat.moments()
        return dict(red=red, blue=blue, u=u, diag=diag)
    if kind == "droplet":
        lat.init_phase(*state["fields"])
        lat.step(c["steps"])
        phi, p = lat.phase_fields()
        rho, u, diag = lat.moments()
        return dict(phi=phi, p=p, u=u, diag=diag)
    if c.get("io") == "populations":
        lat.set_populations(state["f"])
        lat.step(c["steps"])
        return dict(f=lat.get_populations())
    lat.step(c["steps"])
    rho, u, diag = lat.moments()
    out = dict(rho=rho, u=u, diag=diag)
    if kind == "hartmann":
        out["b"], out["j"] = lat.magnetic_fields()
    return out


# floating-point operations per node and step of each collision, and bytes per stored value
FLOPS = dict(flow=310, learned=3900, droplet=450, hartmann=520, bubble=380, rayleigh_taylor=520)
BYTES = dict(fp64=8, fp32=4, fp16=2, bf16=2)


def work(case):
    c, kind = case, case["kind"]
    if kind == "ensemble":
        n = 32 ** 3 + (c["boxes"] - 1) * (48 ** 3 + 64 ** 3 + 96 ** 3) // 3  # the sides' mean
        return dict(bytes=n * c["q"] * 8 + 32 ** 3 * c["q"] * 8,
                    flops=n * c["steps"] * (3900 if c["learned"] else 310 if c["q"] == 19 else 500))
    if kind == "train":
        n, k = c["n"] ** 3, c["samples"]
        return dict(bytes=k * n * (19 * 8 + c["steps"] * 40 + 19 * 4), flops=k * n * c["steps"] * 12000)
    n, eb = c["nx"] * c["ny"] * c["nz"], BYTES[c["precision"]]
    if kind in ("flow", "learned"):
        flops = 500 if c["q"] == 27 else FLOPS[kind]
        io = 2 * c["q"] * 8 if c["io"] == "populations" else 2 * c["q"] * eb + 4 * 8
    else:
        flops = FLOPS[kind]
        io = dict(droplet=(5 + 5) * 8, rayleigh_taylor=(5 + 5) * 8, bubble=2 * 19 * eb + 4 * 8,
                  hartmann=2 * 40 * eb + 10 * 8)[kind]
    return dict(bytes=n * io, flops=n * c["steps"] * flops)


# -- the same in plain torch, 64 bits ----------------------------------------
# Central-moment collision k* = (I - K) k + K k_eq + (I - K/2) R in the monomial
# basis c^e of each lattice, streaming by rolls.

class Basis:
    def __init__(self, exps, c=None):
        self.exps, self.at = exps, {e: i for i, e in enumerate(exps)}
        if c is not None:
            self.c = c
            self.q = len(c)
            self.opp = [c.index(tuple(-v for v in x)) for x in c]
            wt = {0: 2 / 3, 1: 1 / 6}
            w27 = {x: wt[abs(x[0])] * wt[abs(x[1])] * wt[abs(x[2])] for x in c}
            w19 = {0: 1 / 3, 1: 1 / 18, 2: 1 / 36, 3: 0.0}
            self.w = [w27[x] if len(c) == 27 else w19[sum(map(abs, x))] for x in c]
            self._m = None

    def basis(self, c):
        return torch.tensor([[float(x[0] ** e[0] * x[1] ** e[1] * x[2] ** e[2]) for x in c] for e in self.exps],
                            dtype=F64, device=DEV)

    @property
    def m(self):
        if self._m is None:
            self._m = self.basis(self.c)
            self._minv = torch.linalg.inv(self._m)
        return self._m

    @property
    def minv(self):
        return self._minv if self.m is not None else None


_C13 = [(-1, 0, 0), (0, -1, 0), (0, 0, -1), (-1, -1, 0), (-1, 1, 0), (-1, 0, -1), (-1, 0, 1), (0, -1, -1), (0, -1, 1)]
_C27 = _C13 + [(-1, -1, -1), (-1, -1, 1), (-1, 1, -1), (-1, 1, 1)]
_E27 = [(a, b, d) for a in range(3) for b in range(3) for d in range(3)]
_E19 = [e for e in _E27 if min(e) == 0 and sum(e) <= 4 and not (sum(e) == 3 and max(e) == 1)]
Q19 = Basis(_E19, [(0, 0, 0)] + _C13 + [tuple(-v for v in x) for x in _C13])
Q27 = Basis(_E27, [(0, 0, 0)] + _C27 + [tuple(-v for v in x) for x in _C27])
LOW = Basis([(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (2, 0, 0), (0, 2, 0), (0, 0, 2), (1, 1, 0), (1, 0, 1),
             (0, 1, 1)])
HIGH = [(2, 1, 0), (1, 2, 0), (2, 0, 1), (1, 0, 2), (0, 2, 1), (0, 1, 2), (2, 2, 0), (2, 0, 2), (0, 2, 2)]
DIAG = [(2, 0, 0), (0, 2, 0), (0, 0, 2)]
C7 = [(0, 0, 0), (-1, 0, 0), (0, -1, 0), (0, 0, -1), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
W7 = [0.25] + [0.125] * 6


def _mix(a, f):
    return torch.tensordot(a, f, dims=1)


def _pack(lat, m):
    return torch.stack([m[e] for e in lat.exps])


def _mu(p, u):
    return 1.0 if p == 0 else u if p == 1 else u * u + 1.0 / 3.0


def _eq_moments(lat, rho, u):
    return {e: rho * _mu(e[0], u[0]) * _mu(e[1], u[1]) * _mu(e[2], u[2]) for e in lat.exps}


def _shift(lat, m, u):
    """Moments about -u: a binomial sweep along each axis."""
    m = dict(m)
    for a in range(3):
        lower = lambda e, by: tuple(v - (by if k == a else 0) for k, v in enumerate(e))  # noqa: E731
        new = {}
        for e in lat.exps:
            if e[a] == 0:
                new[e] = m[e]
            elif e[a] == 1:
                new[e] = m[e] + u[a] * m[lower(e, 1)]
            else:
                new[e] = m[e] + u[a] * (2 * m[lower(e, 1)] + u[a] * m[lower(e, 2)])
        m = new
    return m


def _force_moments(lat, F, u=None):
    """Gaussian rule sum_a p_a F_a m_(e - e_a) on the equilibrium's moments: central ones, or raw ones with u."""
    mom = lambda e: ([1.0, 0.0, 1.0 / 3.0][e[0]] * [1.0, 0.0, 1.0 / 3.0][e[1]] * [1.0, 0.0, 1.0 / 3.0][e[2]]  # noqa: E731
                     if u is None else _mu(e[0], u[0]) * _mu(e[1], u[1]) * _mu(e[2], u[2]))
    out = {}
    for e in lat.exps:
        r = 0.0
        for a in range(3):
            if e[a]:
                v = mom(tuple(x - (k == a) for k, x in enumerate(e)))
                if not (isinstance(v, float) and v == 0.0):
                    r = r + e[a] * F[a] * v
        out[e] = r
    return out


def _relax(lat, f, meq, u, R, omega, bulk=1.0, hi=None, raw=False):
    """One collision; hi: the non-equilibrium central moments -> the nine higher rates, or None."""
    m = _mix(lat.m, f)
    n = {e: m[i] - meq[e] for i, e in enumerate(lat.exps)}
    if not raw:
        n = _shift(lat, n, [-v for v in u])
    rates = hi(n) if callable(hi) else ([hi] * 9 if hi is not None else None)
    p = {}
    tr_n, tr_r = sum(n[e] for e in DIAG), sum(R[e] for e in DIAG)
    for e in lat.exps:
        if e in DIAG:
            p[e] = ((1 - omega) * (n[e] - tr_n / 3) + (1 - 0.5 * omega) * (R[e] - tr_r / 3)
                    + ((1 - bulk) * tr_n + (1 - 0.5 * bulk) * tr_r) / 3)
        else:
            k = omega if sum(e) == 2 else 1.0
            if rates is not None and e in HIGH:
                k = rates[HIGH.index(e)]
            p[e] = (1 - k) * n[e] + (1 - 0.5 * k) * R[e] + torch.zeros_like(n[e])
    if not raw:
        p = _shift(lat, p, u)
    return _mix(lat.minv, torch.stack([p[e] + meq[e] for e in lat.exps]))


def _macro(lat, f, F):
    rho = f.sum(0)
    u = []
    for a in range(3):
        j = sum(lat.c[i][a] * f[i] for i in range(lat.q) if lat.c[i][a])
        u.append((j + 0.5 * F[a]) / rho)
    return rho, u


def _plain_collide(lat, f, omega, F=(0.0, 0.0, 0.0), bulk=1.0, hi=None, raw=False):
    rho, u = _macro(lat, f, F)
    rates = (lambda n: hi(n, rho)) if callable(hi) else hi
    return _relax(lat, f, _eq_moments(lat, rho, u), u, _force_moments(lat, F, u if raw else None), omega, bulk, rates,
                  raw)


def _stream(lat, fs, walls=False):
    return torch.stack([_pull(fs, i, lat.c[i], lat.opp[i], walls) for i in range(lat.q)])


def _pull(fs, i, c, opp, walls, wall_value=None):
    out = torch.roll(fs[i], shifts=(c[2], c[1], c[0]), dims=(0, 1, 2))
    if walls and c[1]:
        row = 0 if c[1] > 0 else fs.shape[2] - 1
        back = fs[opp][:, row] if wall_value is None else wall_value - fs[opp][:, row]
        out[:, row] = back
    return out


def _by_planes(f, fn, extra=None, nodes=4_000_000):
    """fn over runs of z planes (it is local to each node), to bound its temporaries."""
    nz, per = f.shape[1], max(1, nodes // (f.shape[2] * f.shape[3]))
    out = torch.empty_like(f)
    for z in range(0, nz, per):
        cut = slice(z, min(nz, z + per))
        out[:, cut] = fn(f[:, cut], None if extra is None else extra[:, cut])
    return out


def _diag(rho, u):
    u = torch.stack(list(u))
    j = [float((rho * v).sum()) for v in u]
    u2 = u.square().sum(0)
    return np.array([float(rho.sum())] + j + [0.5 * float((rho * u2).sum()), float(u2.max().sqrt())])


def _net(P, x):
    W = lambda a, o, i: P[a:a + o * i].reshape(o, i)  # noqa: E731
    b = lambda a, o: P[a:a + o].reshape(o, 1, 1, 1)  # noqa: E731
    h = torch.relu(_mix(W(0, 32, 11), x) + b(352, 32))
    h = torch.relu(_mix(W(384, 32, 32), h) + b(1408, 32))
    return _mix(W(1440, 9, 32), h) + b(1728, 9)


def _learned_rates(P):
    scales = torch.tensor(np.float32(SCALES).astype(np.float64), device=DEV).reshape(11, 1, 1, 1)

    def rates(n, rho):
        x = torch.stack([rho - 1, sum(n[e] for e in DIAG) / rho] + [n[e] / rho for e in HIGH])
        return 1 + _net(P, x / scales)
    return rates


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "train":
        return _exact_train(c, seed)
    with torch.no_grad():
        return dict(flow=_exact_flow, learned=_exact_flow, droplet=_exact_droplet, hartmann=_exact_hartmann,
                    bubble=_exact_bubble, rayleigh_taylor=_exact_rayleigh_taylor,
                    ensemble=_exact_ensemble)[c["kind"]](c, seed)


def _exact_flow(c, seed):
    lat = Q27 if c["q"] == 27 else Q19
    rho, u, force = _flow_fields(c, seed)
    F = torch.zeros((3,) + rho.shape, dtype=F64, device=DEV) if force is None else force
    if c["force"] == "uniform":
        F[0], F[2] = 1e-6, 2e-7
    elif c["force"] == "kolmogorov":
        F[0] = 1e-6 * torch.sin(2 * math.pi * _axes(1, c["ny"], 1)[1] / c["ny"])
    f = _by_planes(torch.empty((lat.q,) + rho.shape, dtype=F64, device=DEV),
                   lambda _, e: _mix(lat.minv, _pack(lat, _eq_moments(lat, e[0], e[1:]))),
                   torch.cat([rho[None], u]))
    del rho, u
    hi = c.get("omega_hi")
    if c["kind"] == "learned":
        hi = _learned_rates(torch.tensor(_network(seed).astype(np.float64), device=DEV))
    om, bulk, raw = _omega(c["nu"]), c.get("omega_bulk", 1.0), c.get("moments") == "raw"
    for _ in range(c["steps"]):
        f = _stream(lat, _by_planes(f, lambda g, e: _plain_collide(lat, g, om, e, bulk, hi, raw), F), c["walls"])
    if c["io"] == "populations":
        return dict(f=f)
    rho, u = _macro(lat, f, F)
    return dict(rho=rho, u=torch.stack(u), diag=_diag(rho, u))


def _neighbours(phi, walls=False):
    """phi(x + c_i), i = 0..18; beyond a wall the wall-side row stands in."""
    out = []
    for x in Q19.c:
        p = torch.roll(phi, shifts=(-x[2], -x[1], -x[0]), dims=(0, 1, 2))
        if walls and x[1]:
            row = phi.shape[1] - 1 if x[1] > 0 else 0
            p[:, row] = torch.roll(phi, shifts=(-x[2], -x[0]), dims=(0, 2))[:, row]
        out.append(p)
    return out


def _gradient(phin):
    return [3 * sum(Q19.w[i] * Q19.c[i][a] * phin[i] for i in range(19) if Q19.c[i][a]) for a in range(3)]


def _exact_droplet(c, seed):
    phi, p, u = _droplet_fields(c, seed)
    rl, dr = PHASE["rho_light"], PHASE["rho_heavy"] - PHASE["rho_light"]
    W, om = PHASE["width"], 1.25
    beta, kappa = 12 * PHASE["sigma"] / W, 1.5 * PHASE["sigma"] * W
    wphi = 1 / (PHASE["mobility"] / 0.25 + 0.5)
    rest = _mix(Q19.m, torch.tensor(Q19.w, dtype=F64, device=DEV))

    def eq(rho, u, Pi):
        m = _eq_moments(Q19, rho, u)
        return {e: m[e] + (Pi - rho) * rest[i] for i, e in enumerate(Q19.exps)}

    def h_eq(phi, u):
        return torch.stack([phi * W7[i] * (1 + 4 * sum(C7[i][a] * u[a] for a in range(3))) for i in range(7)])

    def fields(g, h):
        phi = h.sum(0)
        phin = _neighbours(phi)
        gr = _gradient(phin)
        lap = 6 * sum(Q19.w[i] * (phin[i] - phi) for i in range(1, 19))
        mu = 4 * beta * phi * (phi - 1) * (phi - 0.5) - kappa * lap
        rho = rl + phi * dr
        F = [mu * v for v in gr]
        j = _mix(Q19.m, g)
        u = [(j[Q19.at[e]] + 0.5 * F[a]) / rho for a, e in enumerate([(1, 0, 0), (0, 1, 0), (0, 0, 1)])]
        S0 = dr * sum(u[a] * gr[a] for a in range(3))
        return phi, gr, rho, F, u, S0, g.sum(0) + 0.5 * S0

    g = _mix(Q19.minv, _pack(Q19, eq(rl + phi * dr, u, 3 * p)))
    h = h_eq(phi, u)
    for _ in range(c["steps"]):
        phi, gr, rho, F, u, S0, Pi = fields(g, h)
        R = _force_moments(Q19, F)
        R[(0, 0, 0)] = S0
        for a, e in enumerate([(1, 0, 0), (0, 1, 0), (0, 0, 1)]):
            R[e] = R[e] - u[a] * S0
        for e in Q19.exps:
            if sum(e) == 2:
                ax = [a for a in range(3) for _ in range(e[a])]
                R[e] = dr / 3 * (u[ax[0]] * gr[ax[1]] + u[ax[1]] * gr[ax[0]]) + (S0 / 3 if ax[0] == ax[1] else 0.0)
        gs = _relax(Q19, g, eq(rho, u, Pi), u, R, om)
        gn = sum(v * v for v in gr).sqrt()
        nrm = [torch.where(gn > 0, v / gn.clamp(min=1e-300), 0.0) for v in gr]
        he = h_eq(phi, u)
        th = 4 / W * phi * (1 - phi)
        hs = torch.stack([h[i] - wphi * (h[i] - he[i])
                          + (1 - 0.5 * wphi) * W7[i] * th * sum(C7[i][a] * nrm[a] for a in range(3)) for i in range(7)])
        g = _stream(Q19, gs)
        h = torch.stack([_pull(hs, i, C7[i], i, False) for i in range(7)])
    phi, gr, rho, F, u, S0, Pi = fields(g, h)
    return dict(phi=phi, p=Pi / 3, u=torch.stack(u), diag=_diag(rho, u))


def _exact_hartmann(c, seed):
    b0, fx, rho, u, b = _hartmann(c, seed)
    bw, om, wm = (0.0, b0, 0.0), 1.25, 1 / (0.1 / 0.25 + 0.5)
    opp = [0, 4, 5, 6, 1, 2, 3]

    def g_eq(b, u):
        return [torch.stack([W7[i] * (b[a] + 4 * sum(C7[i][k] * (u[k] * b[a] - b[k] * u[a]) for k in range(3)))
                             for i in range(7)]) for a in range(3)]

    def fields(f, g):
        rho, u0 = _macro(Q19, f, (0.0, 0.0, 0.0))
        b = [v.sum(0) for v in g]
        lam = [[g[a][4 + k] - g[a][1 + k] - (u0[k] * b[a] - b[k] * u0[a]) for a in range(3)] for k in range(3)]
        j = [-4 * wm * (lam[1][2] - lam[2][1]), -4 * wm * (lam[2][0] - lam[0][2]), -4 * wm * (lam[0][1] - lam[1][0])]
        F = [j[1] * b[2] - j[2] * b[1] + fx, j[2] * b[0] - j[0] * b[2], j[0] * b[1] - j[1] * b[0]]
        return rho, [u0[a] + 0.5 * F[a] / rho for a in range(3)], b, j, F

    f, g = _mix(Q19.minv, _pack(Q19, _eq_moments(Q19, rho, u))), g_eq(b, u)
    for _ in range(c["steps"]):
        rho, u, b, j, F = fields(f, g)
        f = _stream(Q19, _plain_collide(Q19, f, om, F), True)
        ge = g_eq(b, u)
        gs = [v - wm * (v - e) for v, e in zip(g, ge)]
        g = [torch.stack([_pull(gs[a], i, C7[i], opp[i], True, 2 * W7[i] * bw[a]) for i in range(7)]) for a in range(3)]
    rho, u, b, j, F = fields(f, g)
    return dict(rho=rho, u=torch.stack(u), diag=_diag(rho, u), b=torch.stack(b), j=torch.stack(j))


def _exact_bubble(c, seed):
    rho, u = _bubble_fields(c, seed)

    def force(rho):
        psi = 1 - torch.exp(-rho)
        return [5.0 / 3.0 * psi * v for v in _gradient(_neighbours(psi))]

    f = _mix(Q19.minv, _pack(Q19, _eq_moments(Q19, rho, u)))
    for _ in range(c["steps"]):
        f = _stream(Q19, _plain_collide(Q19, f, _omega(0.0333), force(f.sum(0))))
    rho, u = _macro(Q19, f, force(f.sum(0)))
    return dict(rho=rho, u=torch.stack(u), diag=_diag(rho, u))


def _exact_rayleigh_taylor(c, seed):
    prm, om, rr, rb, u = _rayleigh_taylor(c, seed)
    c2 = [sum(map(abs, x)) for x in Q19.c]
    part = lambda v: torch.tensor([v[k] for k in c2], dtype=F64, device=DEV)  # noqa: E731
    a1, a0 = part([1.0, -1 / 12, -1 / 24]), part([0.0, 1 / 12, 1 / 24])
    w, B = torch.tensor(Q19.w, dtype=F64, device=DEV), part([-1 / 3, 1 / 18, 1 / 36])
    ma, mb = _mix(Q19.m, a1), _mix(Q19.m, a0 - w)

    def macro(f):
        tot = f[0] + f[1]
        rr, rb = f[0].sum(0), f[1].sum(0)
        F = [(rr + rb - prm["rho_ref"]) * v for v in prm["gravity"]]
        return tot, rr, rb, (rr * prm["alpha_red"] + rb * prm["alpha_blue"]) / (rr + rb), F, _macro(Q19, tot, F)[1]

    def eq(rho, u, al):
        m = _eq_moments(Q19, rho, u)
        return {e: m[e] + rho * (al * ma[i] + mb[i]) for i, e in enumerate(Q19.exps)}

    rho = rr + rb
    he = _mix(Q19.minv, _pack(Q19, eq(rho, u, (rr * prm["alpha_red"] + rb * prm["alpha_blue"]) / rho)))
    f = [rr / rho * he, rb / rho * he]
    for _ in range(c["steps"]):
        tot, rr, rb, al, F, u = macro(f)
        rho = rr + rb
        gr = _gradient(_neighbours((rr - rb) / rho, True))
        fs = _relax(Q19, tot, eq(rho, u, al), u, _force_moments(Q19, F), om)
        gn = sum(v * v for v in gr).sqrt()
        on, safe = gn > 0, gn.clamp(min=1e-300)
        red, blue = [], []
        for i, x in enumerate(Q19.c):
            cg = sum(x[a] * gr[a] for a in range(3)) / safe
            v = fs[i] + torch.where(on, 0.5 * prm["A"] * gn * (w[i] * cg * cg - B[i]), 0.0)
            cos = torch.where(on, cg / math.sqrt(c2[i]), 0.0) if c2[i] else torch.zeros_like(gn)
            bias = prm["beta"] * rr * rb / rho * cos * (al * a1[i] + a0[i])
            red.append(rr / rho * v + bias)
            blue.append(rb / rho * v - bias)
        f = [_stream(Q19, torch.stack(red), True), _stream(Q19, torch.stack(blue), True)]
    tot, rr, rb, al, F, u = macro(f)
    return dict(red=rr, blue=rb, u=torch.stack(u), diag=_diag(rr + rb, u))


def _exact_ensemble(c, seed):
    lat = Q27 if c["q"] == 27 else Q19
    hi = _learned_rates(torch.tensor(_network(seed).astype(np.float64), device=DEV)) if c["learned"] else None
    ke, mass, box0 = [], [], None
    for b, (n, nu) in enumerate(_box_list(c, seed)):
        rho = torch.ones((n, n, n), dtype=F64, device=DEV)
        f = _mix(lat.minv, _pack(lat, _eq_moments(lat, rho, _turbulence(n, seed + b))))
        for _ in range(c["steps"]):
            f = _stream(lat, _plain_collide(lat, f, _omega(nu), hi=hi))
        d = _diag(*_macro(lat, f, (0.0, 0.0, 0.0)))
        ke.append(d[4])
        mass.append(d[0])
        box0 = f.cpu().numpy() if box0 is None else box0
    return dict(ke=np.array(ke), mass=np.array(mass), box0=box0)


def _exact_train(c, seed):
    P = torch.tensor(_network(seed).astype(np.float64), device=DEV, requires_grad=True)
    hi, om, steps, out = _learned_rates(P), _omega(c["nu"]), c["steps"], []
    low = LOW.basis(Q19.c)
    energy = lambda m: 0.5 * (m[1:4].square().sum(0) / m[0]).sum()  # noqa: E731
    for f19, targets, sigma, weight in _train_inputs(c, seed):
        f = f0 = f19.clone().requires_grad_(True)
        sig, loss, per = torch.tensor(sigma, device=DEV).reshape(10, 1, 1, 1), 0.0, []
        for k in range(steps):
            f = _stream(Q19, _plain_collide(Q19, f, om, hi=hi))
            m, t = _mix(low, f), targets[k].double()
            lk = ((m - t) / sig).square().sum(0).mean()
            loss = loss + weight[k] / steps * lk
            if c["energy"]:
                loss = loss + c["energy"] / steps * ((energy(m) - energy(t)) / energy(t)).square()
            per.append(float(lk.detach()))
        loss.backward()
        out.append(dict(loss=float(loss.detach()), per_step=np.array(per), dstate=f0.grad))
    return dict(samples=out, grad=P.grad)
