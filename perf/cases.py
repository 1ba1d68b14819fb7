"""Performance cases of the FermiNet VMC path: what a program calls, on the
inputs it has, with the work each call cannot do without.

listed() are the cases that are followed, draw() gives further ones of the
same ranges, prepare() makes a program's state from a seed, run() is one pass
through the public entry points and exact() the same outputs from the plain
formulas in 64 bits (torch on the GPU, no code of the package).

Systems and network sizes are those of paper_2401_10287_amd.inputs: He and H2
(2 layers 32/8, 2 determinants), LiH, LiF, H20 and the atoms and ions of the
serving mix (4 layers 256/32, 16 determinants).  Parameters are seeded normal
matrices as there, the envelope's near 1 and the identity.  Walkers start
about their nuclei and take some Metropolis moves of the plain network, so
that they sit where sampling puts them and not on the nodes of psi.
"""
import math

import numpy as np
import torch

from paper_2401_10287_amd import fnvmc
from paper_2401_10287_amd import inputs as I
from paper_2401_10287_amd.train import VMCTrainer

SIGMA = 0.2              # Metropolis step, bohr
SETTLE_MOVES = 16        # moves of the plain network before a walker counts as a sample
TRAIN_MOVES = 10         # moves between two parameter updates
DEVICE = "cuda:0"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: log|psi| of a two-electron atom, all launch latency
        {"name": "he-log-psi-fp64", "op": "log_psi", "system": "He", "precision": "fp64", "walkers": 256},
        # a whole training iteration of the small FP64 networks (sampling, energies, gradient, Adam)
        {"name": "he-training-step-fp64", "op": "train", "system": "He", "precision": "fp64", "walkers": 256},
        # the headline: forward-Laplacian local energy of LiH with BF16 weights
        {"name": "lih-energy-bf16w", "op": "energy", "system": "LiH", "precision": "bf16w", "walkers": 4096},
        # the same network in FP64, the precision results are checked in
        {"name": "lih-energy-fp64", "op": "energy", "system": "LiH", "precision": "fp64", "walkers": 1024},
        # the three calls of a LiF training step: sampling, energies, gradient
        {"name": "lif-moves-bf16w", "op": "moves", "system": "LiF", "precision": "bf16w", "walkers": 4096,
         "moves": 10},
        {"name": "lif-energy-bf16w", "op": "energy", "system": "LiF", "precision": "bf16w", "walkers": 4096},
        {"name": "lif-gradient-bf16w", "op": "gradient", "system": "LiF", "precision": "bf16w", "walkers": 4096},
        # plain FP32 at a batch that is no multiple of anything
        {"name": "lif-energy-fp32", "op": "energy", "system": "LiF", "precision": "fp32", "walkers": 999},
        # the largest: 20 electrons, 8192 walkers
        {"name": "h20-energy-bf16w", "op": "energy", "system": "H20", "precision": "bf16w", "walkers": 8192},
        # serving: one quantum of a gang of equal jobs, and the energy estimate of a small ion job
        {"name": "ne-group-moves-bf16x6", "op": "group", "system": "Z10q+0", "precision": "bf16x6", "walkers": 256,
         "jobs": 8, "moves": 5},
        {"name": "f2+-energy-bf16x6", "op": "energy", "system": "Z9q+2", "precision": "bf16x6", "walkers": 257},
        # pretraining on orbital targets in FP32
        {"name": "lih-pretrain-fp32", "op": "pretrain", "system": "LiH", "precision": "fp32", "walkers": 1000},
    ]


def draw(rng):
    """One more case: every call, every system, the precisions each is used
    in, batches from a single walker to the largest listed one."""
    op = rng.choice(["energy", "energy", "energy", "log_psi", "moves", "group", "gradient", "pretrain", "train"])
    if op == "train":
        return {"op": op, "system": "He" if rng.random() < 0.5 else "H2-%.2f" % rng.uniform(1.0, 2.0),
                "precision": "fp64", "walkers": _log_uniform(rng, 64, 1024)}
    kind = rng.choice(["small", "LiH", "LiH", "LiF", "LiF", "H20", "atom", "atom"])
    if kind == "small":
        system = "He" if rng.random() < 0.5 else "H2-%.2f" % rng.uniform(1.0, 2.0)
        precision, most = rng.choice(["fp64", "fp32"]), 4096
    elif kind == "atom":
        z, q = rng.choice([(z, q) for z, q in I.serving_job_types() if z - q >= 2])
        system = "Z%dq%+d" % (z, q)
        precision, most = rng.choice(["bf16x6", "bf16x6", "bf16w", "fp32", "fp64"]), 4096
    else:
        system = kind
        precision = rng.choice(["bf16w", "bf16w", "bf16x6", "fp32", "fp64"])
        most = {"LiH": 4096, "LiF": 4096, "H20": 2048}[kind]
    # the pair stage of these sizes does not fit LDS in FP64 and is refused
    n = _system({"system": system}).n_elec
    if precision == "fp64" and n > {"energy": 10, "gradient": 19, "pretrain": 19}.get(op, 20):
        precision = "fp32"
    if precision == "fp64" and kind != "small":
        most = {"LiH": 1024, "atom": 512, "LiF": 256, "H20": 64}[kind]
    case = {"op": op, "system": system, "precision": precision}
    if op == "group":
        case["jobs"] = rng.randint(2, 8)
        most = max(1, most // case["jobs"])
    if op in ("moves", "group"):
        case["moves"] = rng.randint(1, 10)
    case["walkers"] = _log_uniform(rng, 1, most)
    if rng.random() < 0.25:
        case["isotropic"] = True
    return case


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def _system(case):
    name = case["system"]
    if name == "He":
        s = I.he()
    elif name.startswith("H2-"):
        s = I.h2(float(name[3:]))
    elif name == "LiH":
        s = I.lih()
    elif name == "LiF":
        s = I.lif()
    elif name == "H20":
        s = I.h_chain(20)
    else:
        z, q = name[1:].split("q")
        s = I.atom_ion(int(z), int(q))
    return I.isotropic(s) if case.get("isotropic") else s


def _batch(case):
    return case["walkers"] * case.get("jobs", 1)


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------
def _rounded(s, theta, precision):
    """The parameters as the network of that precision has them, in FP64."""
    if precision == "fp64":
        return theta
    theta = theta.float().double()
    if precision == "bf16w":           # layer and head weights are BF16 numbers
        for name, (o, shape) in I.param_offsets(s).items():
            if name.startswith("V") or name in ("w_up", "w_dn"):
                n = int(np.prod(shape))
                theta[o:o + n] = theta[o:o + n].float().bfloat16().double()
    return theta


def _inputs(case, seed):
    s = _system(case)
    g = torch.Generator().manual_seed(seed)
    parts = []
    for name, shape, fan_in in I.param_tensors(s):
        v = torch.randn(shape, generator=g, dtype=torch.float64)
        if name.startswith("pi_"):
            v = 1.0 + 0.1 * v
        elif name.startswith("sig_"):
            v = 0.05 * v + (1.0 if s.envelope else torch.eye(3, dtype=torch.float64))
        else:
            v = v / math.sqrt(fan_in)
        parts.append(v.reshape(-1))
    theta = torch.cat(parts).to(DEVICE)
    b = _batch(case)
    centres = torch.tensor(s.nuc_xyz[np.array(s.electron_site, dtype=np.int64)])
    x = (centres + s.init_scale * torch.randn((b, s.n_elec, 3), generator=g, dtype=torch.float64)).to(DEVICE)
    exact_theta = _rounded(s, theta.clone(), case["precision"])
    net = _Net(s, exact_theta)
    gd = torch.Generator(device=DEVICE).manual_seed(seed + 1)
    lp = net.log_psi(x)[0]
    for _ in range(SETTLE_MOVES):
        xp = x + 0.3 * torch.randn(x.shape, generator=gd, dtype=torch.float64, device=DEVICE)
        u = torch.rand(b, generator=gd, dtype=torch.float64, device=DEVICE)
        lpp = net.log_psi(xp)[0]
        keep = torch.log(u) <= 2.0 * (lpp - lp)
        x = torch.where(keep[:, None, None], xp, x)
        lp = torch.where(keep, lpp, lp)
    inp = {"s": s, "theta": theta, "exact_theta": exact_theta, "x": x.contiguous(), "seed": seed % (1 << 30) + 1}
    if case["op"] == "gradient":
        # local energies about a mean, as a batch of samples has them
        e0 = -float(np.sum(s.nuc_z ** 2)) * 0.5
        inp["e_loc"] = e0 + torch.randn(b, generator=gd, dtype=torch.float64, device=DEVICE)
    if case["op"] == "pretrain":
        inp["targets"] = [0.3 * torch.randn((b, s.n_det, n, n), generator=gd, dtype=torch.float64, device=DEVICE)
                          if n else None for n in (s.n_up, s.n_dn)]
    if case["op"] in ("moves", "group"):
        inp["log_abs"] = lp.clone()
    return inp


def prepare(case, seed):
    inp = _inputs(case, seed)
    s, op = inp["s"], case["op"]
    if op == "train":
        return {"op": op, "trainer": VMCTrainer(s, case["precision"], inp["theta"].cpu().numpy(),
                                                inp["x"].cpu().numpy(), sigma=SIGMA, mc_steps=TRAIN_MOVES,
                                                seed=inp["seed"])}
    cfg = fnvmc.Config(s, case["precision"])
    st = {"op": op, "cfg": cfg, "theta": inp["theta"].to(cfg.param_dtype), "x": inp["x"],
          "ws": fnvmc.Workspace(torch.device(DEVICE))}
    if op == "gradient":
        st["e_loc"] = inp["e_loc"]
    elif op == "pretrain":
        st["targets"] = inp["targets"]
    elif op in ("moves", "group"):
        st["log_abs"] = inp["log_abs"]
        st["moves"], st["seed"], st["step"] = case["moves"], inp["seed"], 0
        st["n_accept"] = torch.zeros(_batch(case), dtype=torch.int32, device=DEVICE)
        st["jobs"], st["job_walkers"] = case.get("jobs", 1), case["walkers"]
    return st


def run(st):
    op = st["op"]
    if op == "train":
        t = st["trainer"]
        stats = t.step()
        return {"theta": t.theta, "x": t.x, "log_abs": t.log_abs, "n_accept": t.n_accept,
                "energy": stats.energy, "variance": stats.variance, "std_error": stats.std_error}
    cfg, theta, x, ws = st["cfg"], st["theta"], st["x"], st["ws"]
    if op == "log_psi":
        lp, sign = fnvmc.fn_log_psi(cfg, theta, x, ws=ws)
        return {"log_abs": lp, "sign": sign}
    if op == "energy":
        e, lp, parts = fnvmc.fn_local_energy(cfg, theta, x, ws=ws)
        return {"e_loc": e, "log_abs": lp, "parts": parts}
    if op == "gradient":
        grad, stats = fnvmc.fn_param_grad(cfg, theta, x, st["e_loc"], ws=ws)
        return {"grad": grad, "stats": stats}
    if op == "pretrain":
        loss, grad = fnvmc.fn_pretrain_grad(cfg, theta, x, st["targets"][0], st["targets"][1], ws=ws)
        return {"loss": loss, "grad": grad}
    step = st["step"]
    st["step"] = step + st["moves"]
    if op == "moves":
        fnvmc.vmc_metropolis_step(cfg, theta, x, st["log_abs"], st["moves"], SIGMA, seed=st["seed"], step0=step,
                                  n_accept=st["n_accept"], ws=ws)
    else:
        jobs = [(st["job_walkers"], st["seed"] + q, step, q) for q in range(st["jobs"])]
        fnvmc.vmc_metropolis_step_group(cfg, theta, jobs, x, st["log_abs"], st["moves"], SIGMA,
                                        n_accept=st["n_accept"], ws=ws)
    return {"x": x, "log_abs": st["log_abs"], "n_accept": st["n_accept"]}


# ---------------------------------------------------------------------------
# the work of a pass
# ---------------------------------------------------------------------------
def work(case):
    """Bytes: parameters and walkers read once, results written once.  FLOPs:
    the products of the layers, pair layers and head over the rows a walker
    has (1, or 3N + 2 with derivatives), and the determinants; a gradient
    counts its forward pass and two products per product."""
    s, op = _system(case), case["op"]
    b, n, k = _batch(case), s.n_elec, s.n_det
    pbytes = 8 if case["precision"] == "fp64" else 4
    params = I.param_count(s)
    spins = [m for m in (s.n_up, s.n_dn) if m]

    def flops(rows):
        f = 0
        for l in range(s.n_layers):
            dh, dp, _ = I.layer_dims(s, l)
            f += 2 * n * rows * (dh + 2 * dp) * s.w1 + 2 * rows * 2 * dh * s.w1
            if l + 1 < s.n_layers:
                f += 2 * n * (n - 1) * min(rows, 8) * dp * s.w2     # a pair depends on six coordinates
        f += sum(2 * m * rows * s.w1 * k * m for m in spins)
        f += sum(k * (2 * m ** 3 / 3 if rows == 1 else 2 * m ** 3 + 2 * rows * m ** 3) for m in spins)
        return f

    x = 24 * n
    if op == "log_psi":
        return {"bytes": params * pbytes + b * (x + 9), "flops": b * flops(1)}
    if op == "energy":
        return {"bytes": params * pbytes + b * (x + 48), "flops": b * flops(3 * n + 2)}
    if op in ("gradient", "pretrain"):
        extra = 8 if op == "gradient" else 8 * k * sum(m * m for m in spins)
        return {"bytes": 2 * params * pbytes + b * (x + extra), "flops": 3 * b * flops(1)}
    if op == "train":
        return {"bytes": 7 * params * pbytes + b * (2 * x + 20),
                "flops": b * ((TRAIN_MOVES + 4) * flops(1) + flops(3 * n + 2))}
    return {"bytes": params * pbytes + b * (2 * x + 24), "flops": b * case["moves"] * flops(1)}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits, from the formulas
# ---------------------------------------------------------------------------
class _Net:
    """The network in FP64.  Activations carry a leading row axis: the value
    alone, or value, 3N derivatives and Laplacian (forward mode)."""

    def __init__(self, s, theta):
        self.s, self.theta = s, theta
        self.p = {name: theta[o:o + int(np.prod(shape))].reshape(shape)
                  for name, (o, shape) in I.param_offsets(s).items() if name != "_total"}
        self.R = torch.tensor(s.nuc_xyz, device=theta.device)
        self.spins = [(0, 0, s.n_up, "up"), (1, s.n_up, s.n_dn, "dn")]

    def chunk(self, fl):
        n = self.s.n_elec
        rows = 3 * n + 2 if fl else 1
        return max(1, int(6e9 / (8 * rows * n * (n * self.s.w2 + 3 * self.s.w1))))

    @staticmethod
    def _tanh(z):
        y = torch.tanh(z[:1])
        if z.shape[0] == 1:
            return y
        d = 1.0 - y * y
        src = (z[1:-1] ** 2).sum(0, keepdim=True)
        return torch.cat([y, d * z[1:-1], d * z[-1:] - 2.0 * y * d * src])

    def _features(self, x, fl):
        """(electron-nucleus [T][B][N][4M], electron-electron [T][B][N][N][4])."""
        b, n = x.shape[:2]
        m = self.R.shape[0]
        rows = 3 * n + 2 if fl else 1
        d = x[:, :, None, :] - self.R
        r = d.norm(dim=-1, keepdim=True)
        h = x.new_zeros((rows, b, n, m, 4))
        h[0] = torch.cat([d, r], -1)
        dd = x[:, :, None, :] - x[:, None, :, :]
        eye = torch.eye(n, dtype=torch.bool, device=x.device)
        rr = torch.where(eye, 1.0, (dd * dd).sum(-1)).sqrt()
        other = (~eye).double()
        p = x.new_zeros((rows, b, n, n, 4))
        p[0, ..., :3] = dd
        p[0, ..., 3] = rr * other
        if fl:
            for e in range(n):
                for a in range(3):
                    t = 1 + 3 * e + a
                    h[t, :, e, :, a] = 1.0
                    h[t, :, e, :, 3] = d[:, e, :, a] / r[:, e, :, 0]
                    p[t, :, e, :, a] += other[e]
                    p[t, :, :, e, a] -= other[e]
                    p[t, :, e, :, 3] += dd[:, e, :, a] / rr[:, e] * other[e]
                    p[t, :, :, e, 3] -= dd[:, :, e, a] / rr[:, :, e] * other[e]
            h[-1, ..., 3] = 2.0 / r[..., 0]
            p[-1, ..., 3] = 4.0 / rr * other
        return h.reshape(rows, b, n, 4 * m), p

    def _mean(self, v, dim):
        """Means over the spin-up and the spin-down electrons of an axis."""
        nu, nd = self.s.n_up, self.s.n_dn
        up, dn = v.narrow(dim, 0, nu), v.narrow(dim, nu, nd)
        return [q.sum(dim) / max(1, q.shape[dim]) for q in (up, dn)]

    def _envelope(self, x, tag, fl):
        """Envelope [B][n][K n], its gradient [3] and its Laplacian."""
        pi, sig = self.p["pi_" + tag], self.p["sig_" + tag]
        val = grad = lap = 0.0
        for m in range(self.R.shape[0]):
            d = x - self.R[m]
            if self.s.envelope:
                sd = sig[:, m, None] * d[:, :, None, :]
                q = sd.norm(dim=-1)
            else:
                sd = torch.matmul(d, sig[:, m].reshape(-1, 3).T).reshape(*d.shape[:2], -1, 3)
                q = sd.norm(dim=-1)
            e = pi[:, m] * torch.exp(-q)
            val = val + e
            if fl:
                if self.s.envelope:
                    gq = sig[:, m, None] * sd / q[..., None]
                    tr = 3.0 * sig[:, m] ** 2
                else:
                    gq = (sd[..., None] * sig[:, m]).sum(-2) / q[..., None]
                    tr = (sig[:, m] ** 2).sum((-1, -2))
                g2 = (gq * gq).sum(-1)
                grad = grad - e[..., None] * gq
                lap = lap + e * (g2 - (tr - g2) / q)
        return val, grad, lap

    def orbitals(self, x, fl):
        """Per spin the orbital matrices [T][B][K][n (orbital)][n (electron)]."""
        s, p = self.s, self.p
        h, pair = self._features(x, fl)
        for l in range(s.n_layers):
            dh, dp, _ = I.layer_dims(s, l)
            V = p["V%d" % l]
            gu, gd = self._mean(h, 2)
            piu, pid = self._mean(pair, 3)
            z = torch.matmul(h, V[:dh])
            z = z + (torch.matmul(gu, V[dh:2 * dh]) + torch.matmul(gd, V[2 * dh:3 * dh]))[:, :, None]
            z = z + torch.matmul(piu, V[3 * dh:3 * dh + dp]) + torch.matmul(pid, V[3 * dh + dp:])
            z = torch.cat([z[:1] + p["b%d" % l], z[1:]])
            y = self._tanh(z)
            h = y + h if l else y
            if l + 1 < s.n_layers:
                z = torch.matmul(pair, p["W2_%d" % l])
                z = torch.cat([z[:1] + p["c2_%d" % l], z[1:]])
                y = self._tanh(z)
                pair = y + pair if l else y
        out = []
        for _, j0, n, tag in self.spins:
            if n == 0:
                out.append(None)
                continue
            a = torch.matmul(h[:, :, j0:j0 + n], p["w_" + tag])
            a = torch.cat([a[:1] + p["g_" + tag], a[1:]])
            e, ge, le = self._envelope(x[:, j0:j0 + n], tag, fl)
            A = a * e
            if fl:
                own = torch.zeros_like(A)
                own[-1] = a[0] * le
                for j in range(n):
                    for c in range(3):
                        t = 1 + 3 * (j0 + j) + c
                        own[t, :, j] = a[0, :, j] * ge[:, j, :, c]
                        own[-1, :, j] += 2.0 * a[t, :, j] * ge[:, j, :, c]
                A = A + own
            out.append(A.reshape(*A.shape[:3], s.n_det, n).permute(0, 1, 3, 4, 2))
        return out

    @staticmethod
    def _inverse(A):
        """(inverse, sign, log|det|) by Gauss-Jordan elimination with row pivoting."""
        n = A.shape[-1]
        W = torch.cat([A, torch.eye(n, dtype=A.dtype, device=A.device).expand_as(A)], -1).clone()
        sign = torch.ones(A.shape[:-2], dtype=A.dtype, device=A.device)
        logdet = torch.zeros_like(sign)
        for k in range(n):
            r = W[..., k:, k].abs().argmax(-1) + k
            idx = r[..., None, None].expand(*r.shape, 1, 2 * n)
            pr, kr = W.gather(-2, idx), W[..., k:k + 1, :].clone()
            W.scatter_(-2, idx, kr)
            W[..., k:k + 1, :] = pr
            piv = pr[..., 0, k]
            sign = sign * torch.where(r == k, 1.0, -1.0) * torch.sign(piv)
            logdet = logdet + piv.abs().log()
            row = pr / piv[..., None, None]
            f = W[..., :, k:k + 1].clone()
            f[..., k, 0] = 0.0
            W = W - f * row
            W[..., k:k + 1, :] = row
        return W[..., n:], sign, logdet

    def _sum(self, inv):
        """(log|psi|, sign, weights psi_k / psi) from per-spin (inverse, sign, log)."""
        sk = math.prod([v[1] for v in inv if v is not None])
        lk = sum([v[2] for v in inv if v is not None])
        top = lk.max(-1, keepdim=True).values
        t = sk * torch.exp(lk - top)
        tot = t.sum(-1, keepdim=True)
        return (top + tot.abs().log())[:, 0], torch.sign(tot)[:, 0], t / tot

    def log_psi(self, x):
        out = []
        for xc in x.split(self.chunk(False)):
            with torch.no_grad():
                inv = [None if A is None else self._inverse(A[0]) for A in self.orbitals(xc, False)]
                out.append(self._sum(inv)[:2])
        return torch.cat([o[0] for o in out]), torch.cat([o[1] for o in out])

    @torch.no_grad()
    def energy(self, x):
        s = self.s
        Z = torch.tensor(s.nuc_z, device=x.device)
        nn = sum(float(s.nuc_z[i] * s.nuc_z[j] / np.linalg.norm(s.nuc_xyz[i] - s.nuc_xyz[j]))
                 for i in range(s.n_nuc) for j in range(i))
        es, ls, ps = [], [], []
        for xc in x.split(self.chunk(True)):
            orb = self.orbitals(xc, True)
            inv = [None if A is None else self._inverse(A[0]) for A in orb]
            lp, _, om = self._sum(inv)
            tr, lap = 0.0, 0.0
            for A, v in zip(orb, inv):
                if A is None:
                    continue
                M = torch.matmul(v[0], A[1:])
                t = M.diagonal(dim1=-2, dim2=-1).sum(-1)
                tr = tr + t[:-1]
                lap = lap + t[-1] - (M[:-1] * M[:-1].transpose(-1, -2)).sum((0, -1, -2))
            lap = lap + (tr * tr).sum(0)
            kin = -0.5 * (om * lap).sum(-1)
            i, j = torch.triu_indices(s.n_elec, s.n_elec, 1, device=x.device)
            ee = (1.0 / (xc[:, i] - xc[:, j]).norm(dim=-1)).sum(-1)
            en = -(Z / (xc[:, :, None] - self.R).norm(dim=-1)).sum((-1, -2))
            parts = torch.stack([kin, ee, en, torch.full_like(kin, nn)], -1)
            es.append(parts.sum(-1))
            ls.append(lp)
            ps.append(parts)
        return torch.cat(es), torch.cat(ls), torch.cat(ps)

    def _accumulate(self, x, surrogate):
        theta = self.theta.clone().requires_grad_(True)
        net = _Net(self.s, theta)
        total, o = torch.zeros_like(theta), 0
        for xc in x.split(self.chunk(False) // 4 + 1):
            g, = torch.autograd.grad(surrogate(net, xc, o), theta)
            total += g
            o += xc.shape[0]
        return total

    def gradient(self, x, coeff):
        """sum_p coeff_p d log|psi_p| / d theta."""
        def surrogate(net, xc, o):
            orb = net.orbitals(xc, False)
            inv = [None if A is None else self._inverse(A[0].detach()) for A in orb]
            om = self._sum(inv)[2]
            return sum((coeff[o:o + xc.shape[0], None] * om * (v[0].transpose(-1, -2) * A[0]).sum((-1, -2))).sum()
                       for A, v in zip(orb, inv) if A is not None)
        return self._accumulate(x, surrogate)

    def pretrain(self, x, targets):
        loss = []

        def surrogate(net, xc, o):
            orb = net.orbitals(xc, False)
            v = sum(((A[0] - t[o:o + xc.shape[0]]) ** 2).sum() for A, t in zip(orb, targets) if A is not None)
            v = v / x.shape[0]
            loss.append(v.detach())
            return v
        g = self._accumulate(x, surrogate)
        return torch.stack(loss).sum().reshape(1), g


def _philox(d, walker, step, stream, seed):
    """Philox4x32-10 words [4][...] (int64 holding 32 bits)."""
    m = 0xFFFFFFFF
    c = [d & m, walker & m, torch.full_like(d, step & m), torch.full_like(d, stream & m)]
    k0, k1 = seed & m, (seed >> 32) & m
    for _ in range(10):
        # 32 x 32 -> 64 bit products: int64 wraps, which keeps both halves once masked
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & m) ^ c[1] ^ k0, p1 & m, ((p0 >> 32) & m) ^ c[3] ^ k1, p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c


def _unit(a, b):
    return (((a << 21) | (b >> 11)) + 1).double() * 2.0 ** -53


def _walk(net, x, lp, moves, seed, step0, stream):
    b, n3 = x.shape[0], 3 * net.s.n_elec
    w = torch.arange(b, device=x.device)
    acc = torch.zeros(b, dtype=torch.int32, device=x.device)
    for k in range(moves):
        d = torch.arange((n3 + 1) // 2, device=x.device)
        c = _philox(*torch.broadcast_tensors(d[None, :], w[:, None]), step0 + k, stream, seed)
        rad = torch.sqrt(-2.0 * torch.log(_unit(c[0], c[1])))
        ang = 2.0 * math.pi * _unit(c[2], c[3])
        z = torch.stack([rad * torch.cos(ang), rad * torch.sin(ang)], -1).reshape(b, -1)[:, :n3]
        a = _philox(torch.full_like(w, 0xFFFFFFFF), w, step0 + k, stream, seed)
        xp = x + SIGMA * z.reshape(x.shape)
        lpp = net.log_psi(xp)[0]
        keep = torch.isfinite(lpp) & (torch.log(_unit(a[0], a[1])) <= 2.0 * (lpp - lp))
        x = torch.where(keep[:, None, None], xp, x)
        lp = torch.where(keep, lpp, lp)
        acc += keep.int()
    return x, lp, acc


def _stats(e):
    mean, var = e.mean(), e.var(unbiased=False)
    return torch.stack([mean, var, (var / e.shape[0]).sqrt()]), 2.0 * (e - mean) / e.shape[0]


def exact(case, seed):
    inp = _inputs(case, seed)
    s, op, x = inp["s"], case["op"], inp["x"]
    net = _Net(s, inp["exact_theta"])
    if op == "log_psi":
        lp, sign = net.log_psi(x)
        return {"log_abs": lp, "sign": sign.to(torch.int8)}
    if op == "energy":
        e, lp, parts = net.energy(x)
        return {"e_loc": e, "log_abs": lp, "parts": parts}
    if op == "gradient":
        stats, coeff = _stats(inp["e_loc"])
        return {"grad": net.gradient(x, coeff), "stats": stats}
    if op == "pretrain":
        loss, grad = net.pretrain(x, inp["targets"])
        return {"loss": loss, "grad": grad}
    if op == "train":
        x, lp, acc = _walk(net, x, net.log_psi(x)[0], TRAIN_MOVES, inp["seed"], 0, 0)
        e, _, _ = net.energy(x)
        stats, coeff = _stats(e)
        g = net.gradient(x, coeff)
        # the first Adam update: bias-corrected moments are g and g^2
        theta = net.theta - 1e-3 * g / (g.abs() + 1e-8)
        lp = _Net(s, theta).log_psi(x)[0]
        mean, var, err = (float(v) for v in stats)
        return {"theta": theta, "x": x, "log_abs": lp, "n_accept": acc, "energy": mean, "variance": var,
                "std_error": err}
    if op == "moves":
        x, lp, acc = _walk(net, x, inp["log_abs"], case["moves"], inp["seed"], 0, 0)
        return {"x": x, "log_abs": lp, "n_accept": acc}
    b, got = case["walkers"], []
    for q in range(case["jobs"]):
        got.append(_walk(net, x[q * b:(q + 1) * b], inp["log_abs"][q * b:(q + 1) * b], case["moves"],
                         inp["seed"] + q, 0, q))
    return {k: torch.cat([v[i] for v in got]) for i, k in enumerate(("x", "log_abs", "n_accept"))}
