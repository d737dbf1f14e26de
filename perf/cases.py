"""The work that users of this library have it do, as timed cases.

listed() names the cases, draw() gives more of the same ranges, prepare()
makes what a program holds before the call (a lattice or a job server on the
GPU, started and a few sweeps old), run() is one call or a short sequence of
calls of the public interface, work() what such a call cannot do without, and
exact() the same outputs from plain torch arithmetic in 64 bits.

Kinds of case:
  sweep       Lattice.sweep(n, beta): updating sweeps without measurement,
              what the paper times.  Returns the links.
  measure     Lattice.sweep_measure(n, beta): sweeps with the plaquette after
              each.  Returns the plaquettes and the links.
  betas       Lattice.sweep_betas(n, b0, b1) and the Polyakov loops: a
              double-layered torus with one coupling per layer.
  plaquette   Lattice.plaquette(): the measurement with the check of every
              link, as after loading a configuration.
  counts      Lattice.sweep and Lattice.counters: several attempts per
              subgroup, with the acceptance read after the call.
  checkpoint  Lattice.set_links and Lattice.get_links: resuming from and
              writing a configuration in host memory.
  serve       serve.Server: a batch of jobs submitted at once and run to the
              end, as a scan over couplings and sizes.
Links come back as the library keeps them on the device (rows 0 and 1 of each
matrix in tiles of 16 links), in floating point.
"""
import math

import numpy as np
import torch

WARM_SWEEPS = 2  # sweeps after the hot start, before the timed call
SERVING_SIZES = (8, 10, 12, 16, 20, 24)


def _case(kind, L, n, *, name=None, nlat=1, flip=0, precision=64, nhit=1, beta=5.7, beta1=0.0, jobs=0):
    c = {"kind": kind, "L0": L[0], "L1": L[1], "L2": L[2], "L3": L[3], "n": n, "nlat": nlat, "flip": flip,
         "precision": precision, "nhit": nhit, "beta": beta, "beta1": beta1, "jobs": jobs}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one sweep and its plaquette per call on the smallest lattice of the paper's tables: a
        # thermalisation loop that looks at every value; one update's latency and the launches count
        _case("measure", (8, 8, 8, 8), 1, name="measure-8x4-f64-1"),
        # the paper's smallest lattice swept without measurement
        _case("sweep", (8, 8, 8, 8), 8, name="sweep-8x4-f64"),
        # a ragged box with several attempts per subgroup and its acceptance count
        _case("counts", (6, 10, 14, 18), 4, nhit=3, beta=5.9, name="counts-ragged-f64-3hit"),
        # the 16^4 lattice of the paper's tables, measured, in the working precision
        _case("measure", (16, 16, 16, 16), 8, name="measure-16x4-f64"),
        # the same lattice in the FP32 tier, swept only
        _case("sweep", (16, 16, 16, 16), 8, precision=32, name="sweep-16x4-f32"),
        # the double-layered torus of the paper's tables, per-layer plaquettes after every sweep
        _case("measure", (16, 16, 16, 16), 8, nlat=2, flip=7, name="measure-2x16x4-f64"),
        # the same torus with a hot and a cold layer, and its Polyakov loops
        _case("betas", (16, 16, 16, 16), 4, nlat=2, flip=7, beta=5.5, beta1=6.2, name="betas-2x16x4-f64"),
        # the benchmark's lattice: production sweeps with the plaquette after each, both precisions
        _case("measure", (32, 32, 32, 32), 4, name="measure-32x4-f64"),
        _case("measure", (32, 32, 32, 32), 4, precision=32, name="measure-32x4-f32"),
        # the largest lattice of the paper's plans at its weaker coupling
        _case("sweep", (64, 64, 64, 64), 1, beta=6.0, name="sweep-64x4-f64"),
        # a configuration read back in: plaquette and unitarity check of every link
        _case("plaquette", (32, 32, 32, 32), 1, name="plaquette-32x4-f64"),
        # a batch of mixed FP32 jobs run to the end
        _case("serve", (0, 0, 0, 0), 30, precision=32, jobs=24, name="serve-24-jobs-f32"),
    ]


def _extent(rng, lo, hi):
    """An even extent in [lo, hi], even in its logarithm."""
    return max(lo, min(hi, 2 * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 2)))


def draw(rng):
    kind = rng.choice(["sweep", "sweep", "measure", "measure", "betas", "plaquette", "counts", "checkpoint", "serve"])
    beta = round(rng.uniform(5.5, 6.2), 4)
    if kind == "serve":
        return _case(kind, (0, 0, 0, 0), rng.randint(8, 40), precision=rng.choice([32, 32, 64]),
                     jobs=rng.randint(4, 24), beta=beta)
    hi = {"betas": 32, "checkpoint": 20, "counts": 32}.get(kind, 64)
    if rng.random() < 0.4:  # a symmetric lattice, as in the paper
        a = _extent(rng, 6, hi)
        L = [a, a, a, a]
    else:
        L = [_extent(rng, 4, hi) for _ in range(4)]
    nlat = 2 if kind == "betas" else rng.choice([1, 1, 2])
    if nlat == 2 and max(L) > 48:
        L = [min(x, 48) for x in L]
    flip = rng.choice([7, 7, 15, rng.randint(0, 15)]) if nlat == 2 else 0
    V = nlat * L[0] * L[1] * L[2] * L[3]
    most = 1 << 24
    n = max(1, min(rng.randint(1, 16), most // V))
    nhit = rng.choice([2, 3, 4]) if kind == "counts" else 1
    return _case(kind, L, n, nlat=nlat, flip=flip, precision=rng.choice([64, 64, 32]), nhit=nhit, beta=beta,
                 beta1=round(rng.uniform(5.5, 6.2), 4) if kind == "betas" else 0.0)


def _extents(case):
    return case["L0"], case["L1"], case["L2"], case["L3"]


def _serve_jobs(case, seed):
    """The jobs of a batch: sizes, couplings and sweep counts as a scan has them, from the case alone; the keys from the seed."""
    g = np.random.default_rng(1000 * case["jobs"] + case["n"])
    return [{"L": int(g.choice(SERVING_SIZES)), "beta": float(g.uniform(5.5, 6.2)),
             "nsweeps": int(g.integers(max(1, case["n"] // 2), case["n"] + 1)), "seed": int(seed) * 4096 + k + 1}
            for k in range(case["jobs"])]


def prepare(case, seed):
    from paper_0904_1179_amd import serve, su3hb

    if case["kind"] == "serve":
        jobs = [serve.make_job(j["L"], j["beta"], j["nsweeps"], j["seed"], precision=case["precision"])
                for j in _serve_jobs(case, seed)]
        need = sum(sum(su3hb.su3_footprint(j.params)) + 512 for j in jobs)
        return {"case": case, "server": serve.Server(need + (16 << 20), max_active=64), "jobs": jobs}
    lat = su3hb.Lattice(_extents(case), nlat=case["nlat"], flip_mask=case["flip"], precision=case["precision"],
                        nhit=case["nhit"], seed=int(seed) + 1)
    lat.links_buf.zero_()  # the buffer's padding, which no kernel writes, comes back with the links
    lat.start(True)
    if case["kind"] == "betas":
        lat.sweep_betas(WARM_SWEEPS, case["beta"], case["beta1"])
    else:
        lat.sweep(WARM_SWEEPS, case["beta"])
    state = {"case": case, "lat": lat,
             "links": lat.links_buf.view(torch.float64 if case["precision"] == 64 else torch.float32)}
    if case["kind"] == "checkpoint":
        state["host"] = lat.get_links()
    return state


def run(state):
    case = state["case"]
    kind, n, beta = case["kind"], case["n"], case["beta"]
    if kind == "serve":
        srv, ids = state["server"], [state["server"].submit(j) for j in state["jobs"]]
        active = queued = 1
        while active or queued:
            active, queued, _ = srv.run(8)
        out = []
        for jid in ids:
            r = srv.poll(jid)
            srv.release(jid)
            out.append(r)
        return {"plaquette": np.array([r["plaquette"] for r in out]),
                "attempts": np.array([r["kp_attempts"] for r in out], dtype=np.int64),
                "accepts": np.array([r["kp_accepts"] for r in out], dtype=np.int64),
                "bad_links": np.array([r["bad_links"] for r in out], dtype=np.int64)}
    lat = state["lat"]
    if kind == "sweep":
        lat.sweep(n, beta)
        return {"links": state["links"]}
    if kind == "measure":
        return {"plaquette": lat.sweep_measure(n, beta), "links": state["links"]}
    if kind == "betas":
        lat.sweep_betas(n, beta, case["beta1"])
        return {"polyakov": lat.polyakov(), "links": state["links"]}
    if kind == "plaquette":
        return {"plaquette": lat.plaquette()}
    if kind == "counts":
        lat.sweep(n, beta)
        _, attempts, accepts = lat.counters()
        return {"attempts": attempts, "accepts": accepts, "links": state["links"]}
    lat.set_links(state["host"])
    return {"links": lat.get_links()}


# One link update: twelve 3x3 complex products and six sums for the staple, one product with the
# link, three subgroups of about 250 operations each, and the reunitarisation.
UPDATE_FLOPS = 12 * 198 + 5 * 18 + 198 + 3 * 250 + 80


def work(case):
    real = case["precision"] // 8
    if case["kind"] == "serve":
        js = _serve_jobs(case, 0)
        return {"bytes": sum(4 * j["L"] ** 4 * 12 * real for j in js),
                "flops": sum(4 * j["L"] ** 4 * j["nsweeps"] * UPDATE_FLOPS for j in js)}
    L = _extents(case)
    links = 4 * case["nlat"] * L[0] * L[1] * L[2] * L[3]
    lattice = links * 12 * real
    if case["kind"] == "plaquette":
        return {"bytes": lattice, "flops": links // 4 * 6 * (2 * 198 + 36)}
    if case["kind"] == "checkpoint":
        return {"bytes": 2 * (links * 18 * 8 + lattice), "flops": links * 2 * 42}
    return {"bytes": 2 * lattice, "flops": links * case["n"] * UPDATE_FLOPS}


# ---------------------------------------------------------------------------
# exact(): the same chain in 64 bits with plain torch operations.  Fields are
# tensors of shape (nlat, L3, L2, L1, L0, ...) over all sites.
# ---------------------------------------------------------------------------
_M32 = (1 << 32) - 1


def _signed(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _hi32(x):
    return (x >> 32) & _M32


def _mulhilo(a, m):
    m0, m1 = m & _M32, m >> 32
    a0, a1 = a & _M32, _hi32(a)
    p = a0 * m0
    t = a0 * m1 + _hi32(p)
    u = a1 * m0 + (t & _M32)
    return (u << 32) | (p & _M32), a1 * m1 + _hi32(t) + _hi32(u)


def _philox(c0, c1, c2, c3, seed):
    """Philox4x64-10 with key (seed, 0); c0 an int64 tensor, the others whole numbers."""
    c = [c0] + [torch.full_like(c0, _signed(v)) for v in (c1, c2, c3)]
    k0, k1 = seed, 0
    for _ in range(10):
        la, ha = _mulhilo(c[0], 0xD2E7470EE14C6C93)
        lb, hb = _mulhilo(c[2], 0xCA5A826395121157)
        c = [hb ^ c[1] ^ _signed(k0), lb, ha ^ c[3] ^ _signed(k1), la]
        k0, k1 = k0 + 0x9E3779B97F4A7C15, k1 + 0xBB67AE8584CAA73B
    return c


def _u52(w):
    return (((w >> 12) & ((1 << 52) - 1)).double() + 0.5) * 2.0 ** -52


def _u32(h):
    return (h.double() + 0.5) * 2.0 ** -32


def _mm(a, b):
    c = a[..., :, 0, None] * b[..., 0, None, :]
    for k in (1, 2):
        c = c + a[..., :, k, None] * b[..., k, None, :]
    return c


def _dag(a):
    return a.conj().transpose(-1, -2)


def _shift(f, mu, s, flip):
    """f(x + s mu); across a flipped boundary the other layer's value."""
    dim = 4 - mu
    g = torch.roll(f, -s, dims=dim)
    if flip >> mu & 1:
        at = g.select(dim, g.shape[dim] - 1 if s > 0 else 0)
        at.copy_(at.flip(0))
    return g


def _row2(r0, r1):
    return torch.linalg.cross(r0, r1, dim=-1).conj()


def _reunit(u):
    r0, r1 = u[..., 0, :], u[..., 1, :]
    r0 = r0 / (r0.abs() ** 2).sum(-1, keepdim=True).sqrt()
    r1 = r1 - (r0.conj() * r1).sum(-1, keepdim=True) * r0
    r1 = r1 / (r1.abs() ** 2).sum(-1, keepdim=True).sqrt()
    return torch.stack([r0, r1, _row2(r0, r1)], -2)


class _Exact:
    def __init__(self, L, nlat, flip, nhit, seed, device):
        self.L, self.nlat, self.flip, self.nhit, self.seed = L, nlat, flip, nhit, seed
        shape = (nlat, L[3], L[2], L[1], L[0])
        V = L[0] * L[1] * L[2] * L[3]
        self.site = torch.arange(nlat * V, device=device).reshape(shape)
        x = [torch.arange(L[mu], device=device).reshape([-1 if 4 - mu == d else 1 for d in range(5)]) for mu in range(4)]
        self.parity = (x[0] + x[1] + x[2] + x[3]) % 2 + torch.zeros_like(self.site)
        self.layer = torch.arange(nlat, device=device).reshape(-1, 1, 1, 1, 1) + torch.zeros_like(self.site)
        self.sweep_index, self.attempts, self.accepts = 0, 0, 0
        self.U = [self._haar(4 * self.site + mu) for mu in range(4)]

    def _haar(self, lid):
        z = []
        for d in range(3):
            w = _philox(lid, 0, d, 1, self.seed)
            for p in (0, 2):
                r, phi = (-2.0 * _u52(w[p]).log()).sqrt(), 2.0 * math.pi * _u52(w[p + 1])
                z.append(torch.complex(r * phi.cos(), r * phi.sin()))
        rows = torch.stack(z, -1).reshape(lid.shape + (2, 3))
        return _reunit(rows)

    def _staple(self, mu, w):
        A = 0
        for nu in range(4):
            if nu == mu:
                continue
            up = _mm(_mm(_shift(self.U[nu], mu, 1, self.flip), _dag(_shift(self.U[mu], nu, 1, self.flip))), _dag(self.U[nu]))
            f = _shift(self.U[nu], nu, -1, self.flip)
            d = _shift(f, mu, 1, self.flip)
            dn = _mm(_mm(_dag(d), _dag(_shift(self.U[mu], nu, -1, self.flip))), f)
            if w is not None:
                up = up * w[..., None, None]
                dn = dn * _shift(w, nu, -1, self.flip)[..., None, None]
            A = A + up + dn
        return A

    def _pass(self, mu, par, beta, w):
        here = self.parity == par
        A = self._staple(mu, w)
        lid = (4 * self.site + mu)[here]
        U, W = self.U[mu][here], _mm(self.U[mu], A)[here]
        for sub, (i, j) in enumerate(((0, 1), (1, 2), (0, 2))):
            v = torch.stack([(W[:, i, i] + W[:, j, j]).real, -(W[:, i, j] + W[:, j, i]).imag,
                             (W[:, j, i] - W[:, i, j]).real, (W[:, j, j] - W[:, i, i]).imag], -1) / 2
            k = (v * v).sum(-1).sqrt()
            alpha = 2.0 * beta * k / 3.0
            todo, got = k > 0, torch.zeros_like(k, dtype=torch.bool)
            a = torch.zeros_like(v)
            for t in range(self.nhit):
                r = _philox(lid, self.sweep_index, sub << 32 | t, 0, self.seed)
                u1, u3 = _u52(r[0]), _u52(r[1])
                u2, u4, u5, u6 = _u32(r[2] & _M32), _u32(_hi32(r[2])), _u32(r[3] & _M32), _u32(_hi32(r[3]))
                lam = -(u1.log() + torch.cos(2.0 * math.pi * u2) ** 2 * u3.log()) / (2.0 * alpha)
                ok = todo & (u4 * u4 <= 1.0 - lam)
                self.attempts += int(todo.sum())
                self.accepts += int(ok.sum())
                a0 = 1.0 - 2.0 * lam
                rho, cth = (1.0 - a0 * a0).clamp(min=0.0).sqrt(), 2.0 * u5 - 1.0
                sth, phi = (1.0 - cth * cth).sqrt(), 2.0 * math.pi * u6
                new = torch.stack([a0, rho * sth * phi.cos(), rho * sth * phi.sin(), rho * cth], -1)
                a = torch.where(ok[:, None], new, a)
                todo, got = todo & ~ok, got | ok
            p = [self._su2(q) for q in (a, v / k.clamp(min=1e-300)[:, None])]
            r = p[0] @ p[1]
            r = torch.where(got[:, None, None], r, torch.eye(2, dtype=r.dtype, device=r.device))
            for m in (U, W):
                mi, mj = m[:, i, :].clone(), m[:, j, :].clone()
                m[:, i, :] = r[:, 0, 0, None] * mi + r[:, 0, 1, None] * mj
                m[:, j, :] = r[:, 1, 0, None] * mi + r[:, 1, 1, None] * mj
        self.U[mu][here] = _reunit(U)

    @staticmethod
    def _su2(q):
        a, b = torch.complex(q[:, 0], q[:, 3]), torch.complex(q[:, 2], q[:, 1])
        return torch.stack([torch.stack([a, b], -1), torch.stack([-b.conj(), a.conj()], -1)], -2)

    def sweep(self, n, beta, beta1=None):
        w = None if beta1 is None else beta + (beta1 - beta) * self.layer.double()
        for _ in range(n):
            for mu in range(4):
                for par in (0, 1):
                    self._pass(mu, par, beta if w is None else 1.0, w)
            self.sweep_index += 1

    def plaquette(self):
        s = torch.zeros(self.nlat, dtype=torch.float64, device=self.site.device)
        for mu in range(4):
            for nu in range(mu + 1, 4):
                P = _mm(self.U[mu], _shift(self.U[nu], mu, 1, self.flip))
                Q = _mm(self.U[nu], _shift(self.U[mu], nu, 1, self.flip))
                s += (P * Q.conj()).real.sum((1, 2, 3, 4, 5, 6))
        per = s / (18.0 * self.site[0].numel())
        return np.concatenate([[float(per.mean())], per.cpu().numpy()])

    def polyakov(self):
        P, ly = None, torch.arange(self.nlat, device=self.site.device)
        for _ in range(2 if self.flip >> 3 & 1 else 1):
            for x3 in range(self.L[3]):
                u = self.U[3][ly, x3]
                P = u if P is None else _mm(P, u)
            ly = ly.flip(0) if self.flip >> 3 & 1 else ly
        per = P.diagonal(dim1=-2, dim2=-1).sum(-1).mean((1, 2, 3)) / 3.0
        return np.concatenate([[complex(per.mean())], per.cpu().numpy()])

    def canonical(self):
        """(4 site + mu, 18) doubles, as Lattice.get_links."""
        u = torch.stack(self.U, 5)
        return torch.view_as_real(u.resolve_conj()).reshape(-1, 18)

    def tiled(self, precision):
        """The device image of the links, the padding zero."""
        n = self.site.numel() // 2
        stride = (n + 63) // 64 * 64 + 64
        out = torch.zeros((4, 2, stride, 6, 2), dtype=torch.float64, device=self.site.device)
        for mu in range(4):
            rows = torch.view_as_real(self.U[mu][..., :2, :].resolve_conj()).reshape(self.site.shape + (6, 2))
            for par in (0, 1):
                out[mu, par, :n] = rows[self.parity == par]
        return out.reshape(4, 2, stride // 16, 16, 6, 2).transpose(3, 4).reshape(-1)


def exact(case, seed):
    """Links and plaquettes of the same chain in 64 bits.  (The FP32 tier's accept decisions part from it
    now and then; its long served chains all do, and have no exact value.)"""
    if case["kind"] == "serve":
        return None
    L, nlat = _extents(case), case["nlat"]
    V, gpu = nlat * L[0] * L[1] * L[2] * L[3], torch.cuda.is_available()
    if V * (WARM_SWEEPS + case["n"]) > ((1 << 23) if gpu else (1 << 18)):
        return None
    e = _Exact(L, nlat, case["flip"], case["nhit"], int(seed) + 1, "cuda" if gpu else "cpu")
    kind, n, beta = case["kind"], case["n"], case["beta"]
    if kind == "betas":
        e.sweep(WARM_SWEEPS + n, beta, case["beta1"])
        return {"polyakov": e.polyakov(), "links": e.tiled(64)}
    e.sweep(WARM_SWEEPS, beta)
    if kind == "plaquette":
        return {"plaquette": e.plaquette()}
    if kind == "checkpoint":
        return {"links": e.canonical()}
    plaq = []
    for _ in range(n):
        e.sweep(1, beta)
        if kind == "measure":
            plaq.append(e.plaquette())
    if kind == "measure":
        return {"plaquette": np.array(plaq), "links": e.tiled(64)}
    if kind == "counts":
        return {"attempts": e.attempts, "accepts": e.accepts, "links": e.tiled(64)}
    return {"links": e.tiled(64)}
