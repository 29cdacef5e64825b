"""Performance cases of the emulator: the calls that a variational chemistry
program makes, over the range of problems it makes them on.

A case is a dict of plain values:

* ``kind``: which entry points one pass goes through (see ``run``);
* ``n``, ``na``, ``nb``: qubits, alpha and beta electrons;
* ``ops``: ansatz length (sampled from the singles and doubles pool without
  replacement; 0: the whole pool in its canonical order);
* ``rank``: number of symmetric factors the two-electron integrals are built
  from (8: the synthetic Hamiltonians of the benchmark, 0: as many as orbital
  pairs, the full rank that integrals read from an FCIDUMP file have);
* ``precision`` (0 FP64, 1 FP32 amplitudes), ``ordering`` (0 interleaved, 1
  blocked qubits), ``qeb`` (qubit instead of fermionic excitations), ``dets``
  (determinants of a warm start; 0: the reference determinant), ``pool`` (size
  of a screened operator pool), ``count`` (instances of a batch).

Integrals, excitation lists, angles and start states are drawn from the seed.
``exact`` evaluates the same quantities in plain FP64 torch from the operator
definitions, without the emulator.
"""

from math import comb

import numpy as np
import torch

import paper_2405_11567_amd as fsv

BASE = {"kind": "grad", "n": 24, "na": 6, "nb": 6, "ops": 200, "rank": 8, "precision": 0, "ordering": 0,
        "qeb": False, "dets": 0, "pool": 0, "count": 0}


def _case(**kw):
    c = dict(BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a 4-electron toy or embedded fragment, where the
        # optimiser's time per step is launches and host work
        _case(name="grad_8q", n=8, na=2, nb=2, ops=0),
        # a whole UCCSD ansatz on a small molecule: many operators, a state
        # that fits on the chip
        _case(name="grad_16q_uccsd", n=16, na=4, nb=4, ops=0),
        # a growing ADAPT ansatz of qubit excitations on an open-shell system,
        # blocked qubit order, warm-started from a selected-CI expansion
        _case(name="grad_22q_qeb_warm", n=22, na=5, nb=4, ops=80, ordering=1, qeb=True, dets=1000),
        # the benchmark's workload: one optimiser step at 24 qubits
        _case(name="grad_24q"),
        # the same with FP32 amplitudes
        _case(name="grad_24q_fp32", precision=1),
        # an ordinary molecule: integrals of full rank, as read from a file
        _case(name="grad_24q_full_rank", ops=100, rank=0),
        # the largest state a user runs on one GPU day to day
        _case(name="grad_30q", n=30, na=7, nb=7, ops=500),
        # a serving loop that may not allocate
        _case(name="grad_noalloc_20q", kind="noalloc", n=20, na=5, nb=5, ops=100),
        # forward only: a large state prepared for reading, and its energy
        _case(name="state_energy_28q", kind="state", n=28, na=6, nb=6, ops=100),
        # one outer iteration of the self-consistent loop: new one-body
        # potential, a gradient step, the state, its energy and its density
        _case(name="scf_step_24q", kind="scf", ops=100),
        # one ADAPT growth step: the whole pool screened at the current state
        _case(name="pool_24q", kind="pool", ops=60, pool=1818, qeb=True),
        # many small independent problems at once (geometries, fragments)
        _case(name="batch_256", kind="batch", n=0, na=0, nb=0, ops=0, count=256),
    ]


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["grad"] * 5 + ["noalloc", "state", "scf", "pool", "batch"])
    if kind == "batch":
        return _case(kind="batch", n=0, na=0, nb=0, ops=0, count=int(round(2 ** rng.uniform(3, 8))))
    top = {"grad": 24, "noalloc": 22, "state": 28, "scf": 24, "pool": 24}[kind]
    n = 2 * rng.randint(4, top // 2)
    if n in (14, 26):  # 14: a size whose direct-product tests are skipped; 26: plans that take 10 s to build
        n += 2
    if kind == "grad" and rng.random() < 0.2:
        n = rng.choice([28, 30])
    m = n // 2
    na = min(m - 1, max(2, m // 2 + rng.randint(-1, 1)))
    nb = max(1, na - rng.randint(0, 2))
    if n == 24 and comb(m, na) * comb(m, nb) > 900000:
        nb = na - 2
    size = len(pool_of(m, na, nb))
    ops = min(size, int(round(2 ** rng.uniform(4, 7.7 if n < 28 else 6.5))))
    big = n >= 28
    return _case(kind=kind, n=n, na=na, nb=nb, ops=ops,
                 rank=8 if big else rng.choice([8, 8, 0]),
                 precision=1 if kind == "grad" and rng.random() < 0.2 else 0,
                 ordering=rng.randint(0, 1), qeb=rng.random() < 0.4,
                 dets=0 if big or kind != "grad" else rng.choice([0, 0, 50, 500]) if comb(m, na) * comb(m, nb) > 1000 else 0,
                 pool=0 if kind != "pool" else min(size, rng.randint(50, 1500)))


# ------------------------------------------------------------------ inputs ----
class Problem:
    """The attributes a plan reads, and the angles."""

    def __init__(self, n, na, nb, h, g, ops, theta, e_core, ordering, qeb):
        self.n_qubits, self.n_alpha, self.n_beta = n, na, nb
        self.h, self.g, self.ops, self.theta = h, g, ops, theta
        self.e_core, self.ordering, self.excitation = e_core, ordering, int(qeb)


def pool_of(m, na, nb):
    """Spin-conserving singles and doubles out of the reference determinant:
    (a, b, j, i) spin-orbital labels 2 p + s, singles (a, -1, -1, i)."""
    occ, vir = (range(na), range(nb)), (range(na, m), range(nb, m))
    out = [(2 * a + s, -1, -1, 2 * i + s) for s in (0, 1) for i in occ[s] for a in vir[s]]
    for s in (0, 1):
        out += [(2 * a + s, 2 * b + s, 2 * j + s, 2 * i + s) for i in occ[s] for j in occ[s] if j > i
                for a in vir[s] for b in vir[s] if b > a]
    out += [(2 * a, 2 * b + 1, 2 * j + 1, 2 * i) for i in occ[0] for j in occ[1] for a in vir[0] for b in vir[1]]
    return np.array(out, dtype=np.int32).reshape(-1, 4)


def symmetric(rng, m, std):
    u = np.triu(rng.normal(0.0, std, (m, m)))
    return u + np.triu(u, 1).T


def integrals(rng, m, rank):
    h = symmetric(rng, m, 0.1)
    h[np.diag_indices(m)] = np.linspace(-1.0, 0.5, m)
    r = rank or m * (m + 1) // 2
    # factors that fall off as those of a Cholesky-decomposed molecule do
    f = np.stack([symmetric(rng, m, 0.05 * (1.0 if rank else 0.9 ** k)) for k in range(r)]).reshape(r, m * m)
    return h, (f.T @ f).reshape(m, m, m, m)


def problem(rng, n, na, nb, ops, rank, ordering, qeb, replace=False):
    m = n // 2
    h, g = integrals(rng, m, rank)
    pool = pool_of(m, na, nb)
    if ops:
        pool = pool[rng.integers(0, len(pool), ops) if replace else rng.choice(len(pool), ops, replace=False)]
    theta = rng.normal(0.0, 0.1 if n <= 24 else 0.05, len(pool))
    return Problem(n, na, nb, h, g, np.ascontiguousarray(pool), theta, 0.7 * m, ordering, qeb)


def batch_of(count, seed):
    """10 to 20 qubits, around half filling, 50 to 150 operators each (the
    sizes from the count alone, everything else from the seed)."""
    sizes, rng = np.random.default_rng((4, count)), np.random.default_rng((seed, 9))
    out = []
    for _ in range(count):
        n = 2 * int(sizes.integers(5, 11))
        ne, k = n // 2 + int(sizes.integers(-2, 3)), int(sizes.integers(50, 151))
        out.append(problem(rng, n, (ne + 1) // 2, ne // 2, k, 8, 0, False, replace=True))
    return out


def inputs(case, seed):
    """Everything of one case that comes from the seed, on the host."""
    if case["kind"] == "batch":
        return {"problems": batch_of(case["count"], seed)}
    rng = np.random.default_rng((seed, case["n"], case["na"], case["nb"], case["ops"]))
    p = problem(rng, case["n"], case["na"], case["nb"], case["ops"], case["rank"], case["ordering"], case["qeb"])
    m = case["n"] // 2
    out = {"problem": p, "v": symmetric(rng, m, 0.02)}
    if case["pool"]:
        every = pool_of(m, case["na"], case["nb"])
        out["pool"] = every[rng.choice(len(every), min(case["pool"], len(every)), replace=False)]
    if case["dets"]:
        a, b = strings(m, case["na"]), strings(m, case["nb"])
        at = rng.choice(len(a) * len(b), min(case["dets"], len(a) * len(b)), replace=False)
        at[0] = 0 if 0 not in at else at[0]
        coef = rng.normal(size=len(at)) * 0.02
        coef[0] = 1.0
        out["at"], out["coef"] = at, coef / np.linalg.norm(coef)
        xa, xb = qubits(a, case["n"], 0, case["ordering"]), qubits(b, case["n"], 1, case["ordering"])
        out["dets"] = (xa[at // len(b)] | xb[at % len(b)]).astype(np.uint64)
    return out


def prepare(case, seed):
    d = inputs(case, seed)
    if case["kind"] == "batch":
        return {"kind": "batch", "batch": fsv.Batch(d["problems"]),
                "theta": np.concatenate([p.theta for p in d["problems"]])}
    p = d["problem"]
    plan = fsv.Plan(p, precision=case["precision"])
    s = {"kind": case["kind"], "plan": plan, "theta": p.theta, "v": d["v"], "psi": plan.new_state()}
    if case["kind"] != "state":
        s["lam"] = plan.new_state()
    if case["dets"]:
        plan.set_initial_state(d["dets"], d["coef"])
    if case["pool"]:
        s["pool"] = plan.pool(d["pool"])
    return s


def run(s):
    kind, plan = s["kind"], s.get("plan")
    if kind == "batch":
        return s["batch"].energy_grad(s["theta"])
    if kind == "grad":
        return plan.energy_grad(s["theta"], s["psi"], s["lam"])
    if kind == "noalloc":
        return plan.energy_grad_noalloc(s["theta"], s["psi"], s["lam"])
    if kind == "state":
        psi = plan.ansatz_apply(s["theta"], s["psi"])
        return psi, plan.energy(psi)
    if kind == "pool":
        return s["pool"].gradients(s["theta"], s["psi"], s["lam"])
    plan.set_onebody_potential(s["v"])
    e, g = plan.energy_grad(s["theta"], s["psi"], s["lam"])
    psi = plan.ansatz_apply(s["theta"], s["psi"])
    return e, g, psi, plan.energy(psi), plan.rdm1(psi)


# -------------------------------------------------------------------- work ----
def _pairs(m, n, part):
    """Strings of one spin that an operator with (annihilated, created) = part moves."""
    d, c = part
    return comb(m, n) if d + c == 0 else comb(m - d - c, n - d) if n >= d else 0


def _mean_pairs(m, na, nb):
    """Active amplitude pairs of a pool operator, averaged over the pool."""
    va, vb = m - na, m - nb
    kinds = [(na * va, (1, 1), (0, 0)), (nb * vb, (0, 0), (1, 1)), (comb(na, 2) * comb(va, 2), (2, 2), (0, 0)),
             (comb(nb, 2) * comb(vb, 2), (0, 0), (2, 2)), (na * va * nb * vb, (1, 1), (1, 1))]
    total = sum(k for k, _, _ in kinds)
    return sum(k * _pairs(m, na, a) * _pairs(m, nb, b) for k, a, b in kinds) / max(total, 1), total


def _plan_work(m, na, nb, ops, rank, size, sweeps, products, pool=0):
    """size: bytes of a stored amplitude; sweeps: rotated vectors (1 forward,
    3 with the adjoint pair); products: applications of H."""
    pairs, total = _mean_pairs(m, na, nb)
    k = ops or total
    dim = comb(m, na) * comb(m, nb)
    ea, eb = na * (m - na) + 1, nb * (m - nb) + 1  # excitations of a string, its own term once
    ab = min(ea * eb, 8 * (ea + eb)) if rank == 8 else ea * eb
    same = sum(1 + e * (v - e) + comb(e, 2) * comb(v - e, 2) for e, v in ((na, m), (nb, m)))
    flops = k * pairs * (6.0 if sweeps == 1 else 21.0) + products * 2.0 * dim * (ab + same) + 4.0 * pool * pairs
    # psi written by the forward sweep; read and H psi written by the product; both read by the adjoint sweep
    moved = dim * size * (1.0 + 2.0 * min(products, 1) + (2.0 if sweeps == 3 or pool else 0.0))
    return moved, flops


def work(case):
    if case["kind"] == "batch":
        b = f = 0.0
        for n in range(10, 21, 2):  # the mean instance of each size
            ne = n // 2
            x, y = _plan_work(n // 2, (ne + 1) // 2, ne // 2, 100, 8, 8, 3, 1)
            b, f = b + x, f + y
        return {"bytes": b * case["count"] / 6, "flops": f * case["count"] / 6}
    m, na, nb, kind = case["n"] // 2, case["na"], case["nb"], case["kind"]
    size = 4 if case["precision"] else 8
    dim, full = comb(m, na) * comb(m, nb), 16.0 * 2 ** case["n"]
    sweeps = 3 if kind in ("grad", "noalloc", "scf") else 1
    b, f = _plan_work(m, na, nb, case["ops"], case["rank"], size, sweeps, 1, case["pool"])
    if kind == "state":
        return {"bytes": full + 16.0 * dim, "flops": f}
    if kind == "scf":  # besides: the dense state, its energy and its density
        x, y = _plan_work(m, na, nb, case["ops"], case["rank"], size, 1, 1)
        return {"bytes": b + full + 32.0 * dim, "flops": f + y + 2.0 * dim * (na * (m - na) + nb * (m - nb))}
    return {"bytes": b, "flops": f}


# ------------------------------------------------- plain FP64 evaluation ----
def strings(m, k):
    """Occupation masks of k electrons in m orbitals, ascending."""
    x = np.arange(1 << m, dtype=np.int64)
    return x[np.bitwise_count(x) == k]


def qubits(s, n, spin, ordering):
    """Qubit strings of orbital strings s of one spin."""
    out = np.zeros_like(s)
    for p in range(n // 2):
        out |= ((s >> p) & 1) << (2 * p + spin if ordering == 0 else p + spin * (n // 2))
    return out


class Plain:
    """The sector state as an FP64 matrix over alpha x beta strings (creation
    operators of all alpha orbitals before those of all beta orbitals)."""

    def __init__(self, p, device):
        self.p, self.dev, self.kept = p, device, {}
        self.m = p.n_qubits // 2
        self.a, self.b = strings(self.m, p.n_alpha), strings(self.m, p.n_beta)
        # sign between this order of creation operators and ascending qubits:
        # one transposition for each alpha orbital above a beta orbital
        if p.ordering == 0:
            cnt = np.zeros((len(self.a), len(self.b)), dtype=np.int8)
            for q in range(self.m):
                below = np.bitwise_count(self.b & ((1 << q) - 1))
                cnt += ((self.a >> q) & 1).astype(np.int8)[:, None] * (below & 1).astype(np.int8)[None, :]
            self.phase = torch.from_numpy((1.0 - 2.0 * (cnt & 1))).to(device)
        else:
            self.phase = torch.ones(len(self.a), len(self.b), dtype=torch.float64, device=device)

    def start(self, at=None, coef=None):
        c = torch.zeros(len(self.a), len(self.b), dtype=torch.float64, device=self.dev)
        if at is None:
            c[0, 0] = self.phase[0, 0]
        else:
            i = torch.from_numpy(at).to(self.dev)
            c.view(-1)[i] = torch.from_numpy(coef).to(self.dev) * self.phase.view(-1)[i]
        return c

    def _moves(self, op):
        """tau = a+_a a+_b a_j a_i on the strings: (sources, targets, signs) of each spin, and a common sign."""
        cur = [self.a.copy(), self.b.copy()]
        sgn = [np.ones(len(self.a)), np.ones(len(self.b))]
        ok = [np.ones(len(self.a), bool), np.ones(len(self.b), bool)]
        common, n_alpha = 1.0, self.p.n_alpha
        a, b, j, i = (int(v) for v in op)
        for lab, up in ((i, 0), (j, 0), (b, 1), (a, 1)):
            if lab < 0:
                continue
            q, s = divmod(lab, 2)
            bit = 1 << q
            ok[s] &= ((cur[s] & bit) != 0) == (up == 0)
            sgn[s] *= 1.0 - 2.0 * (np.bitwise_count(cur[s] & (bit - 1)) & 1)
            cur[s] ^= bit
            if s:
                common *= -1.0 if n_alpha & 1 else 1.0
            else:
                n_alpha += 1 if up else -1
        out = []
        for s, all_s in ((0, self.a), (1, self.b)):
            src = np.flatnonzero(ok[s])
            dst = np.searchsorted(all_s, cur[s][src])
            out.append([torch.from_numpy(x).to(self.dev) for x in (src, dst, sgn[s][src])])
        return out[0], out[1], common

    def pairs(self, op, qeb):
        """Flat source and target positions of tau's pairs, and the sign of each."""
        key = tuple(int(v) for v in op)
        if key in self.kept:
            return self.kept[key]
        (ia, ja, sa), (ib, jb, sb), common = self._moves(op)
        nb = len(self.b)
        src = (ia[:, None] * nb + ib[None, :]).view(-1)
        dst = (ja[:, None] * nb + jb[None, :]).view(-1)
        if qeb:
            f = self.phase.view(-1)
            out = src, dst, f[src] * f[dst]
        else:
            out = src, dst, (common * sa[:, None] * sb[None, :]).reshape(-1)
        if len(self.a) * nb < 1 << 17:  # small states: each operator's pairs once
            self.kept[key] = out
        return out

    @staticmethod
    def rotate(c, pairs, theta):
        src, dst, sg = pairs
        v = c.view(-1)
        x, y = v[src], v[dst]
        co, si = np.cos(theta), np.sin(theta)
        v[src] = co * x - si * (sg * y)
        v[dst] = co * y + si * (sg * x)

    @staticmethod
    def bracket(lam, c, pairs):
        """2 Re<lam| tau - tau+ |c>."""
        src, dst, sg = pairs
        l, v = lam.view(-1), c.view(-1)
        return 2.0 * float((sg * (l[dst] * v[src] - l[src] * v[dst])).sum())

    def forward(self, theta, at=None, coef=None):
        c = self.start(at, coef)
        for op, t in zip(self.p.ops, theta):
            self.rotate(c, self.pairs(op, self.p.excitation), t)
        return c

    def single(self, spin, p, q):
        """a+_p a_q on the strings of one spin: (sources, targets, signs)."""
        s = self.b if spin else self.a
        src = np.flatnonzero((((s >> q) & 1) == 1) & ((((s >> p) & 1) == 0) | (p == q)))
        x = s[src]
        y = x & ~(1 << q)
        sg = 1.0 - 2.0 * ((np.bitwise_count(x & ((1 << q) - 1)) + np.bitwise_count(y & ((1 << p) - 1))) & 1)
        dst = np.searchsorted(s, y | (1 << p))
        return [torch.from_numpy(v).to(self.dev) for v in (src, dst, sg)]

    def add_single(self, out, c, p, q, scale=1.0):
        """out += scale (E_pq of both spins) c."""
        src, dst, sg = self.single(0, p, q)
        out.index_add_(0, dst, c[src] * (scale * sg)[:, None])
        src, dst, sg = self.single(1, p, q)
        out.index_add_(1, dst, c[:, src] * (scale * sg)[None, :])

    def product(self, c, v=None):
        """H c with H = e_core + sum h'_pq E_pq + 1/2 sum (pq|rs) E_pq E_rs."""
        m, g = self.m, self.p.g
        h = self.p.h if v is None else self.p.h + v
        h1 = h - 0.5 * np.einsum("prrq->pq", g)
        out = self.p.e_core * c
        parts = torch.zeros((m * m,) + tuple(c.shape), dtype=torch.float64, device=self.dev)
        for p in range(m):
            for q in range(m):
                self.add_single(parts[p * m + q], c, p, q)
                out += float(h1[p, q]) * parts[p * m + q]
        mat = torch.from_numpy(np.ascontiguousarray(g.reshape(m * m, m * m))).to(self.dev)
        flat = parts.view(m * m, -1)
        for lo in range(0, flat.shape[1], 1 << 20):
            flat[:, lo:lo + (1 << 20)] = mat @ flat[:, lo:lo + (1 << 20)].contiguous()
        for p in range(m):
            for q in range(m):
                self.add_single(out, parts[p * m + q], p, q, 0.5)
        return out

    def gradient(self, theta, c, lam):
        grad = np.zeros(len(theta))
        for k in range(len(theta) - 1, -1, -1):
            pr = self.pairs(self.p.ops[k], self.p.excitation)
            grad[k] = self.bracket(lam, c, pr)
            self.rotate(c, pr, -theta[k])
            self.rotate(lam, pr, -theta[k])
        return grad

    def density(self, c):
        out = np.zeros((2, self.m, self.m), dtype=np.complex128)
        for p in range(self.m):
            for q in range(self.m):
                src, dst, sg = self.single(0, p, q)
                out[0, p, q] = float((c[dst] * c[src] * sg[:, None]).sum())
                src, dst, sg = self.single(1, p, q)
                out[1, p, q] = float((c[:, dst] * c[:, src] * sg[None, :]).sum())
        return out

    def dense(self, c):
        p = self.p
        x = qubits(self.a, p.n_qubits, 0, p.ordering)[:, None] | qubits(self.b, p.n_qubits, 1, p.ordering)[None, :]
        out = torch.zeros(1 << p.n_qubits, dtype=torch.complex128, device=self.dev)
        out[torch.from_numpy(x.reshape(-1)).to(self.dev)] = (c * self.phase).view(-1).to(torch.complex128)
        return out


def exact(case, seed):
    dev = "cuda:0" if torch.cuda.is_available() else "cpu"
    d = inputs(case, seed)
    kind = case["kind"]
    if kind == "batch":
        es, gs = [], []
        for p in d["problems"]:
            w = Plain(p, "cpu")  # small states: faster on the host
            c = w.forward(p.theta)
            lam = w.product(c)
            es.append(float((c * lam).sum()))
            gs.append(w.gradient(p.theta, c, lam))
        return np.array(es), np.concatenate(gs)
    p = d["problem"]
    w = Plain(p, dev)
    c = w.forward(p.theta, d.get("at"), d.get("coef"))
    lam = w.product(c, d["v"] if kind == "scf" else None)
    e = float((c * lam).sum())
    if kind == "state":
        return w.dense(c), e
    if kind == "pool":
        return e, np.array([w.bracket(lam, c, w.pairs(op, case["qeb"])) for op in d["pool"]])
    if kind == "scf":
        psi, gamma = w.dense(c), w.density(c)
        return e, w.gradient(p.theta, c, lam), psi, e, gamma
    return e, w.gradient(p.theta, c, lam)
