"""The workloads whose speed this framework is judged by.

Each case is one piece of an iQCC calculation as a program makes it through
paper_2603_08883_amd: QMF energies and angle gradients of a resident
Hamiltonian, screening of DIS candidates, dressing (out of place, in place,
taped for reverse mode, many small Hamiltonians at once), a whole iQCC
iteration, and the term limit with its export.  The Hamiltonians are synthetic
but built like the real ones: Jordan-Wigner strings of local one- and two-body
excitations (flips on up to four spin orbitals, Z strings between them, an even
number of Y's), grown by XOR with DIS-form generators where more terms are
wanted than the plain Hamiltonian has, with coefficients over several decades.

  listed()              the listed cases
  draw(rng)             one more case of the same ranges
  prepare(case, seed)   inputs, stores and handles a program holds, on the GPU
  run(state)            one pass through the public entry points
  work(case)            bytes and operations a pass cannot do without
  exact(case, seed)     what run() returns, from plain torch in 64 bits
"""
import math

import numpy as np
import torch

from paper_2603_08883_amd import autograd, iqcc

DEV = "cuda"
EPS = 1e-8           # compression threshold of the chains (the benchmark's value)
BAND = 6             # locality of the orbital pairs (the banded Hamiltonians' value)

_ctx = None


def context():
    """The one library context of the program."""
    global _ctx
    if _ctx is None:
        _ctx = iqcc.Context(0)
    return _ctx


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest call: the energy of an H2-sized Hamiltonian inside an
        # optimiser's line search, where only latency counts
        {"name": "energy_8q", "kind": "energy", "nq": 8, "n": 361, "angles": "random"},
        # energy of a large resident Hamiltonian after a long chain
        {"name": "energy_124q", "kind": "energy", "nq": 124, "n": 16_000_001, "angles": "random"},
        # reverse mode of the energy: all Bloch-angle gradients and the
        # cotangent of every coefficient
        {"name": "angle_gradient_124q", "kind": "gradient", "nq": 124, "n": 4_000_003, "angles": "random"},
        # the screening step of an iteration: a thousand generators against a
        # Hamiltonian of a million terms
        {"name": "dis_screen_100q", "kind": "dis", "nq": 100, "n": 1_000_003, "n_cand": 1000, "w_max": 12,
         "angles": "random"},
        # the gradients of the handful of generators an iteration applies
        {"name": "dis_few_40q", "kind": "dis", "nq": 40, "n": 233_001, "n_cand": 5, "w_max": 8, "angles": "random"},
        # out-of-place dressing with the energy carried along, as the
        # iteration's ping-pong makes it
        {"name": "dress_40q", "kind": "dress", "nq": 40, "n": 233_001, "steps": 4},
        # in-place chain of a small molecule: a copy of H0 and every step is
        # launches and latency
        {"name": "inplace_chain_24q", "kind": "inplace", "nq": 24, "n": 12_007, "steps": 10},
        # the headline path at production size: copy of H0, ten in-place steps
        # with the energy after each, angle gradients of the result
        {"name": "inplace_chain_124q", "kind": "inplace", "nq": 124, "n": 1_119_607, "steps": 10},
        # one gradient step of the joint optimisation of angles and amplitudes:
        # taped chain forward, reverse sweep
        {"name": "train_step_40q", "kind": "train", "nq": 40, "n": 50_021, "steps": 8},
        # one whole iQCC iteration from a freshly loaded Hamiltonian
        {"name": "iteration_24q", "kind": "iteration", "nq": 24, "n": 12_007, "w_max": 4, "n_select": 4},
        # many small Hamiltonians of uneven size in one captured launch, then
        # their energies
        {"name": "batch_32h", "kind": "batch", "n_ham": 32, "q_lo": 16, "q_hi": 64, "lo": 1000, "hi": 500_000},
        # the maximum-terms limit of a long run, and the limited Hamiltonian
        # taken out (a checkpoint)
        {"name": "term_limit_100q", "kind": "limit", "nq": 100, "n": 3_000_017, "keep": 0.8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["energy", "gradient", "dis", "dress", "inplace", "train", "iteration", "batch", "limit"])
    # qubits: one word to four, the short ones more often
    nq = rng.choice([rng.randint(8, 63), rng.randint(24, 64), rng.randint(65, 128), rng.randint(65, 128),
                     rng.randint(129, 200)])
    angles = "random" if rng.random() < 0.8 else "reference"
    if kind == "energy":
        return {"kind": kind, "nq": nq, "n": _log(rng, 100, 8e6 if nq <= 128 else 4e6), "angles": angles}
    if kind == "gradient":
        # (at the poles every angle gradient of a number-conserving sum vanishes)
        return {"kind": kind, "nq": nq, "n": _log(rng, 100, 3e6), "angles": "random"}
    if kind == "dis":
        n = _log(rng, 1000, 1e6)
        return {"kind": kind, "nq": nq, "n": n, "n_cand": _log(rng, 1, min(1000, 5e8 / n)),
                "w_max": rng.randint(6, 12), "angles": angles}
    if kind == "dress":
        return {"kind": kind, "nq": nq, "n": _log(rng, 300, 1e6), "steps": rng.randint(1, 5)}
    if kind == "inplace":
        return {"kind": kind, "nq": nq, "n": _log(rng, 300, 8e5), "steps": rng.randint(2, 9)}
    if kind == "train":
        return {"kind": kind, "nq": min(nq, 128), "n": _log(rng, 300, 1.5e5), "steps": rng.randint(2, 8)}
    if kind == "iteration":
        return {"kind": kind, "nq": rng.randint(10, 40), "n": _log(rng, 300, 15_000), "w_max": 4,
                "n_select": rng.randint(1, 5)}
    if kind == "batch":
        lo = _log(rng, 300, 3000)
        return {"kind": kind, "n_ham": rng.randint(3, 40), "q_lo": 16, "q_hi": rng.choice([32, 64]),
                "lo": lo, "hi": lo * _log(rng, 4, 150)}
    return {"kind": kind, "nq": nq, "n": _log(rng, 300, 2.5e6), "keep": round(rng.uniform(0.3, 0.95), 3)}


# ---------------------------------------------------------------------------
# inputs (torch, from the seed alone)
# ---------------------------------------------------------------------------

def words(nq):
    return (nq + 63) // 64


def _bit(q, W):
    """(W, N) words with bit q[i] set in column i."""
    w = torch.arange(W, device=DEV).unsqueeze(1)
    return torch.where((q >> 6) == w, torch.ones_like(q) << (q & 63), torch.zeros_like(q))


def _below(q, W):
    """(W, N) words with the bits below q[i] set."""
    w = torch.arange(W, device=DEV).unsqueeze(1)
    k = (q - 64 * w).clamp(0, 64)
    return torch.where(k >= 64, torch.full_like(k, -1), (torch.ones_like(k) << k.clamp(max=63)) - 1)


_M = (0x5555555555555555, 0x3333333333333333, 0x0F0F0F0F0F0F0F0F)


def _pop(v):
    """Set bits of each int64."""
    v = v - ((v >> 1) & _M[0])
    v = (v & _M[1]) + ((v >> 2) & _M[1])
    v = (v + (v >> 4)) & _M[2]
    return ((v * 0x0101010101010101) >> 56) & 0xFF


def _count(a):
    """Set bits of each column of (W, N) words."""
    return _pop(a).sum(0)


def _mix(h):
    """A bijective 64-bit finaliser (multiplications and logical shifts)."""
    h = (h ^ ((h >> 32) & 0xFFFFFFFF)) * -2960836687051489901
    h = (h ^ ((h >> 29) & 0x7FFFFFFFF)) * -7723592293110705685
    return h ^ ((h >> 32) & 0xFFFFFFFF)


def _hash(x, z):
    """A 64-bit mix of each column's key."""
    h = torch.zeros_like(x[0])
    for w in range(x.shape[0]):
        h = _mix(_mix(h + x[w] * -7046029254386353131) ^ (z[w] * 2870177450012600261))
    return h


def _distinct(x, z, c):
    h, order = torch.sort(_hash(x, z), stable=True)
    keep = torch.ones_like(h, dtype=torch.bool)
    keep[1:] = h[1:] != h[:-1]
    at = order[keep]
    return x[:, at], z[:, at], c[at]


def _excitations(nq, k, gen):
    """k Jordan-Wigner strings of local one- and two-body excitations, with repeats."""
    W, no = words(nq), nq // 2

    def ri(hi):
        return torch.randint(0, hi, (k,), generator=gen, device=DEV)

    p, r = ri(no), ri(no)
    q = (p + ri(2 * BAND + 1) - BAND).clamp(0, no - 1)
    s = (r + ri(2 * BAND + 1) - BAND).clamp(0, no - 1)
    u, v = ri(2), ri(2)
    two = ri(16) > 0
    x = torch.zeros((W, k), dtype=torch.int64, device=DEV)
    z = torch.zeros_like(x)
    for mode, on in ((2 * p + u, None), (2 * r + v, two), (2 * s + v, two), (2 * q + u, None)):
        b, t = _bit(mode, W), _below(mode, W) ^ (_bit(mode, W) * ri(2))
        x = x ^ (b if on is None else torch.where(on, b, torch.zeros_like(b)))
        z = z ^ (t if on is None else torch.where(on, t, torch.zeros_like(t)))
    # an even number of Y's (real coefficients)
    odd = (_count(x & z) & 1).bool()
    first = torch.zeros_like(odd)
    for w in range(W):
        here = odd & ~first & (x[w] != 0)
        z[w] = torch.where(here, z[w] ^ (x[w] & -x[w]), z[w])
        first |= here
    d = ((p - q).abs() + (r - s).abs()).double()
    c = torch.randn(k, generator=gen, device=DEV, dtype=torch.float64) * 0.1 * torch.exp(-d / 3)
    return x, z, c


def generators(x, nq, count, w_max, seed):
    """`count` distinct DIS-form generators on the host, (count, W) uint64 each:
    the flip set of a term, one Y, X elsewhere, Z's outside it, weight 2 .. w_max."""
    rng = np.random.default_rng(seed)
    W = words(nq)
    some = x[:, torch.from_numpy(rng.integers(0, x.shape[1], 40 * count + 200)).to(DEV)].cpu().numpy()
    out, seen = [], set()
    for col in range(some.shape[1]):
        f = [64 * w + b for w in range(W) for b in range(64) if (int(some[w, col]) >> b) & 1]
        if not 1 <= len(f) <= w_max:
            continue
        xs, zs = sum(1 << q for q in f), 1 << f[rng.integers(len(f))]
        rest = [q for q in range(nq) if q not in f]
        more = int(rng.integers(max(2, len(f)), w_max + 1)) - len(f) if len(f) < w_max else 0
        for q in rng.choice(rest, size=min(more, len(rest)), replace=False):
            zs |= 1 << int(q)
        if (xs, zs) not in seen:
            seen.add((xs, zs))
            out.append((xs, zs))
        if len(out) == count:
            break
    m = (1 << 64) - 1
    gx = np.array([[(a >> (64 * w)) & m for w in range(W)] for a, _ in out], dtype=np.uint64)
    gz = np.array([[(b >> (64 * w)) & m for w in range(W)] for _, b in out], dtype=np.uint64)
    return gx, gz


def _column(g):
    return torch.from_numpy(g.view(np.int64).copy()).to(DEV).unsqueeze(1)


def hamiltonian(nq, n, seed):
    """(x, z, c): at most n (and mostly exactly n) distinct terms, (W, n) int64 words."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    x, z, c = _distinct(*_excitations(nq, min(4 * n, 600_000), gen))
    gx, gz = generators(x, nq, 48, 8, seed + 1)
    for j in range(400):
        if x.shape[1] >= n:
            break
        pick = torch.rand(x.shape[1], generator=gen, device=DEV) < 0.5
        u = torch.rand(int(pick.sum()), generator=gen, device=DEV, dtype=torch.float64) * 0.4 - 0.2
        j %= len(gx)
        x, z, c = _distinct(torch.cat([x, x[:, pick] ^ _column(gx[j])], 1),
                            torch.cat([z, z[:, pick] ^ _column(gz[j])], 1), torch.cat([c, c[pick] * u]))
    at = torch.randperm(x.shape[1], generator=gen, device=DEV)[:n]
    return x[:, at].contiguous(), z[:, at].contiguous(), c[at].contiguous()


def qmf_angles(nq, seed, how="random"):
    """Bloch angles: anywhere on the sphere, or the reference determinant's (poles)."""
    rng = np.random.default_rng(seed + 2)
    theta, phi = rng.uniform(0, np.pi, nq), rng.uniform(0, 2 * np.pi, nq)
    if how == "reference":
        theta = np.where(np.arange(nq) < nq // 2, np.pi, 0.0)
    return torch.from_numpy(theta).to(DEV), torch.from_numpy(phi).to(DEV)


def amplitudes(k, seed):
    return np.random.default_rng(seed + 3).uniform(-0.2, 0.2, k)


def batch_inputs(case, seed):
    """One (nq, x, z, c, px, pz, tau, theta, phi) per Hamiltonian."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(case["n_ham"]):
        nq = 2 * int(rng.integers(case["q_lo"] // 2, case["q_hi"] // 2 + 1))
        n = int(np.exp(rng.uniform(np.log(case["lo"]), np.log(case["hi"]))))
        x, z, c = hamiltonian(nq, n, seed + 100 * (i + 1))
        px, pz = generators(x, nq, 1, 8, seed + 100 * (i + 1) + 7)
        theta, phi = qmf_angles(nq, seed + i)
        out.append((nq, x, z, c, px[0], pz[0], float(rng.uniform(-0.2, 0.2)), theta, phi))
    return out


# ---------------------------------------------------------------------------
# one pass of each kind
# ---------------------------------------------------------------------------

def _store(nq, max_terms, flags=0):
    return iqcc.Store(context(), nq, max(int(max_terms), 16), flags)


def _loaded(nq, x, z, c, max_terms=None, flags=0):
    st = _store(nq, max_terms or x.shape[1], flags)
    iqcc.iqcc_store_load(context().handle, st.handle, x, z, c)
    return st


def _room(n, nq, steps):
    """Terms a store needs after `steps` dressing steps (measured growth: 1.4 to 1.5 a step)."""
    return int(min(n * min(2.0 ** steps, 1.6 * 1.45 ** steps), 4.0 ** nq))


def prepare(case, seed):
    kind = case["kind"]
    ctx = context().handle
    if kind == "batch":
        rows = batch_inputs(case, seed)
        ins = [_loaded(nq, x, z, c) for nq, x, z, c, *_ in rows]
        outs = [_store(nq, 2 * x.shape[1]) for nq, x, *_ in rows]
        batch = iqcc.iqcc_batch_create(ctx, [s.handle for s in ins], [s.handle for s in outs],
                                       np.stack([r[4] for r in rows]), np.stack([r[5] for r in rows]),
                                       np.array([r[6] for r in rows]), EPS)
        torch.cuda.synchronize()
        return {"kind": kind, "ins": ins, "outs": outs, "batch": Batch(batch), "angles": [(r[7], r[8]) for r in rows],
                "energy": torch.zeros(len(rows), dtype=torch.float64, device=DEV)}
    nq, n = case["nq"], case["n"]
    x, z, c = hamiltonian(nq, n, seed)
    n = x.shape[1]
    theta, phi = qmf_angles(nq, seed, case.get("angles", "random"))
    s = {"kind": kind, "theta": theta, "phi": phi}
    if kind in ("energy", "gradient", "dis"):
        s["h"] = _loaded(nq, x, z, c)
    if kind == "gradient":
        s["lam"] = torch.zeros(iqcc.iqcc_store_rows(s["h"].handle), dtype=torch.float64, device=DEV)
    elif kind == "dis":
        gx, gz = generators(x, nq, case["n_cand"], case["w_max"], seed + 5)
        s["cx"], s["cz"] = iqcc.to_device_words(gx), iqcc.to_device_words(gz)
    elif kind in ("dress", "inplace", "train"):
        gx, gz = generators(x, nq, case["steps"], 8, seed + 5)
        s["ents"] = list(zip(gx, gz))
        s["taus"] = amplitudes(len(gx), seed)
        room = _room(n, nq, len(gx))
        if kind == "dress":
            s["h"] = _loaded(nq, x, z, c)
            s["a"], s["b"] = _store(nq, room), _store(nq, room)
            s["energies"] = torch.zeros(len(gx), dtype=torch.float64, device=DEV)
        elif kind == "inplace":
            s["h"] = _loaded(nq, x, z, c)
            s["work"] = _store(nq, room, iqcc.IQCC_STORE_INPLACE)
            s["energies"] = torch.zeros(len(gx), dtype=torch.float64, device=DEV)
        else:
            s["chain"] = autograd.DressingChain(context(), nq, *(iqcc.from_device_words(t) for t in (x, z)),
                                                c.cpu().numpy(), s["ents"], EPS)
            s["tau"] = torch.from_numpy(s["taus"]).to(DEV)
    elif kind == "iteration":
        s["x"], s["z"], s["c"] = x, z, c
        room = _room(n, nq, case["n_select"])
        s["h"], s["spare"] = _store(nq, room), _store(nq, room)
        s["w_max"], s["n_select"] = case["w_max"], case["n_select"]
    elif kind == "limit":
        s["h"], s["out"] = _loaded(nq, x, z, c), _store(nq, n)
        s["keep"] = int(case["keep"] * n)
    torch.cuda.synchronize()
    return s


class Batch:
    """A captured batch, given back with its state."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        try:
            iqcc.iqcc_batch_destroy(context().handle, self.handle)
        except Exception:
            pass


def run(s):
    ctx, kind = context().handle, s["kind"]
    theta, phi = s.get("theta"), s.get("phi")
    if kind == "energy":
        return iqcc.iqcc_qmf_energy(ctx, s["h"].handle, theta, phi)
    if kind == "gradient":
        dtheta, dphi = iqcc.iqcc_qmf_energy_backward(ctx, s["h"].handle, theta, phi, None, s["lam"])
        return {"dtheta": dtheta, "dphi": dphi, "lambda": s["lam"]}
    if kind == "dis":
        return iqcc.iqcc_dis_gradients(ctx, s["h"].handle, theta, phi, s["cx"], s["cz"])
    if kind == "dress":
        e, src, dst, free = s["energies"], s["h"], s["a"], s["b"]
        for j, (px, pz) in enumerate(s["ents"]):
            if j == 0:
                iqcc.iqcc_dress(ctx, src.handle, px, pz, s["taus"][j], EPS, dst.handle, theta, phi, e[0:1])
            else:
                iqcc.iqcc_dress_energy_update(ctx, src.handle, px, pz, s["taus"][j], EPS, dst.handle, theta, phi,
                                              e[j - 1:j], e[j:j + 1])
            src, dst, free = dst, free, dst
        dtheta, dphi = iqcc.iqcc_qmf_energy_backward(ctx, src.handle, theta, phi)
        return {"energies": e, "dtheta": dtheta, "dphi": dphi}
    if kind == "inplace":
        e, h = s["energies"], s["work"].handle
        iqcc.iqcc_store_copy(ctx, s["h"].handle, h)
        for j, (px, pz) in enumerate(s["ents"]):
            iqcc.iqcc_dress_inplace(ctx, h, px, pz, s["taus"][j], EPS, theta, phi, e[j - 1:j] if j else None,
                                    e[j:j + 1])
        dtheta, dphi = iqcc.iqcc_qmf_energy_backward(ctx, h, theta, phi)
        return {"energies": e, "dtheta": dtheta, "dphi": dphi}
    if kind == "train":
        th, ph, ta = (t.detach().requires_grad_(True) for t in (theta, phi, s["tau"]))
        energy = autograd.qmf_chain_energy(th, ph, ta, s["chain"])
        energy.backward()
        return {"energy": energy.detach(), "dtheta": th.grad, "dphi": ph.grad, "dtau": ta.grad}
    if kind == "iteration":
        iqcc.iqcc_store_load(ctx, s["h"].handle, s["x"], s["z"], s["c"])
        got = iqcc.iqcc_qcc_iteration(ctx, s["h"], s["spare"], theta, phi, s["w_max"], s["n_select"], EPS)
        return {"x": got["sel_x"].view(np.int64), "z": got["sel_z"].view(np.int64), "g": got["sel_g"],
                "tau": got["sel_tau"], "energy": got["energy"], "n_candidates": got["n_candidates"]}
    if kind == "batch":
        iqcc.iqcc_batch_launch(ctx, s["batch"].handle)
        e = s["energy"]
        for i, (st, (th, ph)) in enumerate(zip(s["outs"], s["angles"])):
            iqcc.iqcc_qmf_energy(ctx, st.handle, th, ph, e[i:i + 1])
        return e
    iqcc.iqcc_truncate_top(ctx, s["h"].handle, s["keep"], s["out"].handle)
    x, z, c = iqcc.iqcc_store_export(ctx, s["out"].handle)
    return {"x": x, "z": z, "c": c}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Keys and coefficients read once, results written once; one multiplication
    per qubit of a product state value (per support qubit of a screened pair),
    two per rotated coefficient.  Chains grow by about 1.4 a step and half of
    the terms anticommute with a generator."""
    kind, n, nq = case["kind"], case.get("n", 0), case.get("nq", 0)
    row = 16 * words(nq) + 8
    if kind == "energy":
        return {"bytes": n * row, "flops": n * (nq + 1)}
    if kind == "gradient":
        return {"bytes": n * (row + 8) + 16 * nq, "flops": n * 3 * nq}
    if kind == "dis":
        pairs = n * case["n_cand"]
        return {"bytes": n * row + 8 * case["n_cand"], "flops": pairs * (case["w_max"] / 2 + 2)}
    if kind == "limit":
        keep = int(case["keep"] * n)
        return {"bytes": 8 * n + keep * row * 3, "flops": 0}
    if kind == "batch":
        mean = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"]) if case["hi"] > case["lo"] else case["lo"]
        m = case["n_ham"] * mean
        return {"bytes": m * 24 * (1 + 1.4 + 1.4), "flops": m * (1 + 1.4 * 40)}
    steps = case.get("steps", case.get("n_select"))
    size = [n * 1.4 ** j for j in range(steps + 1)]
    if kind == "dress":
        b = sum((size[j] + size[j + 1]) * row for j in range(steps)) + size[-1] * row
        return {"bytes": b, "flops": sum(size[1:]) * nq + size[-1] * 3 * nq}
    if kind == "inplace":
        b = 2 * n * row + sum(size[j] * (row + 4) + (size[j + 1] - size[j]) * row for j in range(steps)) + size[-1] * row
        return {"bytes": b, "flops": sum(size[:-1]) * nq + size[-1] * 3 * nq}
    if kind == "train":
        fwd = sum((size[j] + size[j + 1]) * row + 8 * size[j] for j in range(steps))
        bwd = sum(size[j] * 24 + size[j + 1] * 8 for j in range(steps)) + size[-1] * 2 * row
        return {"bytes": fwd + bwd, "flops": sum(size) * 4 + size[-1] * 4 * nq}
    # iteration: load, screening of the flip sets' generators, n_select steps
    cand = min(n, nq * 40)
    b = 2 * n * row + sum((2 * size[j] + size[j + 1]) * row for j in range(steps)) + n * row
    return {"bytes": b, "flops": n * cand * 6 + sum(size) * nq}


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ---------------------------------------------------------------------------

def _factors(theta, phi):
    """(nq, 4): <I>, <X>, <Z>, <Y> of every qubit (bit 0 = x, bit 1 = z)."""
    one = torch.ones_like(theta)
    st, ct = torch.sin(theta), torch.cos(theta)
    return torch.stack([one, st * torch.cos(phi), ct, st * torch.sin(phi)], 1)


def _op(x, z, q):
    return ((x[q >> 6] >> (q & 63)) & 1) | (((z[q >> 6] >> (q & 63)) & 1) << 1)


def _expect(x, z, b):
    p = torch.ones(x.shape[1], dtype=torch.float64, device=DEV)
    for q in range(b.shape[0]):
        p *= b[q][_op(x, z, q)]
    return p


def _angle_gradient(x, z, c, theta, phi):
    nq, b = theta.numel(), _factors(theta, phi)
    st, ct, sp, cp = torch.sin(theta), torch.cos(theta), torch.sin(phi), torch.cos(phi)
    zero = torch.zeros_like(theta)
    bt, bp = torch.stack([zero, ct * cp, -st, ct * sp], 1), torch.stack([zero, -st * sp, zero, st * cp], 1)
    dt, dp = torch.zeros_like(theta), torch.zeros_like(theta)
    for i in range(0, x.shape[1], 1 << 18):
        xs, zs, cs = x[:, i:i + (1 << 18)], z[:, i:i + (1 << 18)], c[i:i + (1 << 18)]
        ops = [_op(xs, zs, q) for q in range(nq)]
        pre = [cs]
        for q in range(nq - 1):
            pre.append(pre[-1] * b[q][ops[q]])
        suf = torch.ones_like(cs)
        for q in range(nq - 1, -1, -1):
            v = pre[q] * suf
            dt[q] += (v * bt[q][ops[q]]).sum()
            dp[q] += (v * bp[q][ops[q]]).sum()
            suf = suf * b[q][ops[q]]
    return dt, dp


def _mod4(xa, za, xb, zb):
    """e of A B = i^e Q."""
    return (_count(xa & za) + _count(xb & zb) + 2 * _count(za & xb) - _count((xa ^ xb) & (za ^ zb))) & 3


def _dress(x, z, c, px, pz, tau, eps):
    """The dressed, merged and compressed terms; differentiable in c and tau."""
    px, pz = _column(px), _column(pz)
    anti = (_count((x & pz) ^ (z & px)) & 1).bool()
    xa, za, ca = x[:, anti], z[:, anti], c[anti]
    sign = torch.where(_mod4(px, pz, xa, za) == 3, 1.0, -1.0).double()
    cos, sin = (torch.cos(tau), torch.sin(tau)) if torch.is_tensor(tau) else (math.cos(tau), math.sin(tau))
    ax, az = torch.cat([x, xa ^ px], 1), torch.cat([z, za ^ pz], 1)
    v = torch.cat([torch.where(anti, c * cos, c), sign * (ca * sin)])
    h, at = torch.sort(_hash(ax, az))
    new = torch.ones_like(h, dtype=torch.bool)
    new[1:] = h[1:] != h[:-1]
    where = torch.cumsum(new, 0) - 1
    total = torch.zeros(int(new.sum()), dtype=torch.float64, device=DEV).index_add(0, where, v[at])
    keep = total.detach().abs() >= eps
    first = at[new][keep]
    return ax[:, first], az[:, first], total[keep]


def _dis(x, z, c, gx, gz, b):
    """g of every generator (host words): Im <Omega| H P |Omega>."""
    n, nq = x.shape[1], b.shape[0]
    pk, nzero = torch.ones(n, dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.int64, device=DEV)
    for q in range(nq):
        f = b[q][_op(x, z, q)]
        nzero += f == 0
        pk *= torch.where(f == 0, 1.0, f)
    pk *= c
    g = torch.zeros(len(gx), dtype=torch.float64, device=DEV)
    for a in range(len(gx)):
        px, pz = _column(gx[a]), _column(gz[a])
        v, left = pk, nzero
        for q in range(nq):
            p = ((int(gx[a][q >> 6]) >> (q & 63)) & 1) | (((int(gz[a][q >> 6]) >> (q & 63)) & 1) << 1)
            if p:
                k = _op(x, z, q)
                row = torch.stack([b[q][i ^ p] for i in range(4)])
                ratio = torch.where(b[q] == 0, row, row / torch.where(b[q] == 0, 1.0, b[q]))
                v = v * ratio[k]
                left = left - (b[q] == 0).long()[k]
        e = _mod4(x, z, px, pz)
        g[a] = torch.where((left == 0) & (e == 1), v, torch.where((left == 0) & (e == 3), -v, 0.0)).sum()
    return g


def _energy(x, z, c, theta, phi):
    return (c * _expect(x, z, _factors(theta, phi))).sum()


def _exact_iteration(case, x, z, c, theta, phi):
    """Every generator of every small flip set by |g|, then closed-form steps."""
    nq, b, W = case["nq"], _factors(theta, phi), words(case["nq"])
    if W > 1:
        return None
    w = _count(x)
    sets = torch.unique(x[0][(w >= 1) & (w <= case["w_max"])]).cpu().tolist()
    gx, gz = [], []
    for f in sets:
        for q in range(nq):
            if (f >> q) & 1:
                gx.append(f)
                gz.append(1 << q)
    if len(gx) * x.shape[1] > 1e9 or len(gx) > 20_000:
        return None
    gx, gz = np.array(gx, np.uint64).reshape(-1, 1), np.array(gz, np.uint64).reshape(-1, 1)
    g = _dis(x, z, c, gx, gz, b).cpu().numpy()
    take = np.argsort(-np.abs(g), kind="stable")[:case["n_select"]]
    energy, taus = [float(_energy(x, z, c, theta, phi))], []
    for a in take:
        px, pz = _column(gx[a]), _column(gz[a])
        anti = (_count((x & pz) ^ (z & px)) & 1).bool()
        eb = float((c * _expect(x, z, b))[anti].sum())
        ec = float(_dis(x, z, c, gx[a:a + 1], gz[a:a + 1], b)[0])
        taus.append(math.atan2(-ec, -eb))
        x, z, c = _dress(x, z, c, gx[a], gz[a], taus[-1], EPS)
        energy.append(float(_energy(x, z, c, theta, phi)))
    return {"x": gx[take].view(np.int64), "z": gz[take].view(np.int64), "g": g[take], "tau": np.array(taus),
            "energy": np.array(energy), "n_candidates": len(gx)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "limit":
        return None   # copies of the input's values
    if kind == "batch":
        e = [_energy(*_dress(x, z, c, px, pz, tau, EPS), th, ph)
             for _, x, z, c, px, pz, tau, th, ph in batch_inputs(case, seed)]
        return torch.stack(e)
    nq = case["nq"]
    x, z, c = hamiltonian(nq, case["n"], seed)
    theta, phi = qmf_angles(nq, seed, case.get("angles", "random"))
    if kind == "energy":
        return _energy(x, z, c, theta, phi)
    if kind == "gradient":
        dt, dp = _angle_gradient(x, z, c, theta, phi)
        return {"dtheta": dt, "dphi": dp, "lambda": None}
    if kind == "dis":
        gx, gz = generators(x, nq, case["n_cand"], case["w_max"], seed + 5)
        return _dis(x, z, c, gx, gz, _factors(theta, phi))
    if kind == "iteration":
        return _exact_iteration(case, x, z, c, theta, phi)
    gx, gz = generators(x, nq, case["steps"], 8, seed + 5)
    taus = amplitudes(len(gx), seed)
    if kind == "train":
        tau = torch.from_numpy(taus).to(DEV).requires_grad_(True)
        for j in range(len(gx)):
            x, z, c = _dress(x, z, c, gx[j], gz[j], tau[j], EPS)
        energy = _energy(x, z, c, theta, phi)
        energy.backward()
        dt, dp = _angle_gradient(x, z, c.detach(), theta, phi)
        return {"energy": energy.detach(), "dtheta": dt, "dphi": dp, "dtau": tau.grad}
    energies = []
    for j in range(len(gx)):
        x, z, c = _dress(x, z, c, gx[j], gz[j], float(taus[j]), EPS)
        energies.append(_energy(x, z, c, theta, phi))
    dt, dp = _angle_gradient(x, z, c, theta, phi)
    return {"energies": torch.stack(energies), "dtheta": dt, "dphi": dp}
