"""Workloads for timing the library: what a user of POLFED has it do, through
the public entry points of ``paper_2005_09534_amd.polfed``.

A case is a dict of plain values; its ``kind`` names the call:

* ``filter``   -- ``apply_filter``: Y = P^K_sigma(H~) X, the bulk of every solve;
* ``apply_h``  -- ``apply_h``: Y = H X (Rayleigh-Ritz, residuals);
* ``project``  -- ``gram`` and ``update``: one Gram-Schmidt pass of a block
  against the Lanczos basis, C = Q^T U, U <- U - Q C;
* ``moments``  -- ``dos_moments``: Chebyshev moments for the density of states;
* ``entropy``  -- ``entanglement``: S_E of eigenvectors for every half-ring cut;
* ``solve``    -- ``solve``: the N_ev eigenpairs nearest the target, one chain;
* ``batch``    -- ``solve_batch``: the eigenvalues of many disorder realisations.

The chains are the paper's: J1 = 1, fields uniform on [-W, W], periodic, with
(J1-J2) or without (XXZ) second-neighbour bonds.  Vectors are standard normal
columns scaled to unit length, as the blocks of a Lanczos basis are.
"""

import math

import numpy as np
import torch

from paper_2005_09534_amd import polfed as pf

_HANDLE = []


def _handle():
    """The program's one library context."""
    if not _HANDLE:
        _HANDLE.append(pf.Context(0))
    return _HANDLE[0]


def listed():
    return [
        # the filter of the smallest workload (L = 12, 20 eigenpairs): 924
        # rows, where a step costs its launch
        dict(name="filter_L12_s4_fp64", kind="filter", L=12, J2=0.0, Delta=1.0, W=3.0, nvec=4,
             precision="fp64", K=200),
        # one realisation of a disorder average, FP32 filter
        dict(name="filter_L16_s8_fp32", kind="filter", L=16, J2=0.0, Delta=1.0, W=2.0, nvec=8,
             precision="fp32", K=1201),
        # the J1-J2 chain of medium length, all FP64
        dict(name="filter_L18_j1j2_s16_fp64", kind="filter", L=18, J2=1.0, Delta=1.0, W=2.0,
             nvec=16, precision="fp64", K=501),
        # the FP32 filter where a block no longer fits the caches twice
        dict(name="filter_L22_s32_fp32", kind="filter", L=22, J2=0.0, Delta=1.0, W=5.0, nvec=32,
             precision="fp32", K=200),
        # the longest chain, a full block of 64 columns in FP64
        dict(name="filter_L26_s64_fp64", kind="filter", L=26, J2=0.0, Delta=1.0, W=4.0, nvec=64,
             precision="fp64", K=11),
        # H applied to the columns of a Rayleigh-Ritz block
        dict(name="apply_h_L22_s64_fp64", kind="apply_h", L=22, J2=1.0, Delta=0.55, W=4.0, nvec=64,
             precision="fp64"),
        # reorthogonalisation early in a short chain's run, and late in a long one's
        dict(name="project_L14_p104_q8", kind="project", L=14, p=104, q=8),
        dict(name="project_L22_p480_q32", kind="project", L=22, p=480, q=32),
        # the density of states that sizes a filter
        dict(name="moments_L20", kind="moments", L=20, J2=1.0, Delta=0.55, W=4.0, nmom=256, nvec=4),
        # entropies of one solve's eigenvectors
        dict(name="entropy_L16", kind="entropy", L=16, nvec=20),
        # a whole solve of the smallest workload
        dict(name="solve_L12", kind="solve", L=12, J2=0.0, Delta=1.0, W=3.0, nev=20, block=4, K=200),
        # a disorder average over chains of uneven length, away from the middle
        dict(name="batch_L14_16_18", kind="batch", lengths="14,16,18", R=12, J2=0.0, Delta=1.0,
             W=3.0, nev=20, target=0.2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["filter", "filter", "filter", "filter", "apply_h", "project", "project",
                       "moments", "entropy", "solve", "batch"])
    J2 = rng.choice([0.0, 1.0])
    model = dict(J2=J2, Delta=rng.choice([1.0, 0.55]), W=round(rng.uniform(0.5, 8.0), 2))
    if kind == "filter":
        L = rng.choice([10, 12, 14, 16, 18, 20, 22, 24])
        nvec = rng.choice([1, 2, 4, 8, 16, 32, 64])
        # about as much work per pass at every length, longer orders on short chains
        most = max(4, min(4000, int(2.0e10 / (pf.dim(L) * nvec * (1 + J2)))))
        return dict(kind=kind, L=L, nvec=nvec, precision=rng.choice(["fp64", "fp32"]),
                    K=_log_int(rng, max(3, most // 20), most), **model)
    if kind == "apply_h":
        L = rng.choice([12, 14, 16, 18, 20, 22, 24])
        return dict(kind=kind, L=L, nvec=rng.choice([1, 4, 8, 32, 64]),
                    precision=rng.choice(["fp64", "fp32"]), **model)
    if kind == "project":
        L = rng.choice([12, 14, 16, 18, 20, 22])
        q = rng.choice([1, 4, 8, 16, 32, 64])
        p = _log_int(rng, q, max(q, min(1000, pf.dim(L) // 6)))
        return dict(kind=kind, L=L, p=p, q=q)
    if kind == "moments":
        return dict(kind=kind, L=rng.choice([12, 14, 16, 18, 20, 22]), nmom=_log_int(rng, 31, 512),
                    nvec=rng.choice([1, 3, 4, 10]), **model)
    if kind == "entropy":
        return dict(kind=kind, L=rng.choice([10, 12, 14, 16]), nvec=_log_int(rng, 1, 60))
    if kind == "solve":
        return dict(kind=kind, L=rng.choice([10, 12]), nev=rng.choice([5, 10, 20]),
                    block=rng.choice([2, 4, 8]), K=0, **model)
    return dict(kind=kind, lengths=rng.choice(["12", "12,14", "14,16", "16", "14,16,18"]),
                R=rng.choice([3, 5, 8, 12]), nev=rng.choice([10, 20]),
                target=round(rng.uniform(0.2, 0.3), 3), **model)


# ------------------------------------------------------------- inputs --


def _fields(case, seed, L=None):
    return np.random.default_rng([seed, 11]).uniform(-case["W"], case["W"], L or case["L"])


def _columns(n, s, seed, dtype=torch.float64):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    X = torch.randn((n, s), generator=g, device="cuda", dtype=torch.float64)
    X /= math.sqrt(n)
    return X.to(dtype)


def _enclosure(case, h):
    """A bound on |E| for every eigenvalue: row sums of |H|, field by field."""
    J = 1.0 + abs(case["J2"])
    return J * case["L"] * (0.25 * abs(case["Delta"]) + 0.25) + 0.5 * float(np.abs(h).sum())


def _sigma(seed):
    """A target near the middle of the spectrum, in rescaled units."""
    return float(np.random.default_rng([seed, 12]).uniform(-0.06, 0.06))


def _members(case, seed):
    lengths = [int(x) for x in case["lengths"].split(",")]
    rng = np.random.default_rng([seed, 13])
    return [(L, rng.uniform(-case["W"], case["W"], L))
            for L in (lengths[r % len(lengths)] for r in range(case["R"]))]


def _dtype(case):
    return torch.float64 if case["precision"] == "fp64" else torch.float32


def prepare(case, seed):
    kind = case["kind"]
    state = dict(case=case, ctx=_handle())
    if kind in ("filter", "apply_h", "moments", "solve"):
        h = _fields(case, seed)
        state["model"] = pf.make_model(case["L"], 1.0, case["J2"], case["Delta"], h)
    if kind in ("filter", "apply_h"):
        state["X"] = _columns(pf.dim(case["L"]), case["nvec"], seed, _dtype(case))
    if kind == "moments":
        state["X"] = torch.sign(_columns(pf.dim(case["L"]), case["nvec"], seed))
    if kind in ("filter", "moments"):
        state["E"] = _enclosure(case, h)
    if kind == "filter":
        state["sigma"] = _sigma(seed)
    if kind == "project":
        n = pf.dim(case["L"])
        state["Q"] = _columns(n, case["p"], seed)
        state["U"] = _columns(n, case["q"], seed + (1 << 20))
    if kind == "entropy":
        V = _columns(pf.dim(case["L"]), case["nvec"], seed)
        state["V"] = V / V.norm(dim=0)
    if kind == "batch":
        state["models"] = [pf.make_model(L, 1.0, case["J2"], case["Delta"], h)
                           for L, h in _members(case, seed)]
    return state


# --------------------------------------------------------------- passes --


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "filter":
        return ctx.apply_filter(state["model"], -state["E"], state["E"], state["sigma"],
                                case["K"], state["X"])
    if kind == "apply_h":
        return ctx.apply_h(state["model"], state["X"])
    if kind == "project":
        C = ctx.gram(state["Q"], state["U"])
        ctx.update(state["Q"], C, state["U"], alpha=-1.0, beta=1.0)
        return C, state["U"]
    if kind == "moments":
        return ctx.dos_moments(state["model"], -state["E"], state["E"], case["nmom"], R=state["X"])
    if kind == "entropy":
        return ctx.entanglement(case["L"], state["V"])
    if kind == "solve":
        # (the residual norms, rounding noise by design, are not a result of their own)
        r = ctx.solve(state["model"], case["nev"], block_size=case["block"], K=case["K"])
        return dict(E=r["E"], V=r["V"], status=r["status"])
    r = ctx.solve_batch(state["models"], case["nev"], precision=1, target=case["target"])
    return dict(E=r["E"], status=np.array(r["status"]))


# ----------------------------------------------------------------- work --


def _hv_flops(L, J2, s):
    """One H~ application to s columns: on average L/2 (1 + 1/(L-1)) antiparallel
    pairs a row and bond range, a multiply and an add each, and the diagonal."""
    return pf.dim(L) * s * 2.0 * ((0.5 * L * L / (L - 1.0)) * (2 if J2 else 1) + 1)


def _filter_work(L, J2, s, b, K):
    n = pf.dim(L)
    block = float(n) * s * b
    # within the 256 MB Infinity Cache the recurrence need not leave the chip;
    # beyond it each step reads b_{k+1}, b_{k+2} and X and writes b_k
    moved = 2 * block if 2 * block <= 256e6 else (K + 1) * 4 * block
    return moved + 12.0 * n, (K + 1) * (_hv_flops(L, J2, s) + 4.0 * n * s)


def _order(L, J2, nwin):
    """Roughly the filter order whose main lobe holds nwin states mid-spectrum."""
    return max(8, int(1.2 * pf.dim(L) / nwin))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        lengths = [int(x) for x in case["lengths"].split(",")]
        nbytes = flops = 0.0
        for r in range(case["R"]):
            L = lengths[r % len(lengths)]
            n, cols = pf.dim(L), 6 * case["nev"]
            _, f = _filter_work(L, case["J2"], cols, 4, _order(L, case["J2"], 1.5 * case["nev"]) // 2)
            nbytes += 8.0 * n * cols
            flops += f + 4.0 * n * cols * cols
        return dict(bytes=nbytes, flops=flops)
    n = pf.dim(case["L"])
    if kind == "filter":
        nbytes, flops = _filter_work(case["L"], case["J2"], case["nvec"],
                                     8 if case["precision"] == "fp64" else 4, case["K"])
    elif kind == "apply_h":
        b = 8 if case["precision"] == "fp64" else 4
        nbytes, flops = 2.0 * n * case["nvec"] * b + 12.0 * n, _hv_flops(case["L"], case["J2"], case["nvec"])
    elif kind == "project":
        p, q = case["p"], case["q"]
        # Q once for both products only where it stays on the chip in between
        passes = 1 if 8.0 * n * p <= 256e6 else 2
        nbytes, flops = 8.0 * n * (passes * p + 2 * q), 4.0 * n * p * q
    elif kind == "moments":
        nbytes, flops = _filter_work(case["L"], case["J2"], case["nvec"], 8, case["nmom"] // 2)
    elif kind == "entropy":
        h = case["L"] // 2
        pairs = case["nvec"] * h
        nbytes = 8.0 * n * case["nvec"]
        flops = pairs * sum((2.0 + 4.0 / 3.0) * math.comb(h, k) ** 3 for k in range(h + 1))
    else:
        K = case["K"] or _order(case["L"], case["J2"], 1.5 * case["nev"])
        cols = 6 * case["nev"]
        _, f = _filter_work(case["L"], case["J2"], cols, 8, K)
        nbytes, flops = 8.0 * n * (cols + case["nev"]), f + 4.0 * n * cols * cols
    return dict(bytes=nbytes, flops=flops)


# ---------------------------------------------------------------- exact --


def _chain(L, J2, Delta, h):
    """H of one chain in plain torch, FP64: its diagonal, and for every bond
    (weight, row of the state with the pair swapped, 1 where antiparallel)."""
    s = torch.arange(1 << L, device="cuda", dtype=torch.int32)
    pop = torch.zeros_like(s)
    for i in range(L):
        pop += (s >> i) & 1
    s = s[pop == L // 2]
    row = torch.full((1 << L,), -1, device="cuda", dtype=torch.int32)
    row[s.long()] = torch.arange(s.numel(), device="cuda", dtype=torch.int32)
    del pop
    d = torch.zeros(s.numel(), device="cuda", dtype=torch.float64)
    for i in range(L):
        d += float(h[i]) * (((s >> i) & 1).double() - 0.5)
    bonds = []
    for l, J in ((1, 1.0), (2, J2)):
        if J == 0.0:
            continue
        for i in range(L):
            j = (i + l) % L
            anti = ((s >> i) ^ (s >> j)) & 1
            d += 0.25 * J * Delta * (1.0 - 2.0 * anti.double())
            swapped = torch.where(anti.bool(), s ^ ((1 << i) | (1 << j)), s)
            bonds.append((0.5 * J, row[swapped.long()], anti.double()))
    return d, bonds


def _times(op, V, a=1.0, b=0.0):
    d, bonds = op
    Y = (a * d + b)[:, None] * V
    for w, idx, anti in bonds:
        Y.addcmul_(V[idx.long()], (a * w * anti)[:, None])
    return Y


def _dense(L, J2, Delta, h):
    """Eigenvalues and vectors of H from a dense matrix."""
    d, bonds = _chain(L, J2, Delta, h)
    n = d.numel()
    H = torch.diag(d)
    r = torch.arange(n, device="cuda")
    for w, idx, anti in bonds:
        H.index_put_((r, idx.long()), w * anti, accumulate=True)
    w, V = np.linalg.eigh(H.cpu().numpy())
    return w, V


def _nearest(w, sigma, nev):
    return np.sort(np.argsort(np.abs(w - sigma), kind="stable")[:nev])


def exact(case, seed):
    kind = case["kind"]
    if kind == "filter":
        h = _fields(case, seed)
        op, E, sigma, K = _chain(case["L"], case["J2"], case["Delta"], h), _enclosure(case, h), _sigma(seed), case["K"]
        if K * len(op[1]) > 120000 or (pf.dim(case["L"]) > 2e6 and K * case["nvec"] > 2000):
            return None
        k = np.arange(K + 1)
        c = np.sqrt(4.0 - 3.0 * (k == 0)) * np.cos(k * math.acos(sigma))
        D = float(np.sum(c * np.cos(k * math.acos(sigma))))
        t0 = _columns(pf.dim(case["L"]), case["nvec"], seed, _dtype(case)).double()
        Y = t0 * (c[0] / D)
        t1 = _times(op, t0, 1.0 / E)
        for j in range(1, K + 1):
            Y.add_(t1, alpha=float(c[j] / D))
            if j < K:
                t2 = _times(op, t1, 1.0 / E).mul_(2.0).sub_(t0)
                t0, t1 = t1, t2
        return Y
    if kind == "apply_h":
        op = _chain(case["L"], case["J2"], case["Delta"], _fields(case, seed))
        return _times(op, _columns(pf.dim(case["L"]), case["nvec"], seed, _dtype(case)).double())
    if kind == "project":
        n = pf.dim(case["L"])
        Q, U = _columns(n, case["p"], seed), _columns(n, case["q"], seed + (1 << 20))
        C = Q.T.contiguous() @ U
        return C, U - Q @ C
    if kind == "moments":
        h = _fields(case, seed)
        op, E = _chain(case["L"], case["J2"], case["Delta"], h), _enclosure(case, h)
        t0 = torch.sign(_columns(pf.dim(case["L"]), case["nvec"], seed))
        r, norm, mu = t0, float((t0 * t0).sum()), []
        t1 = _times(op, t0, 1.0 / E)
        for j in range(case["nmom"]):
            mu.append(float((r * t0).sum()) / norm)
            t0, t1 = t1, _times(op, t1, 1.0 / E).mul_(2.0).sub_(t0)
        return np.array(mu)
    if kind == "entropy":
        L, hL = case["L"], case["L"] // 2
        V = prepare(case, seed)["V"].cpu().numpy()
        s = np.arange(1 << L)
        s = s[np.array([bin(x).count("1") for x in s]) == hL]
        S = np.zeros((case["nvec"], hL))
        for x in range(hL):
            t = ((s >> x) | (s << (L - x))) & ((1 << L) - 1)
            psi = np.zeros((case["nvec"], 1 << hL, 1 << hL))
            psi[:, t >> hL, t & ((1 << hL) - 1)] = V.T
            lam = np.linalg.svd(psi, compute_uv=False) ** 2
            S[:, x] = -np.sum(np.where(lam > 1e-300, lam * np.log(np.maximum(lam, 1e-300)), 0.0), axis=1)
        return S
    if kind == "solve":
        w, V = _dense(case["L"], case["J2"], case["Delta"], _fields(case, seed))
        at = _nearest(w, 0.5 * (w[0] + w[-1]), case["nev"])
        V = V[:, at]
        V = V * np.sign(V[np.argmax(np.abs(V), axis=0), np.arange(len(at))])
        return dict(E=w[at], V=V, status=None)
    E = np.empty((case["R"], case["nev"]))
    for r, (L, h) in enumerate(_members(case, seed)):
        if L > 12:
            return None
        w, _ = _dense(L, case["J2"], case["Delta"], h)
        E[r] = w[_nearest(w, w[0] + case["target"] * (w[-1] - w[0]), case["nev"])]
    return dict(E=E, status=None)
