"""The work that a user of this framework has it do, as cases that can be timed.

Two kinds of pass, both through the public entry points of the package:

* ``simulate``: feature rows -> MPS batch -> kernel matrix, as a program does
  with new points (the batch itself has a gauge freedom, so what comes back
  is the kernel matrix of the states it holds and their bond dimensions);
* ``gram``: the kernel matrix of MPS batches that the program already holds:
  the symmetric training matrix, a test x train block, one inference row, or
  a fold of the training set gathered and packed anew.

Features are a two-class Gaussian mixture scaled to [0, 1]; the states of the
``gram`` cases are left-canonical MPS with a decaying Schmidt spectrum around
two class centres, so the matrix holds ones, mid-range values and zeros.
"""
import math

import numpy as np
import torch

import paper_2411_09336_amd as q

# bytes of one complex tensor entry in each operand form
FORM_BYTES = {"fp64": 16, "fp32": 8, "split_bf16": 16, "split_i8": 8}


def _sim(name, n, m, d, reps, chi, cutoff, coef_z=2.0, coef_xx=2.0, graph=False):
    return {"name": name, "kind": "simulate", "n": n, "m": m, "d": d, "reps": reps, "chi": chi, "cutoff": cutoff,
            "coef_z": coef_z, "coef_xx": coef_xx, "graph": graph}


def _gram(name, rows, cols, m, chi, form, fold=False):
    """cols = 0: the symmetric matrix of the rows."""
    return {"name": name, "kind": "gram", "rows": rows, "cols": cols, "m": m, "chi": chi, "form": form, "fold": fold}


def listed():
    return [
        # a few new points of a 20-feature problem (d = 1, chi 16): latency
        _sim("sim_20q_d1", 8, 20, 1, 2, 16, 1e-10),
        # the classification circuit (165 features, d = 1, gamma 0.1): a block
        # of the points of a support vector machine's training set
        _sim("sim_165q_d1", 512, 165, 1, 2, 64, 1e-8, 0.2, 0.01 * math.pi),
        # 50 qubits, d = 2, chi 32: an ordinary batch, as recorded graph replays
        _sim("sim_50q_d2", 128, 50, 2, 2, 32, 1e-10, graph=True),
        # 60 qubits, d = 3, chi 32: more points than a small batch, deeper circuit
        _sim("sim_60q_d3", 300, 60, 3, 2, 32, 1e-10),
        # the bandwidth of the full-scale circuit (d = 8, chi 64) on a short
        # chain: saturated bonds, SWAP networks, truncation at every gate
        _sim("sim_18q_d8", 16, 18, 8, 1, 64, 1e-8),
        # a bond cap of 128: bonds above 64 in the middle of the chain
        _sim("sim_16q_chi128", 4, 16, 5, 2, 128, 1e-10),
        # the full-scale states (165 qubits, chi 64): training matrix in FP64
        # and in the two split forms
        _gram("gram_165q_fp64", 64, 0, 165, 64, "fp64"),
        _gram("gram_165q_bf16", 128, 0, 165, 64, "split_bf16"),
        # test x train block at 100 qubits, odd sizes
        _gram("gram_100q_i8", 61, 301, 100, 64, "split_i8"),
        # a fold of the 50-qubit training set: gathered, packed, multiplied
        _gram("fold_50q_fp32", 160, 0, 50, 32, "fp32", fold=True),
        # one new point against a training set at bond 2 (d = 1 states)
        _gram("row_165q_d1", 1, 1000, 165, 2, "fp64"),
        # bonds up to 128: the widest kernels
        _gram("gram_40q_chi128", 24, 0, 40, 128, "fp64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        if rng.random() < 0.45:
            c = _sim(None, _log_int(rng, 1, 400), _log_int(rng, 5, 165), rng.choice([1, 1, 2, 2, 3, 4]),
                     rng.choice([1, 2]), rng.choice([8, 16, 32, 48, 64, 128]), rng.choice([1e-8, 1e-10]),
                     *rng.choice([(2.0, 2.0), (0.2, 0.01 * math.pi), (1.0, 0.8)]), graph=rng.random() < 0.3)
        else:
            form = rng.choice(["fp64", "fp64", "fp32", "split_bf16", "split_i8"])
            chi = rng.choice([2, 4, 13, 16, 32, 45, 64] + ([100, 128] if form in ("fp64", "fp32") else []))
            fold = rng.random() < 0.2
            c = _gram(None, _log_int(rng, 1, 300), 0 if fold else rng.choice([0, _log_int(rng, 1, 1000)]),
                      _log_int(rng, 6, 165), chi, form, fold)
        del c["name"]
        if _seconds(c) < 0.7:
            return c


# ---------------------------------------------------------------- inputs

def _features(case, seed):
    """Balanced two-class mixture, min-max scaled per feature (seeded)."""
    rng = np.random.default_rng(seed)
    n, m = case["n"], case["m"]
    u = rng.standard_normal(m)
    mu = 0.5 * u / np.linalg.norm(u)
    lab = np.where(np.arange(n) < n // 2, 1.0, -1.0)
    # scaled over a population larger than the block, as a program scales by
    # its training set
    x = rng.standard_normal((max(n, 64), m))
    x[:n] += lab[:, None] * mu
    lo, hi = x.min(axis=0), x.max(axis=0)
    return np.ascontiguousarray(((x - lo) / (hi - lo))[:n])


def _bonds(m, chi):
    return [min(chi, 2 ** min(l, m - l, 30)) for l in range(m + 1)]


def _distinct(case):
    """Distinct states made for a matrix; the rest are copies at their own
    addresses (the work depends on the bond profile alone)."""
    return max(2, min(case["rows"] + case["cols"], 40 * 64 * 50 // (case["m"] * min(case["chi"], 128)), 24))


def _states(case, seed, device):
    """Left-canonical states as one (k, D_l, 2, D_{l+1}) tensor per site, on
    the device: every site's columns orthonormalised by Cholesky, twice."""
    m, k = case["m"], _distinct(case)
    dims = _bonds(m, case["chi"])
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    eps = 0.5 / math.sqrt(m)
    out = []
    for l in range(m):
        dl, dr = dims[l], dims[l + 1]
        shape = (dl * 2, dr)
        g = torch.view_as_complex(torch.randn((2,) + shape + (2,), generator=gen, device=device, dtype=torch.float64))
        e = torch.view_as_complex(torch.randn((k,) + shape + (2,), generator=gen, device=device, dtype=torch.float64))
        x = g[torch.arange(k, device=device) % 2] + eps * e
        # rows of decreasing weight: the Schmidt values fall by 1e-4 over a bond
        w = torch.exp(torch.linspace(0.0, -9.0 if dl > 2 else 0.0, dl, device=device, dtype=torch.float64))
        x = x * w.repeat_interleave(2)[:, None]
        x = x / x.abs().pow(2).sum(dim=1, keepdim=True).sqrt()
        for _ in range(3):
            xh = x.mH.resolve_conj().contiguous()
            c = torch.linalg.cholesky(xh @ x)
            x = torch.linalg.solve_triangular(c, xh, upper=False).mH.resolve_conj().contiguous()
        out.append(x.reshape(k, dl, 2, dr))
    return out


def _layout(case):
    """Which state each row and column of the matrix is."""
    k = _distinct(case)
    rows = [(3 * i + i // k) % k for i in range(case["rows"])]
    cols = rows if case["cols"] == 0 else [(i + i // k) % k for i in range(case["cols"])]
    return rows, cols


def prepare(case, seed):
    if case["kind"] == "simulate":
        spec = q.CircuitSpec(case["m"], case["d"], case["reps"], case["coef_z"], case["coef_xx"])
        return {"case": case, "x": torch.tensor(_features(case, seed), device="cuda"), "spec": spec}
    sites = [s.cpu().numpy() for s in _states(case, seed, "cuda")]
    base = q.import_batch([[s[i] for s in sites] for i in range(sites[0].shape[0])])
    rows, cols = _layout(case)
    if case["fold"]:
        # the fold is gathered out of the stored batch in the pass itself
        return {"case": case, "base": base, "fold": np.array(rows, dtype=np.int64)}
    form = case["form"]
    base.pack(form)
    a = base.gather(rows, (form,))
    b = None if case["cols"] == 0 else base.gather(cols, (form,))
    return {"case": case, "a": a, "b": b}


def run(state):
    case = state["case"]
    if case["kind"] == "simulate":
        batch = q.simulate(state["x"], state["spec"], case["chi"], case["cutoff"],
                           graph_circuits=0 if case["graph"] else None)
        return {"K": q.gram(batch), "bonds": batch.bond_dims()}
    if case["fold"]:
        return q.gram(state["base"].gather(state["fold"]), precision=case["form"])
    return q.gram(state["a"], state["b"], precision=case["form"])


# ---------------------------------------------------------------- work

def _gates(m, d, reps):
    """The circuit: per repetition Rz on every qubit, then for each qubit i
    the Rxx with i + 1 .. i + d, reached by SWAPs and carried back."""
    out = []
    for _ in range(reps):
        out += [("z", i, i, -1) for i in range(m)]
        for i in range(m - 1):
            for k in range(1, min(d, m - 1 - i) + 1):
                out += [("s", p, -1, -1) for p in range(i, i + k - 1)]
                out.append(("x", i + k - 1, i, i + k))
                out += [("s", p, -1, -1) for p in range(i + k - 2, i - 1, -1)]
    return out


def _sim_bonds(case):
    """Bond bound of the circuit's states: doubled by every Rxx over a cut."""
    m, d = case["m"], case["d"]
    cap = min(case["chi"], 2 ** min(30, case["reps"] * d * (d + 1) // 2))
    return _bonds(m, cap)


def _two_qubit_bonds(case):
    """The larger outer bond at every two-qubit gate."""
    dims = _sim_bonds(case)
    return [max(dims[g[1]], dims[g[1] + 2]) for g in _gates(case["m"], case["d"], case["reps"]) if g[0] != "z"]


def _exact_seconds(case):
    """Rough time of the numpy simulation of one point."""
    return sum(6e-5 + 9e-4 * (b / 64.0) ** 3 for b in _two_qubit_bonds(case))


def _seconds(case):
    """Rough time of one pass, to keep drawn cases below the largest listed."""
    m = case["m"]
    if case["kind"] == "simulate":
        sim = sum(4.5e-2 if b > 64 else 1.5e-4 + 2.0e-3 * (b / 64.0) ** 2 for b in _two_qubit_bonds(case))
        sim *= 1 + case["n"] // 257
        return sim + case["n"] ** 2 / 2 * m / 165 / 3.4e4
    rate = 4e3 if case["chi"] > 64 else {"fp64": 3.4e4, "fp32": 6e4, "split_bf16": 9e4, "split_i8": 17e4}[case["form"]]
    return case["rows"] * (case["cols"] or case["rows"] / 2) * m / 165 / rate


def work(case):
    if case["kind"] == "simulate":
        dims, n, m = _sim_bonds(case), case["n"], case["m"]
        tensors = sum(2 * dims[l] * dims[l + 1] for l in range(m))
        flops = 0.0
        for g in _gates(m, case["d"], case["reps"]):
            if g[0] == "z":
                continue
            a, c, b = dims[g[1]], dims[g[1] + 1], dims[g[1] + 2]
            s = 2 * min(a, b)
            # two-site product, its singular values and vectors, projection
            flops += 8.0 * (4 * a * b * c + 4.0 * a * b * s * 4 + 4 * a * b * c)
        entry = 16.0 * sum(2 * dims[l] * dims[l + 1] * dims[l + 1] for l in range(m))
        return {"bytes": n * m * 8 + 16 * n * tensors + 8 * n * n, "flops": n * flops + n * (n + 1) / 2 * entry}
    dims, m, rows = _bonds(case["m"], case["chi"]), case["m"], case["rows"]
    cols = case["cols"] or rows
    entries = rows * (rows + 1) / 2 if case["cols"] == 0 else rows * cols
    states = rows + case["cols"]
    entry = sum(16.0 * dims[l] * dims[l + 1] * (dims[l] + dims[l + 1]) for l in range(m))
    tensors = sum(2 * dims[l] * dims[l + 1] for l in range(m))
    size = FORM_BYTES[case["form"]] + (16 if case["fold"] else 0)
    return {"bytes": states * tensors * size + 8 * rows * cols, "flops": entries * entry}


# ---------------------------------------------------------------- in 64 bits

def _exact_state(x, case):
    """Truncated MPS simulation of one point in numpy (complex128)."""
    m, chi, cutoff = case["m"], case["chi"], case["cutoff"]
    A = [np.full((1, 2, 1), math.sqrt(0.5), dtype=np.complex128) for _ in range(m)]
    gates = _gates(m, case["d"], case["reps"])
    two = [g for g in gates if g[0] != "z"]
    centre, done = 0, 0

    def right(l):
        dl, _, dr = A[l].shape
        u, r = np.linalg.qr(A[l].reshape(dl * 2, dr))
        A[l] = u.reshape(dl, 2, -1)
        A[l + 1] = np.tensordot(r, A[l + 1], axes=(1, 0))

    def left(l):
        dl, _, dr = A[l].shape
        u, r = np.linalg.qr(A[l].reshape(dl, 2 * dr).conj().T)
        A[l] = u.conj().T.reshape(-1, 2, dr)
        A[l - 1] = np.tensordot(A[l - 1], r.conj().T, axes=(2, 0))

    for op, p, i, j in gates:
        if op == "z":
            h = 0.5 * case["coef_z"] * x[i]
            A[p] = A[p] * np.exp(np.array([-1j * h, 1j * h]))[None, :, None]
            continue
        while centre < p:
            right(centre)
            centre += 1
        while centre > p + 1:
            left(centre)
            centre -= 1
        t = np.tensordot(A[p], A[p + 1], axes=(2, 0))
        if op == "s":
            t = t.transpose(0, 2, 1, 3)
        else:
            h = 0.5 * case["coef_xx"] * (1.0 - x[i]) * (1.0 - x[j])
            t = math.cos(h) * t - 1j * math.sin(h) * t[:, ::-1, ::-1, :]
        a, b = t.shape[0], t.shape[3]
        u, s, v = np.linalg.svd(t.reshape(2 * a, 2 * b), full_matrices=False)
        w = s * s
        tail = np.concatenate([np.cumsum(w[::-1])[::-1], [0.0]])
        k = max(1, min(chi, int(np.argmax(tail <= cutoff * w.sum()))))
        s = s[:k] / math.sqrt(w[:k].sum())
        done += 1
        nxt = two[done][1] if done < len(two) else None
        if nxt is None or nxt > p:
            A[p], A[p + 1] = u[:, :k].reshape(a, 2, k), (s[:, None] * v[:k]).reshape(k, 2, b)
            centre = p + 1
        else:
            A[p], A[p + 1] = (u[:, :k] * s).reshape(a, 2, k), v[:k].reshape(k, 2, b)
            centre = p
    while centre < m - 1:
        right(centre)
        centre += 1
    A[-1] = A[-1] / np.linalg.norm(A[-1])
    return A


def _matrix(sites):
    """|<i|j>|^2 of k states given as one (k, D_l, 2, D_{l+1}) tensor per
    site: row i against every state at once."""
    k = sites[0].shape[0]
    K = np.zeros((k, k))
    for i in range(k):
        e = torch.ones((k, 1, 1), dtype=torch.complex128, device=sites[0].device)
        for s in sites:
            _, dl, _, dr = s.shape
            t = torch.bmm(e, s.reshape(k, dl, 2 * dr)).reshape(k, 2 * dl, dr)
            e = torch.matmul(s[i].reshape(2 * dl, dr).mH.resolve_conj().contiguous(), t)
        K[i] = e[:, 0, 0].abs().pow(2).cpu().numpy()
    return K


def exact(case, seed):
    if case["kind"] == "simulate":
        if case["n"] * _exact_seconds(case) > 14.0:
            return None
        states = [_exact_state(x, case) for x in _features(case, seed)]
        sites = []
        for l in range(case["m"]):
            dl, dr = (max(s[l].shape[ax] for s in states) for ax in (0, 2))
            t = np.zeros((len(states), dl, 2, dr), dtype=np.complex128)
            for i, s in enumerate(states):
                t[i, : s[l].shape[0], :, : s[l].shape[2]] = s[l]
            sites.append(torch.from_numpy(t).cuda())
        return {"K": _matrix(sites), "bonds": None}
    rows, cols = _layout(case)
    return _matrix(_states(case, seed, "cuda"))[np.ix_(rows, cols)]
