"""Gram kernels by bond dimension: four pairs per wave at bonds up to 4
(FP64), one pair per wave at bonds up to 16 and 32, one pair per workgroup
above (E in LDS up to bond 64, in global scratch beyond, with 16-row blocks
that the bonds fill or not).  Bonds at the edges of each, ragged blocks,
single rows, fewer rows than a pair tile, and jobs of several kernels in one
call, against the oracle's overlaps of the same left-canonical states.

Tolerances: FP64 1e-12 (rounding of 15 sites of at most 127 x 127 products,
~1e-14, with a wide margin); FP32 1e-5 (15 sites x 2 products x sqrt(2 x 127)
roundings of 6e-8 at most 3e-5 one way, random signs sqrt(30 x 254) x 6e-8 =
5e-6 on K <= 1).
"""
import numpy as np
import pytest

from oracle import gram as ogram
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}
# split forms: 31-bit codes of two operands at 2 x 13 products, 2^-31 each way
# on |<a|b>|, twice that on K: 4 x 26 x 2^-31 = 4.8e-8
SPLIT_TOL = {"split_bf16": 5e-8, "split_i8": 5e-8}


def random_mps(rng, m, bond, near=None, eps=0.05):
    """Left-canonical MPS with bonds min(bond, 2^l, 2^(m-l)); close to
    `near` when given, so that off-diagonal entries are not all zero."""
    out = []
    for l in range(m):
        dl, dr = (min(bond, 2 ** min(x, m - x)) for x in (l, l + 1))
        z = rng.standard_normal((2 * dl, dr)) + 1j * rng.standard_normal((2 * dl, dr))
        if near is not None:
            z = near[l].reshape(2 * dl, dr) + eps * z / np.sqrt(2 * dl)
        u, r = np.linalg.qr(z)
        u = u * (np.diag(r) / np.abs(np.diag(r)))[None, :]
        out.append(u.reshape(dl, 2, dr))
    return out


@pytest.mark.parametrize("bond", [1, 2, 3, 4, 5, 8, 16, 17, 31, 32, 33, 47, 48, 49, 64, 65, 81, 100, 127])
def test_bonds_vs_oracle(bond):
    import paper_2411_09336_amd as q
    require_gpu()
    rng = np.random.default_rng(bond)
    m = 13 if bond <= 64 else 15
    base = random_mps(rng, m, bond)
    mps = [random_mps(rng, m, bond, base) for _ in range(11)]
    K_ref = np.array([[abs(ogram.overlap(a, b)) ** 2 for b in mps] for a in mps])
    b = q.import_batch(mps)
    for prec, tol in TOL.items():
        K = q.gram(b, precision=prec).cpu().numpy()
        print(bond, prec, "max|dK|", np.abs(K - K_ref).max(), "off-diagonal", K_ref[0, 1])
        assert np.abs(K - K_ref).max() < tol
        # a single row, and ragged blocks around the four-pair units
        for a0, na, b0, nb in ((3, 1, 0, 11), (0, 11, 10, 1), (2, 5, 3, 7), (9, 2, 1, 3)):
            Kb = q.gram_block(b, a0, na, b, b0, nb, precision=prec).cpu().numpy()
            assert np.abs(Kb - K_ref[a0:a0 + na, b0:b0 + nb]).max() < tol


@pytest.mark.parametrize("bond", [1, 2, 5, 15, 16, 17, 31, 32])
def test_split_bonds(bond):
    """The split forms at one pair per wave: against the oracle, and the bits
    of the workgroup kernel, which takes the same states when a state of bond
    40 stands beside them in the batch (so does FP32)."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    rng = np.random.default_rng(1000 + bond)
    m, n = 13, 9
    base = random_mps(rng, m, bond)
    mps = [random_mps(rng, m, bond, base) for _ in range(n)]
    K_ref = np.array([[abs(ogram.overlap(a, c)) ** 2 for c in mps] for a in mps])
    small = q.import_batch(mps)
    mixed = q.import_batch(mps + [random_mps(rng, m, 40)])
    for prec in ("split_bf16", "split_i8", "fp32"):
        K = q.gram(small, precision=prec)
        assert torch.equal(K, q.gram(mixed, precision=prec)[:n, :n])
        row = q.gram_block(small, 2, 1, small, 2, 7, precision=prec)
        assert torch.equal(K[2:3, 2:], row)
        err = np.abs(K.cpu().numpy() - K_ref).max()
        print(bond, prec, "max|dK|", err)
        assert err < SPLIT_TOL.get(prec, 1e-5)


@pytest.mark.parametrize("n,m", [(1, 1), (2, 2), (3, 3), (5, 6), (37, 9)])
def test_sites_and_sizes(n, m):
    """Chains shorter than the sites loaded ahead, and triangles that end
    inside a tile."""
    import paper_2411_09336_amd as q
    require_gpu()
    rng = np.random.default_rng(100 * n + m)
    for bond in (2, 4, 12):
        base = random_mps(rng, m, bond)
        mps = [random_mps(rng, m, bond, base) for _ in range(n)]
        K_ref = np.array([[abs(ogram.overlap(a, c)) ** 2 for c in mps] for a in mps])
        b = q.import_batch(mps)
        for prec, tol in {**TOL, **SPLIT_TOL}.items():
            assert np.abs(q.gram(b, precision=prec).cpu().numpy() - K_ref).max() < tol


def test_scaled_states():
    """Unnormalised states (every site scaled by 1e-3 or 1e3): the rescaling
    by powers of two of each pair keeps FP64 and FP32 in range."""
    import paper_2411_09336_amd as q
    require_gpu()
    rng = np.random.default_rng(5)
    for bond in (4, 16, 32):
        mps = [random_mps(rng, 13, bond) for _ in range(3)]
        scaled = [[t * f for t in a] for a, f in zip(mps, (1e-3, 1.0, 1e3))]
        norms = np.array([1e-3 ** 13, 1.0, 1e3 ** 13])
        K_ref = np.array([[abs(ogram.overlap(a, c)) ** 2 for c in mps] for a in mps])
        b = q.import_batch(scaled)
        for prec, tol in TOL.items():
            K = q.gram(b, precision=prec).cpu().numpy() / np.outer(norms, norms) ** 2
            assert np.abs(K - K_ref).max() < 2 * tol


def test_jobs_of_several_kernels():
    """Jobs at bonds 2, 16, 32 and 40 in one call: the bits of separate
    calls, for every form that takes them."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    rng = np.random.default_rng(9)
    batches = []
    for bond, m in ((2, 7), (16, 11), (32, 12), (40, 13)):
        base = random_mps(rng, m, bond)
        batches.append(q.import_batch([random_mps(rng, m, bond, base) for _ in range(6)]))
    for prec in ("fp64", "fp32", "split_bf16", "split_i8"):
        jobs = []
        for b in batches:
            jobs.append(dict(a=b, b=b, na=6, nb=6, upper_only=True,
                             out=torch.zeros((6, 6), dtype=torch.float64, device="cuda")))
            jobs.append(dict(a=b, b=b, a0=1, na=2, b0=0, nb=5,
                             out=torch.zeros((2, 5), dtype=torch.float64, device="cuda")))
        q.gram_multi(jobs, precision=prec)
        for k, b in enumerate(batches):
            assert torch.equal(jobs[2 * k]["out"], q.gram(b, precision=prec))
            assert torch.equal(jobs[2 * k + 1]["out"], q.gram_block(b, 1, 2, b, 0, 5, precision=prec))


@pytest.mark.parametrize("bonds", [(33, 33), (64, 64), (17, 64), (64, 3), (48, 33), (49, 63)])
def test_split_edge_tiles(bonds):
    """The split forms' workgroup kernels leave out the tiles beyond the bonds
    of either operand: bras and kets of other bonds than each other."""
    import paper_2411_09336_amd as q
    require_gpu()
    rng = np.random.default_rng(64 * bonds[0] + bonds[1])
    m = 13
    base = random_mps(rng, m, min(bonds))
    wide = random_mps(rng, m, max(bonds))
    bras, kets = ([(random_mps(rng, m, bd, base) if bd == min(bonds) else random_mps(rng, m, bd, wide))
                   for _ in range(3)] for bd in bonds)
    K_ref = np.array([[abs(ogram.overlap(a, c)) ** 2 for c in kets] for a in bras])
    a, b = q.import_batch(bras), q.import_batch(kets)
    for prec, tol in SPLIT_TOL.items():
        err = np.abs(q.gram(a, b, precision=prec).cpu().numpy() - K_ref).max()
        print(bonds, prec, "max|dK|", err)
        assert err < tol
