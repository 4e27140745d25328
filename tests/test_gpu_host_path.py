"""The host side of small calls: work queues and step lists that travel in
kernel arguments, in several of them, or as one copy; the allocation-free
Gram recorded into a graph; sizes of freed batches."""
import numpy as np
import pytest

from oracle import gram as ogram
from tests.gpu_util import require_gpu
from tests.test_gpu_gram_small import random_mps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 37, 250, 420, 700])
def test_work_queue_sizes(n):
    """Symmetric matrices whose tile lists take one kernel argument block
    (up to ~200 tiles of 16 x 16), several, and a copy (above ~1,300):
    states are repeats of eight, so every entry is known."""
    import paper_2411_09336_amd as q
    require_gpu()
    rng = np.random.default_rng(n)
    base = random_mps(rng, 6, 4)
    mps = [random_mps(rng, 6, 4, base) for _ in range(8)]
    idx = np.arange(n) % 8
    K_ref = np.array([[abs(ogram.overlap(a, b)) ** 2 for b in mps] for a in mps])[np.ix_(idx, idx)]
    b = q.import_batch(mps).gather(idx)
    assert np.abs(q.gram(b).cpu().numpy() - K_ref).max() < 1e-12


def test_noalloc_gram_in_a_graph():
    """A recorded allocation-free Gram gives the eager result at every replay,
    with eager calls and synchronisations between the replays."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    rng = np.random.default_rng(2)
    base = random_mps(rng, 8, 12)
    b = q.import_batch([random_mps(rng, 8, 12, base) for _ in range(20)])
    for prec in ("fp64", "split_i8"):
        b.pack(prec)
        ref = q.gram(b, precision=prec)
        out = torch.zeros_like(ref)
        q.gram_block_noalloc(b, 0, 20, b, 0, 20, out, precision=prec, upper_only=True)   # warm-up
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            q.gram_block_noalloc(b, 0, 20, b, 0, 20, out, precision=prec, upper_only=True)
        for _ in range(4):
            out.fill_(-1.0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, ref)
            assert torch.equal(q.gram(b, precision=prec), ref)


def test_batch_used_on_another_stream():
    """A simulated batch can be multiplied on any stream at once."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    x = torch.rand((6, 9), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    b = q.simulate(x, q.CircuitSpec(9, 2, 1), 16, 1e-10, stream=side)
    K = q.gram(b)
    torch.cuda.synchronize()
    assert torch.equal(K, q.gram(b))
    assert np.allclose(np.diag(K.cpu().numpy()), 1.0, atol=1e-12)


def test_freed_batch_is_refused():
    import paper_2411_09336_amd as q
    require_gpu()
    rng = np.random.default_rng(3)
    a = q.import_batch([random_mps(rng, 4, 2) for _ in range(2)])
    b = q.import_batch([random_mps(rng, 4, 2) for _ in range(3)])
    assert (a.n, a.m, b.n) == (2, 4, 3)
    b.free()
    for call in (lambda: b.n, lambda: q.gram(a, b), lambda: q.gram(b), lambda: b.bond_dims()):
        with pytest.raises(q.QKError):
            call()
