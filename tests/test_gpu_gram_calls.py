"""What a Gram call promises around its kernels: planes packed on first use
and read on another stream."""
import numpy as np
import pytest

from tests.gpu_util import require_gpu
from tests.test_gpu_gram_small import random_mps

pytestmark = pytest.mark.gpu


def _batch(n, m, bond, seed):
    import paper_2411_09336_amd as q
    rng = np.random.default_rng(seed)
    base = random_mps(rng, m, bond)
    return q.import_batch([random_mps(rng, m, bond, base) for _ in range(n)])


@pytest.mark.parametrize("prec", ["fp32", "split_bf16", "split_i8"])
def test_first_use_packs_for_every_stream(prec):
    """The planes that a Gram call builds are complete when it returns, also
    where its stream has earlier work to do: the next call may be on another
    stream."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    ref = q.gram(_batch(12, 10, 20, 1), precision=prec)
    b = _batch(12, 10, 20, 1)
    side = torch.cuda.Stream()
    first = torch.empty_like(ref)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)   # about 0.1 s
        q.gram(b, precision=prec, out=first)
    other = q.gram(b, precision=prec)
    torch.cuda.synchronize()
    assert torch.equal(other, ref)
    assert torch.equal(first, ref)


@pytest.mark.parametrize("prec", ["fp64", "split_i8"])
def test_allocating_calls_are_refused_under_capture(prec):
    """Calls that draw their work queue (and planes) from the allocator cannot
    be recorded: a replay would use memory that has gone back to it.  They say
    so before any launch, so the capture and the batch stay usable."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    ref = q.gram(_batch(6, 8, 12, 2), precision=prec)
    b = _batch(6, 8, 12, 2)
    out = torch.zeros((6, 6), dtype=torch.float64, device="cuda")
    flag = torch.zeros(1, device="cuda")
    job = dict(a=b, b=b, na=6, nb=6, upper_only=True, out=out)
    calls = [lambda: q.gram(b, precision=prec, out=out),
             lambda: q.gram_block(b, 0, 2, b, 1, 3, precision=prec, out=out[:2, :3]),
             lambda: q.gram_multi([job], precision=prec),
             lambda: q.autotune(b, prec, sample=4)]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        flag.add_(1.0)
        for call in calls:
            with pytest.raises(q.QKError) as e:
                call()
            assert "capture" in str(e.value)
    g.replay()
    torch.cuda.synchronize()
    assert flag.item() == 1.0 and not out.any()
    assert torch.equal(q.gram(b, precision=prec), ref)


def test_largest_allocation_free_queue():
    """724 x 724 pair tiles of side 16: 8,386,816 bytes of tiles, to which the
    counters and the job of one kernel add 656, in the 8,388,608 of the
    allocation-free scratch."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    x = torch.tensor([[0.3], [0.9], [0.1]], dtype=torch.float64, device="cuda")
    few = q.simulate(x, q.CircuitSpec(1, 1, 2), 2, 0.0)
    n = 16 * 724
    idx = torch.arange(n, device="cuda") % 3
    b = few.gather(idx.cpu().numpy())
    out = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    q.gram_block_noalloc(b, 0, n, b, 0, n, out)
    assert torch.equal(out, q.gram_block(few, 0, 3, few, 0, 3)[idx][:, idx])


@pytest.mark.parametrize("rows,cols", [(1, 256), (1, 500), (3, 200), (5, 37), (8, 8), (1, 3), (9, 130)])
@pytest.mark.parametrize("bond", [33, 64])
def test_rows_over_the_queues(bond, rows, cols):
    """Few rows with a queue per XCD (split-int8): the pairs lie in tiles of
    at most 16 columns, so that every queue has its share."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    few = _batch(3, 13, bond, 3)
    few.pack("split_i8")
    i, j = torch.arange(rows) % 3, torch.arange(cols) % 3
    a, b = few.gather(i.numpy(), ("split_i8",)), few.gather(j.numpy(), ("split_i8",))
    st = {}
    K = q.gram(a, b, precision="split_i8", stats=st)
    assert st["tiles"] == -(-rows // 16) * -(-cols // 16) and st["entries"] == rows * cols
    assert torch.equal(K.cpu(), q.gram_block(few, 0, 3, few, 0, 3, precision="split_i8").cpu()[i][:, j])


def test_few_pairs_of_the_split_forms():
    """No more pairs than the workgroup kernel holds at once: split-int8 from
    bond 17, and any call with a bond above 32, is one launch of that kernel,
    whose bits are those of a wave per pair."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    batches = {bond: _batch(4, 13, bond, bond) for bond in (3, 12, 20, 32, 40)}
    idx = torch.arange(44) % 4   # 990 pairs of the triangle, 1,936 of the block
    for prec in ("split_bf16", "split_i8"):
        ref = {}
        for bond, b in batches.items():
            b.pack(prec)
            st = {}
            K = q.gram(b, precision=prec, stats=st)
            assert st["block"] == (64 if bond > (16 if prec == "split_i8" else 32) else 32)
            many = q.gram(b.gather(idx.numpy(), (prec,)), precision=prec, stats=st)
            assert st["block"] == (64 if bond > 32 else 32)
            ref[bond] = many[:4, :4]
            assert torch.equal(K, ref[bond])
            # every ordered pair, as the triangle of repeats contracts them
            full = q.gram_block(b, 0, 4, b, 0, 4, precision=prec).cpu()[idx][:, idx]
            assert torch.equal(torch.triu(many.cpu()), torch.triu(full))
        for bonds in ((3, 12, 20, 40), (12, 32), (3, 40)):
            outs = {x: torch.zeros((4, 4), dtype=torch.float64, device="cuda") for x in bonds}
            q.gram_multi([dict(a=batches[x], b=batches[x], na=4, nb=4, upper_only=True, out=outs[x]) for x in bonds],
                         precision=prec)
            for x in bonds:
                assert torch.equal(outs[x], ref[x])


def test_longest_queue_has_its_workgroups():
    """1 x 400 split-int8 pairs are 25 tiles of 16 over eight queues, of which
    one has four: 64 pairs, as many as an eighth of the full grid."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    few = _batch(3, 9, 40, 7)
    few.pack("split_i8")
    j = torch.arange(400) % 3
    st = {}
    K = q.gram(few.gather([1], ("split_i8",)), few.gather(j.numpy(), ("split_i8",)), precision="split_i8", stats=st)
    assert st["workgroups"] // 8 >= 64
    assert torch.equal(K.cpu(), q.gram_block(few, 1, 1, few, 0, 3, precision="split_i8").cpu()[:, j])


def test_tuned_choice_is_a_different_launch_of_its_kernel():
    """The tuner chooses among launches that differ: at bonds up to 32, whose
    kernels have one queue and one block, tile sides alone; and a choice made
    for one kernel leaves the others alone."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    rng = np.random.default_rng(11)
    # 33 states: a triangle that sides of 8, 16 and 32 fill differently
    by_bond = {}
    for bond in (2, 12, 32, 40):
        few = _batch(3, 13, bond, bond)
        by_bond[bond] = few.gather(rng.integers(0, 3, 33))
    try:
        for prec in ("fp64", "fp32", "split_bf16", "split_i8"):
            default = (64, 16, 8 if prec == "split_i8" else 1)
            st = {}
            for bond in (32, 40):
                rep = q.autotune(by_bond[bond], prec, sample=33)
                chosen = (rep["maxp"], rep["tile_side"], rep["queues"])
                print(prec, bond, chosen, flush=True)
                assert rep["n_candidates"] == (12 if prec in ("fp64", "fp32") and bond <= 32 else 6)
                if chosen != default and bond <= 32:
                    assert rep["maxp"] == 64 and rep["queues"] == 1 and rep["tile_side"] != 16
                q.gram(by_bond[bond], precision=prec, stats=st)
                assert st["tile_side"] == rep["tile_side"]
                assert st["queues"] == (1 if bond <= 32 or st["tiles"] < 8 else rep["queues"])
            for bond in (2, 12) if prec == "fp64" else (12,):
                q.gram(by_bond[bond], precision=prec, stats=st)
                assert st["tile_side"] == 16 and st["queues"] == 1
    finally:
        q.autotune_reset()


# One kernel argument block carries 3,584 bytes: 512 of counters, a job of 144
# and 183 tiles; six of them 1,303 tiles, beyond which the queue is copied.
@pytest.mark.parametrize("rows,cols,tiles", [(48, 976, 183), (128, 368, 184), (224, 1488, 1302), (128, 2608, 1304),
                                             (800, 800, 2500)])
def test_queues_by_arguments_and_by_copy(rows, cols, tiles):
    """Work queues just within and beyond one argument block and all of them,
    drawn from the allocator and in the allocation-free scratch."""
    import paper_2411_09336_amd as q
    torch = require_gpu()
    few = _batch(7, 4, 4, 5)
    idx = torch.arange(max(rows, cols)) % 7
    b = few.gather(idx.numpy())
    st = {}
    K = q.gram_block(b, 0, rows, b, 0, cols, stats=st)
    assert st["tiles"] == tiles
    ref = q.gram_block(few, 0, 7, few, 0, 7).cpu()
    assert torch.equal(K.cpu(), ref[idx[:rows]][:, idx[:cols]])
    out = torch.zeros_like(K)
    q.gram_block_noalloc(b, 0, rows, b, 0, cols, out)
    assert torch.equal(out, K)
