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
