"""GPU parity at the sizes where a launch rule or a kernel variant changes: edges of units, workgroups and grids,
remainders, and the smallest and largest array of each variant.  Oracle and tolerances as in test_gpu_parity.py."""
import numpy as np
import pytest

import oracle
from paper_1511_04561_amd import workloads
from tests.test_gpu_parity import Guarded, check_error_stats, dev, same_bits  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dq8():
    if not torch.cuda.is_available():
        pytest.fail("these tests need a GPU (select them with -m gpu on a GPU box)")
    from paper_1511_04561_amd import dq8 as mod
    mod.lib()  # a missing library is an error, not a skip
    mod.init()
    oracle.set_threads(16)
    return mod


@pytest.mark.parametrize("n,block", [
    (1, 0), (11 * 1024 + 5, 0),         # one workgroup of twelve wavefronts, some of them without work
    (12 * 1024, 0), (13 * 1024 + 1, 0),  # exactly one workgroup, and one wavefront more
    (40 * 5120 + 3, 5120),              # blocks that end inside a workgroup's runs: it holds several at the end
    (800 * 100, 100), (2500 * 1100 + 7, 1100),  # a block or two per wavefront; more blocks than the last workgroup has threads
    (12 * 1024 * 512 + 4099, 0),        # two units per wavefront, the grid full
    (12 * 1024 * 512 * 2 + 1, 6144 * 1024)])
def test_error_stats_shared_blocks(dq8, n, block):
    """Wavefronts that share blocks: combined in the workgroup, merged by atomics, means by the workgroup that ends last."""
    rng = np.random.Generator(np.random.PCG64(6100 + n % 97))
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-6, 0, n))).astype(np.float32)
    x[::17] = 0.0
    check_error_stats(dq8, 0, x, block, tag="shared")
    nb = oracle.dq8_oracle.n_blocks(n, block)
    check_error_stats(dq8, 3, x, block, given=np.full(nb, 4.0, np.float32), tag="shared, given")
