"""Block-sign's first pass on the quarters of a chunk that are not whole ones of one block: where the row ends inside the quarter
(still one sum, columns beyond the row as they were), and where blocks end inside it (round by round).  Bit for bit against
the oracle, as every operation is fixed."""
import numpy as np
import pytest
import torch

from paper_2205_05632_amd import binding as B

from parity import Pair
from test_gpu_pages import offsets, values

pytestmark = pytest.mark.gpu
KINDS = ["plain", "zeros", "wide", "special", "ends"]


def run(n, d, size, kind, ld=None):
    p = Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=offsets(d, size), ld=ld)
    beyond = torch.arange(p.gpu.ld - d, device=p.gpu.device, dtype=torch.float32) + 7.0
    p.gpu.e[:, d:] = beyond
    rng = np.random.default_rng(d + size)
    for t in range(3):
        p.step(values(rng, n, d, kind), 1e-3, label=f"{n} x {d} / {size} {kind} step {t}", with_e=t == 2)
        assert bool((p.gpu.e[:, d:] == beyond).all()), "columns beyond the row were written"
    assert all(p.exact.values()), p.exact
    p.close()


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("d", [5, 1023, 1025, 2 * 1024 + 255, 3 * 1024 + 258, 4 * 1024 + 771, 9 * 4096 + 1021])
def test_row_ends_inside_a_quarter(d, kind):
    run(3, d, 1 << 30, kind, ld=B.padded_ld(d) + 64)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("size", [64, 256, 300, 1000, 1500])
def test_blocks_end_inside_quarters(size, kind):
    run(2, 3 * 4096 + 517, size, kind)
