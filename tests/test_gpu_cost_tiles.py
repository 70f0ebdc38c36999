"""The cost kernel covers a matrix in tiles of up to 256 columns and 32 rows:
all four matrices against the oracle where a tile is cut (one row or column,
one column past a tile, rows that do not fill the last tile), with several
replicas, tied embeddings on two stages, many stages on one side, failed ranks
whose stand-ins lie one and two replicas on, and replicas that lost a rank in
any of their words of the bitmap."""
import numpy as np
import pytest

from paper_2607_04749_amd import etc
from paper_2607_04749_amd.workloads import GPT, LLAMA, ModelShape, Parallel as P

pytestmark = pytest.mark.gpu

TIED = ModelShape(GPT, 4, 24, 12, 12, 36, 24, 8, 1)
UNTIED = ModelShape(LLAMA, 4, 24, 12, 12, 36, 24, 0, 0)
TIED16 = ModelShape(GPT, 16, 24, 12, 12, 36, 24, 8, 1)
UNTIED16 = ModelShape(LLAMA, 16, 24, 12, 12, 36, 24, 0, 0)


@pytest.mark.parametrize("model,src,dst,failed", [
    (TIED, P(1, 1, 1), P(1, 1, 1), []),
    (TIED, P(1, 1, 2), P(1, 1, 257), []),
    (UNTIED, P(1, 1, 257), P(1, 1, 1), [0, 2]),
    (UNTIED, P(3, 1, 1), P(2, 2, 1), []),
    (TIED, P(3, 2, 3), P(2, 4, 5), [0, 1, 2, 6]),
    (TIED, P(2, 2, 65), P(4, 1, 64), [0, 1, 4, 5, 259]),
    (UNTIED, P(4, 4, 16), P(4, 4, 33), [31, 32]),
    (UNTIED, P(1, 4, 64), P(2, 2, 64), list(range(8))),
    (TIED, P(2, 1, 4), P(1, 2, 7), [6, 0, 1]),  # stand-ins past the last replica
    # the only lost rank of a replica in a later word of the bitmap than its first: ranks 0 to 63, and 30 to 35
    (UNTIED16, P(4, 16, 2), P(4, 8, 2), [40]),
    (TIED16, P(4, 16, 2), P(2, 16, 3), [63, 97]),
    (UNTIED, P(3, 2, 7), P(2, 2, 7), [33]),
    (TIED16, P(1, 16, 1), P(1, 1, 1), []),  # many source stages of one target stage
    (TIED16, P(2, 1, 2), P(1, 16, 3), [1]),
    (UNTIED16, P(2, 16, 3), P(4, 2, 2), [5, 40]),
    (UNTIED16, P(4, 8, 1), P(3, 16, 1), []),
])
@pytest.mark.parametrize("placed", [False, True])
def test_matrices_at_tile_edges(model, src, dst, failed, placed):
    from gpu_util import check_matrices
    pair = None
    if placed:  # new ranks on live old GPUs in any order, across replicas
        rng = np.random.default_rng(src.world * 1000 + dst.world)
        live = np.setdiff1d(np.arange(src.world), failed)
        n = min(len(live), dst.world)
        pair = np.full(dst.world, -1, np.int32)
        pair[rng.permutation(dst.world)[:n]] = rng.permutation(live)[:n]
    print("[gpu] matrices", src, "->", dst, "failed", failed, "placed", placed, flush=True)
    plan = etc.etc_plan(model, src, dst, rank=int(np.setdiff1d(np.arange(src.world), failed)[0]), pair=pair,
                        failed=failed)
    check_matrices(plan, model, src, dst, pair=pair, failed=failed)
