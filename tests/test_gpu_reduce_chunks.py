"""The reduction's chunks (4,096 paths) at their edges: nodes of one path more
or less than a chunk, of none and of more chunks than a wave has lanes, in one
launch and in launches that cut them, against exact sums of the records: to
1e-12 of the summed magnitudes, the counts exactly. Without the caller's
records (one launch then reduces and ends the statistics at once), the same bits."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("cap", [0, 4096, 10007])
@pytest.mark.parametrize("counts", [[4096, 1, 4097, 4095], [4097], [0, 8193, 0, 8192, 0], [5, 65 * 4096 + 1, 5]])
def test_chunk_edges(counts, cap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = pdd.Context(0)
    prob = pdd.Problem(ctx, W.unit_square_problem(seed=0))
    counts = np.array(counts, dtype=np.uint64)
    nodes = W.unit_square_nodes()[:len(counts)]
    rec = pdd.alloc_records(int(counts.sum()))
    st = pdd.stats_to_numpy(pdd.solve_nodes(prob, nodes, dt=4e-3, n_paths_per_node=counts, records=rec,
                                            tuning=(256, 0, 64, cap)))
    scratch = pdd.stats_to_numpy(pdd.solve_nodes(prob, nodes, dt=4e-3, n_paths_per_node=counts, tuning=(256, 0, 64, cap)))
    assert scratch.tobytes() == st.tobytes()
    phis, words = rec["phi"].cpu().numpy(), rec["steps"].cpu().numpy().view(np.uint32)
    prob.close()
    ctx.close()
    ends = np.cumsum(counts.astype(np.int64))
    for i, end in enumerate(ends):
        phi, word = phis[end - int(counts[i]):end], words[end - int(counts[i]):end]
        assert st["n"][i] == counts[i]
        assert st["steps_sum"][i] == int((word & 0x7FFFFFFF).astype(np.int64).sum())
        assert st["n_capped"][i] == int((word >> 31).sum())
        for q, terms in ((0, phi), (2, phi * phi)):
            total = st["sums"][i][q] + st["sums"][i][q + 1]
            assert abs(total - math.fsum(terms)) <= 1e-12 * math.fsum(np.abs(terms))
