"""Replays whose rows take another work-unit size than the rows they were sized by:
the size follows the row count and the slots that the rows lie in (at reach 3, 128 rows a
unit up to 524,288 rows in many slots, 512 from about 1.8e6 on, or from 3,584 rows a slot
on) in an insert and in a replay alike, so that both sum in one order."""
import numpy as np
import pytest

from gpu_cases import cuda

pytestmark = pytest.mark.gpu


def _bits(m):
    ijk, alpha = m.export()
    return ijk.cpu().numpy(), alpha.cpu().numpy().view(np.uint32)


# (rows of the sizing insert, rows of the replays, margin): a step down, a step up,
# the widest steps, and a step down without margin, where the shorter units of
# fewer rows outnumber the sizing insert's; in a small box, whose few slots give longer
# units, and in a large one
@pytest.mark.parametrize("edge", [1.5, 9.0])
@pytest.mark.parametrize("B", [4, 8])
@pytest.mark.parametrize("n0,n1,margin", [(600_000, 500_000, 0.5), (500_000, 600_000, 0.5),
                                          (2_000_000, 300_000, 0.5), (530_000, 520_000, 0.0),])
def test_replays_with_other_row_counts_equal_the_insert(n0, n1, margin, B, edge):
    import torch
    from paper_1909_04631_amd import SemanticMap
    print(f"[case] units B={B} box {edge} sized by {n0} rows, replayed with {n1}", flush=True)
    n, K = max(n0, n1), 3
    rng = np.random.default_rng(n1 + B)
    xyz = cuda(rng.uniform(0.0, edge, size=(n, 3)).astype(np.float32))
    lab = rng.integers(1, K, size=n).astype(np.int32)

    def labels(rows):   # (the hits without a label make no row)
        y = lab.copy()
        y[rng.permutation(n)[:n - rows]] = -1
        return y

    offs, org = [0, n // 3, n], [(0.0, 0.0, 0.0)] * 2
    new = lambda: SemanticMap(0.1, B, 0.3, 0.1, K, 1e-3, initial_blocks=1 << 12)  # noqa: E731
    y = cuda(labels(n0))
    m, ref = new(), new()
    b = m.batch_capture(xyz, y, offs, org, 0.0, margin=margin)
    for rows in (n1, n0, n1):
        y.copy_(cuda(labels(rows)))
        m.reset()
        b.replay(offs, org)
        m.sync()
        ref.reset()
        ref.insert_scans(xyz, y, offs, org, 0.0)
        torch.cuda.synchronize()
        a, r = m.stats(), ref.stats()
        assert a["n_hits"] == r["n_hits"] == rows
        assert a["n_units"] == r["n_units"] and a["n_pairs"] == r["n_pairs"]
        for u, v in zip(_bits(m), _bits(ref)):
            assert np.array_equal(u, v), rows
    b.close()
