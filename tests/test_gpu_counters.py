"""Insert counters of the splat's work: the pairs it examines and the lane-iterations
it issues, recomputed from the rows of each (class, block)."""
import itertools

import numpy as np
import pytest

from gpu_cases import cuda

pytestmark = pytest.mark.gpu

RES = 0.125   # (a power of two: cells follow from the rows without rounding)


def _offsets(lv, octant):
    """Voxel offsets within lv (in cells) of some point of a cell, or of its first octant."""
    L, r = lv + 1e-4, 5
    lo = (lambda o: o - 0.5 if o >= 1 else float(-min(o, 0))) if octant else (lambda o: max(0.0, abs(o) - 0.5))
    return sum(sum(lo(o) ** 2 for o in v) < L * L for v in itertools.product(range(-r, r + 1), repeat=3))


@pytest.mark.parametrize("budget", [0, 100])
@pytest.mark.parametrize("lv,B", [(0.4, 4), (0.8, 2), (1.0, 4), (1.5, 4), (1.5, 16), (1.7, 4), (3.0, 8)])
def test_pairs_examined_and_lane_iterations(lv, B, budget):
    import torch
    from paper_1909_04631_amd import SemanticMap
    print(f"[case] counters l/res={lv} B={B} budget={budget}", flush=True)
    K, n = 3, 3000
    rng = np.random.default_rng(B)
    xyz = np.concatenate([rng.uniform(0.0, 8.0, size=(n // 2, 3)), rng.uniform(1.0, 2.0, size=(n - n // 2, 3))])
    xyz, lab = xyz.astype(np.float32), rng.integers(0, K, size=n).astype(np.int32)
    m = SemanticMap(RES, B, lv * RES, 0.1, K, 1e-3, unit_budget=budget)
    pts, labels = cuda(xyz), cuda(lab)
    m.insert_scan(pts, labels, (0.0, 0.0, 0.0), 0.0)
    torch.cuda.synchronize()
    st = m.stats()
    blocks = np.floor(xyz / RES).astype(np.int64) // B
    _, rows = np.unique(np.column_stack([lab, blocks]), axis=0, return_counts=True)
    chunk = budget or 128   # (3,000 rows: never longer)
    ceil = lambda a, b: -(-a // b)  # noqa: E731
    assert st["n_units"] == ceil(rows, chunk).sum()
    full = _offsets(lv, False)
    if full <= 33:   # 64 rows at a time, the offsets three by three; up to 16 rows one by one
        unit = lambda r: np.where(r <= 16, r, ceil(r, 64) * ceil(full, 3) * 3)  # noqa: E731
        want = n * full, 64 * (rows // chunk * unit(chunk) + unit(rows % chunk)).sum()
    else:            # one row at a time, the offsets of its octant in steps of 64 lanes
        octant = _offsets(lv, True)
        want = n * octant, n * ceil(octant, 64) * 64
    assert (st["n_candidates"], st["n_lane_slots"]) == want
    assert st["n_pairs"] <= st["n_candidates"] <= st["n_lane_slots"]
    b = m.batch_capture(pts, labels, [0, n], [(0.0, 0.0, 0.0)], 0.0, margin=0.5)
    m.reset()
    b.replay([0, n], [(0.0, 0.0, 0.0)])
    m.sync()
    rp = m.stats()
    assert all(rp[k] == st[k] for k in ("n_units", "n_pairs", "n_candidates", "n_lane_slots"))
    b.close()
