"""Units of few rows at small stencils: their rows are splatted one by one up to 16 of
them, then by lanes over rows, 16 rows at a time through the LDS table."""
import numpy as np
import pytest

import oracle
from gpu_cases import ALPHA_RTOL, compare_map, cuda

pytestmark = pytest.mark.gpu

RES, K = 0.2, 3


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("lv,B", [(0.4, 4), (0.8, 2), (1.0, 8), (1.5, 4), (1.5, 16)])
def test_rows_per_unit(lv, B, soft):
    # one block per row count, three blocks apart: 1 .. 17, around a table's 16 rows and
    # a set's 64, a unit's 128
    import torch
    from paper_1909_04631_amd import SemanticMap
    print(f"[case] small units l/res={lv} B={B} soft={soft}", flush=True)
    rng = np.random.default_rng(int(10 * lv) + B)
    counts = list(range(1, 18)) + [31, 32, 33, 48, 63, 64, 65, 79, 80, 81, 127, 128, 129, 145]
    xyz, edge = [], B * RES
    for i, n in enumerate(counts):
        # a block's rows in a few of its cells, on both sides of every axis; some share a cell
        p = rng.uniform(0.0, edge, size=(n, 3))
        p[n // 2:] = p[0] + rng.uniform(-0.05, 0.05, size=(n - n // 2, 3))
        xyz.append(np.clip(p, 0.001, edge - 0.001) + [3 * edge * i, -3 * edge * (i % 2), 0.0])
    xyz = np.concatenate(xyz).astype(np.float32)
    n = xyz.shape[0]
    f32 = lambda v: float(np.float32(v))  # noqa: E731
    m = SemanticMap(RES, B, lv * RES, 0.1, K, 1e-3)
    om = oracle.OracleMap(res=f32(RES), l=f32(lv * RES), sigma0=f32(0.1), alpha0=f32(1e-3), K=K, block_size=B)
    if soft:
        w = np.zeros((n, K), np.float32)
        w[:, 1] = rng.uniform(0.1, 1.0, size=n)
        m.insert_scan_soft(cuda(xyz), cuda(w), (0.0, 0.0, 0.0), 0.0)
        om.insert_scan_soft(xyz, w, (0.0, 0.0, 0.0), 0.0, 0)
    else:
        lab = np.ones(n, np.int32)
        m.insert_scan(cuda(xyz), cuda(lab), (0.0, 0.0, 0.0), 0.0)
        om.insert_scan(xyz, lab, (0.0, 0.0, 0.0), 0.0, 0)
    torch.cuda.synchronize()
    assert m.stats()["n_hits"] == n
    compare_map(m, om, K, rtol=ALPHA_RTOL)


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("lv", [0.4, 1.0, 1.5])
def test_few_rows_have_the_bits_of_many(lv, soft):
    # rows in one corner of a block, alone (a unit of few rows) and with 16 rows in the
    # opposite corner: the voxels around the first corner hold the same bits
    import torch
    from paper_1909_04631_amd import SemanticMap
    print(f"[case] few rows l/res={lv} soft={soft}", flush=True)
    rng = np.random.default_rng(int(10 * lv))
    B = 16
    for n in (1, 2, 5, 9, 16):
        xyz = np.concatenate([rng.uniform(0.0, 4 * RES, size=(n, 3)),
                              rng.uniform(11 * RES, 15.9 * RES, size=(16, 3))]).astype(np.float32)
        ijk = cuda(np.stack(np.meshgrid(*[np.arange(-3, 7)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.int32))
        w = np.zeros((n + 16, K), np.float32)
        w[:, 1] = rng.uniform(0.1, 1.0, size=n + 16)
        got = []
        for rows in (n, n + 16):
            m = SemanticMap(RES, B, lv * RES, 0.1, K, 1e-3)
            if soft:
                m.insert_scan_soft(cuda(xyz[:rows]), cuda(w[:rows]), (0.0, 0.0, 0.0), 0.0)
            else:
                m.insert_scan(cuda(xyz[:rows]), cuda(np.ones(rows, np.int32)), (0.0, 0.0, 0.0), 0.0)
            got.append(m.query(ijk)["alpha"])
            assert m.stats()["n_hits"] == rows
        torch.cuda.synchronize()
        assert torch.equal(got[0], got[1]), n
