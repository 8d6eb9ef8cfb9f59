"""Readouts of some of the outputs hold what a readout of all of them holds."""
import itertools

import numpy as np
import pytest

from gpu_cases import cuda

pytestmark = pytest.mark.gpu

NAMES = ("alpha", "mean", "var", "label", "p_occ")


@pytest.mark.parametrize("K", [4, 33, 65, 255])
def test_subsets_of_the_outputs(K):
    import torch
    from paper_1909_04631_amd import SemanticMap
    print(f"[case] query outputs K={K}", flush=True)
    rng = np.random.default_rng(K)
    xyz = rng.uniform(0.0, 2.0, size=(500, 3)).astype(np.float32)
    m = SemanticMap(0.2, 4, 0.3, 0.5, K, 1e-3)
    m.insert_scan(cuda(xyz), cuda(rng.integers(0, K, size=500).astype(np.int32)), (0.0, 0.0, 0.0), 0.0)
    ijk = cuda(rng.integers(-3, 13, size=(1003, 3)).astype(np.int32))
    full = m.query(ijk)
    for keep in itertools.product([False, True], repeat=len(NAMES)):
        if not any(keep):
            continue
        out = m.query(ijk, **dict(zip(NAMES, keep)))
        for name, k in zip(NAMES, keep):
            if k:
                assert torch.equal(out[name], full[name]), (name, keep)
