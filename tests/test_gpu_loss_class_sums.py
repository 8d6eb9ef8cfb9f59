"""Per-class gradients summed over the queries: up to 8,192 queries in one launch, above
after a fold of the queries to 1,024 rows."""
import numpy as np
import pytest

import oracle
from gpu_cases import cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [2, 66])
@pytest.mark.parametrize("q", [8192, 8193, 9217])
def test_class_sums_around_the_fold(q, K):
    import torch
    from paper_1909_04631_amd.loss import loss_backward_classes, loss_forward_classes
    print(f"[case] class sums queries={q} K={K}", flush=True)
    rng = np.random.default_rng(q + K)
    tx = rng.uniform(-0.8, 0.8, size=(200, 3)).astype(np.float32)
    qx = rng.uniform(-0.8, 0.8, size=(q, 3)).astype(np.float32)
    ty, qy = (rng.integers(0, K, size=m).astype(np.int32) for m in (200, q))
    lk = np.linspace(0.25, 0.45, K).astype(np.float32).astype(np.float64)
    sk = np.linspace(0.2, 0.9, K).astype(np.float32).astype(np.float64)
    a0 = float(np.float32(1e-3))
    ref = oracle.loss_classes(tx, ty, qx, qy, K, lk, sk, a0)
    args = [cuda(v) for v in (tx, ty, qx, qy)] + [lk, sk, a0, K]
    _, aq = loss_forward_classes(*args)
    gl, gs, gt, gq = loss_backward_classes(*args, aq, cuda(np.ones(1, np.float32)))
    torch.cuda.synchronize()
    f = lambda t: t.cpu().numpy().astype(np.float64)  # noqa: E731
    want = np.concatenate([lk * ref["grad_l"], sk * ref["grad_sigma0"]])
    got = np.concatenate([lk * f(gl), sk * f(gs)])
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
    assert np.linalg.norm(f(gt) - ref["grad_train"]) <= 1e-4 * np.linalg.norm(ref["grad_train"])
    assert np.linalg.norm(f(gq) - ref["grad_query"]) <= 1e-4 * np.linalg.norm(ref["grad_query"])
