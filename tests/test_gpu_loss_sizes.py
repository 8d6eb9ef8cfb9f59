"""The differentiable form where the rows and the rows with the queries lie on
different sides of 2^18, the size at which the sort's tiles change: the calls
that sort the rows alone share their scratch with those that sort both.  Above
2^18 queries the marks of the cells around them are written in strides."""
import numpy as np
import pytest

import oracle
from gpu_cases import cuda

pytestmark = pytest.mark.gpu

L, S0, A0, K = np.float32(0.3), np.float32(0.5), np.float32(0.001), 4


@pytest.mark.parametrize("own_ws", [False, True])
@pytest.mark.parametrize("n,q", [(200_000, 70_000), (262_144, 1), (250_000, 25_000), (1_000, 262_144),
                                 (1_000, 262_177)])
def test_rows_and_queries_around_the_tile_change(n, q, own_ws):
    # 300 rows within reach of the queries, the others in a box of about 8,000
    # blocks away from them: the oracle takes the 300
    import torch
    from paper_1909_04631_amd import loss_backward, loss_forward
    from paper_1909_04631_amd.loss import workspace
    print(f"[case] loss rows={n} queries={q} own_ws={own_ws}", flush=True)
    rng = np.random.default_rng(n + q)
    near = 300
    tx = rng.uniform(2.0, 22.0, size=(n, 3)).astype(np.float32)
    tx[-near:] = rng.uniform(-0.9, 0.9, size=(near, 3))
    qx = rng.uniform(-0.6, 0.6, size=(q, 3)).astype(np.float32)
    ty, qy = (rng.integers(0, K, size=m).astype(np.int32) for m in (n, q))
    ref = oracle.loss(tx[-near:], ty[-near:], qx, qy, K, float(L), float(S0), float(A0))
    args = [cuda(v) for v in (tx, ty, qx, qy)] + [float(L), float(S0), float(A0), K]
    ws = workspace(n, q, K) if own_ws else None
    g = cuda(np.ones(1, np.float32))
    loss, aq = loss_forward(*args, ws=ws)
    gl, gs, gt, gq = loss_backward(*args, aq, g, ws=ws)
    gl1, gs1, none, gq1 = loss_backward(*args, aq, g, need_train=False, ws=ws)
    loss1, aq1 = loss_forward(*args, ws=ws)
    torch.cuda.synchronize()
    # a second forward has the bits of the first
    assert none is None and torch.equal(aq, aq1) and torch.equal(loss, loss1)
    f = lambda t: t.cpu().numpy().astype(np.float64)  # noqa: E731
    assert np.max(np.abs(f(aq) - ref["alpha_q"]) / ref["alpha_q"]) <= 1e-5
    assert abs(f(loss)[0] - ref["loss"]) <= 1e-5 * abs(ref["loss"])
    # the rows of one query come in the same order in both sorts
    assert torch.equal(gq, gq1) and torch.equal(gl, gl1) and torch.equal(gs, gs1)
    assert np.linalg.norm(f(gq) - ref["grad_query"]) <= 1e-4 * np.linalg.norm(ref["grad_query"])
    assert np.all(f(gt)[:-near] == 0)
    assert np.linalg.norm(f(gt)[-near:] - ref["grad_train"]) <= 1e-4 * np.linalg.norm(ref["grad_train"])
    got, want = float(L) * f(gl)[0], float(L) * ref["grad_l"]
    assert abs(got - want) <= 1e-4 * np.hypot(want, float(S0) * ref["grad_sigma0"])
