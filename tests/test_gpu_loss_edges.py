"""The differentiable form at the sizes where its kernels can go wrong: row and
query counts around a wavefront, a workgroup and the validation's grid, and
inputs whose only bad row is the last one."""
import numpy as np
import pytest

import oracle
from gpu_cases import cuda

pytestmark = pytest.mark.gpu

L, S0, A0 = np.float32(0.3), np.float32(0.5), np.float32(0.001)


def _rows(n, K, seed, extent=1.5):
    rng = np.random.default_rng(seed)
    return (rng.uniform(-extent, extent, size=(n, 3)).astype(np.float32),
            rng.integers(0, K, size=n).astype(np.int32))


@pytest.mark.parametrize("bad", ["label", "nan", "range"])
@pytest.mark.parametrize("n,q", [(1, 1), (257, 256), (262_145, 65), (300, 262_145)])
def test_last_bad_row_is_an_error(n, q, bad):
    from paper_1909_04631_amd import SmkiError, loss_forward
    tx, ty = _rows(n, 4, n)
    qx, qy = _rows(q, 4, q + 1)
    for which in ("train", "query"):
        x, y = (tx, ty) if which == "train" else (qx, qy)
        x, y = x.copy(), y.copy()
        if bad == "label":
            y[-1] = 4
        else:
            x[-1, 2] = np.nan if bad == "nan" else 4.0e5
        args = (x, y, qx, qy) if which == "train" else (tx, ty, x, y)
        print(f"[case] {bad} in the last {which} row of {n} + {q}", flush=True)
        with pytest.raises(SmkiError) as e:
            loss_forward(*[cuda(v) for v in args], float(L), float(S0), float(A0), 4)
        assert e.value.status == (-6 if bad == "range" else -5)


@pytest.mark.parametrize("per_class", [False, True])
@pytest.mark.parametrize("n,q,K", [(1, 1, 2), (63, 3, 64), (64, 64, 65), (65, 130, 4),
                                   (2_000, 129, 255), (3_000, 65, 20)])
def test_rows_around_a_wavefront_and_many_classes(n, q, K, per_class):
    # 64 rows at a time per query, in up to 18 runs of sorted rows; sums per class
    # in 64, 16 or 8 columns; the box spans the origin so that blocks of either
    # sign meet, and one query lies away from every row
    from paper_1909_04631_amd import (loss_backward, loss_backward_classes, loss_forward,
                                      loss_forward_classes)
    print(f"[case] loss rows={n} queries={q} K={K} per_class={per_class}", flush=True)
    tx, ty = _rows(n, K, n + K, 0.4 if n < 100 else 0.9)
    qx, qy = _rows(q, K, q + K + 1, 0.4 if n < 100 else 0.9)
    qx[-1] = 3.0
    g = np.ones(1, np.float32)
    a = [cuda(v) for v in (tx, ty, qx, qy)]
    if per_class:
        rng = np.random.default_rng(K)
        lk = rng.choice(np.array([0.2, 0.25, 0.3], np.float32), K).astype(np.float64)
        sk = rng.choice(np.array([0.25, 0.5], np.float32), K).astype(np.float64)
        ref = oracle.loss_classes(tx, ty, qx, qy, K, lk, sk, float(A0))
        loss, aq = loss_forward_classes(*a, lk, sk, float(A0), K)
        gl, gs, gt, gq = loss_backward_classes(*a, lk, sk, float(A0), K, aq, cuda(g))
    else:
        lk, sk = np.array([float(L)]), np.array([float(S0)])
        ref = oracle.loss(tx, ty, qx, qy, K, float(L), float(S0), float(A0))
        loss, aq = loss_forward(*a, float(L), float(S0), float(A0), K)
        gl, gs, gt, gq = loss_backward(*a, float(L), float(S0), float(A0), K, aq, cuda(g))
    f = lambda t: t.cpu().numpy().astype(np.float64)  # noqa: E731
    assert np.max(np.abs(f(aq) - ref["alpha_q"]) / ref["alpha_q"]) <= 1e-5
    assert abs(float(loss.cpu()) - ref["loss"]) <= 1e-5 * abs(ref["loss"])
    # one scale for the scalar gradients: they are compared in log parameters
    got = np.concatenate([lk * f(gl).reshape(-1), sk * f(gs).reshape(-1)])
    want = np.concatenate([lk * np.reshape(ref["grad_l"], -1), sk * np.reshape(ref["grad_sigma0"], -1)])
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
    for x, r in ((gt, ref["grad_train"]), (gq, ref["grad_query"])):
        assert np.linalg.norm(f(x) - r) <= 1e-4 * np.linalg.norm(r)


@pytest.mark.parametrize("n,q", [(1, 1), (300, 40), (4_097, 64)])
def test_rows_far_from_queries(n, q):
    # half of the rows lie within reach of a query, the others in a box of about
    # 3.4e6 blocks around them: those are left out of the sort and get a zero
    # gradient.  A workspace of smki_loss_workspace_bytes has no room for the
    # bits of the cells near a query at that size (every row is then sorted);
    # the call's own allocation has: the results agree bit for bit.
    import torch
    from paper_1909_04631_amd import loss_backward, loss_forward
    from paper_1909_04631_amd.loss import workspace
    print(f"[case] far rows n={n} q={q}", flush=True)
    tx, ty = _rows(n, 4, n)
    qx, qy = _rows(q, 4, q + 1, 0.6)
    tx[n // 2:] *= 58.0
    tx[-1] = 89.0
    tx[0] = -89.0
    args = [cuda(v) for v in (tx, ty, qx, qy)] + [float(L), float(S0), float(A0), 4]
    g = cuda(np.ones(1, np.float32))
    ref = oracle.loss(tx, ty, qx, qy, 4, float(L), float(S0), float(A0))
    out = []
    for ws in (None, workspace(n, q, 4)):
        loss, aq = loss_forward(*args, ws=ws)
        out.append([loss, aq, *loss_backward(*args, aq, g, ws=ws)])
    torch.cuda.synchronize()
    for a, b in zip(*out):
        assert torch.equal(a, b)
    loss, aq, _, _, gt, gq = [t.cpu().numpy().astype(np.float64) for t in out[0]]
    assert np.max(np.abs(aq - ref["alpha_q"]) / ref["alpha_q"]) <= 1e-5
    assert abs(loss[0] - ref["loss"]) <= 1e-5 * abs(ref["loss"])
    assert np.all(gt[np.all(ref["grad_train"] == 0, axis=1)] == 0)
    for x, r in ((gt, ref["grad_train"]), (gq, ref["grad_query"])):
        assert np.linalg.norm(x - r) <= 1e-4 * max(np.linalg.norm(r), 1e-30)
