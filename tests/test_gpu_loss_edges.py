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
