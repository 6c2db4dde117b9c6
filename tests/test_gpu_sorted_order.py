"""The sorted order of the force kernels, worked out on the device: exactly the order of a stable
NumPy sort by star and Morton code (10 bits per axis in the star's bounding box), ties by index.

Sizes at the edges of waves, workgroups and tiles of the sort (2048 elements), one star empty or of
one element, coincident elements, a star without extent, coordinates that are not finite or at the
ends of the type's range, in FP32 and FP64, at creation and after a re-sort."""

import numpy as np
import pytest

from gpu_common import print_case, require_gpu

pytestmark = pytest.mark.gpu


def _spread(q):
    out = np.zeros(q.shape, np.uint64)
    for b in range(10):
        out |= ((q >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b)
    return out


def _star(p):
    if len(p) == 0:
        return np.zeros(0, np.int64)
    p = p.astype(np.float64)
    fin = np.isfinite(p)
    lo = np.where(fin, p, 1e300).min(axis=0, initial=1e300)
    hi = np.where(fin, p, -1e300).max(axis=0, initial=-1e300)
    with np.errstate(over="ignore", invalid="ignore"):
        span = np.where(hi > lo, hi - lo, 1.0)
        f = np.where(fin, (p - lo) / span, 0.0)
    f = np.where(f < 0.0, 0.0, f)
    f = np.where(f > 1.0, 1.0, f) * 1024.0
    q = np.where(f < 1023.0, f, 1023.0).astype(np.uint64)
    code = sum(_spread(q[:, d]) << np.uint64(d) for d in range(3))
    return np.argsort(code, kind="stable")


def _reference(p, n1):
    n = len(p)
    p1 = -(-n1 // 256) * 256
    total = max(p1 + -(-(n - n1) // 256) * 256, 256)
    out = np.full(total, -1, np.int64)
    out[:n1] = _star(p[:n1])
    out[p1:p1 + n - n1] = n1 + _star(p[n1:])
    return out


def _positions(n, n1, kind, seed):
    rng = np.random.default_rng(seed)
    p = rng.standard_normal((n, 3))
    p[n1:, 0] += 5.0
    if kind == "ties":
        p = np.round(p * 2.0) / 2.0
    elif kind == "flat":
        p[:n1] = p[0]
        p[n1:, 1] = 0.25
    elif kind == "non-finite":
        p[rng.integers(0, n, max(1, n // 7)), rng.integers(0, 3)] = np.nan
        p[rng.integers(0, n, max(1, n // 9)), rng.integers(0, 3)] = np.inf
        p[rng.integers(0, n, max(1, n // 9)), rng.integers(0, 3)] = -np.inf
    elif kind == "range":
        p[rng.integers(0, n, max(1, n // 5)), 0] = 3e38
        p[rng.integers(0, n, max(1, n // 5)), 1] = -3e38
    return p


@pytest.mark.parametrize("mode", ["kahan", "fp64"])
@pytest.mark.parametrize("n,n1,kind", [
    (1, 1, "plain"), (1, 0, "plain"), (64, 63, "plain"), (257, 1, "ties"), (511, 256, "flat"),
    (2048, 2048, "plain"), (2049, 1000, "ties"), (4095, 0, "plain"), (4097, 2500, "non-finite"),
    (6000, 3000, "range"), (33333, 20001, "plain"), (150001, 100000, "ties")])
def test_order_is_the_stable_morton_order(n, n1, kind, mode):
    import torch

    nb = require_gpu()
    dtype = np.float64 if mode == "fp64" else np.float32
    p = _positions(n, n1, kind, n).astype(dtype)
    print_case("sorted order", n, n1, kind, mode)
    s = nb.System(p, np.zeros_like(p), n1, G=1.0, m=1.0 / n, dt=1e-4, D1=0.05, D2=0.05, q=0.5,
                  mode=mode)
    assert np.array_equal(nb.nb_sorted_order(s.handle, s.stream), _reference(p, n1))
    moved = _positions(n, n1, kind, n + 1).astype(dtype)
    for t, c in zip((s.x, s.y, s.z), moved.T):
        t.copy_(torch.from_numpy(np.ascontiguousarray(c)))
    s.resort()
    assert np.array_equal(nb.nb_sorted_order(s.handle, s.stream), _reference(moved, n1))
    s.close()


@pytest.mark.parametrize("mode", ["kahan", "fp64"])
@pytest.mark.parametrize("n,n1,kind", [
    (2, 1, "plain"), (65, 64, "ties"), (512, 0, "flat"), (513, 300, "ties"), (1023, 511, "non-finite"),
    (1536, 1025, "range"), (1537, 3, "ties"), (2047, 2000, "non-finite"), (2048, 1, "ties")])
def test_order_of_one_sort_tile(n, n1, kind, mode):
    """Systems of at most 2048 elements are sorted by one workgroup: edges of its waves' 512 elements."""
    test_order_is_the_stable_morton_order(n, n1, kind, mode)
