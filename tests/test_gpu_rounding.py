"""Rounding of the FP64 cell rule beyond 48 diameters against extended
precision, next to that of the rule evaluated point by point in double."""
import numpy as np
import pytest

from paper_2110_09214_amd import binding as B
from paper_2110_09214_amd import workloads as W
from gpu_helpers import bind, dev, host

pytestmark = pytest.mark.gpu


def seven_points(v, x, f):
    """Field and potential of the cell v (3, 3) at x (n, 3) by the 7-point rule
    in the type f, without fused operations."""
    v, x, r15 = v.astype(f), x.astype(f), np.sqrt(f(15))
    a, b = (6 - r15) / 21, (6 + r15) / 21
    area = np.sqrt((np.cross(v[1] - v[0], v[2] - v[0]) ** 2).sum()) / 2
    points = [(f(9) / 40, (f(1) / 3, f(1) / 3, f(1) / 3))]
    for t, w in ((a, (155 - r15) / 1200), (b, (155 + r15) / 1200)):
        points += [(w, (1 - 2 * t, t, t)), (w, (t, 1 - 2 * t, t)), (w, (t, t, 1 - 2 * t))]
    E, V = np.zeros_like(x), np.zeros(len(x), f)
    for w, c in points:
        d = x - (c[0] * v[0] + c[1] * v[1] + c[2] * v[2])
        ri = 1 / np.sqrt((d * d).sum(1))
        V += w * area * ri
        E += (w * area * ri * ri * ri)[:, None] * d
    return E, V


@pytest.mark.parametrize("offset", [0.0, 1.0])
@pytest.mark.parametrize("ratio", [(48.1, 60.0), (100.0, 300.0)])
def test_far_rule_rounds_as_its_points(ctx, ratio, offset):
    """Single cells at the origin and a distance of the targets away from it: the
    root mean square errors of field and potential over 12 cells and 24,000
    targets are at most 1.25 of those of the points' own sum in double (which
    has the same seven roundings of distance and root, more of the sum; a form
    that rounds the distance once for all points has 1.6 to 2.3)."""
    rng = np.random.default_rng(int(ratio[0]))
    ke = B.obem_constants()["k_e"]
    err = np.zeros((2, 2))
    for _ in range(12):
        v = rng.normal(size=(3, 3)) * 1e-5
        D = max(np.linalg.norm(v[(k + 1) % 3] - v[k]) for k in range(3))
        u = rng.normal(size=(2000, 3))
        u /= np.linalg.norm(u, axis=1, keepdims=True)
        v += offset * ratio[0] * D * rng.normal(size=3)
        x = v.mean(0) + D * np.exp(rng.uniform(*np.log(ratio), size=(2000, 1))) * u
        m = W.Mesh(v[None, 0], v[None, 1], v[None, 2], np.zeros(1, np.int8), np.ones(1), np.ones(1), np.zeros(1))
        E, V = B.field_eval(ctx, bind(ctx, m), dev(np.ones(1)), None, None, dev(x), 0.0, B.OBEM_FP64, want_v=True)
        Er, Vr = (np.longdouble(ke) * t for t in seven_points(v, x, np.longdouble))
        Ep, Vp = (ke * t for t in seven_points(v, x, np.float64))
        for k, (e, p) in enumerate(((host(E), host(V)), (Ep, Vp))):
            err[k, 0] += float((((e - Er) ** 2).sum(1) / (Er ** 2).sum(1)).sum())
            err[k, 1] += float(((p - Vr) ** 2 / Vr ** 2).sum())
    q = np.sqrt(err[0] / err[1])
    print("field, potential:", np.sqrt(err[0] / 24000), "quotients", q)
    assert (q <= 1.25).all(), q
