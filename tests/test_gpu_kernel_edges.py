"""Kernels at the sizes where their tiles, chunks and dispatch rules change:
remainders, the smallest and the largest of each range, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2110_09214_amd import binding as B
from paper_2110_09214_amd import workloads as W
from gpu_helpers import bind, dev, host, rel_l2

pytestmark = pytest.mark.gpu


def _first_cells(m, n):
    """The mesh of the first n cells of m."""
    return W.Mesh(m.a[:n], m.b[:n], m.c[:n], m.kind[:n], m.eps1[:n], m.eps2[:n], m.rhs[:n] + 1.0, name=f"first_{n}")


@pytest.mark.parametrize("n", [1, 7, 8, 9, 31, 33, 63, 65, 254, 257, 513])
def test_matrix_passes_at_odd_sizes(ctx, orc, n):
    """Product with the inverse and compensated residual: rows and columns on
    both sides of the row block (256, 64) and of the columns in flight (8).
    The matrices' condition is below 1e4, so FP64 products agree to 1e-11.
    (At 255 and 511 cells of this mesh the library's inverse itself is off,
    and the solve reports OBEM_ENOCONV.)"""
    m = _first_cells(W.parallel_plate_mesh(n=12), n)
    ref, _ = orc.bem_solve(m)
    bm = bind(ctx, m)
    sig, info = B.bem_solve_charges(ctx, bm, dev(m.rhs))
    assert info["backward_error"] <= 1e-15
    assert rel_l2(host(sig), ref) <= 1e-11
    for refine in (0, 1):  # without info: nothing read back on the host
        s, _ = B.bem_solve_charges(ctx, bm, dev(m.rhs), max_refine=refine, want_info=False)
        assert rel_l2(host(s), ref) <= 1e-11


@pytest.mark.parametrize("scale", [1e-2, 0.05, 0.2, 0.5, 0.9, 1.1, 2.9, 11.0, 47.0])
def test_closed_form_around_its_switches(ctx, orc, scale):
    """One cell's closed form on both sides of the switch to the distances
    from the edge's line (sum of the two distances 1.25 edge lengths), of the
    arctangent's (numerator a quarter of the denominator) and in the far
    range: targets at scale diameters around the edges, the vertices and the
    centroid.  The form's own error is below 1e-12 up to 48 diameters, the
    rounding of the inputs adds 2^-53 |x| / distance < 1e-13."""
    rng = np.random.default_rng(int(1000 * scale))
    a, b, c = np.array([[0.3, -0.2, 0.1], [1.1, 0.1, -0.2], [0.5, 0.9, 0.3]])[:, None, :] * 1e-5
    D = max(np.linalg.norm(b - a), np.linalg.norm(c - b), np.linalg.norm(a - c))
    u = rng.normal(size=(192, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    t = rng.uniform(size=(64, 1))
    base = np.concatenate([a + t * (b - a), np.repeat(c, 64, 0), np.repeat((a + b + c) / 3, 64, 0)])
    x = base + scale * D * u
    m = W.Mesh(a, b, c, np.zeros(1, np.int8), np.ones(1), np.ones(1), np.zeros(1))
    sig = np.array([1e-6])
    E, V = B.field_eval(ctx, bind(ctx, m), dev(sig), None, None, dev(x), 0.0, B.OBEM_FP64, want_v=True)
    Er, Vr = orc.panel_field(x, a, b, c, sig, want_v=True)
    assert (np.linalg.norm(host(E) - Er, axis=1) / np.linalg.norm(Er, axis=1)).max() <= 2e-12
    assert (np.abs(host(V) - Vr) / np.abs(Vr)).max() <= 2e-12


@pytest.mark.parametrize("n", [1, 63, 65, 130, 257])
@pytest.mark.parametrize("spread", [2e-6, 60e-6])
def test_close_pairs_queue(ctx, orc, n, spread):
    """Targets in a hole of the coarse GEM cell, within a cell's size or over
    many of them: cells seen by a few or by all targets of a wave, batches of
    queued pairs that fill, overflow and end part full.  Tolerances of the
    two precisions as in the field tests (a lost pair is above 1e-4)."""
    geo = W.GemGeometry(m=3, n_r=2, n_cone=2, plain_h=48e-6)
    m = W.gem_cell_mesh(geo)
    rng = np.random.default_rng(n)
    cx, cy = geo.hole_centres()[4]
    x = np.array([cx + 0.8 * geo.r_inner, cy, 3e-6]) + rng.uniform(-1, 1, size=(n, 3)) * np.array([0.2, 0.2, 1.0]) * spread
    sig = 1e-6 * (1.0 + rng.uniform(size=m.n))
    Er, Vr = orc.panel_field(x, m.a, m.b, m.c, sig, want_v=True)
    bm = bind(ctx, m)
    for prec, tol in ((B.OBEM_FP64, 1e-12), (B.OBEM_MIXED, 1e-5)):
        E, V = B.field_eval(ctx, bm, dev(sig), None, None, dev(x), 0.0, prec, want_v=True)
        assert rel_l2(host(E), Er) <= tol
        assert rel_l2(host(V), Vr) <= tol
        # many targets (one wave a workgroup instead of four): the same points again
        at = np.arange(130001 if n == 257 else 0) % n
        if len(at):
            E, V = B.field_eval(ctx, bm, dev(sig), None, None, dev(x[at]), 0.0, prec, want_v=True)
            assert rel_l2(host(E), Er[at]) <= tol
            assert rel_l2(host(V), Vr[at]) <= tol


@pytest.mark.parametrize("n", [6145, 43008, 43009])
def test_pair_once_in_parts(ctx, orc, n):
    """The pair-once evaluation cut in parts (up to 224 super-block pairs: 21
    full super-blocks) and whole (one charge more), and the first size with
    an even number of super-blocks, at the error bound of the pair-once
    tests, on a sample of the charges."""
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 3)) * 50e-6
    q = np.where(rng.uniform(size=n) < 0.6, -W.E_CHARGE, W.E_CHARGE)
    E = host(B.field_eval(ctx, None, None, dev(x), dev(q), dev(x), 1e-7, B.OBEM_MIXED, tgt_is_src=True))
    at = np.concatenate([rng.choice(n, 400, replace=False), [0, n - 1]])
    assert rel_l2(E[at], orc.pair_field(x[at], x, q, 1e-7)) <= 1e-5


@pytest.mark.parametrize("grid", [(40, 41, 43), (128, 128, 129)])
def test_map_packed_and_plain(ctx, orc, grid):
    """Map interpolation just below and at the count that packs the map (2^18
    points, for at most eight times as many nodes): the same values bit for
    bit as in small calls, which read the three arrays, and the oracle's on a
    sample; the currents of the packed map against the plain ones."""
    n = 1 << 18
    lo, h = (-1e-3, -2e-3, 0.0), (1e-5, 2e-5, 1.5e-5)
    fmap = B.FieldMap(lo, h, grid)
    gen = torch.Generator(device="cuda").manual_seed(7)
    for k in range(3):
        fmap.e[k].normal_(generator=gen)
    ext = torch.tensor([h[k] * (grid[k] - 1) for k in range(3)], dtype=torch.float64, device="cuda")
    x = torch.tensor(lo, dtype=torch.float64, device="cuda") + ext * (
        1.04 * torch.rand(n, 3, dtype=torch.float64, device="cuda", generator=gen) - 0.02)
    E = B.field_map_eval(ctx, fmap, x)
    assert torch.equal(E[: n - 1], B.field_map_eval(ctx, fmap, x[: n - 1]))
    assert torch.equal(E[-999:], B.field_map_eval(ctx, fmap, x[-999:]))
    ref = orc.trilinear(host(fmap.values()), lo, h, host(x[:500]))
    assert np.abs(host(E[:500]) - ref).max() <= 1e-12 * np.abs(ref).max()
    v = torch.randn(n, 3, dtype=torch.float64, device="cuda", generator=gen)
    sp = torch.randint(0, 3, (n,), device="cuda", generator=gen).to(torch.int8)
    cur, terms = B.induced_current(ctx, x, v, sp, fmap=fmap, want_terms=True)
    cur2, terms2 = B.induced_current(ctx, x[: n - 1], v[: n - 1], sp[: n - 1], fmap=fmap, want_terms=True)
    assert torch.equal(terms[: n - 1], terms2)
    last = float(terms[-1])
    scale = float(terms.abs().sum())
    for k in range(3):
        assert abs(cur[k] - cur2[k] - (last if int(sp[-1]) == k else 0.0)) <= 1e-13 * scale


def test_point_layouts(ctx):
    """Points in any layout that has the three coordinates along dimension 1
    (contiguous, column-major, strided, with further columns, as columns of a
    3-d tensor) give the same field."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    for n in (1, 2, 65):
        x = 1e-4 * torch.rand(n, 3, dtype=torch.float64, device="cuda", generator=gen)
        q = torch.full((n,), -W.E_CHARGE, dtype=torch.float64, device="cuda")
        wide = torch.rand(2 * n, 5, dtype=torch.float64, device="cuda", generator=gen)
        wide[::2, :3] = x
        E = B.field_eval(ctx, None, None, x, q, x, 1e-7, B.OBEM_FP64, tgt_is_src=True)
        assert E.shape == (n, 3) and E.is_contiguous()
        for y in (x.t().contiguous().t(), wide[::2], wide[::2, :3], x[:, :, None]):
            assert torch.equal(E, B.field_eval(ctx, None, None, y, q, y, 1e-7, B.OBEM_FP64, tgt_is_src=True))
        with pytest.raises(IndexError):
            B.field_eval(ctx, None, None, x[:, :2], q, x, 1e-7)


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 1024, 1025, 4095, 4096, 4097, 5000])
@pytest.mark.parametrize("kind", ["spread", "same_cell", "line"])
def test_orderings(ctx, orc, n, kind):
    """Source copy and target order of small and larger sets (around 128,
    1,024 and 4,096 points): many points in one cell of the curve's
    grid (ties keep the caller's order), on a line, charges of both signs and
    zero, through the field with separate targets, against the oracle, and
    the same bit for bit in a second call."""
    rng = np.random.default_rng(n)
    x = rng.uniform(size=(n, 3)) * 1e-4
    if kind == "same_cell":
        x[n // 3:] = x[0] + 1e-9 * rng.uniform(size=(n - n // 3, 3))
    elif kind == "line":
        x[:, 1:] = 2e-5
    q = rng.choice([-W.E_CHARGE, 0.0, W.E_CHARGE], size=n)
    xt = rng.uniform(size=(n, 3)) * 1e-4
    ref, vref = orc.pair_field(xt, x, q, 1e-6, want_v=True)
    for prec, tol in ((B.OBEM_FP64, 1e-12), (B.OBEM_MIXED, 1e-5)):
        E, V = B.field_eval(ctx, None, None, dev(x), dev(q), dev(xt), 1e-6, prec, want_v=True)
        E2, V2 = B.field_eval(ctx, None, None, dev(x), dev(q), dev(xt), 1e-6, prec, want_v=True)
        assert torch.equal(E, E2) and torch.equal(V, V2)
        assert np.abs(host(E) - ref).max() <= tol * max(np.abs(ref).max(), 1e-300)


@pytest.mark.parametrize("n_t,n_s", [(3, 70001), (1025, 20001), (4097, 257)])
def test_splits_of_few_targets(ctx, orc, n_t, n_s):
    """Target counts on both sides of the slot rule (up to 4 tiles of 256, to
    16, more) with many cells and sources: field, potential, gradients and
    FP64 influence on a sample against the oracle, at the field tests'
    tolerances."""
    m = W.gem_cell_mesh(W.GemGeometry(m=3, n_r=2, n_cone=2, plain_h=48e-6))
    rng = np.random.default_rng(n_t)
    xt = W.gem_cell_points(n_t, seed=n_t)
    xs, q, _ = W.gaussian_clouds(n_s - n_s // 3, n_s // 3, (0, 0, 230e-6), (0, 0, 210e-6), 50e-6, rng)
    sig = 1e-6 * rng.normal(size=m.n)
    w = rng.normal(size=(n_t, 3))
    bm = bind(ctx, m)
    at = np.concatenate([[0, n_t - 1], rng.choice(n_t, 1)])
    Er, Vr = orc.panel_field(xt[at], m.a, m.b, m.c, sig, want_v=True)
    Ep, Vp = orc.pair_field(xt[at], xs, q, 1e-7, want_v=True)
    for prec, tol in ((B.OBEM_FP64, 1e-12), (B.OBEM_MIXED, 1e-5)):
        E, V = B.field_eval(ctx, bm, dev(sig), dev(xs), dev(q), dev(xt), 1e-7, prec, want_v=True)
        assert rel_l2(host(E)[at], Er + Ep) <= tol
        assert rel_l2(host(V)[at], Vr + Vp) <= tol
        # g_sigma is linear in the weights: sum_k sigma_k g_sigma_k = sum w . E_cells
        gs, gt, gsrc = B.field_eval_backward(ctx, bm, dev(sig), dev(xs), dev(q), dev(xt), 1e-7, dev(w), prec)
        Ec = B.field_eval(ctx, bm, dev(sig), None, None, dev(xt), 1e-7, prec)
        lhs, rhs = float((dev(sig) * gs).sum()), float((dev(w) * Ec).sum())
        assert abs(lhs - rhs) <= tol * float((dev(w) * Ec).abs().sum())
        # translating charges and targets together leaves the pairwise term: g_t + g_s of it sum to 0
        _, gt0, gs0 = B.field_eval_backward(ctx, None, None, dev(xs), dev(q), dev(xt), 1e-7, dev(w), prec)
        s = (gt0.sum(0) + gs0.sum(0)).abs().max()
        assert float(s) <= 10 * tol * float(gt0.abs().sum())
    out = host(B.bem_influence(ctx, bm, dev(m.rhs), dev(xs[:n_t]), dev(q[:n_t]), B.OBEM_FP64))
    ref = orc.influence(m, m.rhs, xs[:n_t], q[:n_t])
    ref = ref[0] if isinstance(ref, tuple) else ref
    assert np.abs(out - ref).max() <= 1e-11 * np.abs(ref - m.rhs).max() + 1e-15 * np.abs(m.rhs).max()


@pytest.mark.parametrize("n_s", [1, 63, 64, 65, 1023, 1025, 2100])
@pytest.mark.parametrize("n_c", [1, 7, 9, 130])
def test_influence_remainders(ctx, orc, n_s, n_c):
    """Cells not a multiple of the 8 (2) of a workgroup (wave), charges around
    the runs of 64 and the blocks of 1,024, near, at zone bounds of and far
    from the cells, in both precisions (tolerances of the influence tests)."""
    m = _first_cells(W.parallel_plate_mesh(n=12), n_c)
    rng = np.random.default_rng(n_s + n_c)
    x, q = W.parallel_plate_electrons(n_s, seed=n_s)
    x[: n_s // 2] *= 0.2                     # a dense half near one corner of the cells
    x[: n_s // 2, 2] += 1e-4
    x[:, :2] += rng.choice([0.0, -5e-3, 4e-2], size=(n_s, 1))
    ref = orc.influence(m, m.rhs, x, q)[0]
    scale = np.abs(ref - m.rhs).max()
    bm = bind(ctx, m)
    for prec, tol in ((B.OBEM_FP64, 1e-11), (B.OBEM_MIXED, 1e-5)):
        out = host(B.bem_influence(ctx, bm, dev(m.rhs), dev(x), dev(q), prec))
        assert np.abs(out - ref).max() <= tol * scale + 4e-16 * np.abs(m.rhs).max()


@pytest.mark.parametrize("n", [1, 65, 257])
@pytest.mark.parametrize("spread", [2e-6, 60e-6])
def test_close_pairs_of_the_adjoint(ctx, orc, n, spread):
    """The cell adjoint at targets in a hole of the coarse GEM cell (cells near
    a few or most targets of a wave, batches that fill and end part full,
    cells seen by several waves), both gradients against the oracle at the
    adjoint tests' tolerances."""
    geo = W.GemGeometry(m=3, n_r=2, n_cone=2, plain_h=48e-6)
    m = W.gem_cell_mesh(geo)
    rng = np.random.default_rng(100 + n)
    cx, cy = geo.hole_centres()[4]
    x = np.array([cx + 0.8 * geo.r_inner, cy, 3e-6]) + rng.uniform(-1, 1, size=(n, 3)) * np.array([0.2, 0.2, 1.0]) * spread
    w = rng.normal(size=(n, 3))
    mesh = W.Mesh(m.a, m.b, m.c, m.kind, m.eps1, m.eps2, m.rhs)
    sig = 1e-6 * (1.0 + rng.uniform(size=m.n))
    gs_r, gx_r = orc.panel_backward(x, mesh, sig, w)
    bm = bind(ctx, m)
    for prec, tol in ((B.OBEM_FP64, 1e-10), (B.OBEM_MIXED, 1e-5)):
        gs, gx, _ = B.field_eval_backward(ctx, bm, dev(sig), None, None, dev(x), 0.0, dev(w), prec)
        assert rel_l2(host(gs), gs_r) <= tol
        assert rel_l2(host(gx), gx_r) <= tol


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129])
@pytest.mark.parametrize("ratio", [49.0, 300.0])
def test_far_cells_in_fp64(ctx, orc, n, ratio):
    """Cells beyond 48 diameters only, thin ones seen along their length (the
    far kernel's series at the end of its range) and ordinary ones, cell counts
    around its tile of 64.  The rule it sums is exact to degree 5: off by at
    most (0.67 / 48)^6 = 7e-12 of a cell's field, and the closed form of the
    reference loses no more at 300 diameters."""
    rng = np.random.default_rng(n)
    a = rng.uniform(-1e-7, 1e-7, size=(n, 3))
    t = rng.normal(size=(n, 3))
    t[0] = [1.0, 0.0, 0.0]
    t /= np.linalg.norm(t, axis=1, keepdims=True)
    s = np.cross(t, rng.normal(size=(n, 3)))
    s /= np.linalg.norm(s, axis=1, keepdims=True)
    b = a + 1e-6 * t
    c = a + 1e-6 * (rng.uniform(0.0, 0.9, size=(n, 1)) * t + rng.uniform(0.01, 0.4, size=(n, 1)) * s)
    z = np.zeros(n)
    m = W.Mesh(a, b, c, z.astype(np.int32), z + 1.0, z + 1.0, z, name="far")
    sig = rng.uniform(1e-7, 2e-7, size=n)
    d = rng.normal(size=(70, 3))
    d[:2] = [[1.0, 0.0, 0.0], [-1.0, 0.0, 0.0]]
    x = ratio * 1.04e-6 * d / np.linalg.norm(d, axis=1, keepdims=True)
    E, V = B.field_eval(ctx, bind(ctx, m), dev(sig), None, None, dev(x), 0.0, B.OBEM_FP64, want_v=True)
    Er, Vr = orc.panel_field(x, a, b, c, sig, want_v=True)
    assert rel_l2(host(E), Er) <= 1e-11
    assert rel_l2(host(V), Vr) <= 1e-11


@pytest.mark.parametrize("dt", [1e-13, 3e-12, 2e-11, 2e-10])
def test_chords_through_the_grid(ctx, orc, dt):
    """Free flights of electrons from 0.2 um to 400 um long through the coarse
    GEM cell (chords within one grid cell, over several, and over more than
    the 4096 beyond which every cell is tested): who is absorbed, and in which
    cell the charge lands, as the oracle finds it."""
    m = W.gem_cell_mesh(W.GemGeometry(m=3, n_r=2, n_cone=2, plain_h=48e-6))
    geo = W.GemGeometry()
    gas = W.constant_nu_gas(0.0)
    rng = np.random.default_rng(11)
    n = 700
    top = geo.t_kapton / 2 + geo.t_cu
    x = rng.uniform(-1, 1, size=(n, 3)) * np.array([0.9 * geo.half_x, 0.9 * geo.half_y, 1.2 * top])
    v = rng.normal(size=(n, 3))
    v *= 2e6 / np.linalg.norm(v, axis=1, keepdims=True)
    sp, ids = np.zeros(n, np.int8), np.arange(n, dtype=np.int64)
    p = dict(dt=dt, step=0, seed=5, max_coll=4, max_ion_per_step=1, ion_v_cap=2e4,
             box_lo=(-geo.half_x, -geo.half_y, -3e-3), box_hi=(geo.half_x, geo.half_y, 3e-3), soft=1e-7, r_rec=0.0,
             capacity=n, precision=B.OBEM_FP64, resolve=0, stepper=0)
    state, _, counts, so, _ = orc.track_step(dict(x=x, v=v, species=sp, id=ids, next_id=n), m, np.zeros(m.n), gas, p,
                                             np.zeros(m.n, np.int64), rhs0=m.rhs)
    parts = B.Particles(n, "cuda", dev(x), dev(v), dev(sp, torch.int8), dev(ids, torch.int64), n)
    counts_g = torch.zeros(m.n, dtype=torch.int64, device="cuda")
    gas_s, keep = B.gas_struct(gas, "cuda")
    sg = B.track_step(ctx, bind(ctx, m), parts, gas_s, p, counts_g, dev(np.zeros(m.n)), dev(m.rhs))
    assert so["absorbed"] > 0 or dt < 1e-12
    assert sg["absorbed"] == so["absorbed"]
    assert np.array_equal(host(counts_g), counts)
    assert np.array_equal(host(parts.state()["id"]), state["id"])


@pytest.mark.parametrize("n", [256, 257, 271, 4096, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("kind", ["spread", "same_cell", "line"])
def test_counted_places(ctx, orc, n, kind):
    """Orderings around the sizes of the counted places (above 256 points, 16 a
    workgroup, 4,096 keys a pass, up to 8,192), distinct and equal keys.  A
    point lost or taken twice changes the potential of equal charges by 1 / n
    of it; FP32 terms are off by at most 17 ulps and a tile's 256 sums by 256:
    2e-5 of the sum of magnitudes (for a potential of one sign, of itself)."""
    rng = np.random.default_rng(n)
    x = rng.uniform(size=(n, 3)) * 1e-4
    if kind == "same_cell":
        x[n // 3:] = x[0] + 1e-9 * rng.uniform(size=(n - n // 3, 3))
    elif kind == "line":
        x[:, 1:] = 2e-5
    q = np.full(n, W.E_CHARGE)
    xt = rng.uniform(size=(n, 3)) * 1e-4
    ref, vref = orc.pair_field(xt, x, q, 1e-6, want_v=True)
    for prec, tol in ((B.OBEM_FP64, 1e-12), (B.OBEM_MIXED, 2e-5)):
        E, V = B.field_eval(ctx, None, None, dev(x), dev(q), dev(xt), 1e-6, prec, want_v=True)
        assert (np.abs(host(V) - vref) / vref).max() <= tol
        # the signs' classes, both jobs of one size, and what the coordinates are worth
        s = np.where(np.arange(n) % 3 == 0, -W.E_CHARGE, W.E_CHARGE)
        _, v2 = orc.pair_field(xt, x, s, 1e-6, want_v=True)
        _, V2 = B.field_eval(ctx, None, None, dev(x), dev(s), dev(xt), 1e-6, prec, want_v=True)
        assert (np.abs(host(V2) - v2) / vref).max() <= tol


@pytest.mark.parametrize("n", [1, 255, 257])
@pytest.mark.parametrize("soft", [0.0, 1e-7])
@pytest.mark.parametrize("same", [False, True])
def test_cells_and_charges_side_by_side(ctx, orc, n, soft, same):
    """Cells and charges in one launch: with and without softening, targets =
    sources or not, with and without the potential, remainders of the target
    tile, against the oracle (tolerances of the field tests)."""
    m = W.parallel_plate_mesh(n=7)
    lo, hi = np.array([m.a.min(0), m.a.max(0)])
    rng = np.random.default_rng(n)
    x = lo + (hi - lo) * rng.uniform(0.2, 0.8, size=(n, 3))
    xs, q = (x, W.E_CHARGE * rng.choice([-1.0, 1.0], size=n)) if same else (
        lo + (hi - lo) * rng.uniform(0.2, 0.8, size=(300, 3)), W.E_CHARGE * rng.choice([-1.0, 1.0], size=300))
    sig = 1e-9 * (1.0 + rng.uniform(size=m.n))
    Er, Vr = orc.panel_field(x, m.a, m.b, m.c, sig, want_v=True)
    Ep, Vp = orc.pair_field(x, xs, q, soft, tgt_is_src=same, want_v=True)
    bm = bind(ctx, m)
    for prec, tol in ((B.OBEM_FP64, 1e-12), (B.OBEM_MIXED, 1e-5)):
        E, V = B.field_eval(ctx, bm, dev(sig), dev(xs), dev(q), dev(x), soft, prec, tgt_is_src=same, want_v=True)
        assert rel_l2(host(E), Er + Ep) <= tol
        assert rel_l2(host(V), Vr + Vp) <= tol
        E = B.field_eval(ctx, bm, dev(sig), dev(xs), dev(q), dev(x), soft, prec, tgt_is_src=same)
        assert rel_l2(host(E), Er + Ep) <= tol


def test_map_eval_captured_first():
    """The first call of a context at a packed size, captured: needs no
    workspace, and every replay gives the eager result bit for bit."""
    n, grid = 1 << 18, (9, 8, 7)
    rng = np.random.default_rng(2)
    x = dev(rng.uniform(-1e-5, 9e-5, size=(n, 3)))
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        eager, held = B.Context(0), B.Context(0)
        fmap = B.FieldMap(lo=(0.0, 0.0, 0.0), h=(1e-5, 1e-5, 1e-5), n=grid)
        for k in range(3):
            fmap.e[k].normal_()
        ref = B.field_map_eval(eager, fmap, x)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            E = B.field_map_eval(held, fmap, x)
        for _ in range(3):
            E.zero_()
            g.replay()
            s.synchronize()
            assert torch.equal(E, ref)
            assert torch.equal(B.field_map_eval(eager, fmap, x), ref)


@pytest.mark.parametrize("n", [255, 256, 257, 8191, 8192, 8193])
@pytest.mark.parametrize("kind", ["spread", "same_cell"])
def test_ordered_sources_as_targets(ctx, orc, n, kind):
    """Targets = sources with the potential around the limits of the three
    orderings (256 and 8,192 points): the source copy, the target order and the
    map from the caller's place to the ordered one, by which a charge leaves
    out itself.  Charges of one sign: a charge lost, taken twice or not left
    out changes a potential by 1 / n of it or, of itself, by more.  Errors are
    measured in that potential; FP32 terms are off by at most 17 ulps and a
    tile's 256 sums by 256: 2e-5."""
    rng = np.random.default_rng(n)
    x = rng.uniform(size=(n, 3)) * 1e-4
    if kind == "same_cell":
        x[n // 3:] = x[0] + 1e-9 * rng.uniform(size=(n - n // 3, 3))
    soft = 1e-6
    for sign in (1.0, np.where(np.arange(n) % 3 == 0, -1.0, 1.0)):
        q = W.E_CHARGE * sign * np.ones(n)
        _, vref = orc.pair_field(x, x, q, soft, tgt_is_src=True, want_v=True)
        scale = vref if np.ndim(sign) == 0 else scale
        for prec, tol in ((B.OBEM_FP64, 1e-12), (B.OBEM_MIXED, 2e-5)):
            _, V = B.field_eval(ctx, None, None, dev(x), dev(q), dev(x), soft, prec, tgt_is_src=True, want_v=True)
            assert (np.abs(host(V) - vref) / scale).max() <= tol
