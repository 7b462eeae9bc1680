"""GPU parity of the ion-to-edge distancing against the oracle, through the
C ABI.

Both sides compute the exact point-triangle distance in FP64 on the stored
FP32 values and round it to FP32, with different formulas (the oracle:
plane distance if the foot lies inside by edge cross products, else the
three edges; the GPU: the foot's barycentric weights in dot-product form);
their FP64 values agree to about 1e-15 relative, so the FP32 results are
equal or one ulp apart (at a rounding tie).  Whether a distance is below
the probe distance d_prb is decided on those FP64 values: ions within 1e-6
relative of d_prb may fall on either side.

Cases: a small needle with its inscribed hull at d_prb = 1, 3 and without a
limit; a box surface with ions inside and outside, around 3000 nm; no
triangles, NaN positions, a triangle with an infinite vertex, zero-area
triangles, n = 0; the 7.7e6-ion needle with a 102 912-triangle hull at the
benchmark's d_prb = 2.5 nm.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def gpu():
    import torch

    import paper_2004_05188_amd as aptstat

    assert torch.cuda.is_available()
    aptstat.lib()
    return aptstat, torch, aptstat.Workspace()


def run_edge(gpu, xyz, tri, d_prb):
    aptstat, torch, ws = gpu
    dev = torch.device("cuda:0")
    xyz = np.ascontiguousarray(xyz, np.float32)
    cloud = aptstat.Cloud(torch.from_numpy(xyz).to(dev), torch.zeros(len(xyz), dtype=torch.uint8, device=dev))
    t = torch.from_numpy(np.ascontiguousarray(tri, np.float32).reshape(-1, 3, 3)).to(dev)
    d, st = aptstat.edge_distance(cloud, t, d_prb, ws=ws)
    torch.cuda.synchronize()
    return d.cpu().numpy(), int(st.item())


def compare(g, o, d_prb):
    assert g.shape == o.shape
    assert np.array_equal(np.isnan(g), np.isnan(o))
    fin = np.isfinite(g) & np.isfinite(o)
    ia, ib = g[fin].view(np.int32).astype(np.int64), o[fin].view(np.int32).astype(np.int64)
    ulps = np.abs(ia - ib)
    assert ulps.max(initial=0) <= 1, f"{np.count_nonzero(ulps > 1)} distances differ by more than one ulp"
    # +inf on one side only: allowed within 1e-6 relative of the probe distance
    one = np.isfinite(g) != np.isfinite(o)
    if one.any():
        v = np.where(np.isfinite(g[one]), g[one], o[one]).astype(np.float64)
        assert np.all(np.abs(v - d_prb) <= 1e-6 * d_prb), v[:5]
    return int(np.count_nonzero(ulps)), int(np.count_nonzero(one))


def check(orc, gpu, xyz, tri, d_prb, expect_status=0, method="grid"):
    g, st = run_edge(gpu, xyz, tri, d_prb)
    assert st == expect_status
    o = orc.edge_distance(xyz, tri, d_prb, method=method)
    return g, compare(g, o, d_prb)


@pytest.fixture(scope="module")
def needle(synth):
    spec = synth.clustered_needle(30.0, 10.0, 6.0, seed=7)
    xyz, _, d_an = spec.generate()
    return spec, xyz, d_an, synth.frustum_mesh(spec, 96, 60)


@pytest.mark.parametrize("d_prb", [1.0, 3.0])
def test_needle_hull(gpu, orc, needle, d_prb):
    _say(f"case edge needle d_prb={d_prb}")
    spec, xyz, d_an, mesh = needle
    g, _ = check(orc, gpu, xyz, mesh, d_prb)
    assert np.isfinite(g).sum() > 10000 and np.isinf(g).sum() > 10000


def test_no_probe_limit(gpu, orc, synth):
    _say("case edge no probe limit")
    spec = synth.clustered_needle(12.0, 5.0, 3.0, seed=3)
    xyz, _, d_an = spec.generate()
    mesh = synth.frustum_mesh(spec, 48, 20)
    g, _ = check(orc, gpu, xyz, mesh, float("inf"), method="brute")
    assert np.isfinite(g).all()
    sag = spec.R0 * (1 - np.cos(np.pi / 48))
    assert np.all(np.abs(g.astype(np.float64) - d_an) <= sag + 1e-4)


def _box_mesh(lo, hi):
    c = np.array([[lo[0] if i & 1 == 0 else hi[0], lo[1] if i & 2 == 0 else hi[1], lo[2] if i & 4 == 0 else hi[2]]
                  for i in range(8)], np.float64)
    quads = [(0, 1, 3, 2), (4, 5, 7, 6), (0, 1, 5, 4), (2, 3, 7, 6), (0, 2, 6, 4), (1, 3, 7, 5)]
    tris = []
    for a, b, cc, d in quads:
        tris += [[c[a], c[b], c[cc]], [c[a], c[cc], c[d]]]
    return np.array(tris, np.float32)


def test_box_far_coordinates(gpu, orc):
    _say("case edge box at 3000 nm")
    lo, hi = np.array([3000.0, -2990.0, 3100.0]), np.array([3012.0, -2981.0, 3105.0])
    mesh = _box_mesh(lo, hi)
    rng = np.random.default_rng(21)
    xyz = rng.uniform(lo - 2.0, hi + 2.0, (200_000, 3)).astype(np.float32)
    for d_prb in (0.75, 2.5, float("inf")):
        g, _ = check(orc, gpu, xyz, mesh, d_prb, method="grid" if np.isfinite(d_prb) else "brute")
    P = xyz.astype(np.float64)
    inside = np.all((P >= lo) & (P <= hi), 1)
    expect = np.where(inside, np.minimum(P - lo, hi - P).min(1),
                      np.sqrt((np.maximum(np.maximum(lo - P, 0.0), P - hi) ** 2).sum(1)))
    assert np.all(np.abs(g.astype(np.float64) - expect) <= 1e-6 * np.maximum(expect, 1e-3) + 1e-9)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 1000])
def test_groups_and_cut_triangles(gpu, orc, n):
    """Ions at the edges of a search group (16 and 64), against triangles far larger than the cloud (cut into many
    pieces), thin fans around one point, a sliver of 1e-4 nm, and a hull the ions lie outside of."""
    _say(f"case edge groups n={n}")
    rng = np.random.default_rng(n)
    xyz = (rng.uniform(-3.0, 3.0, (n, 3)) + np.array([40.0, -10.0, 5.0])).astype(np.float32)
    fan = [[[40, -10, 9], [40 + 30 * np.cos(p), -10 + 30 * np.sin(p), 9], [40 + 30 * np.cos(p + 0.05),
            -10 + 30 * np.sin(p + 0.05), 9]] for p in np.arange(0, 6.25, 0.05)]
    big = [[[-400, -300, -8], [500, -250, -9], [30, 600, -7]], [[47, -300, -300], [47, 400, -200], [47, 40, 500]]]
    thin = [[[36, -40, 0], [36, 60, 0], [36, 10, 1e-4]], [[30, -10, 5], [30.5, -10, 5], [30.25, -9.5, 5]]]
    tri = np.array(fan + big + thin, np.float32)
    for d_prb in (0.5, 4.0, 50.0, float("inf")):
        check(orc, gpu, xyz, tri, d_prb, method="brute")
    far = tri + np.float32(300.0)
    for d_prb in (100.0, float("inf")):
        check(orc, gpu, xyz, far, d_prb, method="brute")


def test_edge_cases(gpu, orc, needle):
    _say("case edge edge cases")
    spec, xyz, d_an, mesh = needle
    sub = xyz[:30000].copy()
    # no triangles: every finite ion at +inf
    g, st = run_edge(gpu, sub, np.zeros((0, 3, 3), np.float32), 2.0)
    assert st == 0 and np.isinf(g).all()
    # NaN positions, a triangle with an infinite vertex, zero-area triangles
    sub[[3, 77]] = np.nan
    m = mesh.copy()
    m[10, 2, 0] = np.inf
    m[11] = m[11, [0, 0, 1]]          # a segment
    m[12] = m[12, [2, 2, 2]]          # a point
    g, _ = check(orc, gpu, sub, m, 2.0, expect_status=1)
    assert np.isnan(g[[3, 77]]).all()
    # no ions
    g, st = run_edge(gpu, np.zeros((0, 3), np.float32), mesh, 2.0)
    assert len(g) == 0 and st == 0


def test_frustum7m_hull(gpu, orc, synth):
    _say("case edge frustum7m, 102 912 triangles, d_prb = 2.5")
    spec = synth.frustum7m()
    xyz, _, d_an = spec.generate()
    mesh = synth.frustum_mesh(spec, 256, 200)
    g, (n_ulp, n_edge) = check(orc, gpu, xyz, mesh, 2.5)
    _say(f"[edge] {np.isfinite(g).sum()} ions within 2.5 nm; {n_ulp} one ulp apart, {n_edge} at d_prb")
    # ions inside the analytic surface (its 0.2 nm noise puts some outside,
    # where the analytic distance is negative): within the chords' sagitta
    sag = spec.R0 * (1 - np.cos(np.pi / 256))
    fin = np.isfinite(g) & (d_an > 0)
    assert fin.sum() > 1_000_000
    assert np.all(np.abs(g[fin].astype(np.float64) - d_an[fin]) <= sag + 1e-4)


@pytest.mark.parametrize("d_prb", [25.0, 33.0, float("inf")])
@pytest.mark.parametrize("dims", [(20.0, 20.0, 20.0), (30.0, 20.0, 10.0), (6.0, 40.0, 17.0)])
def test_triangles_at_the_corners(gpu, orc, dims, d_prb):
    """One small triangle at a corner, an edge or a face of the ions' box, nothing else: the search's reach spans the
    box along every axis before it meets the triangle.  Two triangles too, for groups that meet the farther one
    first."""
    _say(f"case edge corners {dims} d_prb={d_prb}")
    rng = np.random.default_rng(5)
    xyz = (rng.random((700, 3)) * dims).astype(np.float32)
    small = np.array([[0.0, 0.0, 0.0], [0.05, 0.0, 0.0], [0.0, 0.05, 0.0]])
    corners = [np.array([i & 1, i >> 1 & 1, i >> 2]) * dims for i in range(8)]
    places = corners + [np.array([0.5, 1.0, 0.0]) * dims, np.array([0.3, 0.6, 1.0]) * dims]
    for p in [[c] for c in places] + [[corners[0], corners[7]], [corners[1], places[9]]]:
        g, _ = check(orc, gpu, xyz, np.stack([small + q for q in p]).astype(np.float32), d_prb, method="brute")
        assert np.isfinite(d_prb) or np.isfinite(g).all()


@pytest.mark.parametrize("cell_occ", [0.1, 1.0, 4.0, 100.0, 1e6])
def test_tuned_cells(gpu, orc, needle, cell_occ):
    """cell_occ sets the ions' cells, from more cells than ions to one cell for all: the distances stay the same."""
    _say(f"case edge cell_occ={cell_occ}")
    _, xyz, _, mesh = needle
    gpu[0].set_tuning(cell_occ=cell_occ)
    try:
        check(orc, gpu, xyz[:20_000], mesh, 1.5)
    finally:
        gpu[0].set_tuning()


@pytest.mark.parametrize("d_prb", [0.4, float("inf")])
@pytest.mark.parametrize("scale", [1e-3, 1e15, 3e17, 1e18, 3e19, 1e30])
def test_coordinates_whose_squares_overflow(gpu, orc, scale, d_prb):
    """Ions and triangles of any finite size (FP32 squares overflow from 1.8e19): both large, or one triangle among
    others, and alone."""
    _say(f"case edge scale={scale} d_prb={d_prb}")
    rng = np.random.default_rng(8)
    xyz = rng.random((400, 3))
    tri = rng.random((60, 1, 3)) * 1.4 - 0.2 + 0.1 * rng.standard_normal((60, 3, 3))
    far = np.array([[0.3, 0.4, 0.5], [0.35, 0.4, 0.5], [0.3, 0.5, 0.55]])[None] * scale
    for ions, t, unit in ((xyz * scale, tri * scale, scale), (xyz, far, scale), (xyz, np.concatenate([tri, far]), 1.0)):
        reach = float(np.float32(d_prb * unit))
        g, _ = check(orc, gpu, ions.astype(np.float32), t.astype(np.float32), reach, method="brute")
        assert np.isfinite(reach) or np.isfinite(g).all()
