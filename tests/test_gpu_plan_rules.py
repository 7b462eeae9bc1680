"""The plan's automatic choice of pair kernels against one target per
wavefront, bit for bit, on both sides of the sizes and densities where the
choice changes (whole numbers and FP32 distances of identical squared
distances: no tolerance)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ANY = 255


def _box(torch, n, frac, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    L = (n / 30.0) ** (1.0 / 3.0)
    xyz = torch.rand((n, 3), generator=g, device="cuda") * L
    lab = (torch.rand(n, generator=g, device="cuda") < frac).to(torch.uint8)
    d = torch.minimum(xyz, L - xyz).amin(1).contiguous()
    return xyz, lab, d


def _both(aptstat, f):
    out = []
    try:
        for policy in (0, 1):
            aptstat.set_tuning(tile_policy=policy)
            out.append(f())
    finally:
        aptstat.set_tuning()
    return out


@pytest.mark.parametrize("n,frac,A,B,k,r_max,d_srf", [
    # neighbours as dense as the targets, around 2^17 and 2^18 targets; equal and nearly equal sets
    ((1 << 17) - 1, 0.5, ANY, ANY, 0, 2.0, 0.0), (1 << 17, 0.5, ANY, ANY, 0, 2.0, 0.0),
    ((1 << 18) + 7, 0.5, ANY, ANY, 10, 2.0, 0.0), ((1 << 18) + 9000, 0.5, ANY, ANY, 16, 1.3, 0.05),
    # few candidates (tiles), and just too many for them, without and with a kNN
    (300_000, 0.01, ANY, 1, 0, 2.0, 0.0), (300_000, 0.03, ANY, 1, 0, 2.0, 0.0),
    (300_000, 0.03, ANY, 1, 10, 2.0, 0.0), (300_000, 0.06, ANY, 1, 10, 2.0, 0.0),
    (4_000, 0.02, ANY, 1, 4, 2.0, 0.0), (270_000, 0.2, ANY, 1, 3, 2.0, 0.0),
])
def test_automatic_mode_equals_one_target_per_wavefront(n, frac, A, B, k, r_max, d_srf):
    import torch

    import paper_2004_05188_amd as aptstat

    print(f"case plan rule n={n} frac={frac} A={A} B={B} k={k} r_max={r_max}", flush=True)
    xyz, lab, d = _box(torch, n, frac, n)
    cloud = aptstat.Cloud(xyz, lab, d)
    ws = aptstat.Workspace()
    if k == 0:
        a, b = _both(aptstat, lambda: aptstat.rdf(cloud, A, B, d_srf, r_max, 200, ws=ws).cpu().numpy())
        assert np.array_equal(a, b) and a.sum() > 0
        return
    a, b = _both(aptstat, lambda: aptstat.knn_rdf(cloud, A, B, d_srf, k, r_max=r_max, ws=ws))
    for x, y in zip((*a.trimmed(), a.knn_hist, a.rdf_hist, a.status), (*b.trimmed(), b.knn_hist, b.rdf_hist, b.status)):
        assert torch.equal(x, y)
    assert int(a.rdf_hist.sum()) > 0


@pytest.mark.parametrize("A,B,k", [(0, 1, 10), (1, 0, 0), (1, 1, 5), (ANY, ANY, 0)])
def test_counting_and_radix_sort_agree(A, B, k):
    """The largest cloud of the counting sort, and one ion more (of a species in no query, or without a finite
    position): the radix sort bins the same ions and every result is the same."""
    import torch

    import paper_2004_05188_amd as aptstat

    n = 1 << (19 if ANY in (A, B) else 20)
    print(f"case counting sort n={n} A={A} B={B} k={k}", flush=True)
    xyz, lab, d = _box(torch, n, 0.02, 5)
    more = torch.full((1, 3), float("nan") if A == ANY else 3.0, device="cuda")
    big = (torch.cat([xyz, more]), torch.cat([lab, torch.full((1,), 7, dtype=torch.uint8, device="cuda")]),
           torch.cat([d, torch.ones(1, device="cuda")]))
    ws = aptstat.Workspace()
    r = []
    for c in ((xyz, lab, d), big):
        cloud = aptstat.Cloud(*c)
        if k == 0:
            r.append((aptstat.rdf(cloud, A, B, 0.5, 2.0, 200, ws=ws),))
        else:
            q = aptstat.knn_rdf(cloud, A, B, 0.5, k, ws=ws)
            r.append((*q.trimmed(), q.knn_hist, q.rdf_hist, q.status))
    assert int(r[0][-1 if k == 0 else -2].sum()) > 0
    for x, y in zip(*r):
        assert torch.equal(x, y)


@pytest.mark.parametrize("n", [1, 2, 63, 4095, 4096, 4097, 70_001])
def test_counting_sort_sizes(orc, n):
    """Clouds around the scan's tile of 4096 keys, stretched so that there are about as many cells as ions, against
    the oracle."""
    import torch

    import paper_2004_05188_amd as aptstat

    print(f"case counting sort sizes n={n}", flush=True)
    rng = np.random.default_rng(n)
    xyz = (rng.random((n, 3)) * np.array([60.0, 40.0, max(1.0, n / 600.0)])).astype(np.float32)
    lab = (rng.random(n) < 0.3).astype(np.uint8)
    d = rng.random(n).astype(np.float32)
    cloud = aptstat.Cloud(*(torch.from_numpy(v).cuda() for v in (xyz, lab, d)))
    for A, B in ((ANY, ANY), (1, 0), (0, ANY)):
        g = aptstat.knn_rdf(cloud, A, B, 0.25, 6, r_max=2.0, n_bins=100, kb_nbins=500)
        t, dist, nid, h = orc.knn(xyz, lab, d, A, B, 0.25, 6, kb_rmax=5.0, kb_nbins=500)
        tid, gd, gn = (v.cpu().numpy() for v in g.trimmed())
        assert np.array_equal(tid, t) and np.array_equal(gn, nid)
        assert np.allclose(gd, dist, rtol=1e-6, atol=0)
        assert np.array_equal(g.knn_hist.cpu().numpy().astype(np.uint64), h)
        assert np.array_equal(g.rdf_hist.cpu().numpy().astype(np.uint64), orc.rdf(xyz, lab, d, A, B, 0.25, 2.0, 100))


@pytest.mark.parametrize("few", [0, 1, 2, 40, 1500, 9000])
@pytest.mark.parametrize("n", [65, 9_000, 131_073])
def test_counting_sort_with_many_ions_per_key(orc, n, few):
    """Cells sized for `few` ions of one species that all others share: counters 1 to 32 places apart, for the targets
    (few neighbours) or the neighbours (few targets), up to the counters that there are; against the oracle."""
    import torch

    import paper_2004_05188_amd as aptstat

    few = min(few, n)
    print(f"case many ions per key n={n} few={few}", flush=True)
    rng = np.random.default_rng(n + few)
    xyz = (rng.random((n, 3)) * (n / 30.0) ** (1.0 / 3.0)).astype(np.float32)
    lab = np.zeros(n, np.uint8)
    lab[rng.permutation(n)[:few]] = 1
    d = rng.random(n).astype(np.float32)
    cloud = aptstat.Cloud(*(torch.from_numpy(v).cuda() for v in (xyz, lab, d)))
    for A, B in ((0, 1), (1, 0), (1, 1), (ANY, 1)):
        g = aptstat.knn_rdf(cloud, A, B, 0.25, 3, r_max=0.6, n_bins=50, kb_nbins=100)
        t, dist, nid, h = orc.knn(xyz, lab, d, A, B, 0.25, 3, kb_rmax=5.0, kb_nbins=100)
        tid, gd, gn = (v.cpu().numpy() for v in g.trimmed())
        assert np.array_equal(tid, t) and np.array_equal(gn, nid)
        assert np.allclose(gd, dist, rtol=1e-6, atol=0)
        assert np.array_equal(g.knn_hist.cpu().numpy().astype(np.uint64), h)
        assert np.array_equal(g.rdf_hist.cpu().numpy().astype(np.uint64), orc.rdf(xyz, lab, d, A, B, 0.25, 0.6, 50))


@pytest.mark.parametrize("n", [64, 700, 30_011])
@pytest.mark.parametrize("every,axes", [(1, 3), (2, 3), (2, 1), (7, 3)])
def test_counting_sort_without_finite_positions(orc, n, every, axes):
    """Every (second, seventh) ion without a finite position, or without a finite x alone: a wavefront's ranks among
    ions that share a counter, beside finite ones and full wavefronts; against the oracle."""
    import torch

    import paper_2004_05188_amd as aptstat

    print(f"case counting sort not finite n={n} every={every} axes={axes}", flush=True)
    rng = np.random.default_rng(n + every)
    xyz = (rng.random((n, 3)) * (n / 30.0) ** (1.0 / 3.0)).astype(np.float32)
    xyz[::every, :axes] = np.nan
    xyz[0, 0] = -np.inf
    lab = rng.integers(0, 2, n).astype(np.uint8)
    d = rng.random(n).astype(np.float32)
    cloud = aptstat.Cloud(*(torch.from_numpy(v).cuda() for v in (xyz, lab, d)))
    for A, B in ((ANY, ANY), (1, 0)):
        g = aptstat.knn_rdf(cloud, A, B, 0.25, 3, r_max=0.6, n_bins=50, kb_nbins=100)
        t, dist, nid, h = orc.knn(xyz, lab, d, A, B, 0.25, 3, kb_rmax=5.0, kb_nbins=100)
        tid, gd, gn = (v.cpu().numpy() for v in g.trimmed())
        assert int(g.status.item()) == aptstat.STATUS_NONFINITE
        assert np.array_equal(tid, t) and np.array_equal(gn, nid)
        assert np.allclose(gd, dist, rtol=1e-6, atol=0)
        assert np.array_equal(g.knn_hist.cpu().numpy().astype(np.uint64), h)
        assert np.array_equal(g.rdf_hist.cpu().numpy().astype(np.uint64), orc.rdf(xyz, lab, d, A, B, 0.25, 0.6, 50))


@pytest.mark.parametrize("blob", [300, 511, 512, 513, 3000])
def test_tiles_with_many_candidates(orc, blob):
    """Dense targets around a tight ball of `blob` neighbours: tiles just inside and beyond what a stage of 512
    records holds (beyond, their targets are left to the one-by-one pass with RDF and kNN), against the oracle."""
    import torch

    import paper_2004_05188_amd as aptstat

    print(f"case tile candidates blob={blob}", flush=True)
    rng = np.random.default_rng(blob)
    n = 120_000
    L = 16.0
    xyz = (rng.random((n, 3)) * L).astype(np.float32)
    lab = (rng.random(n) < 0.002).astype(np.uint8)
    xyz[:blob] = (L / 2 + 0.2 * rng.standard_normal((blob, 3))).astype(np.float32)
    lab[:blob] = 1
    d = np.full(n, 5.0, np.float32)
    cloud = aptstat.Cloud(*(torch.from_numpy(v).cuda() for v in (xyz, lab, d)))
    for k in (3, 10, 16):
        aptstat.set_tuning(tile_policy=2)
        try:
            g = aptstat.knn_rdf(cloud, 0, 1, 1.0, k, r_max=2.0, n_bins=100, kb_nbins=500)
        finally:
            aptstat.set_tuning()
        t, dist, nid, h = orc.knn(xyz, lab, d, 0, 1, 1.0, k, kb_rmax=5.0, kb_nbins=500)
        tid, gd, gn = (v.cpu().numpy() for v in g.trimmed())
        assert np.array_equal(tid, t) and np.array_equal(gn, nid)
        assert np.allclose(gd, dist, rtol=1e-6, atol=0)
        assert np.array_equal(g.knn_hist.cpu().numpy().astype(np.uint64), h)
        assert np.array_equal(g.rdf_hist.cpu().numpy().astype(np.uint64), orc.rdf(xyz, lab, d, 0, 1, 1.0, 2.0, 100))


@pytest.mark.parametrize("kind", ["sc", "fcc", "bcc"])
@pytest.mark.parametrize("k", [1, 4, 5, 8, 10, 12, 13, 16])
def test_tiles_of_a_lattice(orc, kind, k):
    """Exact lattices, where many neighbours share a distance: the tiles keep a few more than k by their leading bits,
    find that the k-th may tie with one left out and leave the target to an exact search.  Every ion, and a random
    tenth of the sites as neighbours; against the oracle."""
    import torch

    import paper_2004_05188_amd as aptstat

    print(f"case lattice {kind} k={k}", flush=True)
    basis = {"sc": [[0, 0, 0]], "fcc": [[0, 0, 0], [.5, .5, 0], [.5, 0, .5], [0, .5, .5]],
             "bcc": [[0, 0, 0], [.5, .5, .5]]}[kind]
    m = {"sc": 26, "fcc": 16, "bcc": 20}[kind]
    cells = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    xyz = ((cells + np.array(basis)).reshape(-1, 3) * 0.5).astype(np.float32)
    rng = np.random.default_rng(k)
    xyz = xyz[rng.permutation(len(xyz))]
    lab = (rng.random(len(xyz)) < 0.1).astype(np.uint8)
    d = rng.random(len(xyz)).astype(np.float32)
    cloud = aptstat.Cloud(*(torch.from_numpy(v).cuda() for v in (xyz, lab, d)))
    for A, B, r_max in ((ANY, ANY, 0.6), (0, 1, 1.2)):
        aptstat.set_tuning(tile_policy=2)
        try:
            g = aptstat.knn_rdf(cloud, A, B, 0.1, k, r_max=r_max, n_bins=60, kb_nbins=500)
        finally:
            aptstat.set_tuning()
        t, dist, nid, h = orc.knn(xyz, lab, d, A, B, 0.1, k, kb_rmax=5.0, kb_nbins=500)
        tid, gd, gn = (v.cpu().numpy() for v in g.trimmed())
        assert np.array_equal(tid, t) and np.array_equal(gn, nid)
        assert np.allclose(gd, dist, rtol=1e-6, atol=0)
        assert np.array_equal(g.knn_hist.cpu().numpy().astype(np.uint64), h)
        assert np.array_equal(g.rdf_hist.cpu().numpy().astype(np.uint64), orc.rdf(xyz, lab, d, A, B, 0.1, r_max, 60))


@pytest.mark.parametrize("n,A,d_srf,n_bins,k", [
    (1 << 18, 1, 0.0, 200, 0), ((1 << 18) + 37, ANY, 0.0, 4000, 0),   # all targets; counters in LDS and global
    (2_000, ANY, 0.1, 200, 0), ((1 << 18) + 1, 1, 0.38, 200, 0), ((1 << 18) + 1, 1, 0.42, 200, 0),   # either side of three targets in five
    ((1 << 19) + 4100, ANY, 0.38, 200, 4), ((1 << 20) + 63, ANY, 0.3, 200, 0),   # chunks split less
])
def test_unordered_pairs_of_one_species(n, A, d_srf, n_bins, k):
    """One species against itself with the neighbour-major RDF (each unordered pair once, weighted by its ends that
    are targets), against one target per wavefront: with ions in the same place, a cell of many chunks, positions
    that are not finite and a last chunk that is not full."""
    import torch

    import paper_2004_05188_amd as aptstat

    print(f"case unordered pairs n={n} A={A} d_srf={d_srf} n_bins={n_bins} k={k}", flush=True)
    xyz, lab, _ = _box(torch, n, 0.9, n)
    g = torch.Generator("cuda").manual_seed(3)
    xyz[:700] = xyz[700] + 0.05 * torch.rand((700, 3), generator=g, device="cuda")
    xyz[1000:1100] = xyz[1100:1200]
    xyz[1500] = float("nan")
    xyz[1501, 1] = float("inf")
    d = torch.rand(n, generator=g, device="cuda")
    cloud = aptstat.Cloud(xyz, lab, d)
    ws = aptstat.Workspace()

    def hist():
        if k:
            return aptstat.knn_rdf(cloud, A, A, d_srf, k, r_max=1.2, n_bins=n_bins, ws=ws).rdf_hist.cpu().numpy()
        return aptstat.rdf(cloud, A, A, d_srf, 1.2, n_bins, ws=ws).cpu().numpy()

    try:
        out = []
        for policy in (4, 1):
            aptstat.set_tuning(tile_policy=policy)
            out.append(hist())
    finally:
        aptstat.set_tuning()
    assert np.array_equal(out[0], out[1]) and out[0].sum() > 0


@pytest.mark.parametrize("n_bins", [1, 200, 2047, 2048, 3072, 4096, 4097])
@pytest.mark.parametrize("r_max", [1.0, float(np.nextafter(np.float32(1.0), np.float32(2.0))), 0.75])
def test_pairs_about_the_last_edge(n_bins, r_max):
    """Pairs at r_max, a rounding step either side of it and up to 1e-4 beyond, whose FP32 bin may be the one after
    the last: every pair kernel against the FP64 distances (whole numbers: no tolerance).  The sizes are the largest
    histograms of each kernel's LDS, and the next."""
    import torch

    import paper_2004_05188_amd as aptstat

    print(f"case last edge n_bins={n_bins} r_max={r_max}", flush=True)
    g = np.mgrid[0:7, 0:7, 0:7].reshape(3, -1).T * 0.25
    rng = np.random.default_rng(n_bins)
    far = np.array([20.0, 0.0, 0.0]) + np.arange(40)[:, None] * np.array([0.0, 8.0, 0.0])
    step = r_max + np.concatenate([np.arange(-10, 10) * 2.0 ** -24, rng.uniform(-1e-4, 1e-4, 20)])
    xyz = np.concatenate([g, far, far + step[:, None] * np.array([0.0, 0.0, 1.0])]).astype(np.float32)
    d = np.sqrt(((xyz[:, None].astype(np.float64) - xyz[None].astype(np.float64)) ** 2).sum(-1))
    d = d[~np.eye(len(xyz), dtype=bool)]
    r = float(np.float32(r_max))
    edges = np.arange(n_bins + 1) * r / n_bins
    b = np.searchsorted(edges, d[d < r], side="right") - 1
    want = np.bincount(np.minimum(b, n_bins - 1), minlength=n_bins)

    cloud = aptstat.Cloud(torch.from_numpy(xyz).cuda(), torch.zeros(len(xyz), dtype=torch.uint8, device="cuda"),
                          torch.ones(len(xyz), device="cuda"))
    ws = aptstat.Workspace()
    try:
        for policy in (0, 1, 2, 3, 4):
            aptstat.set_tuning(tile_policy=policy)
            got = aptstat.rdf(cloud, ANY, ANY, 0.0, r_max, n_bins, ws=ws).cpu().numpy()
            assert np.array_equal(got, want), policy
            got = aptstat.knn_rdf(cloud, ANY, ANY, 0.0, 4, r_max=r_max, n_bins=n_bins, ws=ws).rdf_hist.cpu().numpy()
            assert np.array_equal(got, want), policy
    finally:
        aptstat.set_tuning()


@pytest.mark.parametrize("n,policy,d_srf,r_max,k", [
    ((1 << 17) + 5, 0, 0.0, 2.0, 0), ((1 << 18) + 70, 0, 0.0, 2.0, 10), ((1 << 18) + 70, 0, 0.3, 2.0, 0),
    (5_000, 4, 0.0, 1.0, 0), (63, 4, 0.0, 1.0, 0),
])
def test_candidates_of_one_species_against_itself(n, policy, d_srf, r_max, k):
    """The diagnostic count where the RDF takes unordered pairs (every ion, or the only species, against itself): the
    evaluations of ordered pairs, so the same as for that species against every ion, at least the pairs that the RDF
    counts and at most targets times neighbours."""
    import torch

    import paper_2004_05188_amd as aptstat

    print(f"case candidates of one species n={n} policy={policy} d_srf={d_srf} k={k}", flush=True)
    xyz, _, _ = _box(torch, n, 0.5, n)
    d = torch.rand(n, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    cloud = aptstat.Cloud(xyz, torch.ones(n, dtype=torch.uint8, device="cuda"), d)
    ws = aptstat.Workspace()
    aptstat.set_tuning(tile_policy=policy)
    try:
        got = [int(aptstat.count_candidates(cloud, A, B, d_srf, r_max, 200, k=k, ws=ws).item())
               for A, B in ((ANY, ANY), (1, 1), (1, ANY), (ANY, ANY))]
        pairs = int(aptstat.rdf(cloud, ANY, ANY, d_srf, r_max, 200, ws=ws).sum())
    finally:
        aptstat.set_tuning()
    assert len(set(got)) == 1, got
    assert 0 < pairs <= got[0] <= int((d >= d_srf).sum()) * n
