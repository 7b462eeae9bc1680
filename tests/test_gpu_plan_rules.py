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
