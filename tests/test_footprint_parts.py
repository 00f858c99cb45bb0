"""The footprint estimate of plans whose gridder takes groups in parts: an image per part."""
import numpy as np
import pytest

import paper_2502_17789_amd as aidg
import synth


def sparse(L):
    """2016 baselines of one visibility on one or two centres: parts of three subgrids, the least."""
    wl = synth.config_tiny(5, n_st=64, n_t=1, n_c=1, N=8 * L, L=L, K=L // 4, diameter_m=30.0)
    return wl, dict(grid_size=wl.grid_size, subgrid_size=L, kernel_support=L // 4, pixel_scale=wl.pixel_scale,
                    aterm_interval=3)


@pytest.mark.parametrize("L", [32, 64])
def test_estimate_holds_the_parts_of_sparse_plans(L):
    wl, kw = sparse(L)
    image = 4 * L * L * 8
    table, _ = aidg.partition(aidg.Geometry(**kw), wl.n_stations, wl.baselines, wl.uvw, wl.freqs)
    assert len(table) == 2016
    whole, one = (aidg.footprint(aidg.Geometry(workspace_bytes=w, **kw), wl.n_stations, wl.baselines, wl.uvw, wl.freqs)
                  for w in (0, image))
    images = (whole["plan_bytes"] - one["plan_bytes"]) // image + 1
    assert len(table) // 3 <= images <= 1.25 * (len(table) // 3)


@pytest.mark.gpu
@pytest.mark.parametrize("L", [32, 64, 96])
def test_estimate_against_the_plan(L):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl, kw = sparse(L)
    geo = aidg.Geometry(**kw)
    A = torch.from_numpy(wl.aterms.astype(np.complex64)).cuda()
    f = aidg.footprint(geo, wl.n_stations, wl.baselines, wl.uvw, wl.freqs)
    with aidg.Plan(geo, wl.n_stations, wl.baselines, wl.uvw, wl.freqs, A) as p:
        info = p.info
    assert info["workspace_bytes"] > 100 * info["n_groups"] * 4 * L * L * 8  # in parts
    assert info["device_bytes"] <= f["plan_bytes"] <= 1.25 * info["device_bytes"]
