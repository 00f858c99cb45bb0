"""GPU parity of the paths that sizes and shapes choose: the matrix-core (de)gridder of FP32
plans at the edges of its blocks of 32 visibilities, over w ranges that need every length of
its w series or the general kernels, over data of very different scales and with infinities;
sparse plans' degridder; groups gridded in parts; and the image level's row and column passes.

Bar (tests/gates.py): FP32 <= 1e-5, FP64 <= 1e-10, normwise and for the worst element.
"""
import dataclasses

import numpy as np
import pytest

import synth
from gates import check_grid, check_vis

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = {0: 1e-5, 1: 1e-10}


@pytest.fixture(scope="module")
def aidg():
    import paper_2502_17789_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m.library()
    return m


def dev(x, prec=0):
    return torch.from_numpy(np.ascontiguousarray(x, np.complex128 if prec else np.complex64)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.complex128)


def plan_for(aidg, wl, table=None, precision=0, **kw):
    geo = aidg.Geometry(wl.grid_size, wl.subgrid_size, wl.kernel_support, wl.pixel_scale,
                        aterm_interval=wl.aterm_interval, precision=precision, **kw)
    return aidg.Plan(geo, wl.n_stations, wl.baselines, wl.uvw, wl.freqs, dev(wl.aterms, precision), table=table)


def short_baselines(L, n_t, n_c, n_st=3, seed=31, diameter_m=12.0):
    """Baselines of a few cells: one subgrid per baseline holds all times and channels."""
    return synth.config_tiny(seed, n_st=n_st, n_t=n_t, n_c=n_c, N=4 * L, L=L, K=L // 4, diameter_m=diameter_m,
                             aterm_interval=n_t, f_lo=149e6, f_hi=151e6)


def both_ways(aidg, orc, wl, V, rng, tag, tol=1e-5, **kw):
    """Grid and degrid through the plan's own partition against the oracle on that table."""
    with plan_for(aidg, wl, **kw) as p:
        table = p.subgrids()
        G = synth.random_grid(p.n_wlayers, wl.grid_size, rng)
        got_g, got_v = host(p.grid(dev(V))), host(p.degrid(dev(G)))
    check_grid(got_g, orc.grid(wl, V, table), tol, tag + " grid")
    check_vis(got_v, orc.degrid(wl, G, table), tol, tag + " degrid")
    return table


@pytest.mark.parametrize("L", [32, 64, 96])
@pytest.mark.parametrize("n_t,n_c", [(1, 1), (1, 8), (3, 3), (1, 31), (4, 8), (3, 11), (8, 8), (5, 13), (33, 32)])
def test_block_edges(aidg, orc, L, n_t, n_c):
    wl = short_baselines(L, n_t, n_c)
    rng = np.random.default_rng(n_t * n_c)
    V = synth.random_vis((wl.n_baselines, n_t, n_c), rng)
    table = both_ways(aidg, orc, wl, V, rng, f"L {L}, {n_t} x {n_c}", max_subgrid_vis=2048)
    assert (table["nt"] * table["nc"]).max() == n_t * n_c
    with plan_for(aidg, wl, table=table, max_subgrid_vis=2048) as p:
        G = dev(synth.random_grid(p.n_wlayers, wl.grid_size, rng))
        auto, image = host(p.degrid(G)), host(p.grid(dev(V)))
    # the automatic choice against plans that ask for the general kernels
    with plan_for(aidg, wl, table=table, max_subgrid_vis=2048, reseed_channels=8) as p:
        check_grid(image, host(p.grid(dev(V))), 1e-5, "R = 8 grid")
        check_vis(auto, host(p.degrid(G)), 1e-5, "R = 8 degrid")
    for form in (aidg.DEGRID_RECURRENCE, aidg.DEGRID_DIRECT):
        with plan_for(aidg, wl, table=table, max_subgrid_vis=2048, degrid_form=form) as p:
            check_vis(auto, host(p.degrid(G)), 1e-5, f"form {form}")


@pytest.mark.parametrize("L", [32, 96])
@pytest.mark.parametrize("w", [0.0, 0.3, 3.0, 15.0, 50.0, 150.0, 1e3, 3e5])
@pytest.mark.parametrize("w_mid", [0.0, 1.0])
def test_w_ranges(aidg, orc, L, w, w_mid):
    """Rows at w from (w_mid - 1/2) w to (w_mid + 1/2) w wavelengths in one layer."""
    wl = short_baselines(L, 8, 4)
    uvw = wl.uvw.copy()
    uvw[..., 2] = np.linspace(w_mid - 0.5, w_mid + 0.5, 8) * w * 2.0
    wl = dataclasses.replace(wl, uvw=uvw)
    rng = np.random.default_rng(5)
    V = synth.random_vis((wl.n_baselines, 8, 4), rng)
    both_ways(aidg, orc, wl, V, rng, f"L {L}, w {w} about {w_mid}", w_step=-1.0)


@pytest.mark.parametrize("L", [32, 64])
@pytest.mark.parametrize("rows", ["rising", "falling", "zeros first", "tiny", "huge"])
def test_data_scales(aidg, orc, L, rows):
    """Blocks of one subgrid at different scales (the FP16 split has one scale per subgrid so far)."""
    wl = short_baselines(L, 12, 16)
    rng = np.random.default_rng(6)
    V = synth.random_vis((wl.n_baselines, 12, 16), rng)
    f = {"rising": 2.0 ** np.linspace(-60, 20, 12), "falling": 2.0 ** np.linspace(30, -40, 12),
         "zeros first": np.r_[np.zeros(6), np.ones(6)], "tiny": np.full(12, 2.0 ** -100),
         "huge": np.full(12, 2.0 ** 90)}[rows]
    V *= f[None, :, None, None]
    with plan_for(aidg, wl) as p:
        table = p.subgrids()
        got = host(p.grid(dev(V)))
        check_grid(got, orc.grid(wl, V, table), 1e-5, f"L {L} {rows}")
        scale = f.max()
        G = synth.random_grid(p.n_wlayers, wl.grid_size, rng) * scale
        check_vis(host(p.degrid(dev(G))), orc.degrid(wl, G, table), 1e-5, f"L {L} {rows} degrid")


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_bad_values_stay_in_their_subgrids(aidg, bad):
    """A NaN or infinite visibility reaches its group's window, a grid cell the subgrids whose
    windows hold it, and nothing else changes."""
    wl = synth.config_tiny(41, n_st=7, n_t=6, n_c=8, N=256, diameter_m=300.0)
    rng = np.random.default_rng(8)
    V = synth.random_vis((wl.n_baselines, 6, 8), rng)
    L, N = wl.subgrid_size, wl.grid_size
    with plan_for(aidg, wl, center_lattice=8) as p:
        t = p.subgrids()
        s = t[len(t) // 2]
        Vb = V.copy()
        Vb[s["bl"], s["t0"], s["c0"]] = bad
        Vz = V.copy()
        Vz[s["bl"], s["t0"], s["c0"]] = 0
        got, ref = host(p.grid(dev(Vb))), host(p.grid(dev(Vz)))
        out = np.ones(got.shape, bool)
        out[s["wlayer"], :, s["V0"] - L // 2:s["V0"] + L // 2, s["U0"] - L // 2:s["U0"] + L // 2] = False
        assert out.any() and np.isfinite(got[out]).all()
        check_grid(got[out], ref[out], 1e-6, "outside the window")
        G = synth.random_grid(p.n_wlayers, N, rng).astype(np.complex64)
        ref = host(p.degrid(dev(G)))
        Gb = G.copy()
        Gb[s["wlayer"], 0, s["V0"], s["U0"]] = bad
        got = host(p.degrid(dev(Gb)))
        inside = 0
        for r in t:
            hit = (r["wlayer"] == s["wlayer"] and abs(r["V0"] - s["V0"]) <= L // 2 and abs(r["U0"] - s["U0"]) <= L // 2)
            inside += hit
            if not hit:
                block = np.s_[r["bl"], r["t0"]:r["t0"] + r["nt"], r["c0"]:r["c0"] + r["nc"]]
                np.testing.assert_array_equal(got[block], ref[block])
        assert 0 < inside < len(t)


@pytest.mark.parametrize("L,precision,stokes", [(32, 0, 0), (32, 1, 0), (32, 0, 1), (64, 0, 0), (96, 0, 0), (96, 1, 1)])
def test_groups_in_parts(aidg, orc, L, precision, stokes):
    """Few centres with many subgrids each: the plan grids them in parts; a workspace of two
    images and the executor over ranges that cut groups and parts give the same grid."""
    wl = short_baselines(L, 2, 5, n_st=20, seed=33, diameter_m=2.0 * L)
    rng = np.random.default_rng(9)
    V = synth.random_vis((wl.n_baselines, 2, 5), rng)
    image = 4 * L * L * (16 if precision else 8)
    with plan_for(aidg, wl, precision=precision, stokes_i=stokes, center_lattice=L // 4) as p:
        info, table = p.info, p.subgrids()
        assert info["n_batches"] == 1 and info["workspace_bytes"] > info["n_groups"] * image  # in parts
        got = host(p.grid(dev(V, precision)))
        cuts = [0, 3, len(table) // 3, len(table) // 2 + 1, len(table)]
        for budget in (2 * image, 64 << 20):
            ex = aidg.Executor(workspace_bytes=budget)
            try:
                out = torch.zeros(p.grid_shape(), dtype=torch.complex128 if precision else torch.complex64, device="cuda")
                ex.execute([(p, aidg.DIR_GRID, dev(V, precision), out, a, b) for a, b in zip(cuts[:-1], cuts[1:])])
                check_grid(host(out), got, 1e-12 if precision else 1e-6, f"executor, {budget} bytes")
            finally:
                ex.close()
    ref = orc.grid(wl, V, table)
    if stokes:
        ref = 0.5 * (ref[:, 0:1] + ref[:, 3:4])
    check_grid(got, ref, TOL[precision], f"L {L}, {info['n_groups']} groups of {len(table)}")
    with plan_for(aidg, wl, table=table, precision=precision, stokes_i=stokes, center_lattice=L // 4,
                  workspace_bytes=2 * image) as p:
        assert p.info["n_batches"] > 1
        check_grid(host(p.grid(dev(V, precision))), got, 1e-12 if precision else 1e-6, "two images at a time")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N", [50, 90, 486, 1458, 2000, 2048, 2160, 3000])
def test_image_passes(aidg, orc, N, precision):
    """Rows that are and are not a multiple of a strip, of the longest strip and beyond (column
    steps of every number of passes), Stokes-I and four planes, two layers."""
    wl = synth.config_tiny(51, n_st=3, n_t=2, n_c=2, N=N, diameter_m=60.0, ha0_deg=-60.0)
    stokes = int(N > 500)
    rng = np.random.default_rng(N)
    L, K, P = wl.subgrid_size, wl.kernel_support, 1 if stokes else 4
    with plan_for(aidg, wl, precision=precision, stokes_i=stokes, w_step=4.0) as p:
        w0 = p.wlayers()
        G = rng.standard_normal((p.n_wlayers, P, N, N)) + 1j * rng.standard_normal((p.n_wlayers, P, N, N))
        got_i = host(p.invert(dev(G, precision)))
        got_g = host(p.predict(dev(G[0], precision)))
    check_grid(got_i, orc.invert(G, w0, L, K, wl.pixel_scale), TOL[precision], f"{N} invert, {len(w0)} layers")
    check_grid(got_g, orc.predict(G[0], w0, L, K, wl.pixel_scale), TOL[precision], f"{N} predict")
