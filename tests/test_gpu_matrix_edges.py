"""The matrix-core (de)gridder of FP32 plans where its fixed-size arithmetic could end: byte
offsets of long, wide visibility tables.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def aidg():
    import paper_2502_17789_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m.library()
    return m


def test_rows_beyond_4_gib(aidg):
    """One sub-table of 2048 rows in the last of 65600 channels: its last rows start beyond 2^32
    bytes.  The same rows as a table of that one channel give the same visibilities bit for bit
    (one subgrid, one order of sums) and the same grid."""
    n_t, n_c, L, N = 2048, 65600, 32, 128
    wl = synth.config_tiny(31, n_st=2, n_t=n_t, n_c=1, N=N, L=L, K=8, diameter_m=12.0, aterm_interval=n_t,
                           f_lo=150e6, f_hi=150e6)
    freqs = np.linspace(100e6, wl.freqs[0], n_c)
    freqs[-1] = wl.freqs[0]
    A = torch.from_numpy(wl.aterms.astype(np.complex64)).cuda()
    geo = aidg.Geometry(N, L, 8, wl.pixel_scale, aterm_interval=n_t, w_step=-1.0, max_subgrid_vis=2048)
    table = np.zeros(1, aidg.SUBGRID_DTYPE)
    table["st1"], table["st2"] = wl.baselines[0]
    table["nt"], table["nc"], table["U0"], table["V0"] = n_t, 1, N // 2, N // 2
    wide = table.copy()
    wide["c0"] = wide["vis_offset"] = n_c - 1
    g = torch.Generator(device="cuda").manual_seed(3)
    v = torch.randn((1, n_t, 1, 4), dtype=torch.complex64, device="cuda", generator=g)
    G = torch.randn((1, 4, N, N), dtype=torch.complex64, device="cuda", generator=g)
    with aidg.Plan(geo, 2, wl.baselines, wl.uvw, freqs[-1:], A, table=table) as p:
        ref_v, ref_g = p.degrid(G), p.grid(v)
    with aidg.Plan(geo, 2, wl.baselines, wl.uvw, freqs, A, table=wide) as p:
        got = p.degrid(G)
        assert torch.equal(got[:, :, -1:], ref_v)
        assert not got[:, :, :-1].any()
        vw = torch.zeros((1, n_t, n_c, 4), dtype=torch.complex64, device="cuda")
        vw[:, :, -1:] = v
        assert torch.equal(p.grid(vw), ref_g)
