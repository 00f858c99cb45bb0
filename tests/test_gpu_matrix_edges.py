"""The matrix-core (de)gridder of FP32 plans where its fixed-size arithmetic could end: byte
offsets of long, wide visibility tables, and FP16 operands of the w series under isolated
off-axis sources, their range and their rounding; polarisations of very different sizes;
tables of a caller that the library's own partition would not make; and which kernels plans take.
"""
import numpy as np
import pytest

import synth
from gates import check_grid

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def aidg():
    import paper_2502_17789_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m.library()
    return m


LIGHT = 299792458.0


class Track:
    """Baselines of 16 times and 8 channels that stay within a subgrid about the centre, with w
    from -dw to dw wavelengths in one layer, and identity Jones terms."""

    def __init__(self, aidg, L, fov, dw, n_bl=6, w_mid=0.0, nearby=False):
        self.L, self.N, self.fov, K, n_t = L, 4 * L, fov, L // 4, 16
        self.aidg, self.n_st = aidg, n_bl + 1
        rng = np.random.default_rng(7)
        self.freqs = np.linspace(149.9e6, 150.1e6, 8)
        lam = LIGHT / 150e6
        uv = rng.uniform(-0.2, 0.2, (n_bl, 1, 2)) + rng.uniform(-0.1, 0.1, (n_bl, n_t, 2))
        uv *= (L - K) / fov * (0.2 if nearby else 1.0)  # nearby: one subgrid per baseline
        w = w_mid + np.broadcast_to(np.linspace(-1, 1, n_t), (n_bl, n_t)) * dw / 1.001
        self.uvw = np.concatenate([uv, w[..., None]], -1) * lam
        self.bl = np.array([(i, i + 1) for i in range(n_bl)], np.int32)
        self.A = torch.zeros((1, self.n_st, L, L, 4), dtype=torch.complex64, device="cuda")
        self.A[..., 0] = self.A[..., 3] = 1
        beta = np.pi * K / 4
        f = (np.arange(L) - L // 2) / L
        self.taper = np.i0(beta * np.sqrt(1 - 4 * f * f)) / np.i0(beta)
        self.l = f * fov

    def plan(self, precision=0, table=None, **kw):
        g = self.aidg.Geometry(self.N, self.L, self.L // 4, self.fov / self.N, aterm_interval=16, w_step=-1.0,
                               precision=precision, **kw)
        A = self.A.to(torch.complex128) if precision else self.A
        return self.aidg.Plan(g, self.n_st, self.bl, self.uvw, self.freqs, A, table=table)

    def source(self, x, y):
        """Grid of a source of unit XX and YY at subgrid pixel (x, y) as prediction forms it, its
        visibilities by the measurement equation, and its taper."""
        cell = (np.arange(self.N) - self.N // 2) / self.fov
        T = self.taper[x] * self.taper[y]
        l, m = self.l[x], self.l[y]
        g = np.zeros((1, 4, self.N, self.N), np.complex64)
        g[0, 0] = g[0, 3] = np.outer(np.exp(-2j * np.pi * cell * m), np.exp(-2j * np.pi * cell * l)) / (self.L ** 2 * T)
        w = self.uvw[:, :, None, :] * (self.freqs / LIGHT)[:, None]
        n1 = -(l * l + m * m) / (1 + np.sqrt(1 - l * l - m * m))
        return torch.from_numpy(g).cuda(), np.exp(-2j * np.pi * (w[..., 0] * l + w[..., 1] * m + w[..., 2] * n1)), T


def first_term(aidg, L, fov, first, **kw):
    """A track whose series' first term is up to `first` of the tapered field before the constant
    that the plan takes off b (1.7 to 1.8 times less with it)."""
    n1 = lambda r2: -r2 / (1 + np.sqrt(1 - r2))
    t = Track(aidg, L, fov, 0.0)
    l2 = t.l ** 2
    c = n1(l2[:, None] + l2) - n1(l2)[:, None] - n1(l2)
    return Track(aidg, L, fov, first / (2 * np.pi * (np.outer(t.taper, t.taper) * -c).max()), **kw)


# |w| ranges at which the series takes two and three terms; the last is a narrow field
WIDE = [(32, 0.9, 0.085), (32, 0.9, 0.105), (64, 1.0, 0.2), (64, 1.0, 0.6), (96, 1.2, 0.25), (96, 1.2, 0.7),
        (32, 0.1, 6.5e3), (96, 0.1, 6.3e4)]


@pytest.mark.parametrize("L,fov,dw", WIDE)
def test_series_operands_stay_in_range(aidg, L, fov, dw):
    """A lone off-axis source is the largest value of its rows of the subgrid image: the taper does
    not keep the series' operands small.  Predicted grids carry the rounding of FP32 values of
    1 / T, which the degridder's taper leaves at some 1e-7 / T of the source."""
    t = Track(aidg, L, fov, dw)
    g = torch.Generator(device="cuda").manual_seed(4)
    with t.plan() as p, t.plan(1) as q:
        for x, y in ((0.3, 0.3), (0.41, 0.41), (0.45, 0.2), (0.2, 0.45)):
            x, y = L // 2 + round(x * L), L // 2 - round(y * L)
            G, ref, T = t.source(x, y)
            V = p.degrid(G).cpu().numpy()
            assert np.isfinite(V).all(), (x, y)
            for pol in (0, 3):
                assert np.abs(V[..., pol] - ref).max() <= 1e-5 + 1e-6 / T, (x, y)
        v = torch.randn(p.vis_shape(), dtype=torch.complex64, device="cuda", generator=g)
        check_grid(p.grid(v).cpu().numpy(), q.grid(v.to(torch.complex128)).cpu().numpy(), 1e-5, f"L {L}, {fov} rad")


@pytest.mark.parametrize("L", [32, 64, 96])
@pytest.mark.parametrize("fov", [0.15, 0.58])
@pytest.mark.parametrize("first", [1e-6, 2.4e-5, 1e-4, 4e-4, 1e-3])
def test_sources_over_w_ranges(aidg, L, fov, first):
    """Lone predicted sources over w ranges whose first series term is up to `first` of the tapered
    field.  The rounding of FP32 cells 1 / (L^2 T) and of the subgrid's transform is some 2.5e-8
    of the source after the taper, that of a phasor 1e-7: twice the sum is the bar."""
    t = first_term(aidg, L, fov, first)
    with t.plan() as p:
        for r in (0.1, 0.2, 0.25, 0.3, 0.35, 0.4):
            x = L // 2 + round(r * L)
            G, ref, T = t.source(x, x)
            d = np.abs(p.degrid(G).cpu().numpy()[..., 0] - ref)
            rms = np.sqrt((d ** 2).mean())
            print(f"L {L} fov {fov} first {first} source {r} taper {T:.1e}: rms {rms:.2e}")
            assert rms <= 2 * (1e-7 + 2.5e-8 / T), r


@pytest.mark.parametrize("L", [32, 64, 96])
def test_kernels_that_plans_take(aidg, L):
    """Every length of the series, split and not, and every reason for the general kernels."""
    general, matrix, wide = aidg.KERNEL_GENERAL, aidg.KERNEL_MATRIX, aidg.KERNEL_MATRIX_WIDE
    for first, grid, terms in ((0.0, matrix, 0), (5e-9, matrix, 0), (1e-6, matrix, 1), (2e-5, matrix, 1),
                               (4e-5, wide, 1), (4e-4, wide, 2), (3e-3, general, 0)):
        with first_term(aidg, L, 0.3, first, nearby=True).plan() as p:
            k = p.kernels()
            assert (k["grid_kernel"], k["w_terms"]) == (grid, terms), (first, k)
            assert k["degrid_kernel"] == min(grid, matrix)
            assert (k["n_subgrids_split"] > 0) == (grid == wide)
    t = Track(aidg, L, 0.3, 0.1)
    for kw, grid, degrid in (({}, matrix, matrix), (dict(precision=1), general, general),
                             (dict(reseed_channels=31), general, general), (dict(reseed_channels=96), matrix, matrix),
                             (dict(degrid_form=aidg.DEGRID_RECURRENCE), matrix, general),
                             (dict(degrid_form=aidg.DEGRID_DIRECT), matrix, general)):
        with t.plan(**kw) as p:
            k = p.kernels()
            assert (k["grid_kernel"], k["degrid_kernel"]) == (grid, degrid), (kw, k)
    t.uvw, t.freqs = np.ascontiguousarray(t.uvw[:, :1]), t.freqs[:1]  # one visibility per subgrid
    with t.plan() as p:
        assert p.kernels()["degrid_kernel"] == general
    with Track(aidg, L, 0.9, 0.0, w_mid=3e5).plan() as p:  # FP32 phases of the middle w
        assert p.kernels()["grid_kernel"] == general


@pytest.mark.parametrize("L", [32, 64, 96])
@pytest.mark.parametrize("n_t,n_c", [(2, 1), (2, 4), (3, 3), (4, 8), (11, 3), (16, 8)])
def test_wide_series_at_block_edges(aidg, L, n_t, n_c):
    """The gridder and degridder of split series operands at part-filled steps and blocks: FP32
    sums, 2e-7 of the FP64 plan's, twice that is the bar."""
    t = first_term(aidg, L, 0.3, 3e-4, nearby=True)
    t.uvw, t.freqs = np.ascontiguousarray(t.uvw[:, np.linspace(0, 15, n_t).astype(int)]), t.freqs[:n_c]
    g = torch.Generator(device="cuda").manual_seed(9)
    with t.plan() as p, t.plan(1, table=p.subgrids()) as q:
        assert p.kernels()["grid_kernel"] == aidg.KERNEL_MATRIX_WIDE
        assert len(p.subgrids()) == len(t.bl)
        v = torch.randn(p.vis_shape(), dtype=torch.complex64, device="cuda", generator=g)
        G = torch.randn(p.grid_shape(), dtype=torch.complex64, device="cuda", generator=g)
        for x, y in ((p.grid(v), q.grid(v.to(torch.complex128))), (p.degrid(G), q.degrid(G.to(torch.complex128)))):
            assert float((x - y).norm() / y.norm()) <= 4e-7


@pytest.mark.parametrize("L", [32, 64, 96])
def test_gridder_rounds_no_more_than_the_general_kernel(aidg, L):
    """Sums over a subgrid's visibilities: the matrix gridder adds a step of eight at once, the
    general one (plans that ask for runs below 32 channels) two, so its error against the FP64
    plan is no larger but for the draw's spread, some 5 % over these six."""
    g = torch.Generator(device="cuda").manual_seed(5)
    err = {0: 0.0, 31: 0.0}
    for dw in (0.0, 0.1, 0.6):
        t = Track(aidg, L, 0.3, dw)
        with t.plan() as p, t.plan(reseed_channels=31) as r, t.plan(1) as q:
            for _ in range(2):
                v = torch.randn(p.vis_shape(), dtype=torch.complex64, device="cuda", generator=g)
                ref = q.grid(v.to(torch.complex128))
                for plan, key in ((p, 0), (r, 31)):
                    err[key] += float(((plan.grid(v) - ref).norm() / ref.norm()) ** 2 / 6)
    print(f"L {L}: matrix {err[0] ** 0.5:.3e}, general {err[31] ** 0.5:.3e}")
    assert err[0] <= 1.1 ** 2 * err[31]


@pytest.mark.parametrize("L", [32, 64, 96])
@pytest.mark.parametrize("scales", ["one", "over time", "smallest"])
def test_faint_polarisations_keep_their_digits(aidg, L, scales):
    """With Jones matrices that do not mix them, each polarisation is as exact as if it were alone:
    FP32 sums of 128 visibilities and of the subgrid transform, 2e-7 of each plane; twice that
    is the bar.  Over time: scales that rise, fall and jump between a subgrid's blocks."""
    t = Track(aidg, L, 0.3, 0.3)
    g = torch.Generator(device="cuda").manual_seed(6)
    f = torch.tensor([1.0, 1e-6, 3e-8, 1e4], device="cuda").expand(16, 4).clone()
    if scales == "over time":
        k = torch.arange(16, device="cuda", dtype=torch.float32)
        f = torch.stack([2.0 ** (2 * k), 2.0 ** (-2 * k - 10), 1e-6 * 10.0 ** (k // 4 % 2), (k > 7).float()], dim=1)
    if scales == "smallest":  # about and below the smallest normal FP32 number
        f = torch.full((16, 4), 2.0 ** -125, device="cuda")
    with t.plan() as p, t.plan(1) as q:
        v = torch.randn(p.vis_shape(), dtype=torch.complex64, device="cuda", generator=g) * f[None, :, None, :]
        got, ref = p.grid(v), q.grid(v.to(torch.complex128))
        G = torch.randn(p.grid_shape(), dtype=torch.complex64, device="cuda", generator=g) * f[-1][None, :, None, None]
        vis, ref_v = p.degrid(G), q.degrid(G.to(torch.complex128))
        for pol in range(4):
            e = float((got[:, pol] - ref[:, pol]).norm() / ref[:, pol].norm())
            d = float((vis[..., pol] - ref_v[..., pol]).norm() / ref_v[..., pol].norm())
            print(f"L {L} {scales} polarisation {pol}: grid {e:.2e}, degrid {d:.2e}")
            assert e <= 4e-7 and d <= 4e-7, pol


@pytest.mark.parametrize("L", [32, 96])
def test_data_between_16_byte_boundaries(aidg, L):
    """Buffers are aligned as complex64, no more: one element on gives the same results."""
    def shifted(x):
        y = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")[1:].view(x.shape)
        assert y.data_ptr() % 16 == 8 and y.is_contiguous()
        return y.copy_(x)
    t = first_term(aidg, L, 0.3, 1e-4, nearby=True)
    t.bl = t.bl[:1]  # one subgrid: one order of the adder's sums
    t.uvw = t.uvw[:1]
    g = torch.Generator(device="cuda").manual_seed(10)
    with t.plan() as p:
        v = torch.randn(p.vis_shape(), dtype=torch.complex64, device="cuda", generator=g)
        G = torch.randn(p.grid_shape(), dtype=torch.complex64, device="cuda", generator=g)
        assert torch.equal(p.grid(shifted(v), shifted(torch.zeros_like(G))), p.grid(v))
        assert torch.equal(p.degrid(shifted(G), shifted(v)), p.degrid(G))
        assert torch.equal(p.invert(shifted(G)), p.invert(G))
        assert torch.equal(p.predict(shifted(G[0])), p.predict(G[0]))


def one_subgrid(t):
    """A caller's table: baseline 0 of a track in one subgrid about the grid's centre."""
    table = np.zeros(1, t.aidg.SUBGRID_DTYPE)
    table["st1"], table["st2"] = t.bl[0]
    table["nt"], table["nc"], table["U0"], table["V0"] = t.uvw.shape[1], len(t.freqs), t.N // 2, t.N // 2
    return table


@pytest.mark.parametrize("L", [32, 96])
def test_channels_in_any_order(aidg, L):
    """The w range of a sub-table is that of all its channels, not of the first and last.  At
    most 1e-6 of the FP64 plan, five times the usual error."""
    t = Track(aidg, L, 0.58, 0.0, w_mid=300.0)
    t.freqs = np.array([150.0, 141.0, 159.0, 148.0, 152.0, 145.0, 155.0, 150.1]) * 1e6
    g = torch.Generator(device="cuda").manual_seed(7)
    with t.plan(table=one_subgrid(t)) as p, t.plan(1, table=one_subgrid(t)) as q:
        v = torch.randn(p.vis_shape(), dtype=torch.complex64, device="cuda", generator=g)
        G = torch.randn(p.grid_shape(), dtype=torch.complex64, device="cuda", generator=g)
        for x, y in ((p.grid(v), q.grid(v.to(torch.complex128))), (p.degrid(G), q.degrid(G.to(torch.complex128)))):
            assert float((x - y).norm() / y.norm()) <= 1e-6


@pytest.mark.parametrize("row", [(np.nan, 0, 0), (0, np.inf, 0), (0, 0, np.nan), (1.6e7 + 5.3, 0, 0), (0, 5.3 - 1.6e7, 0)])
def test_rows_that_have_no_phase_in_fixed_point(aidg, row):
    """Rows that are not finite have no phase and give NaN; rows a long way off the window have one,
    here of up to 2e6 turns (the general kernels count quarter turns in 32 bits)."""
    t = Track(aidg, 32, 0.25, 0.0)
    t.freqs = np.full(1, LIGHT)  # metres are wavelengths
    t.uvw[0, 3] = row
    table = one_subgrid(t)
    g = torch.Generator(device="cuda").manual_seed(8)
    with t.plan(table=table) as p, t.plan(1, table=table) as q:
        v = torch.randn(p.vis_shape(), dtype=torch.complex64, device="cuda", generator=g)
        G = torch.randn(p.grid_shape(), dtype=torch.complex64, device="cuda", generator=g)
        for x, y in ((p.grid(v), q.grid(v.to(torch.complex128))), (p.degrid(G), q.degrid(G.to(torch.complex128)))):
            assert torch.equal(x.isnan(), y.isnan())
            assert x.isnan().any() == (not np.isfinite(row).all())
            x, y = x[~y.isnan()], y[~y.isnan()]
            assert float((x - y).norm()) <= 1e-6 * float(y.norm())


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
