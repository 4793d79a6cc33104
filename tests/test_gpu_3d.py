"""GPU parity of the 3D extension (the paper's future work, Section 5)
against the FP64 oracle: the divergence Gaussian with the z term and the
8-corner level-crossing probability, through the C ABI."""

import numpy as np
import pytest
import torch

import oracle as O
import paper_2510_01190_amd as P
import synth
from gpu_util import TORCH_DT, U32, dev, host64

pytestmark = pytest.mark.gpu

KEYS = ("mean_u", "var_u", "mean_v", "var_v", "mean_w", "var_w")
LCP_TOL = 1e-5

# (nz, ny, nx): one cell wide; strips of 63 (dense rows) and 64 cells
# (line-aligned rows) exact and ragged; two bands of 64 rows; layer counts
# that are and are not multiples of the layers a wave carries (4 or 2)
SHAPES = [(2, 2, 2), (3, 5, 70), (9, 33, 130), (17, 40, 64), (5, 3, 127), (4, 130, 65),
          (6, 7, 2), (2, 66, 190), (3, 4, 129)]
SENTINEL = -7.0  # padding floats of an output must keep this


def _padded(k, shape, pitch=None, gap=0):
    """A [k][nz-1][ny-1][nx-1] view with rows padded to `pitch` floats
    (default: the next multiple of 32) and `gap` extra floats between maps,
    filled with SENTINEL; returns (view, backing buffer)."""
    nz, ny, nx = shape
    pitch = pitch or (nx - 1 + 31) // 32 * 32
    map_ = (nz - 1) * (ny - 1) * pitch
    buf = torch.full((k * (map_ + gap),), SENTINEL, dtype=torch.float32, device="cuda")
    view = buf.as_strided((k, nz - 1, ny - 1, nx - 1),
                          (map_ + gap, (ny - 1) * pitch, pitch, 1))
    return view, buf


def _padding_untouched(view, buf):
    mask = torch.ones_like(buf, dtype=torch.bool)
    idx = torch.arange(buf.numel(), device=buf.device).as_strided(view.shape, view.stride())
    mask[idx.reshape(-1)] = False
    return bool(torch.all(buf[mask] == SENTINEL))


def _field(shape, seed, dt="f32", sigma=(0.05, 0.5)):
    f = synth.gen_moments_3d(*shape, seed, sigma=sigma)
    ts = [dev(f[k], dt) for k in KEYS]
    return f, ts


def _axis_means(st, h):
    """The three axis terms of the oracle's mean, each alone (for the
    rounding bound of the float32 sum)."""
    zero = np.zeros_like(st[0])
    parts = []
    for a in range(3):
        args = [zero] * 6
        args[2 * a], args[2 * a + 1] = st[2 * a], st[2 * a + 1]
        parts.append(O.divergence_gaussian_3d(*args, *h)[0])
    return parts


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_divergence_3d_matches_oracle(shape, dt):
    h = (1.0, 0.5, 2.0)
    _, ts = _field(shape, seed=sum(shape), dt=dt)
    dm, dv = P.divergence_gaussian_3d(*ts, *h)
    st = [host64(t) for t in ts]
    rm, rv = O.divergence_gaussian_3d(*st, *h)
    mx, my, mz = _axis_means(st, h)
    # each axis term: a difference, one coefficient and one product rounded;
    # then two additions
    bound_m = 6 * U32 * (np.abs(mx) + np.abs(my) + np.abs(mz)) + 1e-30
    assert np.all(np.abs(host64(dm) - rm) <= bound_m)
    np.testing.assert_allclose(host64(dv), rv, rtol=8 * U32, atol=0)


def _oracle_div3(ts, h=(1.0, 1.0, 1.0)):
    """The oracle's float32 3D divergence Gaussians of the stored volumes, as
    numpy arrays and device tensors: the pdiv_lcp_3d input of both sides."""
    m, v = O.divergence_gaussian_3d_f32(*[host64(t) for t in ts], *h)
    return m, v, torch.from_numpy(m).cuda(), torch.from_numpy(v).cuda()


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_divergence_3d_rounds_like_the_float32_oracle(shape, dt):
    h = (0.75, 1.0, 2.5)
    _, ts = _field(shape, seed=5 * sum(shape), dt=dt)
    dm, dv = P.divergence_gaussian_3d(*ts, *h)
    m, v, _, _ = _oracle_div3(ts, h)
    assert np.array_equal(dm.cpu().numpy(), m) and np.array_equal(dv.cpu().numpy(), v)


@pytest.mark.parametrize("k", [1, 3, 4, 8, 16, 17])
@pytest.mark.parametrize("shape", SHAPES)
def test_lcp_3d_matches_oracle(shape, k):
    _, ts = _field(shape, seed=7 * sum(shape) + k)
    m, v, dm, dv = _oracle_div3(ts)
    m64, v64 = m.astype(np.float64), v.astype(np.float64)
    iso = np.quantile(m64, np.linspace(0.05, 0.95, k)).astype(np.float32)
    g = host64(P.lcp_3d(dm, dv, iso))
    r = O.lcp_3d(m64, v64, iso)
    err = np.abs(g - r)
    print(f"\n[{shape} K={k}] max |LCP - oracle| = {err.max():.3e}, range [{g.min():.9g}, "
          f"{g.max():.9g}]")
    assert err.max() <= LCP_TOL
    assert np.all((g >= 0) & (g <= 1))


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_fused_equals_two_step(shape, dt):
    """pdiv_lcp_3d_from_moments evaluates Eq. 2-3 on the spot with the same
    operands as the divergence kernel: the maps are bitwise the two-step's."""
    h = (1.0, 0.5, 2.0)
    _, ts = _field(shape, seed=3 * sum(shape), dt=dt)
    dm, dv = P.divergence_gaussian_3d(*ts, *h)
    m = _oracle_div3(ts, h)[0]
    for k in (1, 4, 8, 16, 17):
        iso = np.quantile(m, np.linspace(0.05, 0.95, k)).astype(np.float32)
        two = P.lcp_3d(dm, dv, iso)
        fused = P.lcp_3d_from_moments(*ts, iso, *h)
        assert torch.equal(fused, two), (shape, dt, k)


@pytest.mark.parametrize("shape", SHAPES)
def test_line_aligned_layout_is_bitwise_the_dense_maps(shape):
    """Rows padded to whole 128-byte lines take the 64-cell tile with the
    seam step; the maps are bitwise those of the dense layout (63-cell
    tile), which the oracle test above checks, and the padding is never
    written.  Pitches of 32 (line-aligned) and of nx - 1 + 5 (not aligned),
    with and without a gap between maps."""
    _, ts = _field(shape, seed=11 * sum(shape))
    m, _, dm, dv = _oracle_div3(ts)
    nz, ny, nx = shape
    for k in (1, 2, 3, 4, 8, 16, 17):
        iso = np.quantile(m, np.linspace(0.05, 0.95, k)).astype(np.float32)
        dense = P.lcp_3d(dm, dv, iso)
        for pitch, gap in ((None, 0), (None, 64), ((nx - 1 + 31) // 32 * 32 + 32, 32),
                           (nx - 1 + 5, 3)):
            view, buf = _padded(k, shape, pitch, gap)
            P.lcp_3d(dm, dv, iso, out=view)
            assert torch.equal(view, dense), (shape, k, pitch, gap)
            assert _padding_untouched(view, buf), (shape, k, pitch, gap)


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_fused_line_aligned_layout_equals_two_step(shape, dt):
    h = (0.5, 1.0, 1.5)
    _, ts = _field(shape, seed=13 * sum(shape), dt=dt)
    dm, dv = P.divergence_gaussian_3d(*ts, *h)
    m = _oracle_div3(ts, h)[0]
    for k in (1, 4, 8, 16):
        iso = np.quantile(m, np.linspace(0.05, 0.95, k)).astype(np.float32)
        two = P.lcp_3d(dm, dv, iso)
        view, buf = _padded(k, shape)
        P.lcp_3d_from_moments(*ts, iso, *h, out=view)
        assert torch.equal(view, two), (shape, dt, k)
        assert _padding_untouched(view, buf)


def test_empty_lcp_3d_pads_rows_to_lines():
    shape = (4, 9, 100)
    _, ts = _field(shape, seed=17)
    _, _, dm, dv = _oracle_div3(ts)
    out = P.empty_lcp_3d(3, *shape)
    assert out.stride() == (3 * 8 * 128, 8 * 128, 128, 1) and out.data_ptr() % 128 == 0
    iso = [-0.1, 0.0, 0.1]
    assert torch.equal(P.lcp_3d(dm, dv, iso, out=out), P.lcp_3d(dm, dv, iso))


def test_lcp_3d_end_to_end_float32():
    """From the float64 field through float32 storage and arithmetic."""
    shape = (9, 33, 130)
    f, ts = _field(shape, seed=99)
    iso = np.linspace(-0.6, 0.6, 5).astype(np.float32)
    g = host64(P.lcp_3d(*P.divergence_gaussian_3d(*ts), iso))
    r = O.lcp_3d(*O.divergence_gaussian_3d(*[f[k] for k in KEYS], 1.0, 1.0, 1.0), iso)
    err = float(np.max(np.abs(g - r)))
    print(f"\n[end to end] max |LCP - oracle(float64 field)| = {err:.3e}")
    assert err <= LCP_TOL


def test_zero_variance_is_marching_cubes():
    shape = (6, 20, 70)
    f = synth.gen_moments_3d(*shape, 5)
    ts = [dev(f[k] if k.startswith("mean") else 0.0 * f[k]) for k in KEYS]
    m32, v32, dm, dv = _oracle_div3(ts)
    assert float(np.abs(v32).max()) == 0.0
    m64 = m32.astype(np.float64)
    iso = np.quantile(m64, [0.1, 0.5, 0.9]).astype(np.float32)
    iso[1] = m32[3, 10, 35]  # a tie at a vertex: >= counts as above
    g = host64(P.lcp_3d(dm, dv, iso))
    for q, c in enumerate(iso):
        np.testing.assert_array_equal(g[q], O.crossed_3d(m64, float(c)).astype(np.float64))


def test_nan_reaches_exactly_its_cells():
    shape = (5, 9, 70)
    _, ts = _field(shape, seed=3)
    _, _, dm, dv = _oracle_div3(ts)
    dm[2, 4, 66] = float("nan")
    g = host64(P.lcp_3d(dm, dv, [0.0, 0.3]))
    bad = np.zeros(g.shape[1:], bool)
    bad[1:3, 3:5, 65:67] = True
    assert np.all(np.isnan(g[:, bad]))
    assert not np.any(np.isnan(g[:, ~bad]))


def test_bench_size_sampled_slabs():
    """The benchmark's 3D workload (512^3, float32, 4 isovalues): every cell
    in [0, 1] and finite, and slabs of cell layers at the bottom, middle and
    top of the volume against the oracle."""
    n = 512
    f = synth.gen_moments_3d(n, n, n, synth.SEED_BASE + 30, dtype=np.float32)
    ts = [torch.from_numpy(f[k]).cuda() for k in KEYS]

    def oracle_vertices(k0):
        # vertex planes k0..k0+2 from the z slab around them (planes k0-1 ..
        # k0+3): inside the slab they are differenced as in the whole volume
        a, b = max(0, k0 - 1), min(n, k0 + 4)
        m, v = O.divergence_gaussian_3d(*[f[k][a:b].astype(np.float64) for k in KEYS],
                                        1.0, 1.0, 1.0)
        return m[k0 - a:k0 - a + 3], v[k0 - a:k0 - a + 3]

    iso = np.quantile(oracle_vertices(n // 2 - 2)[0], [0.2, 0.4, 0.6, 0.8]).astype(np.float32)
    dm, dv = P.divergence_gaussian_3d(*ts)
    out = P.lcp_3d(dm, dv, iso)
    assert torch.equal(P.lcp_3d_from_moments(*ts, iso), out)
    # the benchmark's layouts: rows padded to 512 floats, two-step and fused
    padded = P.empty_lcp_3d(4, n, n, n)
    assert torch.equal(P.lcp_3d(dm, dv, iso, out=padded), out)
    assert torch.equal(P.lcp_3d_from_moments(*ts, iso, out=padded), out)
    del padded
    assert not torch.isnan(out).any()
    assert float(out.min()) >= 0.0 and float(out.max()) <= 1.0
    worst = 0.0
    for k0 in (0, n // 2 - 2, n - 3):
        r = O.lcp_3d(*oracle_vertices(k0), iso)
        worst = max(worst, float(np.max(np.abs(host64(out[:, k0:k0 + 2]) - r))))
    print(f"\n[512^3 K=4] max |LCP - oracle(stored volumes)| on sampled slabs = {worst:.3e}")
    assert worst <= LCP_TOL


@pytest.mark.parametrize("shape,k", [((3, 4, 62), 1), ((3, 5, 63), 4), ((2, 3, 123), 8),
                                     ((6, 9, 124), 16), ((9, 2, 61), 2), ((90, 70, 130), 4),
                                     ((70, 260, 130), 1), ((300, 300, 200), 1)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_fused_strips_of_61_cells_and_band_heights(shape, k, dt):
    """The fused walk takes U's neighbours from the adjacent lanes, in strips of
    61 cells: widths of one strip less and more than whole, and volumes whose
    band heights are 1, 2, 4 and 8 rows, bitwise the two-step maps on dense,
    odd and line-aligned rows, padding untouched; the two-step line-aligned and
    dense maps agree, and the lowest cell layer is within 1e-5 of the oracle."""
    rng = np.random.default_rng(sum(shape))
    ts = []
    for q in range(6):
        a = rng.normal(0, 0.3, shape) if q % 2 == 0 else rng.uniform(0.02, 0.2, shape)
        ts.append(dev(a, dt))
    div = P.divergence_gaussian_3d(*ts, dx=0.5, dy=1.0, dz=2.0)
    iso = np.linspace(-0.4, 0.4, k).astype(np.float32)
    ref = P.lcp_3d(*div, iso)
    for pitch in (None, shape[2] - 1, shape[2] + 4):
        view, buf = _padded(k, shape, pitch=pitch, gap=32)
        P.lcp_3d_from_moments(*ts, iso, dx=0.5, dy=1.0, dz=2.0, out=view)
        assert torch.equal(view, ref) and _padding_untouched(view, buf), pitch
        view, buf = _padded(k, shape, pitch=pitch, gap=32)
        P.lcp_3d(*div, iso, out=view)
        assert torch.equal(view, ref) and _padding_untouched(view, buf), pitch
    want = O.lcp_3d(host64(div[0][:2]), host64(div[1][:2]), iso)
    assert np.max(np.abs(host64(ref[:, :1]) - want)) <= LCP_TOL


@pytest.mark.parametrize("shape", [(2, 2, 2), (6, 9, 130)])
def test_every_isovalue_count_3d(shape):
    """Every count's maps, in whatever launches it takes, are bitwise the ones
    computed one isovalue at a time, fused and two-step, dense and
    line-aligned, and nothing is written past the last map."""
    rng = np.random.default_rng(shape[2])
    ts = [dev(rng.normal(0, 0.3, shape) if q % 2 == 0 else rng.uniform(0.02, 0.2, shape), "f32")
          for q in range(6)]
    div = P.divergence_gaussian_3d(*ts)
    iso = rng.uniform(-0.5, 0.5, 25).astype(np.float32)
    ref = torch.cat([P.lcp_3d(*div, [c]) for c in iso])
    assert np.max(np.abs(host64(ref[:2]) - O.lcp_3d(*map(host64, div), iso[:2]))) <= LCP_TOL
    for k in range(2, 26):
        for pitch in (shape[2] - 1, None):
            view, buf = _padded(k, shape, pitch=pitch, gap=64)
            P.lcp_3d(*div, iso[:k], out=view)
            assert torch.equal(view, ref[:k]) and _padding_untouched(view, buf), (k, pitch)
            view, buf = _padded(k, shape, pitch=pitch, gap=64)
            P.lcp_3d_from_moments(*ts, iso[:k], out=view)
            assert torch.equal(view, ref[:k]) and _padding_untouched(view, buf), (k, pitch)


@pytest.mark.parametrize("nz", [3, 4, 5, 7, 8])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_three_layer_groups_3d(nz, dt):
    """Fused launches above 4 isovalues walk three cell layers per wave: the
    last group of one, two and three layers, one group and several, bitwise
    the two-step maps, nothing written past the last layer."""
    shape = (nz, 20, 65)
    rng = np.random.default_rng(nz)
    ts = [dev(rng.normal(0, 0.3, shape) if q % 2 == 0 else rng.uniform(0.02, 0.2, shape), dt)
          for q in range(6)]
    div = P.divergence_gaussian_3d(*ts)
    for k in (5, 6, 7, 8, 16):
        iso = np.linspace(-0.4, 0.4, k).astype(np.float32)
        view, buf = _padded(k, shape, gap=32)
        P.lcp_3d_from_moments(*ts, iso, out=view)
        assert torch.equal(view, P.lcp_3d(*div, iso)) and _padding_untouched(view, buf), k


@pytest.mark.parametrize("shape,dt", [((49, 400, 32), "f32"), ((181, 325, 32), "bf16"),
                                      ((151, 192, 71), "f32"), ((121, 121, 99), "f16"),
                                      ((89, 182, 193), "f32"), ((61, 300, 129), "bf16"),
                                      ((97, 390, 70), "f16"), ((188, 445, 32), "f32"),
                                      ((200, 130, 251), "bf16"), ((83, 160, 240), "f32")])
def test_divergence_shapes_3d(shape, dt):
    """Every walk length and store form the rule picks, with last chunks short
    and whole: the slices of a volume are bitwise those of
    runs of ten of them (but the slices whose z difference a cut makes
    one-sided), whose shape the rule picks by their own size."""
    g = torch.Generator(device="cuda")
    g.manual_seed(shape[0])
    ts = [(torch.randn(shape, generator=g, device="cuda") * 0.3 if q % 2 == 0 else
           torch.rand(shape, generator=g, device="cuda") * 0.2 + 0.01).to(TORCH_DT[dt])
          for q in range(6)]
    whole = P.divergence_gaussian_3d(*ts, dx=0.5, dy=1.0, dz=2.0)
    for a in range(0, shape[0] - 1, 7):
        lo, hi = max(0, a - 1), min(shape[0], a + 9)
        part = P.divergence_gaussian_3d(*[t[lo:hi].contiguous() for t in ts], dx=0.5, dy=1.0, dz=2.0)
        first = 0 if lo == 0 else lo + 1
        last = hi if hi == shape[0] else hi - 1
        for w, p in zip(whole, part):
            assert torch.equal(w[first:last], p[first - lo:last - lo]), (lo, hi)


@pytest.mark.parametrize("nx", [63, 64, 65, 124, 126, 127, 128, 188, 190, 251])
@pytest.mark.parametrize("dt", ["f32", "f16"])
def test_wide_strips_3d(nx, dt):
    """Fused rows of which strips of 63 cells need fewer than strips of 61 (and
    widths just off those): the end lanes' loaded neighbours inside the row and
    at both boundaries, every isovalue count's kernel, rows of few bands and
    many, bitwise the two-step maps, with NaN and infinities at strip ends,
    nothing written outside the cells."""
    shape = (6, 11, nx)
    rng = np.random.default_rng(nx)
    ts = [dev(rng.normal(0, 0.3, shape) if q % 2 == 0 else rng.uniform(0.02, 0.2, shape), dt)
          for q in range(6)]
    ts[0][2, 3, nx - 1] = float("nan")
    ts[0][4, 7, 0] = float("inf")
    for x in (60, 61, 62, 63, 64):
        if x < nx:
            ts[0][x % 6, (3 * x) % 11, x] = float("nan") if x % 2 else float("-inf")
            ts[1][(x + 3) % 6, (5 * x) % 11, x] = float("nan")
    div = P.divergence_gaussian_3d(*ts)
    for k in (1, 2, 3, 4, 5, 6, 7, 8, 16):
        iso = np.linspace(-0.4, 0.4, k).astype(np.float32)
        want = P.lcp_3d(*div, iso)
        view, buf = _padded(k, shape, pitch=nx + 2, gap=32)
        P.lcp_3d_from_moments(*ts, iso, out=view)
        assert torch.equal(torch.isnan(view), torch.isnan(want)), k
        assert torch.equal(torch.nan_to_num(view, nan=-1.0), torch.nan_to_num(want, nan=-1.0)), k
        assert _padding_untouched(view, buf), k


@pytest.mark.parametrize("nx", [63, 64, 65, 124, 126, 127, 128, 188, 190, 251])
@pytest.mark.parametrize("dt", ["f32", "f16"])
def test_wide_strips_in_volumes_that_take_them(nx, dt):
    """As above in a volume whose rounds of bands the wide strips shorten, so
    that the launch takes them (tests/host_checks/launch_rules_test.cpp holds
    the rule to it): bitwise the two-step maps, NaN and infinities at strip
    ends, nothing written outside the cells."""
    shape = (42, 150, nx)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    ts = [(torch.randn(shape, generator=g, device="cuda") * 0.3 if q % 2 == 0 else
           torch.rand(shape, generator=g, device="cuda") * 0.2 + 0.02).to(TORCH_DT[dt])
          for q in range(6)]
    ts[0][2, 3, nx - 1] = float("nan")
    ts[0][40, 149, 0] = float("inf")
    for x in (60, 61, 62, 63, 64, 126, 189):
        if x < nx:
            ts[0][x % 42, (3 * x) % 150, x] = float("nan") if x % 2 else float("-inf")
            ts[1][(x + 3) % 42, (5 * x) % 150, x] = float("nan")
    div = P.divergence_gaussian_3d(*ts)
    for k in (1, 2, 3, 4, 5, 6, 7, 8, 16):
        iso = np.linspace(-0.4, 0.4, k).astype(np.float32)
        want = P.lcp_3d(*div, iso)
        view, buf = _padded(k, shape, pitch=nx + 2, gap=32)
        P.lcp_3d_from_moments(*ts, iso, out=view)
        assert torch.equal(torch.isnan(view), torch.isnan(want)), k
        assert torch.equal(torch.nan_to_num(view, nan=-1.0), torch.nan_to_num(want, nan=-1.0)), k
        assert _padding_untouched(view, buf), k
