"""The LDS-staged paired tile as it runs in production: sizes that the layout
rule sends there (asserted by the rule itself, built from the library's
header), at every band height that exercises its walk, in each storage type,
with every slot filled and with spare slots, into line-aligned rows and rows
that start anywhere, with one-cell last strips -- bitwise the two-step maps."""

import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle as O
import paper_2510_01190_amd as P
from gpu_util import TORCH_DT, host64

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
BANDS = (1, 2, 3, 4, 5, 6, 7, 13, 64)


@pytest.fixture(scope="module")
def paired(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("rule") / "tile_choice")
    src = os.path.join(HERE, "host_checks", "tile_choice.cpp")
    subprocess.run([gxx, "-std=c++17", "-O1", src, "-o", exe], check=True, timeout=300)

    def ask(lines, dt, k, shape):
        slots = k if k <= 4 else 6 if k <= 6 else 8 if k <= 8 else 12 if k <= 12 else 16
        args = [1, int(lines), 4 if dt == "f32" else 2, slots, *shape]
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True)
        return r.stdout.strip() == "1"
    return ask


def _field(shape, dt, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [(torch.randn(shape, generator=g, device="cuda") * 0.3 if q % 2 == 0 else
             torch.rand(shape, generator=g, device="cuda") * 0.2 + 0.01).to(TORCH_DT[dt])
            for q in range(4)]


def _two_step(ts, iso):
    ref = P.lcp(*P.divergence_gaussian(*ts), iso)  # dense rows: the split tile
    # the first cells against the oracle: the cut makes column 258 one-sided
    part = [host64(t[:, :260]) for t in ts]
    want = O.lcp(*O.divergence_gaussian(*part, 1.0, 1.0), iso)[:, :, :257]
    assert np.max(np.abs(host64(ref[:, :, :257]) - want)) <= 1e-5
    return ref


# 163, 256 and 782, 1563 strips of 128 cells and one cell more
LINES = [((61, 20866), 8), ((61, 20866), 16), ((61, 20866), 11), ((61, 20866), 13),
         ((129, 32770), 1), ((129, 32770), 3), ((129, 32770), 4), ((129, 32770), 5)]
OTHER = [((61, 100098), 16), ((61, 100098), 10), ((61, 200066), 8), ((61, 200066), 7)]


@pytest.mark.parametrize("shape,k", LINES)
@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
def test_line_aligned_rows(shape, k, dt, paired):
    assert paired(True, dt, k, shape)
    ts = _field(shape, dt, shape[1] + k)
    iso = np.linspace(-0.4, 0.4, k).astype(np.float32)
    ref = _two_step(ts, iso)
    planar, rows = P.empty_lcp(k, *shape), P.empty_lcp(k, *shape, interleave_rows=True)
    try:
        for band in (0, *BANDS):
            P.set_lcp_band_rows(band)
            for out in (planar, rows) if band in (0, 3) else (planar,):
                out.fill_(-7.0)
                assert torch.equal(P.lcp_from_moments(*ts, iso, out=out), ref), band
    finally:
        P.set_lcp_band_rows(0)


def _other_rows(shape, k, dt):
    ts = _field(shape, dt, shape[1] + k)
    iso = np.linspace(-0.4, 0.4, k).astype(np.float32)
    ref = _two_step(ts, iso)
    ny, nx = shape
    cells = ref.numel()
    try:
        flat = torch.full((cells + 64,), -7.0, device="cuda")
        views = [(flat, flat[1:1 + cells].view(ref.shape)), (flat, flat[:cells].view(ref.shape))]
        odd = torch.full((k, ny - 1, nx + 2), -7.0, device="cuda")
        views.append((odd, odd[:, :, 3:3 + nx - 1]))
        for band in (0, *BANDS):
            P.set_lcp_band_rows(band)
            for buf, view in views if band in (0, 3) else views[1:2]:
                buf.fill_(-7.0)
                P.lcp_from_moments(*ts, iso, out=view)
                assert torch.equal(view, ref), band
                assert int((buf != -7.0).sum()) == cells, band
    finally:
        P.set_lcp_band_rows(0)


@pytest.mark.parametrize("shape,k", OTHER)
@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
def test_rows_that_start_inside_a_line(shape, k, dt, paired):
    assert paired(False, dt, k, shape)
    _other_rows(shape, k, dt)


@pytest.mark.parametrize("k", [1, 2, 4])
def test_few_isovalues_inside_a_line(k, paired):
    """Float32 only: 16-bit maps of so few isovalues keep the split tile."""
    assert paired(False, "f32", k, (61, 200066))
    _other_rows((61, 200066), k, "f32")


@pytest.mark.parametrize("dt,k,n", [("f32", 16, 24), ("f16", 16, 24), ("bf16", 9, 24),
                                    ("f32", 7, 40), ("bf16", 8, 48), ("f32", 3, 64)])
def test_batches_on_lines(dt, k, n):
    """Batches large enough for the paired tile without autotuning: fields of a
    strip and one cell, uneven counts beside the largest, every field bitwise
    its own two-step maps, padding untouched."""
    rng = np.random.default_rng(n + k)
    fields, bufs = [], []
    for i in range(n):
        ny, nx = int(rng.integers(300, 460)), [130, 258, 386, 514, 900][i % 5]
        kk = k if i % 4 else max(1, k - 1)
        m = _field((ny, nx), dt, 100 * n + i)
        iso = np.linspace(-0.4, 0.4, kk).astype(np.float32)
        buf = torch.full((kk, ny - 1, (nx + 30) // 32 * 32 + 32), -3.0, device="cuda")
        fields.append(dict(mean_u=m[0], var_u=m[1], mean_v=m[2], var_v=m[3], iso_host=iso,
                           isovalues=torch.from_numpy(iso).cuda(), lcp=buf[:, :, :nx - 1]))
        bufs.append((buf, nx, m, iso))
    b = P.Batch(fields, graph=False)
    assert b.info()["strip_cells"] == 128, b.info()
    b.launch()
    torch.cuda.synchronize()
    for g, (buf, nx, m, iso) in zip(b.fields, bufs):
        assert torch.equal(g["lcp"], P.lcp(*P.divergence_gaussian(*m), iso))
        assert bool((buf[..., nx - 1:] == -3.0).all())
    b.close()
