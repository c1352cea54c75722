"""GPU parity of the projectors (C ABI through the Python binding) against the oracle.

Tolerance: ||y_gpu - y_oracle||_2 / ||y_oracle||_2 <= 1e-5 per apply in FP32 (the
target for a projector apply); FP64 applies must agree to 1e-12.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

GEOMS = [
    dict(N=64, n_ang=90, n_det=91),                                  # plain FP64 workload
    dict(N=50, n_ang=37, n_det=73),                                  # ragged tiles and waves
    dict(N=40, n_ang=60, n_det=57, ang_range=120.0),                 # limited angle
    dict(N=33, n_ang=0, n_det=49, angles_deg=[0.0, 0.1, 44.99, 45.0, 89.9, 90.0, 90.1,
                                              135.0, 179.9, 30.0, 120.0, 1e-7]),
    dict(N=32, n_ang=30, n_det=48),                                  # even n_det
    dict(N=24, n_ang=17, n_det=31, det_spacing=1.3),
    dict(N=17, n_ang=7, n_det=5),                                    # detector smaller than image
    dict(N=1, n_ang=3, n_det=3),
    dict(N=2, n_ang=4, n_det=1),
    dict(N=300, n_ang=45, n_det=300),                                # > one fwd block per angle
]


def _ids(g):
    return "N{N}_a{a}_d{d}".format(N=g["N"], a=g.get("n_ang") or len(g["angles_deg"]), d=g["n_det"])


def _rel(a, b):
    nb = np.linalg.norm(b)
    return np.linalg.norm(a - b) / (nb if nb > 0 else 1.0)


def _pair(kw):
    import paper_2110_01481_amd as abg
    return O.Geometry(**kw), abg.Geometry(**kw)


@pytest.mark.parametrize("kw", GEOMS, ids=_ids)
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_forward_matches_oracle(gpu_lib, kw, dt):
    import torch
    go, gg = _pair(kw)
    tdt = torch.float64 if dt == "f64" else torch.float32
    tol = 1e-12 if dt == "f64" else 1e-5
    rng = np.random.default_rng(1)
    for x in (rng.uniform(size=go.n), W.ellipse_phantom(go.N, 4, rng) if go.N >= 8 else rng.uniform(size=go.n)):
        want = go.A(x)
        got = gg.fp(torch.tensor(x, dtype=tdt, device="cuda")).double().cpu().numpy()
        assert _rel(got, want) <= tol, (_rel(got, want), np.abs(got - want).max())


@pytest.mark.parametrize("kw", GEOMS, ids=_ids)
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["hat", "adj"])
def test_back_matches_oracle(gpu_lib, kw, dt, kind):
    import torch
    go, gg = _pair(kw)
    tdt = torch.float64 if dt == "f64" else torch.float32
    tol = 1e-12 if dt == "f64" else 1e-5
    rng = np.random.default_rng(2)
    for y in (rng.uniform(size=go.m), go.A(rng.uniform(size=go.n))):
        want = go.back(kind)(y)
        got = gg.bp(torch.tensor(y, dtype=tdt, device="cuda"), kind).double().cpu().numpy()
        assert _rel(got, want) <= tol, (_rel(got, want), np.abs(got - want).max())


@pytest.mark.parametrize("kw", GEOMS[:4], ids=_ids)
def test_gpu_adjoint_identity(gpu_lib, kw):
    """The GPU's ray-driven A and pixel-driven A^T are exact transposes (FP64)."""
    import torch
    _, gg = _pair(kw)
    rng = np.random.default_rng(3)
    x = torch.tensor(rng.standard_normal(gg.n), device="cuda")
    y = torch.tensor(rng.standard_normal(gg.m), device="cuda")
    lhs = float(gg.fp(x) @ y)
    rhs = float(x @ gg.bp(y, "adj"))
    assert abs(lhs - rhs) <= 1e-12 * (abs(lhs) + abs(rhs))


@pytest.mark.parametrize("kw", GEOMS + [dict(N=512, n_ang=7, n_det=725), dict(N=1030, n_ang=6, n_det=1459),
                                 dict(N=600, n_ang=721, n_det=851, ang_range=150.0)],
                         ids=_ids)
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_forward_block_shapes_bit_identical(gpu_lib, kw, dt):
    """The forward projectors' block shapes (one, two or four angles per block) change
    only which rays run together, and a four-angle block that stages its band rows in LDS
    only where its taps are read: every model gives bit-identical sinograms for every
    shape and share of staged blocks (none, three eighths, all), on ragged angle counts
    (waves past the last angle) and ragged detector rows.
    The automatic shape is four angles per block for the 600^2 and 1030^2 geometries
    (600^2 with 721 close angles also stages a share of its blocks in FP64 and FP32),
    two for n_det = 91, 183 or 300, one for the others."""
    import torch
    import paper_2110_01481_amd as abg
    tdt = torch.float64 if dt == "f64" else torch.float32
    rng = np.random.default_rng(5)
    x = torch.tensor(rng.uniform(size=kw["N"] ** 2), dtype=tdt, device="cuda")
    try:
        for model in ("line", "strip", "joseph"):
            if model == "strip" and kw.get("det_spacing", 1.0) > 1.4:
                continue
            gg = abg.Geometry(**kw, model=model)
            abg.fp_force_block_shape(-1)
            auto = gg.fp(x)
            for lg in (0, 1, 2):
                abg.fp_force_block_shape(lg)
                assert torch.equal(gg.fp(x), auto), (model, lg)
            abg.fp_force_block_shape(2)
            for share in (0, 3, 8):
                abg.fp_force_stage_share(share)
                assert torch.equal(gg.fp(x), auto), (model, "stage", share)
            abg.fp_force_stage_share(-1)
            gg.close()
    finally:
        abg.fp_force_block_shape(-1)
        abg.fp_force_stage_share(-1)


# Launches of the staged line-model kernel: four and eight angles per block, plain and tiled
# block order, with ragged numbers of angles, ray groups and rows, and angles too far apart
# for one window (those blocks walk directly).
STAGED_GEOMS = [
    dict(N=200, n_ang=411, n_det=283),                   # four angles, plain (2055 waves)
    dict(N=901, n_ang=103, n_det=1279, ang_range=20.0),  # four angles, tiled (2060 waves)
    dict(N=255, n_ang=2731, n_det=363),                  # eight angles, plain (16386 waves)
    dict(N=897, n_ang=821, n_det=1273),                  # eight angles, tiled (16420 waves)
    dict(N=905, n_ang=105, n_det=1217, det_spacing=1.1), # four angles, tiled, wide steps
]


@pytest.mark.parametrize("kw", STAGED_GEOMS, ids=_ids)
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("model", ["line", "joseph"])
def test_forward_staged_launches_bit_identical(gpu_lib, kw, dt, model):
    """The staged launches write every ray once and give the bits of the direct kernel
    (one angle per block), which the oracle tests pin."""
    import torch
    import paper_2110_01481_amd as abg
    tdt = torch.float64 if dt == "f64" else torch.float32
    rng = np.random.default_rng(6)
    x = torch.tensor(rng.standard_normal(kw["N"] ** 2), dtype=tdt, device="cuda")
    gg = abg.Geometry(**kw, model=model)
    y = torch.full((gg.m,), float("nan"), dtype=tdt, device="cuda")
    try:
        gg.fp(x, out=y)
        abg.fp_force_block_shape(0)
        assert torch.equal(gg.fp(x), y)
    finally:
        abg.fp_force_block_shape(-1)
        gg.close()


# Launches from 8192 waves on whose blocks cannot stage: those walk two bands per trip.
FAR_GEOMS = [
    dict(N=897, n_ang=413, n_det=1275, order="shuffled"),     # 8260 waves, ragged ends
    dict(N=1000, n_ang=401, n_det=1409, order="interleaved"), # some blocks stage in FP64
    dict(N=901, n_ang=1641, n_det=319, det_spacing=4.0),      # 8205 waves of bins of four pixels
]


@pytest.mark.parametrize("kw", FAR_GEOMS, ids=_ids)
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("model", ["line", "joseph"])
def test_forward_far_angles_bit_identical(gpu_lib, kw, dt, model):
    """Two bands per trip add a ray's taps in the order of eight: the bits of the direct kernel,
    from single launches and (line model) from the engine's items."""
    import torch
    import paper_2110_01481_amd as abg
    kw = dict(kw)
    order = kw.pop("order", None)
    if order:
        n = kw["n_ang"]
        a = np.arange(n) * 180.0 / n
        kw["angles_deg"] = np.random.default_rng(9).permutation(a) if order == "shuffled" else np.concatenate([a[i::8] for i in range(8)])
    tdt = torch.float64 if dt == "f64" else torch.float32
    rng = np.random.default_rng(6)
    x = torch.tensor(rng.standard_normal(kw["N"] ** 2), dtype=tdt, device="cuda")
    gg = abg.Geometry(**kw, model=model)
    b = torch.tensor(rng.uniform(size=gg.m), dtype=tdt, device="cuda")
    y = torch.full((gg.m,), float("nan"), dtype=tdt, device="cuda")
    def in_engine():
        p = abg.Problem(g=gg, method="ba", b=b, k_max=2, stop="none")
        return abg.Engine(proj=dt, basis=dt, max_slots=1).run([p])[0].x
    try:
        gg.fp(x, out=y)
        r = in_engine() if model == "line" else None
        abg.fp_force_block_shape(0)
        assert torch.equal(gg.fp(x), y)
        if r is not None:
            assert torch.equal(in_engine(), r)
    finally:
        abg.fp_force_block_shape(-1)
        gg.close()


# Back projections over orbits of four pixels: 16 waves (up to 256 blocks) and 8, even and odd
# images with ragged tiles, angle counts around the 32 of a round, detectors shorter than the
# image diagonal, both ends of the bin spacings.
ORBIT_GEOMS = [
    dict(N=512, n_ang=37, n_det=725),
    dict(N=449, n_ang=32, n_det=301),
    dict(N=481, n_ang=7, n_det=600, det_spacing=1.3),
    dict(N=675, n_ang=33, n_det=957, ang_range=120.0),
    dict(N=700, n_ang=5, n_det=1325, det_spacing=0.75),
]


@pytest.mark.parametrize("kw", ORBIT_GEOMS, ids=_ids)
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_back_orbits_match_oracle(gpu_lib, kw, dt):
    import torch
    go, gg = _pair(kw)
    tdt, tol = (torch.float64, 1e-12) if dt == "f64" else (torch.float32, 1e-5)
    y = np.random.default_rng(12).uniform(size=go.m)
    x = torch.empty(gg.n, dtype=tdt, device="cuda")
    yt = torch.tensor(y, dtype=tdt, device="cuda")
    for kind in ("hat", "adj", "strip_t", "joseph_t"):
        want = go.back(kind)(y)
        x.fill_(float("nan"))
        got = gg.bp(yt, kind, out=x).double().cpu().numpy()
        assert _rel(got, want) <= tol, (kind, _rel(got, want))
    # B_tau drops whole entries at the threshold, so an entry within rounding of it may fall
    # either way; y >= 0 and B_tau y falls with tau, which bounds each pixel by thresholds
    # moved by the entries' rounding (bin positions up to 32, a few units in the last place)
    gg.set_strip_threshold(0.3)
    x.fill_(float("nan"))
    got = gg.bp(yt, "strip_tau", out=x).double().cpu().numpy()
    delta = 64 * np.finfo(np.float64 if dt == "f64" else np.float32).eps * 4
    lo, hi = go.B_tau(0.3 + delta)(y), go.B_tau(0.3 - delta)(y)
    slack = tol * np.abs(hi).max()
    assert np.all(got >= lo - slack) and np.all(got <= hi + slack)
    # AB-GMRES takes B's output straight in the forward projector's copies: one step gives
    # x_1 = (<b, A B b> / ||A B b||^2) B b
    import paper_2110_01481_amd as abg
    r = abg.gmres("ab", gg, yt, 1)
    bb = gg.bp(yt)
    q = gg.fp(bb)
    want = (torch.dot(yt.double(), q.double()) / torch.dot(q.double(), q.double()) * bb.double()).cpu().numpy()
    assert _rel(r.x.double().cpu().numpy(), want) <= tol


def test_back_projection_of_a_sinogram_over_2gib(gpu_lib):
    """The back projectors read a sinogram of less than 2 GiB through one buffer resource
    with 31-bit offsets, a larger one through clamped 64-bit addresses. A 16^2 image with
    4.1M angles x 65 bins in FP64 (2.15 GB) takes the second path; its back projection
    (interpolating and matched) must equal the sum of the back projections of four blocks
    of its angles (each under 2 GiB, the first path), up to summation order."""
    import torch
    import paper_2110_01481_amd as abg
    N, n_det = 16, 65
    n_ang = (1 << 31) // (8 * n_det) + 64
    theta = (np.arange(n_ang, dtype=np.float64) * 180.0) / n_ang
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    y = torch.randn(n_ang * n_det, dtype=torch.float64, device="cuda", generator=gen)
    big = abg.Geometry(N, n_ang, n_det)
    cuts = np.linspace(0, n_ang, 5).astype(int)
    parts = [abg.Geometry(N, 0, n_det, angles_deg=theta[lo:hi]) for lo, hi in zip(cuts[:-1], cuts[1:])]
    for kind in ("hat", "adj"):
        whole = big.bp(y, kind).cpu().numpy()
        summed = sum(g.bp(y[lo * n_det:hi * n_det].contiguous(), kind).cpu().numpy()
                     for g, lo, hi in zip(parts, cuts[:-1], cuts[1:]))
        assert _rel(whole, summed) <= 1e-12, (kind, _rel(whole, summed))
    for g in parts + [big]:
        g.close()
    del y
    torch.cuda.empty_cache()


def test_forward_deterministic_and_stream_ordered(gpu_lib):
    import torch
    _, gg = _pair(dict(N=128, n_ang=64, n_det=183))
    x = torch.rand(gg.n, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        y1 = gg.fp(x)
        y2 = gg.fp(x)
    s.synchronize()
    assert torch.equal(y1, y2)


def test_config2_full_size_f32(gpu_lib):
    """Full-size image and sinogram of the single-solve workload (512^2, 720 x 725)."""
    import torch
    w = W.CONFIG2
    go, gg = _pair(dict(N=w.N, n_ang=w.n_ang, n_det=w.n_det))
    x = w.phantom()
    want = go.A(x)
    got = gg.fp(torch.tensor(x, dtype=torch.float32, device="cuda")).double().cpu().numpy()
    assert _rel(got, want) <= 1e-5
    for kind in ("hat", "adj"):
        want_b = go.back(kind)(want)
        got_b = gg.bp(torch.tensor(want, dtype=torch.float32, device="cuda"), kind).double().cpu().numpy()
        assert _rel(got_b, want_b) <= 1e-5, kind


def test_config3_sampled_f32(gpu_lib):
    """Large workload (2048^2, 1800 x 2897): the GPU applies the full operators; the
    oracle recomputes sampled sinogram rows (a geometry holding only those angles) and
    sampled pixels of the back projections."""
    import torch
    w = W.CONFIG3
    import paper_2110_01481_amd as abg
    gg = abg.Geometry(w.N, w.n_ang, w.n_det)
    go_full = O.Geometry(w.N, w.n_ang, w.n_det)
    x = w.phantom()
    y = gg.fp(torch.tensor(x, dtype=torch.float32, device="cuda")).double().cpu().numpy()
    rows = [0, 1, 449, 450, 899, 900, 901, 1349, 1799]
    sub = O.Geometry(w.N, 0, w.n_det, angles_deg=go_full.theta[rows])
    want_rows = sub.A(x).reshape(len(rows), w.n_det)
    got_rows = y.reshape(w.n_ang, w.n_det)[rows]
    assert _rel(got_rows, want_rows) <= 1e-5
    rng = np.random.default_rng(4)
    pix = np.concatenate([rng.integers(0, w.N * w.N, 150), [0, w.N - 1, w.N * w.N - 1, w.N * (w.N // 2) + w.N // 2]])
    yt = torch.tensor(y, dtype=torch.float32, device="cuda")
    ysn = yt.double().cpu().numpy()
    for kind in ("hat", "adj"):
        got = gg.bp(yt, kind).double().cpu().numpy()[pix]
        want = go_full.back_pixels(kind, ysn, pix)
        assert _rel(got, want) <= 1e-5, kind
    # partition of unity holds for every pixel at any size
    ones = torch.ones(gg.m, dtype=torch.float32, device="cuda")
    xb = gg.bp(ones, "hat")
    assert float((xb - w.n_ang).abs().max()) <= 1e-5 * w.n_ang


@pytest.mark.parametrize("n_ang,span,ds", [(65, 120.0, 1.0), (188, 120.0, 1.4), (100, 180.0, 1.0), (90, 90.0, 0.75)])
@pytest.mark.parametrize("kind", ["hat", "adj", "strip_t", "joseph_t"])
def test_back_orbits_are_as_accurate_as_tiles(gpu_lib, kind, n_ang, span, ds):
    """FP32 against FP64: the relative error of a back projection depends on the angles, not on
    the image's size, so 507^2 (orbits of four pixels) may be no further off than 352^2 (tiles).
    Over 25000 pixels and more the norms of two such errors differ by a few percent: 5%."""
    import torch
    import paper_2110_01481_amd as abg
    err = {}
    for N in (352, 507):
        gg = abg.Geometry(N, n_ang, int(1.42 * N / ds) | 1, ang_range=span, det_spacing=ds)
        y = torch.tensor(np.random.default_rng(N).uniform(size=gg.m).astype(np.float32), device="cuda")
        want = gg.bp(y.double(), kind)
        err[N] = float((gg.bp(y, kind).double() - want).norm() / want.norm())
        gg.close()
    assert err[507] <= 1.05 * err[352], err


@pytest.mark.parametrize("N", [1, 31, 32, 33, 64])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_forward_scratch_contents_do_not_matter(gpu_lib, N, dt):
    """The padding of the scratch copies is written with them, in the tiles at the image's
    edges: A x over a scratch full of NaN equals A x over a scratch of zeros, bit for bit, at
    images below, at and past a tile's size, for the line and the strip model (whose taps
    reach furthest past the edge)."""
    import torch
    abg = gpu_lib
    tdt = torch.float64 if dt == "f64" else torch.float32
    x = torch.tensor(np.random.default_rng(3).uniform(size=N * N), dtype=tdt, device="cuda")
    for model in ("line", "strip"):
        gg = abg.Geometry(N, 24, 2 * N + 3, model=model)
        gg.fp(x)
        (ws,) = gg._fp_ws.values()
        ws.fill_(0)
        want = gg.fp(x).clone()
        ws.fill_(255)
        got = gg.fp(x)
        assert torch.equal(got, want) and bool(torch.isfinite(got).all())
        gg.close()
