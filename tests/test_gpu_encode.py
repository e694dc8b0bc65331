"""GPU parity of the expanded encoding operators (FP32 form) against the FP64
oracle: whole-output comparisons at small sizes that span several tiles and
ragged tails, the adjoint identity, and
bitwise determinism.  Tolerance: relative l2 error <= 1e-5 (FP32 form)."""
import numpy as np
import pytest

import synth
from oracle import encoding
from tests.gpu_common import Case, c64, rel

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _ee():
    import paper_2211_07532_amd as ee
    return ee


def test_sh_basis_matches_oracle():
    import torch
    ee = _ee()
    for n, ny, fov, z0, nb in ((32, 32, 0.222, 0.0, 9), (148, 148, 0.222, 0.003, 16), (13, 7, 0.1, -0.006, 16)):
        b = ee.sh_basis(n, ny, fov, fov * ny / n, z0, nb, device="cuda").cpu().numpy()
        ref = encoding.sh_basis(n, fov, z0, nb, ny=ny, fov_y=fov * ny / n)
        assert np.max(np.abs(b - ref)) <= 1e-15 * np.max(np.abs(ref)) + 1e-300


@pytest.mark.parametrize("sh", [False, True], ids=["maps", "sh"])
@pytest.mark.parametrize("name", ["tiny", "ragged", "onecoil-nofield", "40coils"])
def test_forward_adjoint_whole_output(name, sh):
    import torch
    ee = _ee()
    if name == "tiny":
        w = synth.TINY
        case = Case(w, sh=sh)
        batch = 2
    elif name == "ragged":
        w = synth.Workload("ragged", 13, 0.1, 5, 333, 3e-6, 2.0, 16, 120.0, 20.0, 5, "haar", 1, 21)
        case = Case(w, z0=0.004, sh=sh)
        batch = 3
    elif name == "onecoil-nofield":
        w = synth.Workload("c1", 24, 0.2, 1, 600, 2e-6, 2.0, 3, 0.0, 20.0, 5, "haar", 1, 22)
        case = Case(w, with_dw0=False, nbasis=0, sh=sh)
        batch = 1
    else:
        w = synth.Workload("c40", 20, 0.2, 40, 700, 2e-6, 2.0, 9, 80.0, 20.0, 5, "haar", 1, 23)
        case = Case(w, sh=sh)
        batch = 1
    print(f"[case] {name} n={w.n} T={w.nsamples} C={case.smaps.shape[0]} L={case.coef.shape[1]} B={batch}",
          flush=True)
    x = c64(synth.random_complex((batch, w.npix), 31))
    x[0] = case.x_noisy
    y_ref = encoding.forward(x, *case.oracle_args())
    y = ee.forward(case.to_dev(x), case.op).cpu().numpy()
    assert y.shape == y_ref.shape
    assert rel(y, y_ref) <= TOL
    g = c64(synth.random_complex(y_ref.shape, 32))
    x_ref = encoding.adjoint(g, *case.oracle_args())
    xa = ee.adjoint(case.to_dev(g), case.op).cpu().numpy()
    assert rel(xa, x_ref) <= TOL
    # adjoint identity on the GPU results
    for b in range(batch):
        lhs = np.vdot(g[b], y[b])
        rhs = np.vdot(xa[b], x[b])
        assert abs(lhs - rhs) / (np.linalg.norm(y[b]) * np.linalg.norm(g[b])) <= 1e-6
    torch.cuda.synchronize()


def test_bitwise_determinism():
    ee = _ee()
    case = Case(synth.TINY)
    x = case.to_dev(case.x_noisy)
    y1 = ee.forward(x, case.op).cpu().numpy()
    y2 = ee.forward(x, case.op).cpu().numpy()
    assert np.array_equal(y1.view(np.uint32), y2.view(np.uint32))
    g = case.to_dev(y1)
    a1 = ee.adjoint(g, case.op).cpu().numpy()
    a2 = ee.adjoint(g, case.op).cpu().numpy()
    assert np.array_equal(a1.view(np.uint32), a2.view(np.uint32))


def test_invalid_arguments_raise():
    import torch
    ee = _ee()
    case = Case(synth.TINY)
    bad = torch.zeros(5, dtype=torch.complex64, device="cuda")
    with pytest.raises((ValueError, RuntimeError)):
        ee.forward(bad, case.op)


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1, 1, 1), (1, 7, 17, 3, 4, 2), (5, 3, 300, 2, 0, 1),
                                   (17, 2, 5, 17, 2, 1)],
                         ids=["1x1-T1-C1", "1x7-T17-C3-B2", "5x3-nofield", "17x2-T5-C17"])
def test_degenerate_shapes(shape, prec):
    """Degenerate geometries against the oracle: a single pixel and sample,
    a one-column image, no field terms, more coils than samples (basis given
    as maps, so any nx x ny)."""
    import torch
    ee = _ee()
    nx, ny, T, C, L, B = shape
    R = nx * ny
    rng = np.random.default_rng(7 + nx + 10 * ny + T)
    smaps = c64(synth.random_complex((C, R), 41 + C))
    coef = rng.normal(0.0, 2.0, (T, L))
    basis = rng.uniform(-1.0, 1.0, (L, R))
    time = np.arange(T, dtype=np.float64) * 2e-6
    dw0 = rng.uniform(-600.0, 600.0, R)
    x = c64(synth.random_complex((B, R), 43))
    dev = torch.device("cuda")
    op = ee.Operator(nx, ny, torch.from_numpy(smaps.astype(np.complex64)).to(dev), torch.from_numpy(coef).to(dev),
                     torch.from_numpy(time).to(dev), torch.from_numpy(basis).to(dev), torch.from_numpy(dw0).to(dev))
    print(f"[case] degenerate {nx}x{ny} T={T} C={C} L={L} B={B} {prec}", flush=True)
    bar = TOL if prec == "fp32" else 1e-3
    y_ref = encoding.forward(x, smaps, coef, time, basis, dw0)
    y = ee.forward(torch.from_numpy(x.astype(np.complex64)).to(dev), op, precision=prec).cpu().numpy()
    assert y.shape == y_ref.shape and rel(y, y_ref) <= bar
    g = c64(synth.random_complex(y_ref.shape, 44))
    xa = ee.adjoint(torch.from_numpy(g.astype(np.complex64)).to(dev), op, precision=prec).cpu().numpy()
    x_ref = encoding.adjoint(g, smaps, coef, time, basis, dw0)
    assert xa.shape == x_ref.shape and rel(xa, x_ref) <= bar


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1, 1), (3, 17, 40, 2, 1), (17, 3, 33, 5, 2), (33, 20, 100, 4, 1)],
                         ids=["1x1-T1", "3x17", "17x3-B2", "33x20"])
def test_degenerate_shapes_sh(shape, prec):
    """The solid-harmonic kind (the library evaluates the basis from the grid
    geometry and, in the split forms, runs the polynomial kernels) on
    degenerate and non-square grids with rectangular fields of view, 16 terms
    and dB0, against the oracle's basis on the same geometry."""
    import torch
    ee = _ee()
    nx, ny, T, C, B = shape
    fx, fy, z0, L = 0.1, 0.07, 0.003, 16
    R = nx * ny
    rng = np.random.default_rng(100 + nx + 10 * ny + T)
    basis = encoding.sh_basis(nx, fx, z0, L, ny=ny, fov_y=fy)
    scale = 3.0 / np.maximum(np.abs(basis).max(axis=1), 1e-12)   # a few radians per term at most
    coef = rng.normal(0.0, 1.0, (T, L)) * scale[None, :]
    time = np.arange(T, dtype=np.float64) * 2e-6
    dw0 = rng.uniform(-600.0, 600.0, R)
    smaps = c64(synth.random_complex((C, R), 51 + C))
    x = c64(synth.random_complex((B, R), 52))
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    op = ee.Operator(nx, ny, t(smaps.astype(np.complex64)), t(coef), t(time), None, t(dw0), sh_grid=(fx, fy, z0))
    print(f"[case] degenerate sh {nx}x{ny} T={T} C={C} B={B} {prec}", flush=True)
    bar = TOL if prec == "fp32" else 1e-3
    y_ref = encoding.forward(x, smaps, coef, time, basis, dw0)
    y = ee.forward(t(x.astype(np.complex64)), op, precision=prec).cpu().numpy()
    assert y.shape == y_ref.shape and rel(y, y_ref) <= bar
    g = c64(synth.random_complex(y_ref.shape, 53))
    xa = ee.adjoint(t(g.astype(np.complex64)), op, precision=prec).cpu().numpy()
    x_ref = encoding.adjoint(g, smaps, coef, time, basis, dw0)
    assert xa.shape == x_ref.shape and rel(xa, x_ref) <= bar


@pytest.mark.parametrize("sh", [False, True], ids=["maps", "sh"])
@pytest.mark.parametrize("T", [255, 257, 800])
def test_field_tables_at_tile_remainders(T, sh):
    """One-direction field setup (each call prepares only the tables it reads)
    where the sample axis ends inside an anchor workgroup's 512 samples and
    the pixel axis inside a tile; rectangular slice offset, two images for the
    FP32 form.  FP32 and fp16-split sums of a few hundred terms: 2e-6; a bf16
    pair carries 16 bits: 2e-5."""
    import paper_2211_07532_amd as ee
    w = synth.Workload("tables", 19, 0.1, 5, T, 3e-6, 2.0, 16, 120.0, 20.0, 5, "haar", 1, 31)
    case = Case(w, z0=0.004, sh=sh)
    args = case.oracle_args()
    x = c64(synth.random_complex((2, w.npix), 41))
    y = c64(synth.random_complex((2, T, w.ncoils), 42))
    for prec, batch, bar in (("fp32", 2, 2e-6), ("fp16", 1, 2e-6), ("fp16", 2, 2e-6), ("bf16", 1, 2e-5)):
        print(f"[case] tables T={T} sh={sh} {prec} batch={batch}", flush=True)
        f = ee.forward(case.to_dev(x[:batch]), case.op, precision=prec).cpu().numpy()
        a = ee.adjoint(case.to_dev(y[:batch]), case.op, precision=prec).cpu().numpy()
        for b in range(batch):
            assert rel(f[b], encoding.forward(x[b], *args)) <= bar
            assert rel(a[b], encoding.adjoint(y[b], *args)) <= bar


@pytest.mark.parametrize("shape", [
    (5, 200, 500, 3, 16, True, 1.0),       # 16-pixel rows: a workgroup's pixels span 17 image rows
    (100, 3, 1000, 20, 16, True, 1.0),     # fewer image rows than that; sample chunks that end inside an LDS block
    (31, 29, 1000, 33, 16, False, 1.0),    # 17 terms a row (split between LDS and scalar loads), three column groups
    (31, 29, 1000, 7, 9, False, 1.0),
    (31, 29, 1000, 16, 3, False, 1.0),
    (31, 29, 300, 8, 9, True, 1e-25),
    (31, 29, 300, 8, 9, False, 1e25),
], ids=lambda s: "x".join(str(v) for v in s))
def test_fp32_form_edges(shape):
    """The FP32 form's kernel variants (three-way bf16 products, FP64 phases)
    at the edges of their tiles and for operands far from 1, against the
    oracle.  Random sums of up to 1000 FP32 terms: 1e-6 is several times the
    sqrt(n) growth of a 2^-24 rounding."""
    import torch
    ee = _ee()
    nx, ny, T, C, L, sh, scale = shape
    fx, fy, z0 = 0.1, 0.07, 0.003
    R = nx * ny
    rng = np.random.default_rng(7 + nx + T + C + L)
    basis = encoding.sh_basis(nx, fx, z0, L, ny=ny, fov_y=fy)
    coef = rng.normal(0.0, 1.0, (T, L)) * (20.0 / np.maximum(np.abs(basis).max(axis=1), 1e-12))[None, :]
    time = np.arange(T, dtype=np.float64) * 2e-6
    dw0 = rng.uniform(-600.0, 600.0, R)
    smaps = c64(synth.random_complex((C, R), 61))
    x = c64(scale * synth.random_complex((1, R), 62))
    y = c64(scale * synth.random_complex((1, T, C), 63))
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    op = ee.Operator(nx, ny, t(smaps.astype(np.complex64)), t(coef), t(time), None if sh else t(basis), t(dw0),
                     sh_grid=(fx, fy, z0) if sh else None)
    args = (smaps, coef, time, basis, dw0)
    print(f"[case] fp32 edges {shape}", flush=True)
    yf = ee.forward(t(x.astype(np.complex64)), op).cpu().numpy().astype(np.complex128) / scale
    assert rel(yf[0], encoding.forward(x[0] / scale, *args)) <= 1e-6
    xa = ee.adjoint(t(y.astype(np.complex64)), op).cpu().numpy().astype(np.complex128) / scale
    assert rel(xa[0], encoding.adjoint(y[0] / scale, *args)) <= 1e-6


def _small_case(sh, scale=1.0, batch=1, seed=90):
    """A 31 x 29, 8-coil, 9-term operator with its oracle arguments and inputs
    rounded to complex64 after scaling."""
    import torch
    ee = _ee()
    nx, ny, T, C, L = 31, 29, 300, 8, 9
    fx, fy, z0 = 0.1, 0.07, 0.003
    rng = np.random.default_rng(seed)
    basis = encoding.sh_basis(nx, fx, z0, L, ny=ny, fov_y=fy)
    coef = rng.normal(0.0, 1.0, (T, L)) * (20.0 / np.maximum(np.abs(basis).max(axis=1), 1e-12))[None, :]
    time = np.arange(T, dtype=np.float64) * 2e-6
    dw0 = rng.uniform(-600.0, 600.0, nx * ny)
    smaps = c64(synth.random_complex((C, nx * ny), 61))
    x = c64(scale * synth.random_complex((batch, nx * ny), 62))
    y = c64(scale * synth.random_complex((batch, T, C), 63))
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    op = ee.Operator(nx, ny, t(smaps.astype(np.complex64)), t(coef), t(time), None if sh else t(basis), t(dw0),
                     sh_grid=(fx, fy, z0) if sh else None)
    dc = lambda a: t(a.astype(np.complex64))  # noqa: E731
    return op, (smaps, coef, time, basis, dw0), x, y, dc


@pytest.mark.parametrize("sh", [False, True], ids=["maps", "sh"])
@pytest.mark.parametrize("scale", [1e-37, 1e-35, 1e-33, 1e33])
def test_fp32_form_keeps_its_accuracy_over_the_fp32_range(scale, sh):
    """Operands close to the smallest normal FP32 value (and far above 1)
    reach the result with 24 bits: the same 1e-6 as at scale 1.  Two images,
    so that columns of one launch share a scale."""
    ee = _ee()
    op, args, x, y, dc = _small_case(sh, scale, batch=2)
    print(f"[case] fp32 range {scale:g} sh={sh}", flush=True)
    f = ee.forward(dc(x), op).cpu().numpy().astype(np.complex128) / scale
    a = ee.adjoint(dc(y), op).cpu().numpy().astype(np.complex128) / scale
    for b in range(2):
        assert rel(f[b], encoding.forward(x[b] / scale, *args)) <= 1e-6
        assert rel(a[b], encoding.adjoint(y[b] / scale, *args)) <= 1e-6


def test_fp32_normal_equations_keep_their_accuracy_at_small_scale():
    """The residual operand too: conjugate gradients on data of 1e-34 give the
    image of scale 1 times 1e-34 (every step is linear in the data; 20 FP32
    steps on a well-posed system, 1e-5)."""
    ee = _ee()
    op, args, _, _, dc = _small_case(True)
    x = c64(synth.random_complex((1, op.npix), 65))
    y = encoding.forward(x[0], *args)
    ref = ee.cg(dc(y), op, 20).cpu().numpy().astype(np.complex128)
    got = ee.cg(dc(1e-34 * y), op, 20).cpu().numpy().astype(np.complex128)
    assert np.all(np.isfinite(got)) and rel(got / 1e-34, ref) <= 1e-5


@pytest.mark.parametrize("sh", [False, True], ids=["maps", "sh"])
@pytest.mark.parametrize("value", [3.4e38, np.inf, np.nan])
def test_fp32_form_extreme_and_non_finite_operands(value, sh):
    """One element of 3.4e38, infinity or NaN.  The largest values stay finite
    where the result is; an infinity gives the infinities and NaN that real
    arithmetic gives (products of the phase's and the maps' signs, NaN where
    two of opposite sign meet); the other image of the batch is untouched."""
    ee = _ee()
    op, (smaps, coef, time, basis, dw0), x, y, dc = _small_case(sh, 0.0, batch=2)
    x[1] = c64(synth.random_complex((op.npix,), 66))
    y[1] = c64(synth.random_complex(y.shape[1:], 67))
    r0, t0, c0 = 500, 7, 2
    x[0, r0] = y[0, t0, c0] = value
    ph = encoding.phase(coef, time, basis, dw0)
    cs, sn = np.cos(ph), np.sin(ph)
    f = ee.forward(dc(x), op).cpu().numpy()
    a = ee.adjoint(dc(y), op).cpu().numpy()
    args = (smaps, coef, time, basis, dw0)
    # the finite image: 3.4e38 beside it takes the common scale and its bits
    # (2^-128 of the largest value); beside a non-finite one it keeps them
    if not np.isfinite(value):
        assert rel(f[1], encoding.forward(x[1], *args)) <= 1e-6
        assert rel(a[1], encoding.adjoint(y[1], *args)) <= 1e-6
    with np.errstate(all="ignore"):
        z = (smaps[:, r0].real * value, smaps[:, r0].imag * value)
        fr = cs[:, r0, None] * z[0] - sn[:, r0, None] * z[1]
        fi = cs[:, r0, None] * z[1] + sn[:, r0, None] * z[0]
        u = (cs[t0] * value, -sn[t0] * value)
        s = smaps[c0]
        ar, ai = s.real * u[0] + s.imag * u[1], s.real * u[1] - s.imag * u[0]
    clear = np.minimum(np.abs(cs), np.abs(sn)) > 1e-5      # (a sign that a rounded phase cannot change)
    # (a product S x above the FP32 range is infinite in FP32 arithmetic)
    zfits = np.broadcast_to(np.maximum(np.abs(z[0]), np.abs(z[1])) < 3.4e38, fr.shape)
    for got, ref, ok, in_range in ((f[0].real, fr, clear[:, r0], zfits), (f[0].imag, fi, clear[:, r0], zfits),
                                   (a[0].real, ar, clear[t0], None), (a[0].imag, ai, clear[t0], None)):
        got, ref = got[ok].astype(np.float64), ref[ok]
        if np.isfinite(value):
            fits = (np.abs(ref) < 3.4e38) & (True if in_range is None else in_range[ok])
            assert np.all(np.abs(got[fits] - ref[fits]) <= 1e-6 * value)
        else:
            np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("n,coils,T,terms", [(40, 8, 3000, 9), (64, 32, 5000, 16)])
@pytest.mark.parametrize("sh", [False, True], ids=["maps", "sh"])
def test_fp32_form_sums_without_bias(n, coils, T, terms, sh):
    """Random operands, where every output is a sum of many terms that nearly
    cancel, and coil maps that add up the outputs of neighbouring coils: the
    losses of the matrix instruction must neither grow with the sums nor add up
    over splits and coils.  A rounded phase entry is off by 8e-8 (turns rounded
    to FP32 5e-8, sine and cosine 6e-8), the sums and the result by 5e-8 and
    3e-8 more: 1e-7, so 1.5e-7."""
    import torch
    ee = _ee()
    w = synth.Workload("bias", n, 0.222, coils, T, 3e-6, 2.0, terms, 120.0, 20.0, 5, "haar", 1, 77)
    case = Case(w, sh=sh)
    x = c64(synth.random_complex((1, w.npix), 78))
    y = c64(synth.random_complex((1, T, coils), 79))
    args = case.oracle_args()
    f = rel(ee.forward(case.to_dev(x), case.op).cpu().numpy()[0], encoding.forward(x[0], *args))
    a = rel(ee.adjoint(case.to_dev(y), case.op).cpu().numpy()[0], encoding.adjoint(y[0], *args))
    print(f"[case] bias {n} px {coils} coils T={T} sh={sh}: forward {f:.2e}, adjoint {a:.2e}", flush=True)
    assert f <= 1.5e-7 and a <= 1.5e-7
