"""GPU parity of the batched banded solves and the stencil against the oracle
(element by element, FP64).  Every case prints what it runs before the GPU
call so a failure names its case."""
import math

import numpy as np
import pytest

from paper_2101_06550_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def chx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2101_06550_amd import chx as m
    m.load()
    return m


def penta(sigma):
    return (sigma, -4 * sigma, 1 + 6 * sigma, -4 * sigma, sigma)


def kappa_tol(coefs):
    """Forward-error tolerance of one FP64 solve: 20 eps kappa, kappa bounded by
    sum|coef| / (|c| - sum|off|) for diagonally dominant rows, else by 1+16 s."""
    P = len(coefs) // 2
    diag = abs(coefs[P])
    off = sum(abs(v) for k, v in enumerate(coefs) if k != P)
    if diag > off:
        kappa = (diag + off) / (diag - off)
    else:
        kappa = 1 + 16 * coefs[0]
    return max(2e-14, 20 * 2.2e-16 * kappa)


def run_solve(chx, kind, coefs, n, batch, layout, ld=None, periodic=True, seed=3):
    f = inputs.uniform(seed, (n, batch) if layout == 0 else (batch, n), -1, 1)
    if ld is not None:
        shape = (n, ld) if layout == 0 else (batch, ld)
        buf = np.full(shape, 7.25)
        if layout == 0:
            buf[:, :batch] = f
        else:
            buf[:, :n] = f
    else:
        buf = f
    x = torch.tensor(buf, dtype=torch.float64, device="cuda")
    print(f"[case] {kind} n={n} batch={batch} layout={layout} ld={ld} periodic={periodic}",
          flush=True)
    if kind == "penta":
        plan = chx.penta_factor(n, *coefs, periodic=periodic)
        chx.penta_solve_batch(plan, batch, x, ld=x.stride(0), layout=layout)
    else:
        plan = chx.tri_factor(n, *coefs, periodic=periodic)
        chx.tri_solve_batch(plan, batch, x, ld=x.stride(0), layout=layout)
    torch.cuda.synchronize()
    out = x.cpu().numpy()
    if ld is not None:
        pad = out[:, batch:] if layout == 0 else out[:, n:]
        assert np.all(pad == 7.25), "solve wrote outside the systems"
        out = out[:, :batch] if layout == 0 else out[:, :n]
    return f, out


def oracle_lines(orc, kind, coefs, f, layout, periodic=True):
    if periodic:
        direction = 1 if layout == 0 else 0
        if kind == "penta":
            return orc.cpenta_lines(f, direction, coefs)
        return orc.ctri_lines(f, direction, coefs)
    # non-periodic: the oracle's general LR / Thomas line by line
    sys_ = f.T if layout == 0 else f
    out = np.zeros_like(sys_)
    for s in range(sys_.shape[0]):
        n = sys_.shape[1]
        if kind == "penta":
            a, b, c, d, e = (np.full(n, v) for v in coefs)
            out[s] = orc.penta_lr_solve(a, b, c, d, e, sys_[s])
        else:
            a, b, c = (np.full(n, v) for v in coefs)
            out[s] = orc.tri_solve(a, b, c, sys_[s])
    return out.T if layout == 0 else out


def rel(out, ref):
    return np.max(np.abs(out - ref)) / np.max(np.abs(ref))


PENTA_CASES = [
    # (n, batch, sigma)  -- chunked paths need n % 32 == 0
    (1024, 1024, 0.5),      # standalone batched-solve workload
    (32, 64, 0.5), (64, 65, 2.7558), (96, 130, 44.092), (128, 1, 0.17224),
    (8192, 70, 2889.6), (256, 64, 70.547),
    (5, 17, 0.5), (6, 64, 1.0), (7, 3, 2.0), (50, 100, 0.3), (1000, 33, 70.547),
]


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n,batch,sigma", PENTA_CASES)
def test_penta_parity(chx, orc, n, batch, sigma, layout):
    co = penta(sigma)
    f, out = run_solve(chx, "penta", co, n, batch, layout)
    ref = oracle_lines(orc, "penta", co, f, layout)
    assert rel(out, ref) < kappa_tol(co)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n,batch", [(64, 40), (96, 64), (13, 10)])
def test_penta_nonsymmetric_and_ld(chx, orc, n, batch, layout):
    co = (0.21, -0.7, 3.9, 0.45, -0.33)
    f, out = run_solve(chx, "penta", co, n, batch, layout, ld=(batch + 7 if layout == 0 else n + 5))
    ref = oracle_lines(orc, "penta", co, f, layout)
    assert rel(out, ref) < kappa_tol(co)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n,batch,beta", [(1024, 1024, 0.5), (32, 64, 3.0), (96, 65, 0.5),
                                          (8192, 20, 200.0), (3, 5, 1.0), (77, 64, 0.5)])
def test_tri_parity(chx, orc, n, batch, beta, layout):
    co = (-beta, 1 + 2 * beta, -beta)
    f, out = run_solve(chx, "tri", co, n, batch, layout)
    ref = oracle_lines(orc, "tri", co, f, layout)
    assert rel(out, ref) < max(2e-14, 20 * 2.2e-16 * (1 + 4 * beta))


@pytest.mark.parametrize("layout", [0, 1])
def test_tri_nonsymmetric(chx, orc, layout):
    co = (0.4, 2.5, -0.7)
    f, out = run_solve(chx, "tri", co, 64, 33, layout)
    assert rel(out, oracle_lines(orc, "tri", co, f, layout)) < 1e-13


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("kind", ["penta", "tri"])
def test_non_periodic(chx, orc, kind, layout):
    co = penta(1.5) if kind == "penta" else (-1.5, 4.0, -1.5)
    f, out = run_solve(chx, kind, co, 64, 20, layout, periodic=False)
    ref = oracle_lines(orc, kind, co, f, layout, periodic=False)
    assert rel(out, ref) < 1e-13


def test_scaled_batch_sampled(chx, orc):
    """131072 interleaved systems of N = 1024 (1 GiB): every system solved on
    the GPU, a sample of 48 checked against the oracle one by one."""
    n, batch, sigma = 1024, 131072, 0.5
    co = penta(sigma)
    f = inputs.uniform(2, (n, batch), -1, 1)
    x = torch.tensor(f, device="cuda")
    print(f"[case] penta scaled batch n={n} batch={batch}", flush=True)
    plan = chx.penta_factor(n, *co)
    chx.penta_solve_batch(plan, batch, x, layout=0)
    torch.cuda.synchronize()
    cols = np.unique(np.concatenate([np.arange(8), batch - 1 - np.arange(8),
                                     inputs.uniform(9, (32,), 0, batch).astype(np.int64)]))
    out = x[:, torch.tensor(cols, device="cuda")].cpu().numpy()
    for k, s in enumerate(cols):
        ref = orc.cyclic_penta_solve(co, f[:, s])
        assert rel(out[:, k], ref) < kappa_tol(co)


def test_empty_batch_is_noop(chx):
    x = torch.zeros((32, 4), dtype=torch.float64, device="cuda")
    plan = chx.penta_factor(32, *penta(1.0))
    chx.penta_solve_batch(plan, 0, x, ld=4, layout=0)
    torch.cuda.synchronize()
    assert torch.all(x == 0)


def test_workspace_too_small(chx):
    x = torch.zeros((64, 64), dtype=torch.float64, device="cuda")
    plan = chx.penta_factor(64, *penta(1.0))
    ws = torch.empty(64, dtype=torch.uint8, device="cuda")
    with pytest.raises(chx.ChxError) as ei:
        chx.penta_solve_batch(plan, 64, x, layout=0, ws=ws)
    assert ei.value.status == chx.CHX_ENOMEM


def test_repeatable_bitwise(chx):
    f = inputs.uniform(4, (1024, 256), -1, 1)
    plan = chx.penta_factor(1024, *penta(70.547))
    outs = []
    for _ in range(2):
        x = torch.tensor(f, device="cuda")
        chx.penta_solve_batch(plan, 256, x, layout=0)
        torch.cuda.synchronize()
        outs.append(x.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])


# ------------------------------------------------------------------ stencil
STENCIL_CASES = [
    ((64, 64), (1, 1, 1, 1), 1, 0), ((70, 33), (2, 1, 0, 3), 1, 1), ((128, 200), (4, 4, 4, 4), 1, 0),
    ((65, 17), (0, 2, 2, 0), 0, 0), ((40, 130), (3, 3, 1, 1), 0, 1), ((5, 7), (2, 2, 2, 2), 1, 1),
    # fields smaller than the extent (repeated wrap), ragged tiles, one-sided
    # extents in every class
    ((3, 2), (4, 4, 4, 4), 1, 0), ((2, 200), (2, 2, 4, 4), 1, 0), ((1, 1), (1, 1, 1, 1), 1, 1),
    ((130, 65), (0, 3, 2, 1), 1, 1), ((67, 129), (4, 0, 0, 4), 0, 0),
    ((129, 191), (1, 4, 3, 0), 1, 0), ((64, 64), (0, 0, 0, 0), 1, 0),
]


@pytest.mark.parametrize("shape,ext,periodic,premap", STENCIL_CASES)
def test_stencil_parity(chx, orc, shape, ext, periodic, premap):
    ny, nx = shape
    left, right, top, bottom = ext
    x = inputs.uniform(6, shape, -1, 1)
    w = inputs.uniform(7, ((top + bottom + 1) * (left + right + 1),), -1, 1)
    xin = torch.tensor(x, device="cuda")
    xo = torch.full(shape, 3.5, dtype=torch.float64, device="cuda")
    print(f"[case] stencil shape={shape} ext={ext} periodic={periodic} premap={premap}", flush=True)
    chx.stencil2d_apply(xin, xo, list(w), left, right, top, bottom, periodic=bool(periodic),
                        premap=premap)
    torch.cuda.synchronize()
    ref = orc.stencil2d(x, w.reshape(top + bottom + 1, left + right + 1), left, right, top,
                        bottom, periodic=bool(periodic), premap=premap,
                        out=np.full(shape, 3.5))
    np.testing.assert_allclose(xo.cpu().numpy(), ref, rtol=0, atol=1e-13)


@pytest.mark.parametrize("shape,ext,periodic,premap", STENCIL_CASES)
def test_stencil_parity_f32(chx, orc, shape, ext, periodic, premap):
    """FP32 arrays (dtype CHX_F32): against the oracle's FP64 stencil of the
    same FP32 input with the FP32-rounded weights, point by point within the
    rounding bound of an FP32 sum of n products, (n + 4) 2^-24 sum |w| |pre(v)|
    (pre(v) = v^3 - v costs three more roundings)."""
    ny, nx = shape
    left, right, top, bottom = ext
    x = inputs.uniform(6, shape, -1, 1).astype(np.float32)
    w = inputs.uniform(7, ((top + bottom + 1) * (left + right + 1),), -1, 1)
    w32 = w.astype(np.float32).astype(np.float64)
    xin = torch.tensor(x, device="cuda")
    xo = torch.full(shape, 3.5, dtype=torch.float32, device="cuda")
    print(f"[case] stencil f32 shape={shape} ext={ext} periodic={periodic} premap={premap}",
          flush=True)
    chx.stencil2d_apply(xin, xo, list(w), left, right, top, bottom, periodic=bool(periodic),
                        premap=premap)
    torch.cuda.synchronize()
    x64 = x.astype(np.float64)
    W = w32.reshape(top + bottom + 1, left + right + 1)
    ref = orc.stencil2d(x64, W, left, right, top, bottom, periodic=bool(periodic),
                        premap=premap, out=np.full(shape, 3.5))
    mag = np.abs(x64) ** 3 + np.abs(x64) if premap else np.abs(x64)
    scale = orc.stencil2d(mag, np.abs(W), left, right, top, bottom, periodic=bool(periodic),
                          premap=0, out=np.zeros(shape))
    bound = (W.size + 4) * 2.0 ** -24 * scale + 1e-30
    err = np.abs(xo.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= bound), float(np.max(err / bound))


# Rows that are whole 16-byte vectors (2 FP64 or 4 FP32 columns) and rows that
# are not, around the 64 vectors of a tile; fields as wide as the reach, and
# fields that start off a vector's boundary.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,offset", [(4, 4, 0), (8, 15, 0), (64, 16, 0), (66, 17, 0),
                                          (126, 33, 0), (128, 16, 1), (128, 31, 0), (130, 32, 0),
                                          (252, 18, 0), (256, 16, 1), (256, 17, 0), (260, 47, 0),
                                          (261, 16, 0)])
def test_stencil_vectors_and_single_columns(chx, orc, nx, ny, offset, dtype):
    T, eps = (torch.float64, 2.0 ** -53) if dtype == "f64" else (torch.float32, 2.0 ** -24)
    x = torch.tensor(inputs.uniform(16, (ny, nx), -1, 1)).to(T)
    for ext in ((1, 1, 1, 1), (4, 0, 2, 4), (2, 3, 0, 0)):
        left, right, top, bottom = ext
        w = torch.tensor(inputs.uniform(17, ((top + bottom + 1) * (left + right + 1),), -1, 1)).to(T)
        W = w.double().numpy().reshape(top + bottom + 1, left + right + 1)
        for periodic in (True, False):
            print(f"[case] stencil {dtype} {nx}x{ny} ext={ext} periodic={periodic}", flush=True)
            bufs = [torch.full((ny * nx + 5,), 3.5, dtype=T, device="cuda") for _ in range(2)]
            xin, xo = [b[offset:offset + ny * nx].view(ny, nx) for b in bufs]
            xin.copy_(x)
            chx.stencil2d_apply(xin, xo, w.tolist(), left, right, top, bottom, periodic=periodic)
            torch.cuda.synchronize()
            ref = orc.stencil2d(x.double().numpy(), W, left, right, top, bottom,
                                periodic=periodic, out=np.full((ny, nx), 3.5))
            mag = orc.stencil2d(np.abs(x.double().numpy()), np.abs(W), left, right, top, bottom,
                                periodic=periodic, out=np.zeros((ny, nx)))
            err = np.abs(xo.double().cpu().numpy() - ref)
            assert np.all(err <= 2 * (W.size + 1) * eps * mag + 1e-300)
            rest = torch.cat([bufs[1][:offset], bufs[1][offset + ny * nx:]])
            assert torch.all(rest == 3.5)


# widths at which tiles of vectors begin to cover a row as well as single
# columns do, and on either side; heights whose tile counts leave 0 .. 7 tiles
# past eight equal bands
@pytest.mark.parametrize("ny,nx", [(131, 4), (67, 8), (33, 60), (161, 64), (97, 68), (65, 96),
                                   (129, 128), (49, 130), (81, 158), (113, 160), (33, 192),
                                   (145, 196), (17, 200), (177, 256), (35, 260), (21, 640)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_stencil_rows_of_any_width(chx, orc, ny, nx, dtype):
    """Against the oracle, every tile its own values: FP64 to 1e-13, FP32 to
    (terms + 2) eps of the sum of the magnitudes."""
    x = torch.from_numpy(inputs.uniform(41, (ny, nx), -1, 1)).to(dtype)
    for ext in ((1, 1, 1, 1), (2, 0, 1, 3), (0, 0, 2, 2), (4, 4, 4, 4)):
        left, right, top, bottom = ext
        w = torch.from_numpy(inputs.uniform(42, ((top + bottom + 1) * (left + right + 1),), -1,
                                            1)).to(dtype)
        W = w.double().numpy().reshape(top + bottom + 1, left + right + 1)
        for periodic in (True, False):
            print(f"[case] stencil {dtype} {ny}x{nx} ext={ext} periodic={periodic}", flush=True)
            xo = torch.full((ny, nx), 3.5, dtype=dtype, device="cuda")
            chx.stencil2d_apply(x.cuda(), xo, w.tolist(), left, right, top, bottom,
                                periodic=periodic)
            torch.cuda.synchronize()
            kw = dict(periodic=periodic, premap=0)
            ref = orc.stencil2d(x.double().numpy(), W, left, right, top, bottom,
                                out=np.full((ny, nx), 3.5), **kw)
            mag = orc.stencil2d(np.abs(x.double().numpy()), np.abs(W), left, right, top, bottom,
                                out=np.zeros((ny, nx)), **kw)
            tol = 1e-13 if dtype == torch.float64 else \
                (W.size + 2) * np.finfo(np.float32).eps * mag
            assert np.all(np.abs(xo.cpu().double().numpy() - ref) <= tol)


def test_narrow_stencil_is_not_tiled_for_wide_rows(chx):
    """Rows of 4 FP32 columns take about the time of rows of 5, whose length
    rules vectors out (13 us and 14; 76 in tiles of vectors), and rows of 130
    FP64 columns no more than rows of 131."""
    for dtype, ny, nx, ext in ((torch.float32, 100000, 4, 4), (torch.float64, 20000, 130, 0)):
        w = [0.1] * ((2 * ext + 1) * 9)
        best = []
        for n in (nx, nx + 1):
            x = torch.zeros((ny, n), dtype=dtype, device="cuda")
            o = torch.empty_like(x)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            ms = []
            for _ in range(12):
                e0.record()
                for _ in range(20):
                    chx.stencil2d_apply(x, o, w, ext, ext, 4, 4, periodic=False)
                e1.record()
                torch.cuda.synchronize()
                ms.append(e0.elapsed_time(e1) / 20)
            best.append(min(ms))
        print(f"[case] stencil {dtype} {ny}x{nx}: {best[0]:.4f} ms against {best[1]:.4f}",
              flush=True)
        assert best[0] < 1.6 * best[1]


@pytest.mark.parametrize("ext,premap", [((1, 1, 1, 1), 1), ((2, 2, 2, 2), 0), ((4, 4, 4, 4), 0),
                                         ((3, 0, 4, 1), 1)])
def test_stencil_full_size_sampled(chx, orc, ext, premap):
    """The benchmark's 8192 x 8192 periodic field: windows around sampled
    points (the four corners, tile edges, interior points) cut out of the
    field with periodic wrap, solved by the oracle as non-periodic stencils,
    whose interior equals the periodic result at those points."""
    n = 8192
    left, right, top, bottom = ext
    print(f"[case] stencil 8192^2 ext={ext} premap={premap}", flush=True)
    x = inputs.uniform(21, (n, n), -1, 1)
    w = inputs.uniform(22, ((top + bottom + 1) * (left + right + 1),), -1, 1)
    xin = torch.tensor(x, device="cuda")
    xo = torch.empty_like(xin)
    chx.stencil2d_apply(xin, xo, list(w), left, right, top, bottom, periodic=True, premap=premap)
    torch.cuda.synchronize()
    del xin
    half = 6
    for jc, ic in [(0, 0), (0, n - 1), (n - 1, 0), (n - 1, n - 1), (63, 64), (64, 63),
                   (4095, 4160), (5000, 127), (8127, 8128)]:
        rows = np.arange(jc - half - top, jc + half + bottom + 1) % n
        cols = np.arange(ic - half - left, ic + half + right + 1) % n
        win = x[np.ix_(rows, cols)]
        ref = orc.stencil2d(win, w.reshape(top + bottom + 1, left + right + 1), left, right, top,
                            bottom, periodic=False, premap=premap,
                            out=np.zeros_like(win))[top:top + 2 * half + 1,
                                                    left:left + 2 * half + 1]
        orows = np.arange(jc - half, jc + half + 1) % n
        ocols = np.arange(ic - half, ic + half + 1) % n
        got = xo[torch.tensor(orows, device="cuda")][:, torch.tensor(ocols, device="cuda")]
        np.testing.assert_allclose(got.cpu().numpy(), ref, rtol=0, atol=1e-13)


@pytest.mark.parametrize("periodic", [True, False])
def test_stencil_leading_dimension(chx, orc, periodic):
    """Input and output rows padded (ld = nx + 13): the stencil reads and
    writes only the nx columns of each row."""
    ny, nx, ld = 70, 130, 143
    left, right, top, bottom = 2, 1, 3, 2
    x = inputs.uniform(31, (ny, nx), -1, 1)
    w = inputs.uniform(32, ((top + bottom + 1) * (left + right + 1),), -1, 1)
    big_in = torch.full((ny, ld), float("nan"), dtype=torch.float64, device="cuda")
    big_in[:, :nx] = torch.tensor(x, device="cuda")
    big_out = torch.full((ny, ld), 3.5, dtype=torch.float64, device="cuda")
    print(f"[case] stencil ld={ld} periodic={periodic}", flush=True)
    chx.stencil2d_apply(big_in[:, :nx], big_out[:, :nx], list(w), left, right, top, bottom,
                        periodic=periodic, premap=1)
    torch.cuda.synchronize()
    ref = orc.stencil2d(x, w.reshape(top + bottom + 1, left + right + 1), left, right, top,
                        bottom, periodic=periodic, premap=1, out=np.full((ny, nx), 3.5))
    o = big_out.cpu().numpy()
    np.testing.assert_allclose(o[:, :nx], ref, rtol=0, atol=1e-13)
    assert np.all(o[:, nx:] == 3.5)


def test_stencil_eighth_order_example(chx):
    """Thesis Ch.3 "Standard Weights": 8th-order second derivative of sin x
    on 1024 x 512, non-periodic; interior equals -sin x, the 4 boundary
    cells on each side keep their initial zeros."""
    nx, ny = 1024, 512
    dx = 2 * math.pi / nx
    xs = np.arange(nx) * dx
    data = torch.tensor(np.tile(np.sin(xs), (ny, 1)), device="cuda")
    out = torch.zeros_like(data)
    w = np.array([-1 / 560, 8 / 315, -1 / 5, 8 / 5, -205 / 72, 8 / 5, -1 / 5, 8 / 315,
                  -1 / 560]) / dx ** 2
    chx.stencil2d_apply(data, out, list(w), 4, 4, 0, 0, periodic=False)
    o = out.cpu().numpy()
    assert np.abs(o[:, 4:-4] + np.sin(xs)[None, 4:-4]).max() < 1e-9
    assert np.all(o[:, :4] == 0) and np.all(o[:, -4:] == 0)


def test_stencil_argument_errors_leave_the_output_untouched(chx, orc):
    """Through the C-ABI itself: null arrays or weights, an unknown dtype,
    empty or short-pitched fields, extents outside 0..4, an unknown pre-map,
    overlapping input and output, and non-finite weights are refused with
    CHX_EINVAL before any launch; the output keeps its contents and a valid
    call afterwards still matches the oracle."""
    import ctypes
    lib = chx.load()
    ny, nx = 40, 48
    x = inputs.uniform(8, (ny, nx), -1, 1)
    w = inputs.uniform(9, (9,), -1, 1)
    xin = torch.tensor(x, device="cuda")
    xo = torch.full((ny, nx), 3.5, dtype=torch.float64, device="cuda")
    print("[case] stencil argument errors", flush=True)
    wbuf = (ctypes.c_double * 9)(*w)
    wnan = (ctypes.c_double * 9)(*w)
    wnan[4] = float("nan")
    st = chx._stream(None)
    bad = [dict(inp=None), dict(out=None), dict(w=None), dict(dtype=7), dict(nx=0),
           dict(ld=nx - 1), dict(left=-1), dict(bottom=5), dict(premap=2),
           dict(out=xin.data_ptr() + 8), dict(w=wnan)]
    for over in bad:
        g = dict(inp=xin.data_ptr(), out=xo.data_ptr(), nx=nx, ld=nx, dtype=chx.CHX_F64, w=wbuf,
                 left=1, right=1, top=1, bottom=1, premap=0)
        g.update(over)
        rc = lib.stencil2d_apply(g["inp"], g["out"], g["nx"], ny, g["ld"], g["dtype"], g["w"],
                                 g["left"], g["right"], g["top"], g["bottom"], 1, g["premap"], st)
        assert rc == chx.CHX_EINVAL, (over, rc)
    torch.cuda.synchronize()
    assert torch.all(xo == 3.5)
    assert np.array_equal(xin.cpu().numpy(), x)
    rc = lib.stencil2d_apply(xin.data_ptr(), xo.data_ptr(), nx, ny, nx, chx.CHX_F64, wbuf,
                             1, 1, 1, 1, 1, 0, st)
    assert rc == chx.CHX_OK
    torch.cuda.synchronize()
    ref = orc.stencil2d(x, w.reshape(3, 3), 1, 1, 1, 1, periodic=True, premap=0)
    np.testing.assert_allclose(xo.cpu().numpy(), ref, rtol=0, atol=1e-13)
