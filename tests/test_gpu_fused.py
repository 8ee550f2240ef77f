"""Solves and 1D steps of any length on the GPU: systems whose chunks one
workgroup holds (interleaved), rows of any length through LDS (contiguous),
against the oracle at the edges of their ranges -- one chunk, a chunk and a
short one, the shortest remainder, lengths with no even split, the longest
systems a workgroup holds and the first it does not, batches around the tile
widths, padded leading dimensions."""
import math

import numpy as np
import pytest

from paper_2101_06550_amd import inputs
from test_gpu_solves import chx, kappa_tol, oracle_lines, penta, rel, run_solve  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LENGTHS = [3, 5, 6, 7, 9, 31, 33, 34, 37, 38, 63, 65, 95, 97, 256, 257, 993, 997, 1000, 1024,
           1025, 2016, 2047, 2048, 2049, 2050, 4097]


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("n", LENGTHS)
def test_any_length(chx, orc, n, layout):  # noqa: F811
    for kind, co, lo in (("penta", penta(0.5), 5), ("penta", (0.21, -0.7, 3.9, 0.45, -0.33), 5),
                         ("penta", penta(70.547), 5), ("tri", (-0.5, 2.0, -0.5), 3),
                         ("tri", (0.4, 2.5, -0.7), 3)):
        if n < lo:
            continue
        for batch, pad in ((1, 0), (15, 4), (17, 1), (64, 0), (65, 3)):
            ld = (batch if layout == 0 else n) + pad
            f, out = run_solve(chx, kind, co, n, batch, layout, ld=ld)
            ref = oracle_lines(orc, kind, co, f, layout)
            assert rel(out, ref) < kappa_tol(co), (kind, co, batch)


@pytest.mark.parametrize("n,batch", [(1000, 4100), (96, 40000), (64, 70000), (100, 40001)])
@pytest.mark.parametrize("layout", [0, 1])
def test_wide_batches(chx, orc, n, batch, layout):  # noqa: F811
    """Batches wide enough for the larger tiles (32 and 64 systems per
    workgroup, many rows per workgroup), the last tile ragged: sampled."""
    co = penta(2.7558)
    f = inputs.uniform(8, (n, batch) if layout == 0 else (batch, n), -1, 1)
    x = torch.tensor(f, device="cuda")
    print(f"[case] wide batch n={n} batch={batch} layout={layout}", flush=True)
    chx.penta_solve_batch(chx.penta_factor(n, *co), batch, x, layout=layout)
    torch.cuda.synchronize()
    pick = [0, 1, 15, 16, 31, 32, 63, 64, 65, batch // 2, batch - 18, batch - 2, batch - 1]
    out = x.cpu().numpy()
    ref = oracle_lines(orc, "penta", co, f[:, pick] if layout == 0 else f[pick], layout)
    got = out[:, pick] if layout == 0 else out[pick]
    assert rel(got, ref) < kappa_tol(co)


B1D = [(0, 64, 100, 1.0, 1e-9, 1.0, 1.0), (0, 61, 17, 1.0, 1e-9, 1.0, 1.0),
       (0, 7, 5, 1.0, 1e-6, 1.0, 1.0), (0, 101, 70, 1.0, 1e-9, 1.0, 1.0),
       (1, 3, 9, 1.0, 1e-4, 1.0, 1.0), (1, 96, 65, 1.0, 1e-4, 1.0, 1.0),
       (1, 99, 33, 1.0, 1e-4, 1.0, 1.0), (1, 1023, 18, 1.0, 1e-6, 1.0, 1.0),
       (2, 33, 16, 2 * math.pi, 1e-3, 0.01, 1.0), (2, 130, 64, 2 * math.pi, 1e-3, 0.01, 1.0),
       (2, 2048, 20, 2 * math.pi, 1e-5, 0.01, 1.0), (2, 2047, 20, 2 * math.pi, 1e-5, 0.01, 1.0),
       (2, 2050, 20, 2 * math.pi, 1e-5, 0.01, 1.0)]


@pytest.mark.parametrize("kind,n,batch,L,dt,a,D", B1D)
def test_steps_in_one_call(chx, orc, kind, n, batch, L, dt, a, D):  # noqa: F811
    """Five steps in one call, in place in a padded array, against the oracle
    (each step's solve to 20 eps kappa, kappa = 1 + 16 s) and the same steps
    one call at a time, bitwise."""
    x0 = inputs.uniform(70 + kind, (n, batch), -0.1, 0.1)
    b = chx.batch1d_create(kind, n, L, dt, a, D)
    print(f"[case] batch1d five steps kind={kind} n={n} batch={batch}", flush=True)
    outs = []
    for calls, steps in ((1, 5), (5, 1)):
        buf = torch.full((n, batch + 3), 7.25, dtype=torch.float64, device="cuda")
        buf[:, :batch] = torch.from_numpy(x0)
        for _ in range(calls):
            chx.batch1d_step(b, buf[:, :batch], nsteps=steps)
        torch.cuda.synchronize()
        out = buf.cpu().numpy()
        assert np.all(out[:, batch:] == 7.25)
        outs.append(out[:, :batch])
    dx = L / n
    s = {0: a * dt / (2 * dx ** 4), 1: a * dt / (2 * dx ** 2), 2: a * D * dt / dx ** 4}[kind]
    tol = 5 * max(1e-12, 20 * np.finfo(float).eps * (1 + 16 * s))
    assert rel(outs[0], orc.batch1d_step(kind, x0, L, dt, a, D, nsteps=5)) < tol
    if n <= 2048:
        assert np.array_equal(outs[0], outs[1])
