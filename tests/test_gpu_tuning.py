"""Kernel choices of a Cahn-Hilliard handle on the GPU: what a refused, a
repeated and a restored choice leave, and which kernels the choices reach."""
import math

import numpy as np
import pytest

from paper_2101_06550_amd import inputs
from test_gpu_solves import chx, rel  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

L = 2 * math.pi


def stepped(chx, h, c0, n=3):  # noqa: F811
    """State and diagnostics after n steps of one call from c0."""
    c = torch.tensor(c0, device="cuda")
    d = torch.zeros(2 * (n + 1), dtype=torch.float64, device="cuda")
    chx.ch_adi_step(h, c, nsteps=n, diag_out=d)
    torch.cuda.synchronize()
    return c.cpu().numpy(), d.cpu().numpy()


def same(a, b):
    return np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("ny,nx", [(128, 128), (256, 256), (90, 203)])
def test_refused_choice_changes_nothing(chx, ny, nx):  # noqa: F811
    """Unknown choices and values out of range are refused and leave every
    choice, and the steps bit for bit, as they were."""
    c0 = inputs.noise_field(ny, nx, 31)
    h = chx.ch_create(nx, ny, L, L, 1.0, 0.01, 1e-5)
    whats = range(chx.CHX_TUNE_REDUCED_SHAPE, chx.CHX_TUNE_ROW_CHUNK + 1)
    before = [chx.ch_get_tuning(h, w) for w in whats]
    print(f"[case] refused choices {ny}x{nx}", flush=True)
    ref = stepped(chx, h, c0)
    bad = [(99, 0), (-1, 0), (chx.CHX_TUNE_REDUCED_SHAPE, chx.CHX_NUM_REDUCED_SHAPES),
           (chx.CHX_TUNE_REDUCED_SHAPE, -1), (chx.CHX_TUNE_SMALL_PATH, 2),
           (chx.CHX_TUNE_ROW_SPLIT, 0), (chx.CHX_TUNE_ROW_SPLIT, -3),
           (chx.CHX_TUNE_COLUMN_ORDER, chx.CHX_NUM_COLUMN_ORDERS), (chx.CHX_TUNE_GRAPH, 2),
           (chx.CHX_TUNE_COLUMN_CHUNK, 8), (chx.CHX_TUNE_ROW_CHUNK, 64)]
    for what, value in bad:
        with pytest.raises(chx.ChxError) as ei:
            chx.ch_set_tuning(h, value, what=what)
        assert ei.value.status == chx.CHX_EINVAL, (what, value)
        assert [chx.ch_get_tuning(h, w) for w in whats] == before, (what, value)
        assert same(stepped(chx, h, c0), ref), (what, value)


@pytest.mark.parametrize("ny,nx,scheme,two", [
    (64, 64, 0, 1), (128, 128, 0, 1), (1024, 1024, 0, 1), (90, 203, 0, 1), (2048, 64, 0, 0),
    (5, 130, 0, 0), (128, 128, 1, 1), (90, 203, 1, 1), (4096, 1024, 1, 0),
    (1280, 2048, 1, 1), (1312, 2048, 1, 0), (1536, 64, 1, 1), (1568, 64, 1, 0),
    (1568, 1024, 1, 1), (1568, 960, 1, 0), (2048, 70, 1, 1)])
def test_two_launch_choice_is_read_cleared_and_restored(chx, ny, nx, scheme, two):  # noqa: F811
    """CHX_TUNE_TWO_LAUNCH says how unforced steps run; 0 leaves the other
    routes, to rounding; 1 brings the same bits back, and is refused where
    the handle has no such route."""
    c0, p0 = inputs.noise_field(ny, nx, 32), inputs.noise_field(ny, nx, 33)
    h = chx.ch_create(nx, ny, L, L, 1.0, 0.01, 1e-6, scheme=scheme)
    what = chx.CHX_TUNE_TWO_LAUNCH

    def run():
        if scheme == chx.CHX_SCHEME_P1:
            return stepped(chx, h, c0)
        c, p = torch.tensor(c0, device="cuda"), torch.tensor(p0, device="cuda")
        chx.ch_adi_step_p2(h, c, p, nsteps=3)
        torch.cuda.synchronize()
        return c.cpu().numpy(), p.cpu().numpy()

    print(f"[case] two-launch choice {ny}x{nx} scheme {scheme}", flush=True)
    assert chx.ch_get_tuning(h, what) == two
    ref = run()
    chx.ch_set_tuning(h, 0, what=what)
    assert chx.ch_get_tuning(h, what) == 0
    other = run()
    # three steps' solves to 20 eps (1 + 16 s); the thesis scheme doubles
    # what it carries on in every step
    s = 0.01 * 1e-6 / (L / max(nx, ny)) ** 4
    tol = 3 * max(1e-12, 20 * np.finfo(float).eps * (1 + 16 * s)) * (8 if scheme else 1)
    assert np.max(np.abs(other[0] - ref[0])) < tol * np.max(np.abs(ref[0]))
    if two:
        assert not np.array_equal(other[0], ref[0])  # another route did run
        chx.ch_set_tuning(h, 1, what=what)
        assert chx.ch_get_tuning(h, what) == 1
        assert same(run(), ref)
    else:
        assert same(other, ref)
        with pytest.raises(chx.ChxError):
            chx.ch_set_tuning(h, 1, what=what)


@pytest.mark.parametrize("ny,nx", [(128, 128), (256, 256), (64, 4096)])
def test_choices_written_back_restore_the_steps(chx, ny, nx):  # noqa: F811
    """Every choice read, changed and written back in the order of the
    choices: the steps are bit for bit what they were."""
    c0 = inputs.noise_field(ny, nx, 34)
    h = chx.ch_create(nx, ny, L, L, 1.0, 0.01, 1e-6)
    whats = range(chx.CHX_TUNE_REDUCED_SHAPE, chx.CHX_TUNE_TWO_LAUNCH + 1)
    before = [chx.ch_get_tuning(h, w) for w in whats]
    print(f"[case] choices written back {ny}x{nx}", flush=True)
    ref = stepped(chx, h, c0)
    chx.ch_set_tuning(h, 0, what=chx.CHX_TUNE_SMALL_PATH)
    chx.ch_set_tuning(h, -1, what=chx.CHX_TUNE_ROW_SPLIT)
    for w in (chx.CHX_TUNE_COLUMN_CHUNK, chx.CHX_TUNE_ROW_CHUNK):
        chx.ch_set_tuning(h, 32, what=w)
    assert chx.ch_get_tuning(h, chx.CHX_TUNE_TWO_LAUNCH) == 0
    stepped(chx, h, c0)
    split = chx.CHX_TUNE_ROW_SPLIT  # a fused split needs the chunks back first, and they its absence
    for w in sorted(whats, key=lambda w: (w == chx.CHX_TUNE_TWO_LAUNCH, w == split)):
        chx.ch_set_tuning(h, before[w], what=w)
    assert [chx.ch_get_tuning(h, w) for w in whats] == before
    assert same(stepped(chx, h, c0), ref)


def launched(call):
    """Names and counts of what a call did on the device's runtime."""
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return {e.key: e.count for e in p.key_averages()}


@pytest.mark.parametrize("ny,nx,small", [(64, 64, 0), (128, 128, 0), (256, 256, 0), (90, 203, 0),
                                         (128, 128, 1)])
def test_graph_choice_replays_the_two_launch_step(chx, ny, nx, small):  # noqa: F811
    """With CHX_TUNE_GRAPH a call of the two-launch step is one graph launch
    (grids that the single-workgroup path and the chunked passes also take
    among them), the single-workgroup path still launches directly; replays
    with eager work between give the eager bits."""
    c0 = inputs.noise_field(ny, nx, 35)
    h = chx.ch_create(nx, ny, L, L, 1.0, 0.01, 1e-6)
    if small:
        chx.ch_set_tuning(h, 1, what=chx.CHX_TUNE_SMALL_PATH)
    c = torch.empty((ny, nx), dtype=torch.float64, device="cuda")
    d = torch.zeros(8, dtype=torch.float64, device="cuda")
    ws = torch.empty(chx.ch_ws_bytes(h) + 256, dtype=torch.uint8, device="cuda")

    def call():
        chx.ch_adi_step(h, c, nsteps=3, diag_out=d, ws=ws)

    outs = []
    for k in range(5):
        if k == 1:
            chx.ch_set_tuning(h, 1, what=chx.CHX_TUNE_GRAPH)
        print(f"[case] graph {ny}x{nx} small {small} call {k}", flush=True)
        c.copy_(torch.from_numpy(c0))
        d.zero_()
        if k == 3:
            seen = launched(call)
            assert seen.get("hipGraphLaunch", 0) == (0 if small else 1), seen
            assert seen.get("hipLaunchKernel", 0) == (1 if small else 0), seen
        else:
            call()
        torch.cuda.synchronize()
        outs.append((c.cpu().numpy(), d.cpu().numpy()))
    for o in outs[1:]:
        assert same(o, outs[0])


# (ny, nx, two launches, single workgroup, graph): every way a P1 FP64 step runs
WAYS = [(128, 128, 1, 0, 0), (128, 128, 1, 0, 1), (128, 128, 0, 1, 0), (128, 128, 0, 0, 0),
        (128, 128, 0, 0, 1), (1024, 1024, 1, 0, 1), (1024, 1024, 0, 0, 0), (1024, 1024, 0, 0, 1),
        (90, 203, 1, 0, 0), (90, 203, 0, 0, 0)]


def handle_for(chx, ny, nx, two, small, graph, dt):  # noqa: F811
    h = chx.ch_create(nx, ny, L, L, 1.0, 0.01, dt)
    if nx % 64 == 0 and nx * ny <= 16384:
        chx.ch_set_tuning(h, small, what=chx.CHX_TUNE_SMALL_PATH)
    chx.ch_set_tuning(h, two, what=chx.CHX_TUNE_TWO_LAUNCH)
    chx.ch_set_tuning(h, graph, what=chx.CHX_TUNE_GRAPH)
    return h


@pytest.mark.parametrize("ny,nx,two,small,graph", WAYS)
def test_every_way_keeps_to_the_columns_of_a_padded_field(chx, orc, ny, nx, two, small,  # noqa: F811
                                                          graph):
    """Two calls of one step in a field of leading dimension nx + 72: the
    oracle's result, the padding as it was."""
    dt = 1e-6
    c0 = inputs.noise_field(ny, nx, 36)
    h = handle_for(chx, ny, nx, two, small, graph, dt)
    big = torch.full((ny, nx + 72), 7.0, dtype=torch.float64, device="cuda")
    big[:, :nx] = torch.tensor(c0, device="cuda")
    ws = torch.empty(chx.ch_ws_bytes(h) + 256, dtype=torch.uint8, device="cuda")
    print(f"[case] padded field {ny}x{nx} two {two} small {small} graph {graph}", flush=True)
    for _ in range(2):
        chx.ch_adi_step(h, big, nsteps=1, ws=ws)
    torch.cuda.synchronize()
    b = big.cpu().numpy()
    ref = orc.ch_step(orc.ch_step(c0, L, L, 1.0, 0.01, dt), L, L, 1.0, 0.01, dt)
    assert rel(b[:, :nx], ref) < 2e-12
    assert np.all(b[:, nx:] == 7.0)


@pytest.mark.parametrize("ny,nx,two,small,graph", WAYS)
def test_every_way_refuses_bad_arguments_before_it_writes(chx, orc, ny, nx, two, small,  # noqa: F811
                                                          graph):
    """Through the C-ABI: a null field, ld < nx, nsteps < 1 and a workspace
    missing, short or off its alignment are refused with their codes, the
    field and the next valid call are as if they had not been made."""
    lib = chx.load()
    dt = 1e-6
    c0 = inputs.noise_field(ny, nx, 37)
    h = handle_for(chx, ny, nx, two, small, graph, dt)
    c = torch.tensor(c0, device="cuda")
    need = lib.ch_ws_bytes(h.handle)
    ws = torch.zeros(need + 512, dtype=torch.uint8, device="cuda")
    aligned = (ws.data_ptr() + 255) // 256 * 256
    st = chx._stream(None)
    print(f"[case] bad arguments {ny}x{nx} two {two} small {small} graph {graph}", flush=True)
    good = dict(c=c.data_ptr(), ld=nx, nsteps=2, ws=aligned, avail=need)
    for over, code in ((dict(c=None), chx.CHX_EINVAL), (dict(ld=nx - 1), chx.CHX_EINVAL),
                       (dict(nsteps=0), chx.CHX_EINVAL), (dict(nsteps=-3), chx.CHX_EINVAL),
                       (dict(ws=None), chx.CHX_ENOMEM), (dict(avail=need - 8), chx.CHX_ENOMEM),
                       (dict(ws=aligned + 8), chx.CHX_EINVAL)):
        a = dict(good, **over)
        rc = lib.ch_adi_step(h.handle, a["c"], a["ld"], a["nsteps"], None, a["ws"], a["avail"], st)
        assert rc == code, (over, rc)
    torch.cuda.synchronize()
    assert np.array_equal(c.cpu().numpy(), c0)
    assert lib.ch_adi_step(h.handle, good["c"], nx, 2, None, aligned, need, st) == chx.CHX_OK
    torch.cuda.synchronize()
    ref = orc.ch_step(orc.ch_step(c0, L, L, 1.0, 0.01, dt), L, L, 1.0, 0.01, dt)
    assert rel(c.cpu().numpy(), ref) < 2e-12
