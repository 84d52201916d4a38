"""GPU parity of the wavefront kernels over the shapes their dispatch tells
apart: tiles per diagonal (rows 1 to 64), input channels (fused with the
wavefront up to 64, a projection of their own above), storage types,
memory-state matrices, masked layouts, and more rectangles than the one-launch
layout pass looks through."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

RTOL = {"f32": 1e-5, "bf16": 2e-2}  # the parity bounds of test_gpu_layer.py


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(built_lib):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


HEIGHTS = {1: [16, 1, 5], 2: [17, 32, 3], 3: [48, 33, 2], 4: [64, 49, 16]}
SHAPES = [  # hidden, dtype, c_in, memory states
    (4, "f32", 24, False), (8, "f32", 36, False), (16, "f32", 64, False), (16, "f32", 68, False),
    (32, "f32", 33, False), (32, "f32", 8, False), (64, "f32", 12, False), (32, "bf16", 40, False),
    (64, "bf16", 24, False), (64, "bf16", 72, False), (16, "f32", 20, True), (16, "f32", 72, True),
    (32, "f32", 40, True), (32, "f32", 32, True),
]


@pytest.mark.parametrize("nt", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", SHAPES, ids=[f"{d}_H{h}_C{c}{'_mem' if m else ''}" for h, d, c, m in SHAPES])
def test_wavefronts_against_oracle(shape, nt):
    import gpu_run
    import oracle_run
    from conftest import rel_err, rel_max
    from synth.configs import custom_workload

    H, dt, C, mem = shape
    hs, ws = HEIGHTS[nt], [9, 21, 1]
    kind = "padded" if (H + C) % 8 == 4 else "packed"  # some layouts with masked cells
    print(f"case wavefront H={H} C={C} {dt} memory={mem} heights={hs} widths={ws} {kind}", flush=True)
    wl = custom_workload(400 + 16 * SHAPES.index(shape) + nt, hs, ws, 40, C, H, dt)
    xs, params = wl.examples(), wl.params()
    if mem:
        params = (*params, wl.memory_params())
    dys = [wl.dy(k) for k in range(wl.n)]
    gpu = gpu_run.run_layer(xs, params, dys, hs, ws, 40, dtype=dt, kind=kind)
    ref = oracle_run.run_layer(xs, params, dys)
    pairs = [(f"{nm}[{k}]", g, r) for nm in ("Y", "dX") for k, (g, r) in enumerate(zip(gpu[nm], ref[nm]))]
    pairs += [(nm, gpu[nm], ref[nm]) for nm in ("dWx", "dU", "db") + (("dV",) if mem else ())]
    for nm, g, r in pairs:
        e, m = rel_err(g, r), rel_max(g, r)
        assert e <= RTOL[dt] and m <= RTOL[dt], (nm, e, m)


@pytest.mark.parametrize("H,dt,C,mem", [(4, "f32", 8, False), (16, "f32", 8, False), (32, "f32", 20, False),
                                        (64, "f32", 8, False), (32, "bf16", 16, False), (64, "bf16", 8, False),
                                        (16, "f32", 8, True), (32, "f32", 8, True)])
def test_units_of_every_height_in_one_launch(H, dt, C, mem):
    """300 narrow images of 1 to 64 rows: a workgroup runs units of one to four
    tiles one after another in the same LDS."""
    import gpu_run
    import oracle_run
    from conftest import rel_err, rel_max
    from synth.configs import custom_workload

    rng = np.random.default_rng(H)
    hs, ws = rng.integers(1, 65, 300), rng.integers(1, 5, 300)
    hs[:4] = [64, 1, 17, 48]
    print(f"case every height H={H} C={C} {dt} memory={mem}", flush=True)
    wl = custom_workload(640 + H + C + (dt == "bf16"), hs, ws, 200, C, H, dt)
    xs, params = wl.examples(), wl.params()
    if mem:
        params = (*params, wl.memory_params())
    dys = [wl.dy(k) for k in range(wl.n)]
    gpu = gpu_run.run_layer(xs, params, dys, hs, ws, 200, dtype=dt)
    ref = oracle_run.run_layer(xs, params, dys, workers=oracle_run.default_workers())
    pairs = [(nm, np.concatenate([t.ravel() for t in gpu[nm]]), np.concatenate([t.ravel() for t in ref[nm]]))
             for nm in ("Y", "dX")]
    pairs += [(nm, gpu[nm], ref[nm]) for nm in ("dWx", "dU", "db") + (("dV",) if mem else ())]
    for nm, g, r in pairs:
        e, m = rel_err(g, r), rel_max(g, r)
        assert e <= RTOL[dt] and m <= RTOL[dt], (nm, e, m)


@pytest.mark.parametrize("H,dt,C", [(16, "f32", 48), (32, "f32", 20), (64, "bf16", 40)])
def test_per_diagonal_schedule_gives_the_same_bits(H, dt, C):
    """The state read back between launches is the state kept in a unit."""
    import gpu_run
    from paper_1902_11208_amd import api
    from synth.configs import custom_workload

    hs, ws = [50, 17, 3], [12, 20, 7]
    print(f"case per-diagonal H={H} C={C} {dt}", flush=True)
    wl = custom_workload(700 + H, hs, ws, 40, C, H, dt)
    units, place, ch, cw, mask = gpu_run.layout(hs, ws, 40)
    wx, u, b = (gpu_run.to_dev(p, dt) for p in wl.params())
    x = api.pack_data([gpu_run.to_dev(e, dt) for e in wl.examples()], place, ch, cw)
    layer = api.MDLSTMLayer(wx, u, b, ch, cw, units, mask)
    y = layer.forward(x).clone()
    assert torch.equal(y, layer.forward_stepwise(x))


@pytest.mark.parametrize("H,dt,C", [(16, "f32", 48), (64, "f32", 20), (64, "bf16", 40)])
def test_recorded_diagonals_take_the_tensors_of_the_call(H, dt, C):
    """The launches recorded by one per-diagonal call serve the next one's
    inputs, input weights and biases, in other buffers."""
    import gpu_run
    from paper_1902_11208_amd import api
    from synth.configs import custom_workload

    hs, ws = [20, 17], [12, 9]
    print(f"case recorded diagonals H={H} C={C} {dt}", flush=True)
    units, place, ch, cw, mask = gpu_run.layout(hs, ws, 40)
    layer = None
    for seed in (720, 721, 722):
        wl = custom_workload(seed + H, hs, ws, 40, C, H, dt)
        wx, u, b = (gpu_run.to_dev(p, dt) for p in wl.params())
        x = api.pack_data([gpu_run.to_dev(e, dt) for e in wl.examples()], place, ch, cw)
        if layer is None:
            layer = api.MDLSTMLayer(wx, u, b, ch, cw, units, mask)
        layer.wx, layer.b = wx, b  # the same u, workspace and outputs: the same graph
        y = layer.forward(x).clone()
        layer.y.fill_(7)
        assert torch.equal(y, layer.forward_stepwise(x)), seed


def test_more_rectangles_than_the_layout_pass_lists():
    """5000 one-row examples: the ids are painted first and read from there;
    every output against the same examples in two smaller calls, bit for bit,
    and rows outside the rectangles zero."""
    from paper_1902_11208_amd import api

    rng = np.random.default_rng(5)
    ws = rng.integers(1, 4, 5000)
    print("case 5000 rectangles", flush=True)
    H, C = 4, 8
    g = torch.Generator().manual_seed(1)
    wx, u, b = (torch.randn(s, generator=g).mul(0.1).cuda() for s in ((4, 5 * H, C), (4, 5 * H, 2 * H), (4, 5 * H)))
    off = np.concatenate([[0], np.cumsum(ws)])
    pixels = torch.randn((int(off[-1]), C), generator=g).cuda()

    def run(sel):
        """Outputs of the selected examples, 100 to a canvas row."""
        slot = np.arange(len(sel))
        rects = np.stack([2 * (slot // 100), 4 * (slot % 100), np.ones_like(slot), ws[sel]], 1).astype(np.int32)
        ch, cw = 2 * (len(sel) // 100), 400
        idx = np.concatenate([r[0] * cw + r[1] + np.arange(r[3]) for r in rects])
        idx = torch.from_numpy(idx).long().cuda()
        mask = torch.zeros(ch * cw, dtype=torch.uint8, device="cuda")
        mask[idx] = 1
        x = torch.zeros((ch * cw, C), device="cuda")
        x[idx] = pixels[off[sel[0]]:off[sel[-1] + 1]]
        layer = api.MDLSTMLayer(wx, u, b, ch, cw, rects, mask.view(ch, cw))
        y = layer.forward(x.view(ch, cw, C)).view(ch * cw, 4 * H)
        assert not y[mask == 0].any()
        return y[idx]

    whole = run(np.arange(5000))
    halves = torch.cat([run(np.arange(2500)), run(np.arange(2500, 5000))])
    assert torch.equal(whole, halves)


@pytest.mark.parametrize("dt,c", [("f32", 4), ("f32", 5), ("bf16", 8), ("bf16", 4)])
def test_scatter_and_gather_keep_every_byte(dt, c):
    """16-byte copies, and the narrower ones for channels or pointers that are
    not aligned to them."""
    from paper_1902_11208_amd import api

    td = torch.bfloat16 if dt == "bf16" else torch.float32
    hs, ws = [3, 2, 7], [5, 9, 1]
    print(f"case scatter {dt} c={c}", flush=True)
    rects, ch, _ = api.pack_layout(hs, ws, 16)
    for shift in (0, 1):  # 1: examples that start off a 16-byte boundary
        ex = [torch.randn(h * w * c + shift, device="cuda").to(td)[shift:].view(h, w, c) for h, w in zip(hs, ws)]
        canvas = api.pack_data(ex, rects, ch, 16)
        want = torch.zeros((ch, 16, c), dtype=td, device="cuda")
        for e, (y0, x0, h, w) in zip(ex, rects.tolist()):
            want[y0:y0 + h, x0:x0 + w] = e
        assert torch.equal(canvas, want)
        for e, o in zip(ex, api.unpack_data(canvas, rects)):
            assert torch.equal(e, o)


@pytest.mark.parametrize("C", [16, 40])
def test_pre_activations_are_rounded_without_bias(C):
    """Mean error of each candidate tanh(Wx x + b) over 76800 cells, read from
    the workspace, which starts with the activated gates [cell][direction]
    [gate][unit]. Roundings of mean zero leave 2e-8 / sqrt(76800) * 4 = 3e-10
    over the sixteen units of a direction; the tanh's own error, 2.2e-9 towards
    zero, up to 2.2e-9 * 4 times the share by which one sign prevails (below a
    half with these biases). A bias added to a coarse sum, which rounds the same
    way in every cell, left 8e-9 to 1.2e-8."""
    from paper_1902_11208_amd import api

    H, h, w = 16, 48, 1600
    print(f"case bias C={C}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.rand(s, generator=g, device="cuda")  # noqa: E731
    wx, b = (rnd(4, 5 * H, C) - 0.5) * 0.2, (rnd(4, 5 * H) - 0.5) * 0.2
    x = torch.randn((h, w, C), generator=g, device="cuda")
    mask = torch.ones((h, w), dtype=torch.uint8, device="cuda")
    layer = api.MDLSTMLayer(wx, torch.zeros((4, 5 * H, 2 * H), device="cuda"), b, h, w, [[0, 0, h, w]], mask)
    layer.forward(x)
    got = layer.workspace[: h * w * 20 * H * 4].view(torch.float32).view(h * w, 4, 5, H)[:, :, 4].double()
    z = torch.matmul(x.view(-1, C).double(), wx[:, 4 * H:].double().reshape(-1, C).T.contiguous()).view(-1, 4, H)
    mean = (got - (z + b[:, 4 * H:].double()).tanh()).mean(0).norm(dim=1)
    print(mean.tolist())
    assert mean.max() <= 4.5e-9
