"""GPU parity with the float64 oracle where operands are infinite, or states
overflow: NaN and either infinity in the same places, everything else within
the parity bound. fp32 products run on bf16 pieces, which an infinite value
does not have."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

RTOL = {"f32": 1e-5, "bf16": 2e-2}  # the parity bounds of test_gpu_layer.py


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(built_lib):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _same(name, got, ref, tol):
    got, ref = np.asarray(got), np.asarray(ref)
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(got), kind(ref)), (name, kind.__name__, int(kind(got).sum()), int(kind(ref).sum()))
    fin = np.isfinite(ref)
    if fin.any():
        err = np.linalg.norm(got[fin] - ref[fin]) / max(np.linalg.norm(ref[fin]), 1e-30)
        assert err <= tol, (name, err)


SHAPES = [  # hidden, dtype, c_in, memory states, tallest rectangle
    (4, "f32", 8, False, 5), (16, "f32", 24, False, 40), (16, "f32", 72, False, 17), (32, "f32", 40, False, 20),
    (50, "f32", 33, False, 20), (64, "f32", 12, False, 9), (16, "f32", 20, True, 33), (32, "f32", 40, True, 50),
    (32, "bf16", 40, False, 20),
]
IDS = [f"{d}_H{h}_C{c}_h{t}{'_mem' if m else ''}" for h, d, c, m, t in SHAPES]


@pytest.mark.parametrize("where", ["x", "wx", "u", "largest"])
@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_forward_with_infinite_operands(shape, where):
    import gpu_run
    import oracle_run
    from synth.configs import custom_workload

    H, dt, C, mem, tall = shape
    if H == 50 and where != "wx":
        pytest.skip("padded hidden units multiply an infinite value by their zero weights")
    hs, ws = [tall, 3, 4], [7, 9, 5]
    print(f"case infinite {where} H={H} C={C} {dt} memory={mem}", flush=True)
    wl = custom_workload(800 + SHAPES.index(shape), hs, ws, 40, C, H, dt)
    xs = [x.copy() for x in wl.examples()]
    params = [p.copy() for p in wl.params()]
    if where == "x":
        xs[0][1, 2, 3], xs[0][tall - 1, 6, C - 1] = np.inf, -np.inf
        xs[1][2, 4, 0], xs[1][2, 4, C // 2] = np.inf, np.inf  # NaN where their weights differ in sign
        params[0][1, 2 * H + 1, 3] = 0.0  # inf * 0
    elif where == "wx":
        params[0][0, 1, 2], params[0][2, 4 * H + 1, C - 1] = np.inf, -np.inf
        xs[2][1, 1, 2] = 0.0  # inf * 0
    elif where == "u":
        params[1][1, H + 1, 2] = np.inf  # meets h = 0 on the first diagonal
    else:
        xs[0][2, 3, 1] = np.finfo(np.float32).max if dt == "f32" else 3.3895313892515355e38
    if mem:
        params.append(wl.memory_params())
    with np.errstate(all="ignore"):
        ref = oracle_run.run_layer(xs, params, None, backward=False)
    gpu = gpu_run.run_layer(xs, params, None, hs, ws, 40, dtype=dt, backward=False)
    for k in range(3):
        _same(f"Y[{k}]", gpu["Y"][k], ref["Y"][k], RTOL[dt])


@pytest.mark.parametrize("H", [16, 32])
def test_overflowed_states_saturate_their_gates(H):
    """Forget gates near 1 add up both predecessors' states, which pass the
    largest float after some 130 diagonals; the memory-state matrices, all
    positive, then hold the gates at 1."""
    import gpu_run
    import oracle_run
    from synth.configs import custom_workload

    hs, ws = [60, 2], [90, 4]
    print(f"case overflowed states H={H}", flush=True)
    wl = custom_workload(830 + H, hs, ws, 100, 8, H)
    wx, u, b = (p.copy() for p in wl.params())
    b[:, H:3 * H], b[:, 4 * H:] = 30.0, 3.0
    params = (wx, u, b, np.abs(wl.memory_params()))
    ref = oracle_run.run_layer(wl.examples(), params, None, backward=False)
    gpu = gpu_run.run_layer(wl.examples(), params, None, hs, ws, 100, backward=False)
    for k in range(2):
        _same(f"Y[{k}]", gpu["Y"][k], ref["Y"][k], 1e-5)


@pytest.mark.parametrize("H,C,mem,tall", [(8, 12, False, 60), (16, 24, False, 20), (32, 16, False, 40),
                                          (64, 12, False, 9), (64, 68, False, 50), (16, 20, True, 33), (32, 8, True, 60)])
def test_backward_with_infinite_gradients(H, C, mem, tall):
    """Positive weights and inputs: an infinite upstream gradient makes every
    gate gradient of its cell infinite with one sign, and of the cells before
    it, up to those without a left or top predecessor (inf * 0)."""
    import gpu_run
    import oracle_run
    from synth.configs import custom_workload

    hs, ws = [tall, 3, 4], [7, 9, 5]
    print(f"case infinite gradients H={H} C={C} memory={mem} h={tall}", flush=True)
    wl = custom_workload(860 + H + C, hs, ws, 40, C, H)
    xs = [np.abs(x) * 0.1 for x in wl.examples()]
    params = [np.abs(p) * (0.3 / H) for p in wl.params()[:2]] + [wl.params()[2]]
    params[2][:, H:3 * H], params[2][:, 4 * H:] = -1.0, 0.5
    if mem:
        params.append(np.abs(wl.memory_params()) * (0.3 / H))
    dys = [wl.dy(k) for k in range(3)]
    dys[0][tall // 2, 3, 1], dys[0][tall // 2, 3, 2 * H + 1] = np.inf, np.inf
    dys[1][1, 4, H] = np.finfo(np.float32).max  # finite, but beyond the largest bf16
    with np.errstate(all="ignore"):
        ref = oracle_run.run_layer(xs, params, dys)
    gpu = gpu_run.run_layer(xs, params, dys, hs, ws, 40)
    assert np.isinf(ref["dX"][0]).any()
    for k in (1, 2):
        _same(f"dX[{k}]", gpu["dX"][k], ref["dX"][k], 1e-5)
    _same("dX[0]", gpu["dX"][0], ref["dX"][0], 1e-5)
    for nm in ("dWx", "dU", "db") + (("dV",) if mem else ()):
        _same(nm, gpu[nm], ref[nm], 1e-5)
