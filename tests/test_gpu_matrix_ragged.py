"""The matrix kernel's staging of planes that are not whole runs of 8 bytes: the last run of a plane begins where the plane's last 8
bytes do, so it overlaps the one before it.  Against the CPU oracle."""
import numpy as np
import pytest

from helpers import TOL, assert_close
from test_gpu_matrix import _each_output, _layer
from test_gpu_parity import oracle_ref

pytestmark = pytest.mark.gpu

# N, C, K, R, S, H, W, stride, pad.  Planes that lack one, two or three pixels to whole runs; rows of two and three pixels (a run goes over a
# row's end from any of its pixels), planes of one run and a pixel; one chunk of channels and several, one block of runs in flight and two,
# wavefronts that share the tile out and the channels; strides, and no padding.
SHAPES = [("f16", (70, 65, 130, 3, 3, 25, 13, 1, 0)), ("f16", (70, 70, 130, 3, 3, 13, 31, 1, 0)), ("f16", (150, 64, 130, 5, 5, 5, 6, 1, 2)),
          ("f16", (70, 64, 64, 5, 5, 9, 3, 1, 2)), ("f16", (150, 64, 40, 1, 1, 13, 13, 2, 0)), ("f16", (70, 64, 40, 1, 1, 25, 21, 1, 1)),
          ("f16", (3, 64, 130, 2, 2, 13, 2, 1, 1)), ("f16", (150, 64, 64, 3, 3, 1, 5, 1, 1)), ("f16", (150, 300, 130, 1, 3, 9, 6, 1, 0)),
          ("f16", (30, 64, 64, 3, 3, 21, 2, 2, 1)),
          ("f32", (150, 64, 130, 5, 5, 13, 13, 1, 1)), ("f32", (150, 64, 130, 3, 3, 13, 5, 1, 0)), ("f32", (30, 96, 130, 3, 3, 15, 3, 1, 1)),
          ("f32", (150, 200, 130, 1, 1, 5, 9, 2, 1)), ("f32", (150, 64, 130, 2, 2, 15, 3, 1, 1)),
          ("f16", (150, 40, 64, 3, 3, 7, 7, 1, 1)), ("f16", (30, 17, 130, 5, 5, 9, 11, 1, 2)), ("f16", (3, 48, 33, 2, 2, 13, 3, 2, 1)),
          ("f32", (24, 62, 73, 3, 3, 19, 11, 2, 1)), ("f32", (169, 33, 56, 1, 2, 17, 17, 2, 1))]


@pytest.mark.parametrize("dtype,shape", SHAPES, ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_planes_that_are_not_whole_runs(dtype, shape):
    """From an input that starts on 8 bytes and one that does not, the same bits; with a value that is not finite, behind the last whole run
    of the batch's last plane, and (fp32) inputs far above and below their image's window: every output against its own terms."""
    import torch
    N, C, K, R, S, H, W, st, p = shape
    layer, w, m, x = _layer(dtype, shape, 106, 0.9)
    plan = layer.get_matrix_plan(N, H, W, st, p)
    assert plan["runs"] > 0 and H * W % (4 if dtype == "f16" else 2), "the sizes no longer take the staging under test"
    assert layer.check_plan(N, H, W, st, p) == 0
    tdtype = torch.float16 if dtype == "f16" else torch.float32
    if dtype == "f32":
        far = x * np.exp2(np.random.default_rng(107).uniform(-25, 25, x.shape)).astype(np.float32)
        _each_output(layer, w, m, far, st, p, "spread")
    x[N - 1, C - 1, H - 1, W - 1] = np.inf
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oracle_ref(w, m, x, st, p, dtype)
    fin = np.isfinite(ref)
    aligned = torch.from_numpy(x).cuda().to(tdtype)
    want = None
    for off in (0, 1, 2, 3):
        data = torch.empty(aligned.numel() + off, dtype=tdtype, device="cuda")[off:].view(aligned.shape)
        data.copy_(aligned)
        y = layer.forward(data, st, p)
        want = y if want is None else want
        assert torch.equal(torch.nan_to_num(y), torch.nan_to_num(want)), off
    got = want.float().cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    assert_close(got[fin], ref[fin], TOL[dtype], f"{dtype} {shape}")
    layer.close()
