"""The matrix kernel's tiles whose channels eight wavefronts share (binary16), against the CPU oracle."""
import numpy as np
import pytest

import oracle
from helpers import TOL, assert_close
from test_gpu_matrix import _layer
from test_gpu_parity import oracle_ref, run_gpu

pytestmark = pytest.mark.gpu

# MK, NP, steps ahead, blocks of single pixels in flight, blocks of runs in flight (0: it stages single pixels), chunks, and a layer that takes
# it (N, C, K, R, S, H, W, stride, pad): channels off their groups of 16 and off the eight wavefronts' shares (530: a last
# chunk in which most wavefronts have none), rows off their blocks of 32, a last tile that is not full.
VARIANTS = [((1, 1, 2, 2, 0, 5), (9, 530, 33, 2, 2, 1, 3, 1, 1)), ((1, 1, 2, 4, 0, 2), (1, 300, 130, 1, 1, 3, 13, 1, 0)),
            ((1, 1, 2, 6, 0, 1), (30, 130, 40, 1, 1, 9, 1, 2, 1)), ((1, 1, 2, None, 1, 3), (11, 300, 70, 2, 2, 5, 21, 1, 0)),
            ((1, 1, 2, None, 2, 3), (70, 300, 130, 2, 2, 6, 3, 2, 0)), ((1, 1, 3, 2, 0, 3), (3, 300, 70, 3, 3, 5, 8, 1, 1)),
            ((1, 1, 3, 4, 0, 5), (150, 530, 70, 1, 3, 13, 1, 1, 1)), ((1, 1, 3, 6, 0, 2), (30, 130, 33, 3, 3, 3, 1, 2, 1)),
            ((1, 1, 3, None, 1, 3), (9, 530, 70, 1, 3, 7, 21, 1, 0)), ((1, 1, 3, None, 2, 2), (70, 130, 130, 1, 3, 2, 8, 2, 0)),
            ((1, 2, 2, 4, 0, 2), (30, 300, 70, 1, 1, 13, 7, 1, 0)), ((1, 2, 2, None, 1, 2), (70, 200, 70, 2, 2, 8, 13, 1, 1)),
            ((1, 2, 2, None, 2, 1), (150, 200, 40, 1, 2, 5, 9, 1, 0)), ((1, 2, 3, 6, 0, 1), (300, 100, 130, 3, 3, 6, 1, 1, 1)),
            ((1, 2, 3, None, 1, 2), (150, 130, 70, 1, 3, 4, 16, 1, 0)), ((1, 2, 3, None, 2, 2), (70, 130, 130, 3, 3, 5, 16, 1, 0)),
            ((1, 2, 3, None, 1, 4), (230, 512, 513, 3, 3, 2, 2, 1, 1)), ((1, 2, 2, 6, 0, 1), (234, 111, 279, 2, 2, 10, 1, 2, 1)),
            ((1, 2, 3, 4, 0, 3), (176, 364, 108, 3, 1, 15, 1, 1, 0)), ((1, 2, 2, 2, 0, 1), (2, 65, 4770, 1, 2, 1, 32, 1, 0)),
            ((1, 2, 3, 2, 0, 1), (4, 83, 4837, 1, 3, 1, 14, 1, 0))]


@pytest.mark.parametrize("split,shape", VARIANTS, ids=lambda v: "x".join(map(str, v)))
def test_channels_shared_by_eight_wavefronts(split, shape):
    """Plain, with bias and ReLU, from an output off the alignment of the wide stores, and with inputs that are not finite under stored
    weights and pruned ones."""
    import torch
    N, C, K, R, S, H, W, st, p = shape
    layer, w, m, x = _layer("f16", shape, 90, 0.9)
    plan = layer.get_matrix_plan(N, H, W, st, p)
    MK, NP, ahead, fly, runs, chunks = split
    assert plan["KS"] == 8 and (plan["MK"], plan["NP"], plan["ahead"], plan["runs"], plan["nchunks"]) == (MK, NP, ahead, runs, chunks), plan
    assert fly is None or plan["fly"] == fly, plan
    assert layer.check_plan(N, H, W, st, p) == 0
    ref = oracle_ref(w, m, x, st, p, "f16")
    assert_close(run_gpu(layer, x, st, p, "f16"), ref, TOL["f16"], f"{split} {shape}")
    xt = torch.from_numpy(x).cuda().half()
    y = layer.forward(xt, st, p)
    odd = torch.full((y.numel() + 2,), float("nan"), dtype=y.dtype, device="cuda")
    layer.forward(xt, st, p, out=odd[1:-1].view(y.shape))
    assert torch.equal(odd[1:-1].view(y.shape), y) and torch.isnan(odd[[0, -1]]).all()
    bias = np.random.default_rng(5).standard_normal(K).astype(np.float32)
    layer.set_epilogue(bias, relu=True)
    assert_close(run_gpu(layer, x, st, p, "f16"), np.maximum(ref + bias[None, :, None, None], 0.0), TOL["f16"], f"bias, ReLU {shape}")
    layer.set_epilogue(None)
    flat = x.reshape(-1)
    where = np.random.default_rng(7).choice(flat.size, size=6, replace=False)
    flat[where] = (np.inf, -np.inf, np.nan) * 2
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oracle_ref(w, m, x, st, p, "f16")
    got = layer.forward(torch.from_numpy(x).cuda().half(), st, p).float().cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    fin = np.isfinite(ref)
    assert_close(got[fin], ref[fin], TOL["f16"], f"not finite {shape}")
    layer.close()


@pytest.mark.parametrize("H,N,C,K", [(2, 250, 256, 64), (4, 41, 300, 40), (8, 9, 128, 70), (8, 41, 200, 130), (16, 9, 200, 130)])
def test_channels_shared_by_eight_wavefronts_pooled_store(H, N, C, K):
    """A wavefront finishes 32 outputs by itself: whole pairs of rows of up to 16."""
    import torch
    layer, w, m, x = _layer("f16", (N, C, K, 3, 3, H, H, 1, 1), 92, 1.0)
    bias = np.random.default_rng(6).standard_normal(K).astype(np.float32)
    layer.set_epilogue(bias, relu=True, maxpool=True)
    assert layer.get_matrix_plan(N, H, H, 1, 1)["KS"] == 8 and layer.check_plan(N, H, H, 1, 1) == 0
    ref = oracle.maxpool2(oracle.relu((oracle_ref(w, m, x, 1, 1, "f16") + bias[None, :, None, None]).astype(np.float32)))
    assert_close(run_gpu(layer, x, 1, 1, "f16"), ref, TOL["f16"], f"pooled {H}")
    if H <= 8:   # (larger maps: the tile kernel's partial sums are more than the static scratch holds, the call is refused)
        xt = torch.from_numpy(x).cuda().half()
        assert torch.equal(layer.forward_static(xt, 1, 1), layer.forward(xt, 1, 1))
    layer.close()


def test_results_of_eight_wavefronts_do_not_change_from_launch_to_launch():
    """Their sums are added in a fixed order, whoever comes last; captured and replayed as well."""
    import torch
    layer, w, m, x = _layer("f16", (11, 300, 70, 2, 2, 5, 21, 1, 0), 90, 0.9)
    assert layer.get_matrix_plan(11, 5, 21, 1, 0)["KS"] == 8
    a, b = torch.from_numpy(x).cuda().half(), torch.from_numpy(x[::-1].copy()).cuda().half()
    want = [layer.forward(v, 1, 0).clone() for v in (a, b)]
    y = torch.empty_like(want[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer.forward(a, 1, 0, out=y)
    for _ in range(100):
        assert torch.equal(layer.forward(b, 1, 0), want[1])
        y.zero_()
        graph.replay()
        assert torch.equal(y, want[0])
    layer.close()
