"""The matrix kernel's pooled outputs in runs, against those stored one by one and the CPU oracle."""
import numpy as np
import pytest

import oracle
from helpers import TOL, assert_close
from test_gpu_matrix import _layer
from test_gpu_parity import oracle_ref

pytestmark = pytest.mark.gpu

# Bytes of a run in fp32 and in binary16, and N, C, K, H, W: pooled planes of whole runs of 16 bytes, of 8 and of neither; rows of 2 (one
# by one) to 64, rows off their blocks of 32, a last tile that is not full; wavefronts that own 32, 64 and 128 outputs.
STORED = [(0, 0, (301, 192, 70, 12, 2)), (16, 8, (91, 192, 70, 4, 4)), (8, 0, (91, 192, 70, 6, 4)), (16, 16, (91, 192, 250, 8, 4)),
          (16, 8, (93, 128, 130, 2, 8)), (16, 16, (41, 128, 70, 8, 8)), (16, 16, (161, 64, 130, 6, 16)), (16, 16, (35, 128, 130, 16, 16)),
          (16, 16, (33, 48, 65, 10, 32)), (16, 16, (9, 64, 130, 64, 64)),
          (16, 8, (801, 64, 130, 2, 8)), (16, 16, (161, 64, 130, 16, 16)), (16, 8, (1601, 64, 70, 4, 4)), (16, 16, (65, 48, 70, 32, 32))]


# (fp32 wavefronts own 64 outputs at most: no pair of rows of 64)
CASES = [(d, r32 if d == "f32" else r16, s) for r32, r16, s in STORED for d in ("f32", "f16") if d == "f16" or s[4] < 64]


@pytest.mark.parametrize("dtype,runs,shape", CASES, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_matrix_kernel_stores_pooled_runs(dtype, runs, shape):
    """Every output is written and nothing beside them, with the bits that an output off the runs' alignment gets one by one; the first and
    the last images' are the oracle's."""
    import torch
    N, C, K, H, W = shape
    layer, w, m, x = _layer(dtype, (N, C, K, 3, 3, H, W, 1, 1), 92, 1.0)
    bias = np.random.default_rng(6).standard_normal(K).astype(np.float32)
    some = [0, 1, N - 2, N - 1]
    sums = oracle_ref(w, m, x[some], 1, 1, dtype) + bias[None, :, None, None]
    xt = torch.from_numpy(x).cuda().to(torch.float16 if dtype == "f16" else torch.float32)
    size = torch.Size((N, K, H // 2, W // 2))
    for relu in (True, False):
        layer.set_epilogue(bias, relu=relu, maxpool=True)
        assert layer.get_kernel(N, H, W, 1, 1) == "matrix" and layer.check_plan(N, H, W, 1, 1) == 0
        assert layer.get_matrix_out_runs(N, H, W, 1, 1) == runs
        got = []
        for first in (32, 33):                # (a tensor starts at 256 bytes or more)
            room = torch.full((size.numel() + 64,), float("nan"), dtype=xt.dtype, device="cuda")
            y = layer.forward(xt, 1, 1, out=room[first:first + size.numel()].view(size))
            assert torch.isnan(room[:first]).all() and torch.isnan(room[first + size.numel():]).all()
            assert torch.isfinite(y).all()
            got.append(y.clone())
        assert torch.equal(*got)
        ref = oracle.maxpool2((oracle.relu(sums.astype(np.float32)) if relu else sums).astype(np.float32))
        assert_close(got[0][some].float().cpu().numpy(), ref, TOL[dtype], f"{dtype} {shape} relu {relu}")
    layer.close()
