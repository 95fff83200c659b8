"""The matrix kernel (sparse_conv_get_kernel says "matrix") against the CPU oracle at the edges of its tiles: channels off
its groups of 16, rows off its blocks of 32, outputs off its tiles, every variant that is built, pooled stores, inputs that are
not finite, and fp32 inputs and weights of every magnitude (they are cut into two scaled binary16 pieces)."""
import numpy as np
import pytest

import oracle
from helpers import TOL, assert_close, rand_layer
from test_gpu_parity import oracle_ref, run_gpu

pytestmark = pytest.mark.gpu

# N, C, K, R, S, H, W, stride, pad: weights 90 or 100 % dense, so that these sizes take the kernel
SHAPES = [(40, 64, 65, 3, 3, 14, 14, 1, 1), (40, 33, 130, 3, 3, 9, 13, 1, 1), (100, 17, 96, 5, 5, 8, 7, 1, 2), (64, 200, 31, 3, 3, 15, 15, 1, 0),
          (24, 48, 64, 3, 3, 29, 31, 2, 1), (60, 240, 250, 1, 1, 15, 14, 1, 0), (200, 600, 100, 1, 1, 7, 7, 1, 0), (150, 300, 100, 1, 3, 1, 64, 1, 0),
          (600, 512, 128, 3, 3, 2, 2, 1, 1), (64, 256, 256, 3, 3, 4, 4, 1, 1), (4, 16, 64, 3, 3, 65, 120, 1, 1), (100, 80, 48, 2, 2, 18, 18, 2, 3)]


def _layer(dtype, shape, seed, density):
    from paper_2011_06295_amd import binding as B
    N, C, K, R, S, H, W, st, p = shape
    w, m, x = rand_layer(np.random.default_rng(seed), N, C, K, R, S, H, W, density=density)
    return B.SparseConv(w, m, dtype=dtype), w, m, x


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_matrix_kernel_against_the_oracle(dtype, shape):
    import torch
    layer, w, m, x = _layer(dtype, shape, 91, 0.9)
    N, C, K, R, S, H, W, st, p = shape
    # (the fp32 sums of a 5 x 5 filter's chunk are not exact enough for so few channels: the tile kernel's)
    assert layer.get_kernel(N, H, W, st, p) == ("tile" if dtype == "f32" and R == 5 else "matrix"), "the sizes no longer take the kernel under test"
    assert layer.check_plan(N, H, W, st, p) == 0
    ref = oracle_ref(w, m, x, st, p, dtype)
    bias = np.random.default_rng(5).standard_normal(K).astype(np.float32)
    assert_close(run_gpu(layer, x, st, p, dtype), ref, TOL[dtype], f"{dtype} {shape}")
    # an output that starts off the alignment of the wide stores: the same bits
    xt = torch.from_numpy(x).cuda().to(torch.float16 if dtype == "f16" else torch.float32)
    y = layer.forward(xt, st, p)
    odd = torch.full((y.numel() + 2,), float("nan"), dtype=y.dtype, device="cuda")
    layer.forward(xt, st, p, out=odd[1:-1].view(y.shape))
    assert torch.equal(odd[1:-1].view(y.shape), y) and torch.isnan(odd[[0, -1]]).all()
    layer.set_epilogue(bias, relu=True)
    assert_close(run_gpu(layer, x, st, p, dtype), np.maximum(ref + bias[None, :, None, None], 0.0), TOL[dtype], f"bias, ReLU {dtype} {shape}")
    layer.close()


# Every kernel that is built, and every way of sharing output channels out: MK, NP, WK, KS, steps ahead, blocks of single pixels in
# flight, blocks of runs in flight (0: it stages single pixels), and a small layer that takes it (N, C, K, R, S, H, W, stride, pad).
# (Four blocks of single pixels and more are staged one by one on maps of one column and, in fp32 and under 1 x 1 taps, on odd planes.)
VARIANTS = [
    ("f16", (2, 2, 4, 1, 2, 2, 0), (227, 23, 296, 1, 1, 5, 2, 1, 1)),
    ("f16", (2, 2, 4, 1, 2, 4, 0), (5, 32, 54, 5, 1, 47, 1, 2, 0)),
    ("f16", (2, 2, 4, 1, 2, 4, 1), (199, 24, 114, 1, 1, 4, 37, 2, 1)),
    ("f16", (2, 2, 4, 1, 2, 4, 2), (11, 30, 26, 1, 2, 54, 54, 2, 0)),
    ("f16", (2, 2, 4, 1, 2, 6, 0), (122, 54, 98, 5, 1, 5, 1, 1, 1)),
    ("f16", (2, 2, 2, 1, 2, 6, 2), (110, 30, 23, 1, 1, 17, 52, 2, 0)),
    ("f16", (2, 2, 4, 1, 3, 2, 0), (124, 21, 212, 1, 3, 7, 7, 1, 0)),
    ("f16", (2, 2, 4, 1, 3, 4, 0), (27, 29, 137, 3, 3, 3, 1, 1, 1)),
    ("f16", (2, 2, 4, 1, 3, 4, 1), (13, 27, 132, 1, 3, 22, 22, 2, 2)),
    ("f16", (2, 2, 4, 1, 3, 6, 0), (74, 28, 244, 3, 3, 4, 1, 2, 1)),
    ("f16", (2, 2, 4, 1, 3, 6, 2), (3, 31, 169, 3, 1, 34, 34, 2, 2)),
    ("f16", (2, 2, 1, 4, 2, 2, 0), (1, 35, 21, 1, 2, 1, 6, 2, 0)), ("f16", (2, 2, 1, 4, 2, 4, 0), (1, 103, 21, 1, 1, 1, 1, 1, 0)),
    ("f16", (2, 2, 1, 4, 2, 4, 1), (2, 91, 57, 1, 1, 2, 2, 2, 1)), ("f16", (2, 2, 1, 4, 2, 6, 0), (29, 60, 18, 2, 2, 2, 1, 2, 1)),
    ("f16", (2, 2, 1, 4, 2, 6, 2), (233, 38, 22, 2, 2, 2, 4, 1, 0)),
    ("f16", (2, 2, 1, 4, 3, 2, 0), (1, 35, 34, 3, 1, 1, 1, 2, 1)), ("f16", (2, 2, 1, 4, 3, 4, 0), (1, 209, 73, 3, 3, 1, 1, 2, 1)),
    ("f16", (2, 2, 1, 4, 3, 4, 1), (7, 166, 50, 1, 3, 4, 4, 2, 0)),
    ("f16", (2, 2, 1, 4, 3, 6, 0), (14, 44, 16, 3, 3, 4, 1, 2, 1)), ("f16", (2, 2, 1, 4, 3, 6, 2), (2, 74, 20, 3, 3, 6, 6, 1, 0)),
    ("f16", (2, 4, 4, 1, 2, 2, 0), (15, 36, 159, 1, 2, 42, 42, 1, 0)),
    ("f16", (2, 4, 2, 1, 2, 4, 0), (143, 23, 75, 2, 1, 78, 1, 1, 1)),
    ("f16", (2, 4, 4, 1, 2, 4, 1), (10, 24, 142, 1, 2, 50, 50, 1, 0)),
    ("f16", (2, 4, 4, 1, 2, 6, 0), (137, 33, 161, 5, 1, 55, 1, 1, 1)),
    ("f16", (2, 4, 4, 1, 3, 2, 0), (195, 16, 194, 1, 3, 11, 11, 1, 1)),
    ("f16", (2, 4, 2, 1, 3, 4, 0), (158, 21, 66, 3, 1, 85, 1, 1, 1)),
    ("f16", (2, 4, 1, 1, 3, 4, 1), (156, 20, 32, 3, 1, 8, 45, 1, 2)),
    ("f16", (2, 4, 4, 1, 3, 6, 0), (173, 54, 132, 3, 1, 43, 1, 1, 1)),
    ("f32", (1, 2, 4, 1, 2, 1, 0), (147, 27, 119, 1, 2, 39, 3, 1, 0)),
    ("f32", (1, 2, 4, 1, 2, 2, 0), (115, 26, 70, 2, 2, 5, 31, 2, 1)),
    ("f32", (1, 2, 4, 1, 2, 2, 1), (16, 25, 51, 3, 3, 42, 12, 1, 1)),
    ("f32", (1, 2, 4, 1, 2, 3, 0), (10, 25, 47, 2, 2, 49, 49, 2, 1)),
    ("f32", (1, 2, 1, 1, 2, 3, 0), (100, 27, 22, 2, 2, 23, 17, 1, 0)),
    ("f32", (1, 2, 4, 1, 2, 3, 2), (132, 44, 117, 1, 2, 10, 10, 2, 0)),
    ("f32", (1, 2, 4, 1, 3, 1, 0), (21, 20, 279, 1, 3, 12, 20, 1, 0)),
    ("f32", (1, 2, 4, 1, 3, 2, 0), (188, 26, 254, 3, 1, 44, 1, 2, 0)),
    ("f32", (1, 2, 2, 1, 3, 2, 1), (102, 22, 47, 1, 3, 5, 56, 1, 0)),
    ("f32", (1, 2, 4, 1, 3, 3, 0), (24, 16, 151, 3, 3, 21, 21, 2, 0)),
    ("f32", (1, 2, 4, 1, 3, 3, 2), (12, 16, 53, 3, 3, 32, 32, 2, 1)),
    ("f32", (2, 2, 4, 1, 2, 1, 0), (113, 28, 166, 1, 2, 12, 12, 1, 0)),
    ("f32", (2, 2, 2, 1, 2, 2, 0), (9, 31, 105, 2, 1, 47, 47, 1, 0)),
    ("f32", (2, 2, 1, 1, 2, 3, 0), (184, 26, 62, 1, 2, 17, 17, 1, 0)),
    ("f32", (2, 2, 4, 1, 2, 3, 1), (113, 60, 137, 1, 1, 48, 10, 2, 0)),
    ("f32", (2, 2, 4, 1, 3, 1, 0), (70, 25, 215, 1, 3, 38, 4, 1, 1)),
    ("f32", (2, 2, 4, 1, 3, 2, 0), (28, 22, 184, 1, 3, 39, 39, 2, 1)),
    ("f32", (2, 2, 4, 1, 3, 2, 1), (12, 31, 223, 3, 1, 36, 36, 1, 0)),
    ("f32", (2, 2, 4, 1, 3, 3, 0), (31, 25, 224, 3, 1, 59, 15, 2, 1)),
    ("f32", (2, 2, 1, 4, 2, 2, 0), (1, 63, 122, 2, 2, 3, 3, 2, 0)), ("f32", (2, 2, 1, 4, 2, 2, 1), (1, 47, 61, 1, 2, 1, 2, 2, 0)),
    ("f32", (2, 2, 1, 4, 2, 3, 0), (40, 47, 199, 2, 2, 23, 1, 1, 1)),
    ("f32", (2, 2, 1, 4, 2, 3, 1), (15, 54, 244, 2, 2, 62, 3, 2, 1)),
    ("f32", (2, 2, 1, 4, 3, 2, 0), (1, 61, 240, 3, 3, 7, 9, 2, 0)),
    ("f32", (2, 2, 1, 4, 3, 3, 0), (37, 96, 255, 3, 1, 13, 1, 1, 1)),
    ("f32", (2, 2, 1, 4, 3, 3, 1), (13, 60, 141, 3, 1, 26, 5, 1, 1)),
]


@pytest.mark.parametrize("dtype,split,shape", VARIANTS, ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_every_variant_against_the_oracle(dtype, split, shape):
    layer, w, m, x = _layer(dtype, shape, 90, 0.9)
    N, C, K, R, S, H, W, st, p = shape
    plan = layer.get_matrix_plan(N, H, W, st, p)
    assert tuple(plan[k] for k in ("MK", "NP", "WK", "KS", "ahead", "fly", "runs")) == split, "the sizes no longer take the variant under test"
    assert layer.check_plan(N, H, W, st, p) == 0
    assert_close(run_gpu(layer, x, st, p, dtype), oracle_ref(w, m, x, st, p, dtype), TOL[dtype], f"{dtype} {split} {shape}")
    layer.close()


def test_the_variants_are_all_that_is_built():
    """Of four wavefronts (test_kernel_resources.py holds those of eight too against the built library).  Two or three steps ahead; single pixels one, two or three blocks at a time (binary16: twice as many; not one in fp32 where
    wavefronts share the channels) or runs, one block or, where registers allow it, two."""
    built = set()
    for dtype, MK, NP, KS in (("f16", 2, 2, 1), ("f16", 2, 4, 1), ("f16", 2, 2, 4), ("f32", 1, 2, 1), ("f32", 2, 2, 1), ("f32", 2, 2, 4)):
        unit, pieces = (1, 2) if dtype == "f32" else (2, 1)
        for ahead in (2, 3):
            built |= {(dtype, MK, NP, KS, ahead, fly * unit, 0) for fly in (1, 2, 3) if fly > 1 or dtype == "f16" or KS == 1}
            built |= {(dtype, MK, NP, KS, ahead, "any", runs) for runs in (1, 2) if runs == 1 or MK * NP * pieces < 8}
    assert {(d, s[0], s[1], s[3], s[4], "any" if s[6] else s[5], s[6]) for d, s, _ in VARIANTS} == built


# Planes that are whole runs of 16 bytes, of 8 (binary16 14 x 14, fp32 15 x 14) and of neither; rows off their
# blocks of 32, a last tile that is not full, wavefronts that share the tile's outputs or its channels.
# Bytes of a run in fp32 and in binary16, and the layer.
STORED_RUNS = [(16, 8, (41, 64, 65, 3, 3, 14, 14, 1, 1)), (16, 16, (33, 48, 130, 3, 3, 16, 12, 1, 1)), (8, 0, (61, 240, 250, 1, 1, 15, 14, 1, 0)),
               (16, 16, (131, 256, 70, 3, 3, 4, 4, 1, 1)), (16, 8, (1201, 256, 70, 3, 3, 2, 2, 1, 1)), (0, 0, (45, 64, 100, 3, 3, 9, 13, 1, 1))]


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("runs32,runs16,shape", STORED_RUNS, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_matrix_kernel_stores_runs(dtype, runs32, runs16, shape):
    """Every output is written and nothing beside them, with the bits that an output off the runs' alignment gets one by one; the first and
    the last images' are the oracle's."""
    import torch
    layer, w, m, x = _layer(dtype, shape, 97, 0.9)
    N, C, K, R, S, H, W, st, p = shape
    bias = np.random.default_rng(8).standard_normal(K).astype(np.float32)
    layer.set_epilogue(bias, relu=True)
    assert layer.get_kernel(N, H, W, st, p) == "matrix" and layer.check_plan(N, H, W, st, p) == 0
    assert layer.get_matrix_out_runs(N, H, W, st, p) == (runs32 if dtype == "f32" else runs16)
    xt = torch.from_numpy(x).cuda().to(torch.float16 if dtype == "f16" else torch.float32)
    size = torch.Size((N, K, *layer.output_shape(H, W, st, p)))
    got = []
    for first in (32, 33):                # (a tensor starts at 256 bytes or more)
        room = torch.full((size.numel() + 64,), float("nan"), dtype=xt.dtype, device="cuda")
        y = layer.forward(xt, st, p, out=room[first:first + size.numel()].view(size))
        assert torch.isnan(room[:first]).all() and torch.isnan(room[first + size.numel():]).all()
        assert torch.isfinite(y).all()
        got.append(y.clone())
    assert torch.equal(*got)
    some = [0, 1, N - 2, N - 1]
    ref = np.maximum(oracle_ref(w, m, x[some], st, p, dtype) + bias[None, :, None, None], 0.0)
    assert_close(got[0][some].float().cpu().numpy(), ref, TOL[dtype], f"{dtype} {shape}")
    layer.close()


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("H,N,C,K", [(2, 1200, 256, 64), (4, 400, 256, 40), (8, 64, 128, 64), (16, 33, 64, 96), (32, 9, 48, 64), (64, 5, 40, 64)])
def test_matrix_kernel_pooled_store(dtype, H, N, C, K):
    import torch
    shape = (N, C, K, 3, 3, H, H, 1, 1)
    layer, w, m, x = _layer(dtype, shape, 92, 1.0)
    bias = np.random.default_rng(6).standard_normal(K).astype(np.float32)
    layer.set_epilogue(bias, relu=True, maxpool=True)
    # (fp32 wavefronts own 64 outputs: no pair of rows of 64)
    assert layer.get_kernel(N, H, H, 1, 1) == ("tile" if dtype == "f32" and H == 64 else "matrix")
    ref = oracle.maxpool2(oracle.relu((oracle_ref(w, m, x, 1, 1, dtype) + bias[None, :, None, None]).astype(np.float32)))
    assert_close(run_gpu(layer, x, 1, 1, dtype), ref, TOL[dtype], f"pooled {dtype} {H}")
    if H <= 8:   # (larger maps: the tile kernel's partial sums are more than the static scratch holds, the call is refused)
        xt = torch.from_numpy(x).cuda().to(torch.float16 if dtype == "f16" else torch.float32)
        assert torch.equal(layer.forward_static(xt, 1, 1), layer.forward(xt, 1, 1))
    layer.close()


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("shape,pool", [(SHAPES[0], False), (SHAPES[5], False), (SHAPES[8], False), (SHAPES[8], True)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_matrix_kernel_inputs_that_are_not_finite(dtype, shape, pool):
    """The dense table's zeros meet every input of a receptive field: an Inf or NaN must count under stored weights only."""
    import torch
    N, C, K, R, S, H, W, st, p = shape
    layer, w, m, x = _layer(dtype, shape, 93, 0.9)
    rng = np.random.default_rng(7)
    flat = x.reshape(-1)
    where = rng.choice(flat.size, size=40, replace=False)
    flat[where[:15]], flat[where[15:30]], flat[where[30:]] = np.inf, -np.inf, np.nan
    layer.set_epilogue(None, maxpool=pool)
    assert layer.get_kernel(N, H, W, st, p) == "matrix"
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oracle_ref(w, m, x, st, p, dtype)
    xt = torch.from_numpy(x).cuda().to(torch.float16 if dtype == "f16" else torch.float32)
    got = layer.forward(xt, st, p).float().cpu().numpy().astype(np.float64)
    if pool:   # windows without a NaN (one with a NaN gives any of its values)
        win = ref.reshape(N, K, H // 2, 2, W // 2, 2).transpose(0, 1, 2, 4, 3, 5).reshape(N, K, H // 2, W // 2, 4)
        keep = ~np.isnan(win).any(-1)
        got, ref = got[keep], np.where(np.isnan(win), -np.inf, win).max(-1)[keep]
    assert not np.isfinite(ref).all()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    fin = np.isfinite(ref)
    assert_close(got[fin], ref[fin], TOL[dtype], f"not finite {dtype} {shape}")
    layer.close()


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_matrix_kernel_inputs_that_are_not_finite_do_not_stop_it(dtype):
    """Outputs that see such an input are summed one by one.  Measured against the tile kernel, which they do not slow down
    (one NaN: 10 times its time, all NaN: 80 times, when each lane followed a row's mask by itself; 2 and 8 now)."""
    import torch
    layer, w, m, x = _layer(dtype, (128, 256, 256, 3, 3, 14, 14, 1, 1), 99, 0.3)
    assert layer.get_kernel(128, 14, 14, 1, 1) == "matrix"
    xt = torch.from_numpy(x).cuda().to(torch.float16 if dtype == "f16" else torch.float32)
    y = layer.forward(xt, 1, 1)

    def best(data):
        times = []
        for _ in range(5):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            layer.forward(data, 1, 1, out=y)
            e[1].record()
            torch.cuda.synchronize()
            times.append(e[0].elapsed_time(e[1]))
        return min(times)

    one = xt.clone()
    one[5, 3, 4, 4] = float("nan")
    plain, t_one, t_all = best(xt), best(one), best(torch.full_like(xt, float("nan")))
    layer.set_launch(layer.rank_launches(128, 14, 14, 1, 1, 1)[0])
    tile = best(xt)
    print(f"{dtype}: {plain * 1e3:.0f} us, one NaN {t_one * 1e3:.0f} us, all NaN {t_all * 1e3:.0f} us; tile kernel {tile * 1e3:.0f} us", flush=True)
    assert t_one < 5 * tile and t_all < 25 * tile
    layer.close()


# Four wavefronts that share the channels, in one chunk (runs staged) and in three (single pixels; runs); wavefronts that share the
# tile out, in four chunks (runs) and in eight (single pixels).
RANGES = [(24, 64, 64, 3, 3, 14, 14, 1, 1), (48, 192, 100, 3, 3, 5, 5, 1, 1), (40, 240, 130, 1, 1, 15, 14, 1, 0),
          (48, 192, 100, 3, 3, 6, 6, 1, 1), (40, 240, 130, 1, 1, 15, 15, 1, 0)]
CHUNKS = {RANGES[0]: (4, 1, True), RANGES[1]: (4, 3, False), RANGES[2]: (1, 4, True), RANGES[3]: (4, 3, True), RANGES[4]: (1, 8, False)}


def _takes_the_kernel(layer, shape):
    N, C, K, R, S, H, W, st, p = shape
    plan = layer.get_matrix_plan(N, H, W, st, p)
    assert (plan["KS"], plan["nchunks"], plan["runs"] > 0) == CHUNKS[shape], "the sizes no longer take the split under test"


@pytest.mark.parametrize("how", ["tiny", "huge", "late", "early", "zeros first", "rows apart"])
@pytest.mark.parametrize("shape", RANGES, ids=lambda s: "x".join(map(str, s)))
def test_matrix_kernel_fp32_magnitudes(shape, how):
    """The scales of an image's two binary16 pieces come from its first chunk of channels; what a later chunk has above them
    (late; in the one-chunk split what is staged last) is multiplied in a round of its own.  Each output channel's weights have
    a scale of their own ("rows apart"): compared row by row."""
    N, C, K, R, S, H, W, st, p = shape
    layer, w, m, x = _layer("f32", shape, 94, 0.9)
    if how == "tiny":
        x *= np.float32(1e-25)
    elif how == "huge":
        x *= np.float32(1e25)
    elif how == "late":
        x[:, C - 12:] *= np.float32(1e6)
    elif how == "early":
        x[:, :16] *= np.float32(1e4)
    elif how == "zeros first":
        x[:, :C - 16] = 0.0
        x[:, C - 16:] *= np.float32(1e-6)
    elif how == "rows apart":
        from paper_2011_06295_amd import binding as B
        w *= np.logspace(-12, 12, K, dtype=np.float32)[:, None, None, None]
        layer.close()
        layer = B.SparseConv(w, m, dtype="f32")
    _takes_the_kernel(layer, shape)
    ref = oracle_ref(w, m, x, st, p, "f32")
    got = run_gpu(layer, x, st, p, "f32")
    for k in range(K):
        assert_close(got[:, k], ref[:, k], 2e-6, f"{how} row {k}")   # four times the largest error of an fp32 sum of this length
    layer.close()


def _each_output(layer, w, m, x, st, p, what):
    """Every output against the sum of its own terms' magnitudes.  A term is three products, each rounded as it joins the sum:
    3 * 2^-24; both its factors are held to 2^-23 and the product of their low pieces, each 2^-11 of its factor at most, is
    left out: 2 * 2^-23 + 2^-22 = 8 * 2^-24.  (Results may be subnormal: 2^-149 a term.)"""
    K, _, R, S = w.shape
    rowptr, colidx, values = oracle.csr_encode(w, m)
    ref, size = (v.astype(np.float64) for v in oracle.sparse_conv((rowptr, colidx, values), x, K, R, S, st, p, want_abs=True))
    terms = oracle.sparse_conv((rowptr, colidx, np.ones_like(values)), (x != 0).astype(np.float32), K, R, S, st, p)
    got = run_gpu(layer, x, st, p, "f32")
    err = np.abs(got - ref)
    assert (err <= size * (3 * terms + 8) * 2.0 ** -24 + terms * 2.0 ** -149).all(), (what, float((err / np.maximum(size, 1e-300)).max()))
    return got, ref


@pytest.mark.parametrize("ratio", [1e4, 1e6, 1e8, 1e12, 1e25])
@pytest.mark.parametrize("shape", RANGES, ids=lambda s: "x".join(map(str, s)))
def test_matrix_kernel_fp32_images_do_not_depend_on_their_neighbours(shape, ratio):
    """Tiles reach over several images: a loud one takes nothing from the others, not even a bit."""
    N, C, K, R, S, H, W, st, p = shape
    layer, w, m, x = _layer("f32", shape, 96, 0.9)
    _takes_the_kernel(layer, shape)
    x[::3] *= np.float32(ratio)
    got, ref = _each_output(layer, w, m, x, st, p, ratio)
    quiet = np.arange(N) % 3 != 0
    assert np.linalg.norm(got[quiet] - ref[quiet]) <= 1e-6 * np.linalg.norm(ref[quiet])   # (an fp32 sum in order: 4e-7)
    x[::3] = 0.0
    assert np.array_equal(run_gpu(layer, x, st, p, "f32")[quiet], got[quiet])
    layer.close()


# Rows of few weights, by their number, and the split they are multiplied in (MK, KS, chunks).  Both of them in a block's first
# places in the list, in its first row and its last, and behind those places.
SHORT = [((96, 64, 64, 3, 3, 14, 14, 1, 1), {0: 1, 1: 3, 31: 0}, (2, 4, 1)), ((200, 192, 100, 3, 3, 8, 8, 1, 1), {0: 1, 1: 5}, (2, 4, 3)),
         ((80, 240, 130, 1, 1, 15, 14, 1, 0), {0: 1, 1: 5, 31: 0, 40: 20, 129: 3}, (1, 1, 8)),
         ((120, 240, 130, 1, 1, 15, 15, 1, 0), {0: 1, 1: 5, 31: 4, 40: 20, 129: 3}, (2, 1, 4))]


@pytest.mark.parametrize("how", ["normal", "spread", "far apart", "tiny", "not finite"])
@pytest.mark.parametrize("shape,short,split", SHORT, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_matrix_kernel_rows_of_few_weights_are_fp32_sums(shape, short, split, how):
    """Rows of few weights are multiplied as fp32: each term is rounded once as it joins the sum, 2^-24 of at most the sum of the
    terms' magnitudes.  (Two binary16 pieces hold a single product to some 2^-22 only.)"""
    from paper_2011_06295_amd import binding as B
    N, C, K, R, S, H, W, st, p = shape
    rng = np.random.default_rng(105)
    w, m, x = rand_layer(rng, N, C, K, R, S, H, W, density=0.9)
    for k, n in short.items():
        m[k] = 0
        m[k].reshape(-1)[rng.permutation(C * R * S)[:n]] = 1
    if how == "spread":
        x *= np.exp2(rng.uniform(-25, 25, x.shape)).astype(np.float32)
    elif how == "far apart":
        x *= np.where(rng.random(x.shape) < 0.02, 1e20, 1e-15).astype(np.float32)
    elif how == "tiny":
        x *= np.float32(1e-30)
    elif how == "not finite":
        x[1, ::7, H // 2, W // 2] = np.inf
        x[2, 3] = np.nan
    layer = B.SparseConv(w, m, dtype="f32")
    plan = layer.get_matrix_plan(N, H, W, st, p)
    assert (plan["MK"], plan["KS"], plan["nchunks"]) == split, "the sizes no longer take the split under test"
    assert layer.check_plan(N, H, W, st, p) == 0
    got = run_gpu(layer, x, st, p, "f32")
    rows = list(short)
    rowptr, colidx, values = oracle.csr_encode(w[rows], m[rows])
    with np.errstate(invalid="ignore", over="ignore"):
        ref, size = (v.astype(np.float64) for v in oracle.sparse_conv((rowptr, colidx, values), x, len(rows), R, S, st, p, want_abs=True))
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got[:, rows]), fin)
    for i, k in enumerate(rows):
        f = fin[:, i]
        err = np.abs(got[:, k][f] - ref[:, i][f])
        assert (err <= size[:, i][f] * short[k] * 2.0 ** -24 + max(1, short[k]) * 2.0 ** -149).all(), (how, k, float((err / np.maximum(size[:, i][f], 1e-300)).max()))
    layer.close()


@pytest.mark.parametrize("how", ["corner", "channel", "spread", "far apart", "tiny", "subnormal", "late", "late and quiet", "dead first", "one pixel",
                                 "few and quiet"])
@pytest.mark.parametrize("shape", RANGES, ids=lambda s: "x".join(map(str, s)))
def test_matrix_kernel_fp32_inputs_of_every_size(shape, how):
    """Finite inputs of any range within one image, output by output: those that do not see the loud inputs keep fp32's
    precision, those under which a row has no stored weight count for nothing in it."""
    N, C, K, R, S, H, W, st, p = shape
    rng = np.random.default_rng(97)
    w, m, x = rand_layer(rng, N, C, K, R, S, H, W, density=0.9)
    if how == "corner":
        x[:, :, :2, :2] *= np.float32(1e10)
    elif how == "channel":
        x[:, 5] *= np.float32(1e10)
        m[::2, 5] = 0
    elif how == "spread":        # fifty binary orders of magnitude
        x *= np.exp2(rng.uniform(-25, 25, x.shape)).astype(np.float32)
    elif how == "far apart":     # more than one sum holds
        x *= np.where(rng.random(x.shape) < 0.02, 1e20, 1e-15).astype(np.float32)
    elif how == "tiny":
        x *= np.float32(2.0 ** -119)
        w *= np.float32(2.0 ** 12)
    elif how == "subnormal":
        x *= np.exp2(rng.uniform(-149, -120, x.shape)).astype(np.float32)
        w *= np.float32(2.0 ** 60)
    elif how == "late":
        x[:, C // 2:] *= np.float32(1e7)
    elif how == "late and quiet":
        x[:, C // 2:] *= np.float32(1e-9)
        m[::K - 1, :C // 2] = 0        # (two rows that see nothing else)
    elif how == "dead first":
        x[:, :3 * C // 4] = 0.0
        x[:, 3 * C // 4:] *= np.float32(1e-12)
    elif how == "one pixel":
        keep = x[:, C - 1, H - 1, W - 1].copy()
        x[:] = 0.0
        x[:, C - 1, H - 1, W - 1] = keep
    elif how == "few and quiet":  # below the window that no input of the first chunk gives, and near the end of what pieces hold
        x *= (rng.random(x.shape) < 0.5 / (C * R * S)) * np.float32(1e-10)
        w = np.copysign(np.maximum(np.abs(w), np.float32(0.01)), w)
    from paper_2011_06295_amd import binding as B
    layer = B.SparseConv(w, m, dtype="f32")
    _takes_the_kernel(layer, shape)
    _each_output(layer, w, m, x, st, p, how)
    layer.close()


@pytest.mark.parametrize("shape", RANGES, ids=lambda s: "x".join(map(str, s)))
def test_matrix_kernel_fp32_weights_of_every_size(shape):
    """Weights far below their row's largest count in full where they meet the only inputs that are not zero."""
    from paper_2011_06295_amd import binding as B
    N, C, K, R, S, H, W, st, p = shape
    rng = np.random.default_rng(98)
    w, m, x = rand_layer(rng, N, C, K, R, S, H, W, density=0.9)
    for k0 in range(0, K, 32):                               # 1, 2 ... of 32 rows
        flat = w[k0:k0 + 32].reshape(-1)
        flat[rng.choice(flat.size, size=1 + k0 // 32 * 3, replace=False)] *= np.float32(2.0 ** -20)
    small = np.abs(w) < 2.0 ** -19
    m[small] = 1
    alone = x * (rng.random(x.shape) < 0.5 / (C * R * S))    # most outputs see one input or none
    k, c, r, s = np.argwhere(small)[0]
    alone[0], alone[0, c, min(r, H - 1), min(s, W - 1)] = 0.0, 3.0
    layer = B.SparseConv(w, m, dtype="f32")
    _takes_the_kernel(layer, shape)
    assert layer.check_plan(N, H, W, st, p) == 0
    for data in (x, alone, alone * np.float32(1e-30)):
        _each_output(layer, w, m, data, st, p, "small weights")
    layer.close()
    w.reshape(-1)[::50] *= np.float32(1e-7)                  # many: not this kernel's
    layer = B.SparseConv(w, m, dtype="f32")
    assert layer.get_kernel(N, H, W, st, p) == "tile"
    _each_output(layer, w, m, x, st, p, "many small weights")
    layer.close()


def test_matrix_kernel_binary16_subnormals():
    """Inputs and weights below binary16's normal range take part with their value."""
    from paper_2011_06295_amd import binding as B
    rng = np.random.default_rng(95)
    shape = (40, 64, 65, 3, 3, 14, 14, 1, 1)
    for xs, ws in ((2e-6, 1000.0), (1000.0, 2e-6)):
        w, m, x = rand_layer(rng, *shape[:7], density=0.8)
        w, x = w * np.float32(ws), x * np.float32(xs)
        layer = B.SparseConv(w, m, dtype="f16")
        assert layer.get_kernel(40, 14, 14, 1, 1) == "matrix"
        assert_close(run_gpu(layer, x, 1, 1, "f16"), oracle_ref(w, m, x, 1, 1, "f16"), TOL["f16"], f"subnormal {xs} {ws}")
        layer.close()


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(40, 64, 65, 3, 3, 14, 14, 1, 1), (516, 45, 70, 3, 3, 4, 4, 1, 1), (1692, 130, 66, 3, 3, 2, 2, 1, 1), (228, 61, 40, 3, 3, 2, 30, 1, 1),
                                   (24, 48, 64, 3, 3, 29, 32, 2, 1), (134, 200, 80, 1, 3, 1, 36, 1, 0), (60, 240, 252, 1, 1, 16, 14, 1, 0), (52, 40, 64, 3, 3, 3, 44, 1, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_matrix_kernel_stages_runs_and_single_pixels(dtype, shape):
    """Where planes are whole runs of 8 bytes the kernel stages runs, else pixel by pixel: against the oracle, from an input that
    starts on a run's boundary and one that does not, with a value that is not finite and (fp32) one far above the others."""
    import torch
    layer, w, m, x = _layer(dtype, shape, 101, 0.9)
    N, C, K, R, S, H, W, st, p = shape
    x[N // 2, C // 2, H // 2, W // 2] *= np.float32(1e6 if dtype == "f32" else 8)
    x[N - 1, C - 1, H - 1, W - 1] = np.inf
    tdtype = torch.float16 if dtype == "f16" else torch.float32
    aligned = torch.from_numpy(x).cuda().to(tdtype)
    shifted = torch.empty(aligned.numel() + 1, dtype=tdtype, device="cuda")[1:].view(aligned.shape)
    shifted.copy_(aligned)
    plan = layer.get_matrix_plan(N, H, W, st, p)
    assert layer.check_plan(N, H, W, st, p) == 0
    # (one block of single pixels a wavefront, binary16 two, is as fast without)
    assert (plan["runs"] > 0) == (H * W % (2 if dtype == "f32" else 4) == 0 and plan["fly"] > (1 if dtype == "f32" else 2))
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oracle_ref(w, m, x, st, p, dtype)
    fin = np.isfinite(ref)
    assert not fin.all()
    for data in (aligned, shifted):
        got = layer.forward(data, st, p).float().cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
        assert_close(got[fin], ref[fin], TOL[dtype], f"{dtype} {shape}")
    layer.close()


@pytest.mark.parametrize("dtype,shape", [("f32", (516, 64, 70, 3, 3, 4, 4, 1, 1)), ("f32", (40, 64, 65, 3, 3, 14, 14, 1, 1)), ("f32", (60, 240, 252, 1, 1, 16, 14, 1, 0)),
                                         ("f16", (1692, 130, 66, 3, 3, 2, 2, 1, 1)), ("f16", (40, 64, 65, 3, 3, 14, 14, 1, 1)), ("f16", (60, 240, 252, 1, 1, 16, 14, 1, 0))],
                         ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_matrix_kernel_results_do_not_depend_on_the_inputs_address(dtype, shape):
    """An input that starts one element off a run's boundary gives the same bits, also where fp32 values within an image are so
    far apart that the scale its first chunk gives them shows."""
    import torch
    layer, w, m, x = _layer(dtype, shape, 103, 0.9)
    N, C, K, R, S, H, W, st, p = shape
    if dtype == "f32":
        x *= np.exp2(np.random.default_rng(104).uniform(-20, 20, x.shape)).astype(np.float32)
    assert layer.get_matrix_plan(N, H, W, st, p)["runs"] > 0, "the sizes no longer take the staging under test"
    aligned = torch.from_numpy(x).cuda().to(torch.float16 if dtype == "f16" else torch.float32)
    want = layer.forward(aligned, st, p)
    for off in (1, 2, 3):
        shifted = torch.empty(aligned.numel() + off, dtype=aligned.dtype, device="cuda")[off:].view(aligned.shape)
        shifted.copy_(aligned)
        assert torch.equal(layer.forward(shifted, st, p), want), off
    layer.close()
