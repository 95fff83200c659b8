"""Which kernel an automatic forward takes, where the choice carries more than speed.  Needs no GPU."""
import numpy as np
import pytest

from paper_2011_06295_amd import binding as B


def _fp32_layer(kept, K=256, C=256, R=3, unify=False):
    """A layer whose output channels keep these counts of weights in turn."""
    rng = np.random.default_rng(21)
    m = np.zeros((K, C * R * R), dtype=np.uint8)
    for k in range(K):
        m[k, rng.permutation(C * R * R)[:kept[k % len(kept)]]] = 1
    w = rng.standard_normal((K, C, R, R)).astype(np.float32)
    return B.SparseConv(w, m.reshape(w.shape), dtype="f32", unify=unify)


def _masked(K, C, density):
    rng = np.random.default_rng(22)
    w = rng.standard_normal((K, C, 3, 3), dtype=np.float32)
    return w, (rng.random(w.shape, dtype=np.float32) < density).astype(np.uint8)


@pytest.mark.parametrize("unify", [False, True])
@pytest.mark.parametrize("kept,kernel", [([460] * 255 + [9], "matrix"), ([460] * 255 + [1], "matrix"), ([460] * 255 + [60], "matrix"),
                                         ([460] * 255 + [0], "matrix"), ([460] * 31 + [60], "matrix"), ([460] * 3 + [3], "matrix"),
                                         ([460] * 3 + [20], "tile"), ([460] * 3 + [40], "tile")])
def test_short_rows_keep_the_precision_of_fp32_products(kept, kernel, unify):
    """256 -> 256, 14 x 14, 80 %: the matrix kernel holds a weight and an input in two binary16 pieces each, 1.0e-7 of a sum of
    10 terms, where fp32 products leave 0.6e-7 (0.9e-7 and 0.5e-7 of 5 terms; from some 65 terms on it is the more exact one).
    So it multiplies rows of up to 68 as fp32, with or without zero weights that fill them up.  Eight such rows among 32 take
    it too long (160 weights), or are more than it does so (320): the tile kernel's."""
    layer = _fp32_layer(kept, unify=unify)
    assert layer.get_kernel(256, 14, 14, 1, 1) == kernel
    assert layer.check_plan(256, 14, 14, 1, 1) == 0
    layer.close()


@pytest.mark.parametrize("sparsity,kernel", [(80, "matrix"), (85, "matrix"), (88, "matrix"), (90, "tile"), (91, "tile")])
def test_fp32_layers_take_the_matrix_kernel_where_it_was_measured_faster(sparsity, kernel):
    """256 -> 256, 14 x 14, batch 256, us by the matrix and by the tile kernel: 80 %: 169 and 273, 85 %: 167 and 213, 88 %: 165
    and 177; by the tile kernel at 90 %: 153, at 91 %: 142."""
    layer = _fp32_layer([2304 * (100 - sparsity) // 100])
    assert layer.get_kernel(256, 14, 14, 1, 1) == kernel
    layer.close()


# N, C, K, taps, H = W, density.  With inputs that went through a ReLU the matrix kernel's error against 64 bits is 1.15, 1.10, 1.09, 1.08
# and 1.06 of the tile kernel's.
@pytest.mark.parametrize("N,C,K,R,H,density", [(1, 1197, 473, 1, 34, 0.2), (6, 596, 215, 1, 51, 0.2), (50, 22, 21, 3, 57, 0.5),
                                               (20, 363, 44, 1, 39, 0.3), (27, 1250, 498, 1, 9, 0.3)])
def test_fp32_products_are_not_given_up_for_a_few_per_cent(N, C, K, R, H, density):
    """The matrix kernel is estimated 1 to 9 % below the tile launch that is taken, and above 0.85 of the estimate it was measured beside."""
    rng = np.random.default_rng(24)
    w = rng.standard_normal((K, C, R, R), dtype=np.float32)
    order = rng.random((K, C * R * R))
    m = (order <= np.partition(order, int(C * R * R * density) - 1, axis=1)[:, int(C * R * R * density) - 1:][:, :1]).astype(np.uint8)
    layer = B.SparseConv(w, m.reshape(w.shape))
    assert layer.get_kernel(N, H, H, 1, R // 2) == "tile"
    layer.close()


@pytest.mark.parametrize("N", [30, 42, 43, 60])
def test_small_layers_are_priced_as_they_run(N):
    """512 -> 512, 2 x 2, 80 %, binary16 takes 18 us by the matrix kernel and 23 to 32 by the tile kernel from 30 images to 60; an
    estimate of single pixels, which the kernel does not stage there, had it at the tile kernel up to 42."""
    layer = B.SparseConv(*_masked(512, 512, 0.2), dtype="f16")
    assert layer.get_kernel(N, 2, 2, 1, 1) == "matrix"
    layer.close()


def test_binary16_layers_take_the_kernel_that_was_measured_faster():
    """VGG-16's last layer, batch 256 (512 -> 512, 2 x 2, 95 %): 18.7 us by the matrix kernel, 26 by the tile kernel."""
    layer = B.SparseConv(*_masked(512, 512, 0.05), dtype="f16")
    assert layer.get_kernel(256, 2, 2, 1, 1) == "matrix"
    layer.close()


# Layers whose fastest launch by estimate deals the channels over fewer parts than before (4, 2, 2 and 1), or over two, with 40 MB of
# partial sums, where the whole tables were less than the static scratch.  N, C, K, taps, H = W, stride, density, parts at least
CHOICES = [(241, 136, 16, 5, 6, 1, 0.3, 8), (15, 62, 59, 3, 4, 1, 0.2, 4), (4, 44, 19, 5, 108, 1, 0.2, 4), (2, 274, 403, 1, 31, 1, 0.125, 2),
           (14, 487, 192, 3, 40, 1, 0.01, 1)]


@pytest.mark.parametrize("N,C,K,R,H,stride,density,parts", CHOICES)
def test_the_launch_keeps_its_parts_and_fits_the_static_scratch(N, C, K, R, H, stride, density, parts):
    """A sum dealt over parts is the more exact one, and what sparse_conv_forward_static took it still takes."""
    rng = np.random.default_rng(23)
    w = rng.standard_normal((K, C, R, R), dtype=np.float32)
    layer = B.SparseConv(w, (rng.random(w.shape, dtype=np.float32) < density).astype(np.uint8))
    plan = layer.get_launch(N, H, H, stride, R // 2)
    assert layer.check_plan(N, H, H, stride, R // 2) == 0
    assert plan["csplit"] >= parts
    sums = plan["grid"] * plan["threads"] * plan["KW"] * plan["LP"] * plan["V"] * 4 if plan["csplit"] > 1 else 0
    assert plan["entries"] * plan["entry_bytes"] + sums <= 16 << 20
    layer.close()


def _choice(N, C, K, R, H, stride, density, coded=False):
    rng = np.random.default_rng(25)
    order = rng.random((K, C * R * R), dtype=np.float32)
    kept = max(1, int(C * R * R * density))
    m = (order <= np.partition(order, kept - 1, axis=1)[:, kept - 1:kept]).astype(np.uint8).reshape(K, C, R, R)
    if coded:
        layer = B.SparseConv.from_codebook(rng.integers(0, 16, m.shape, dtype=np.uint8), np.sort(rng.standard_normal(16)).astype(np.float32), m)
    else:
        layer = B.SparseConv(rng.standard_normal(m.shape, dtype=np.float32), m)
    plan = layer.get_launch(N, H, H, stride, R // 2)
    assert layer.get_kernel(N, H, H, stride, R // 2) == "tile" and layer.check_plan(N, H, H, stride, R // 2) == 0
    layer.close()
    return plan


# N, C, K, taps, H = W, density
@pytest.mark.parametrize("layer", [(158, 301, 45, 3, 71, 0.1), (58, 160, 17, 5, 105, 0.1), (5, 22, 449, 3, 74, 0.125)])
def test_coded_layers_are_ranked_by_the_kernel_they_run(layer):
    """Weights that are binary16 centroids have a stream a row, whatever the launch: 789 us by two positions a lane and 995 by 16 rows
    a wavefront, 421 and 460, 48 and 56."""
    N, C, K, R, H, density = layer
    plan = _choice(N, C, K, R, H, 1, density, coded=True)
    assert plan["entry_bytes"] == 4 and plan["LP"] == 2 and plan["KW"] <= 4


@pytest.mark.parametrize("layer", [(1, 44, 91, 5, 96, 0.1), (1, 48, 500, 3, 66, 0.09), (2, 81, 101, 3, 106, 0.125)])
def test_a_workgroup_of_more_than_twelve_wavefronts_has_a_cu_to_itself(layer):
    """Its wavefronts go round the SIMDs from the same one on, and no SIMD holds eight of any fp32 kernel on lattice lanes.  28 us by 15
    wavefronts in 456 workgroups and 20 by 16 in 232, 27 by 13 in 504 and 20 by 11, 34 by 14 in 360 and 27 by 7 (the last with stride 2)."""
    N, C, K, R, H, density = layer
    plan = _choice(N, C, K, R, H, 2 if N == 2 else 1, density)
    assert plan["WP"] * plan["WK"] <= 12 or plan["grid"] <= 256


@pytest.mark.parametrize("layer,want", [((1, 500, 393, 5, 63, 0.05), {"V": 1, "LP": 2, "csplit": 2}), ((4, 979, 116, 1, 46, 0.07), {"V": 4, "csplit": 4})])
def test_a_launch_that_may_fit_the_static_scratch_is_not_given_up(layer, want):
    """Tables and partial sums of the launch by rows are about the scratch, so it is a choice whether or not they surely fit: 163 us by it and
    215 by the best that surely does; 28 and 39."""
    N, C, K, R, H, density = layer
    plan = _choice(N, C, K, R, H, 1, density)
    assert {k: plan[k] for k in want} == want


def _split(N, C, K, R, H, density, stride=1):
    rng = np.random.default_rng(26)
    w = rng.standard_normal((K, C, R, R), dtype=np.float32)
    layer = B.SparseConv(w, (rng.random(w.shape, dtype=np.float32) < density).astype(np.uint8), dtype="f16")
    plan = layer.get_matrix_plan(N, H, H, stride, R // 2) if layer.get_kernel(N, H, H, stride, R // 2) == "matrix" else None
    assert layer.check_plan(N, H, H, stride, R // 2) == 0
    layer.close()
    return plan


@pytest.mark.parametrize("C,KS", [(48, 4), (64, 4), (65, 8), (128, 8)])
def test_eight_wavefronts_share_more_than_64_channels(C, KS):
    """With 64 or fewer, half of them have none to multiply."""
    assert _split(1, C, 128, 3, 14, 0.1)["KS"] == KS


@pytest.mark.parametrize("N,C,K,R,H,density", [(63, 118, 26, 3, 38, 0.1), (60, 1489, 31, 1, 47, 0.3)])
def test_eight_wavefronts_take_large_launches_of_few_rows(N, C, K, R, H, density):
    """Of at most 32 output channels four wavefronts multiply 64: 22.7 us by eight and 29.5 by four, 105 and 116."""
    assert _split(N, C, K, R, H, density)["KS"] == 8


@pytest.mark.parametrize("C", [16, 40, 63, 64])
def test_odd_planes_are_staged_in_runs_from_16_channels_on(C):
    """Of 1979 splits of layers with fewer than 64 channels the mean is 12 % faster so."""
    assert _split(150, C, 64, 3, 17, 0.1)["runs"] > 0


@pytest.mark.parametrize("N,C,K,H,density", [(8, 1, 217, 207, 0.3), (47, 3, 82, 133, 0.2), (11, 1, 160, 105, 0.2)])
def test_first_layers_on_odd_planes_stay_with_the_tile_kernel(N, C, K, H, density):
    """us by the tile kernel and by the matrix kernel with runs: 44 and 63, 62 and 72, 22 and 23."""
    assert _split(N, C, K, 3, H, density) is None


def test_runs_of_odd_planes_are_priced_as_they_load():
    """301 -> 45, 71 x 71, batch 158: 354 us in chunks of 32 channels, which leave a CU two workgroups, 319 in chunks of 16."""
    plan = _split(158, 301, 45, 3, 71, 0.1)
    assert plan["runs"] == 1 and plan["CG"] == 2


def test_layers_beyond_the_last_cache_hold_all_loads_in_flight():
    """239 -> 134, 73 x 73, stride 2, fragments of 2 x 4, which have one block of runs in flight and six of single pixels: 397 us by runs
    at batch 247 (650 MB), 382 pixel by pixel; at batch 60 it is staged in runs."""
    plans = [_split(N, 239, 134, 3, 73, 0.1, stride=2) for N in (247, 60)]
    assert [(p["MK"], p["NP"], p["fly"], p["runs"]) for p in plans] == [(2, 4, 6, 0), (2, 4, 6, 1)]
