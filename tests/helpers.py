"""Shared helpers of the test-suite (comparison rule, layer construction)."""
import numpy as np

TOL = {"f32": 1e-5, "f16": 2e-3}


def assert_close(got, ref, tol, what=""):
    """Element-wise |got - ref| <= tol * max|ref|: the stated relative tolerance against the
    largest reference value (an element-wise ratio is undefined where a sum cancels to nearly
    zero); at the largest elements it is exactly the stated relative tolerance."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (what, got.shape, ref.shape)
    scale = float(np.max(np.abs(ref))) if ref.size else 0.0
    err = np.abs(got - ref)
    bound = np.full(err.shape, tol * scale)
    bad = err > bound
    if bad.any():
        idx = np.unravel_index(np.argmax(err - bound), err.shape)
        raise AssertionError(
            f"{what}: {int(bad.sum())}/{bad.size} outside tolerance {tol}; worst at {idx}: "
            f"got {got[idx]!r} ref {ref[idx]!r} (max|ref| {scale})")
    return float(err.max() / scale) if scale > 0 else 0.0


def rand_layer(rng, N, C, K, R, S, H, W, density=0.3, x_dist="normal"):
    w = rng.standard_normal((K, C, R, S)).astype(np.float32)
    m = (rng.random((K, C, R, S)) < density).astype(np.uint8)
    x = rng.standard_normal((N, C, H, W)) if x_dist == "normal" else rng.random((N, C, H, W))
    return w, m, x.astype(np.float32)


# Launches of the tile kernel on batches that leave images of the last group absent (one present, or all but one), several tiles to an
# image: lattice positions as lanes (one and two a lane, banded and whole rows) and outputs, from one and from two image groups.
# dtype, N, H = W, V, WP, WK, KW, Cc, LDS, LP, channel blocks, store, lanes
PARTIAL_GROUPS = [(dtype, n, h, v, *rest, lp, 0, store, lanes) for store in (1, 2) for dtype, n, h, v, rest, lp, lanes in [
    ("f32", 3, 23, 2, (1, 2, 4, 2, 0), 1, 1), ("f32", 5, 23, 4, (1, 2, 4, 2, 0), 1, 1), ("f32", 7, 24, 4, (2, 1, 16, 0, 0), 1, 1),
    ("f32", 5, 23, 4, (1, 2, 4, 2, 0), 2, 1), ("f32", 9, 24, 4, (1, 2, 8, 2, 0), 1, 3), ("f32", 13, 12, 4, (2, 2, 2, 2, 0), 1, 3),
    ("f32", 3, 24, 2, (1, 2, 4, 2, 0), 1, 2), ("f32", 5, 70, 4, (1, 2, 4, 0, 0), 1, 1),
    ("f16", 3, 23, 2, (1, 2, 4, 2, 0), 1, 1), ("f16", 5, 23, 4, (1, 2, 4, 2, 0), 2, 1), ("f16", 9, 23, 8, (1, 2, 4, 2, 0), 1, 1),
    ("f16", 15, 24, 8, (2, 1, 8, 0, 0), 1, 1), ("f16", 9, 24, 8, (1, 2, 4, 2, 0), 1, 2), ("f16", 17, 24, 8, (1, 2, 8, 2, 0), 1, 3),
    ("f16", 7, 24, 4, (2, 2, 2, 2, 0), 1, 3)]]
