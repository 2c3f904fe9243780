"""GPU parity of the tiled forward and input gradient against the float64 oracle,
at the sizes where the plan and the three-part binary32 products can go wrong:
bricks smaller than one wave's tile, one tap plane per pass (strided binary32),
several channel passes, one to three channel units, channels that are not whole
units, one to five N tiles, odd numbers of iterations, and a halo read in place.

Bars: 1e-5 (binary32) and 2e-2 (bf16 data, binary32 sums) of the largest value,
and integer data bit for bit. A binary32 value is three bf16 parts (24 bits), six
products of which keep every term above 2^-24 of the product.
"""
import numpy as np
import pytest

import synth
import shard_cases as cases
from gpu_util import dev, host, log, run_fwd, weights, window_from_tile
from test_gpu_dgrad import _dgrad_case, _same
from test_gpu_fold import INT_DIST, _canary_tile_and_slabs, _folded, build_tile, sc  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [
    # (name, dtype, N, cin, cout, G, parts, K, S)
    ("tiny_brick", "f32", 1, 8, 8, (16, 16), (2, 1), (3, 3), (1, 1)),
    ("one_tap", "f32", 2, 24, 40, (9, 37), (2, 1), (1, 1), (1, 1)),
    ("three_channels_k7", "f32", 1, 3, 32, (40, 45), (2, 1), (7, 7), (1, 1)),
    ("seven_channels_s2", "f32", 1, 7, 100, (21, 45), (1, 2), (3, 3), (2, 2)),
    ("planes_narrow", "f32", 1, 24, 16, (22, 21, 50), (2, 1, 1), (3, 3, 3), (2, 2, 2)),
    ("planes_s3_s1", "f32", 1, 40, 72, (19, 13, 37), (2, 2, 1), (5, 3, 3), (3, 1, 2)),
    ("planes_wide_c140", "f32", 1, 140, 130, (14, 13, 20), (2, 1, 1), (3, 3, 3), (2, 2, 1)),
    ("1d_k4_taps", "f32", 3, 8, 64, (150,), (2,), (5,), (1,)),
    ("eight_channels_3d", "f32", 1, 8, 64, (12, 14, 37), (2, 2, 1), (3, 3, 3), (1, 1, 1)),
    ("eight_channels_3d", "bf16", 1, 8, 48, (12, 14, 37), (2, 2, 1), (3, 3, 3), (1, 1, 1)),
    ("three_channels_s2", "bf16", 2, 3, 64, (39, 46), (2, 1), (7, 5), (2, 2)),
    ("one_channel_three_axes", "bf16", 1, 1, 20, (10, 12, 30), (2, 2, 2), (3, 3, 3), (1, 1, 1)),
]


@pytest.mark.parametrize("case", SHAPES, ids=lambda c: f"{c[1]}_{c[0]}")
def test_forward_and_input_gradient_every_shard(sc, case):  # noqa: F811
    name, dt, N, cin, cout, G, parts, K, S = case
    w = cases.Workload(name, dt, N, cin, cout, G, parts, K, S, (0,) * len(G), x_dist=(synth.UNIFORM, (-1.0, 1.0)),
                       w_dist=(synth.UNIFORM, (-0.5, 0.5)), dy_dist=(synth.UNIFORM, (-1.0, 1.0)))
    for idx in w.shards():
        for dist in (None, INT_DIST):
            log(f"fwd {name} shard {idx} {'int' if dist else 'float'}")
            w_host, w64 = weights(w, dist)
            desc, tile, slabs, sg, full_h = _canary_tile_and_slabs(sc, w, idx, dist)
            xw, origin = window_from_tile(w, sg, full_h)
            ref = cases.expected_fwd(w, sg, xw, origin, w64)
            d2, t2, _, _ = build_tile(sc, w, idx, dist)
            plain = host(run_fwd(sc, w, d2, t2, sg, dev(w_host)))
            folded = host(_folded(sc, w, desc, tile, slabs, sg, dev(w_host), sc.SHARD_REGION_ALL))
            assert plain.tobytes() == folded.tobytes(), idx
            y = _folded(sc, w, desc, tile, slabs, sg, dev(w_host), sc.SHARD_REGION_INTERIOR)
            y = host(_folded(sc, w, desc, tile, slabs, sg, dev(w_host), sc.SHARD_REGION_BOUNDARY, y))
            assert y.tobytes() == plain.tobytes(), idx
            dgot, dref = _dgrad_case(sc, w, idx, dist)
            if dist is INT_DIST:
                assert _same(w, dgot, dref), idx
                assert _same(w, plain, ref), idx
            else:
                assert cases.norm_max_err(cases.as_f64(plain, w), ref) <= cases.TOL[dt], idx
                assert cases.norm_max_err(cases.as_f64(dgot, w), dref) <= cases.TOL[dt], idx


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_f32_forward_special_values(sc, value):  # noqa: F811
    """An input value that has no finite bf16 parts reaches exactly the outputs
    whose window holds it, with the products' own values."""
    import torch
    ext, c, co = (16, 32), 24, 8
    rng = np.random.default_rng(5)
    x = rng.integers(-2, 3, (1,) + ext + (c,)).astype(np.float32)
    x[0, 5, 9, 3] = value
    wt = np.full((co, c, 1, 1), 0.5, np.float32)  # powers of two: the middle and low parts are zero
    wt[1] = -0.25
    desc = sc.tile_desc(1, c, ext)
    y = torch.empty((1,) + ext + (co,), dtype=torch.float32, device="cuda")
    n = sc.shard_conv_workspace_bytes(0, desc, sc.SHARD_F32, co, (1, 1), (1, 1), ext)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    sc.shard_conv_fwd(desc, dev(x), dev(wt), co, (1, 1), (1, 1), (0, 0), ext, y, ws)
    got = host(y)
    with np.errstate(invalid="ignore", over="ignore"):
        want = np.einsum("nhwc,oc->nhwo", x.astype(np.float64), wt[:, :, 0, 0].astype(np.float64))
    if np.isfinite(value):
        assert np.allclose(got, want, rtol=1e-6)
    else:
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[~np.isnan(want)], want[~np.isnan(want)].astype(np.float32))
