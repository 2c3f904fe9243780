"""GPU parity of the any-shape weight gradient against the float64 oracle, at the
sizes where its plan and its indices can go wrong: strides (rows grouped by
residue, residues that no tap meets), tap groups (nine taps, uneven groups, one
kernel row), several ci tiles per workgroup, one to four co tiles, narrow outputs
with the units on two wave halves, bricks past the output, channels that are not
whole vectors, halos folded on one to three axes (the innermost among them).

Bars: 1e-5 (binary32) and 2e-2 (bf16 data, binary32 sums) of the largest value,
and integer data bit for bit. Binary32 data is split into three bf16 parts with
six products: 24 bits, each product good to 2^-24, sums in binary32.
"""
import numpy as np
import pytest

import synth
import shard_cases as cases
from gpu_util import dev, dy_box, host, log, run_wgrad, window_from_tile
from test_gpu_fold import INT_DIST, _canary_tile_and_slabs, _wgrad_folded, build_tile, sc  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [
    # (name, dtype, N, cin, cout, G, parts, K, S)
    ("3d_s2", "bf16", 1, 32, 64, (18, 20, 35), (2, 1, 1), (3, 3, 3), (2, 2, 2)),
    ("3d_s2_f32", "f32", 1, 40, 100, (17, 19, 37), (2, 2, 1), (3, 3, 3), (2, 2, 2)),
    ("3d_s3_narrow_f32", "f32", 2, 24, 16, (22, 21, 50), (2, 1, 1), (3, 3, 3), (2, 3, 2)),
    ("2d_k7_three_channels", "bf16", 1, 3, 32, (40, 45), (2, 1), (7, 7), (1, 1)),
    ("2d_k11", "f32", 1, 4, 8, (30, 41), (2, 1), (11, 11), (1, 1)),
    ("2d_k1_s2_four_ci_tiles", "bf16", 2, 128, 96, (21, 33), (2, 1), (1, 1), (2, 2)),
    ("1d_k3_three_ci_tiles", "f32", 3, 72, 136, (75,), (2,), (3,), (1,)),
    ("2d_k5_s4", "bf16", 1, 48, 72, (37, 50), (2, 2), (5, 5), (4, 3)),
    ("3d_three_axes", "bf16", 1, 32, 32, (12, 18, 70), (2, 2, 2), (3, 3, 3), (1, 1, 1)),
    ("3d_three_axes_f32", "f32", 1, 12, 20, (10, 12, 30), (2, 2, 2), (3, 3, 3), (1, 1, 1)),
    ("2d_wide", "bf16", 1, 136, 136, (19, 70), (2, 1), (3, 3), (1, 1)),
]


@pytest.mark.parametrize("case", SHAPES, ids=lambda c: c[0])
def test_any_shape_wgrad_every_shard(sc, case):  # noqa: F811
    name, dt, N, cin, cout, G, parts, K, S = case
    w = cases.Workload(name, dt, N, cin, cout, G, parts, K, S, (0,) * len(G), x_dist=(synth.UNIFORM, (-1.0, 1.0)),
                       w_dist=(synth.UNIFORM, (-0.5, 0.5)), dy_dist=(synth.UNIFORM, (-1.0, 1.0)))
    for idx in w.shards():
        for dist in (None, INT_DIST):
            log(f"wgrad {name} shard {idx} {'int' if dist else 'float'}")
            desc, tile, slabs, sg, full_h = _canary_tile_and_slabs(sc, w, idx, dist)
            dyh = dy_box(w, sg, dist)
            xw, origin = window_from_tile(w, sg, full_h)
            ref = cases.expected_wgrad(w, sg, xw, origin, cases.to_ncdhw(cases.as_f64(dyh, w)))
            d2, t2, _, _ = build_tile(sc, w, idx, dist)
            for got in (run_wgrad(sc, w, d2, t2, sg, dev(dyh)), _wgrad_folded(sc, w, desc, tile, slabs, sg, dev(dyh))):
                got = host(got).astype(np.float64)
                if dist is INT_DIST:
                    assert np.array_equal(got, ref), idx
                else:
                    assert cases.norm_max_err(got, ref) <= cases.TOL[dt], idx


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_f32_wgrad_special_values(sc, value):  # noqa: F811
    """An input value that has no finite bf16 parts reaches exactly the dw entries
    of its channel, with the products' own values: infinite or NaN where dy
    times the value is, large but finite where it is finite."""
    import torch
    ext, c, co = (16, 32), 8, 8
    rng = np.random.default_rng(5)
    x = rng.integers(-2, 3, (1,) + ext + (c,)).astype(np.float32)
    dy = np.full((1,) + ext + (co,), 0.5, np.float32)  # 0.5: the middle and low parts are zero
    dy[..., 1] = -0.25
    x[0, 5, 9, 3] = value
    desc = sc.tile_desc(1, c, ext)
    dw = torch.empty((co, c, 1, 1), dtype=torch.float32, device="cuda")
    n = sc.shard_conv_workspace_bytes(1, desc, sc.SHARD_F32, co, (1, 1), (1, 1), ext)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    sc.shard_conv_wgrad(desc, dev(x), dev(dy), co, (1, 1), (1, 1), (0, 0), ext, dw, ws)
    got = host(dw)[:, :, 0, 0]
    with np.errstate(invalid="ignore", over="ignore"):
        want = np.einsum("nhwo,nhwc->oc", dy.astype(np.float64), x.astype(np.float64))
    if np.isfinite(value):
        assert np.allclose(got, want, rtol=1e-6)
    else:
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[~np.isnan(want)], want[~np.isnan(want)].astype(np.float32))
