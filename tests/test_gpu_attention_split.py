"""GPU parity of the ring-attention block step where few queries leave the chip idle
and a workgroup's two wave groups take half of the keys each: odd and even numbers
of 32-key blocks, a ragged last block, query counts around the 128-query tile, both
head dims, and a second block merged into the state. Bars as for the other attention tests: output 2e-2 of the largest
value (bf16 probabilities), log-normaliser 1e-4.
"""
import math

import numpy as np
import pytest

from gpu_util import log
from oracle import attention as oat
from test_gpu_attention import _bf16, _check, _state, sc  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [
    # (B, H, Sq, Sk, D)
    (1, 2, 129, 321, 64),
    (1, 1, 128, 352, 128),
    (2, 3, 127, 380, 128),
    (1, 1, 1, 2044, 64),
    (1, 2, 300, 1057, 128),
    (1, 16, 2044, 700, 128),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_two_blocks(sc, shape):  # noqa: F811
    B, H, Sq, Sk, D = shape
    log(f"split attention {shape}")
    rng = np.random.default_rng(sum(shape))
    q, q64 = _bf16(rng, (B, H, Sq, D))
    kv = [(_bf16(rng, (B, H, n, D), 1 + 2 * i), _bf16(rng, (B, H, n, D))) for i, n in enumerate((Sk, Sk - 31))]
    scale = 1 / math.sqrt(D)
    o, lse = _state(B, H, Sq, D)
    for i, ((k, _), (v, _)) in enumerate(kv):
        sc.shard_attn_block(q, k, v, o, lse, scale, i == 0)
    k64 = np.concatenate([k[1] for k, _ in kv], axis=2)
    v64 = np.concatenate([v[1] for _, v in kv], axis=2)
    ref_o, ref_lse = oat.full_attention(q64, k64, v64, scale)
    _check(o, lse, ref_o, ref_lse)
