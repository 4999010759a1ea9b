"""The exact rescoring of an overflowing job at the edges of its LDS layout: up to 128 and up to 256 window
rows (heads of the group times the window), one to eight heads per group, against the oracle."""
import numpy as np
import pytest

from oracle import prefill as OP
from test_gpu_prefill import gen, run_case

pytestmark = pytest.mark.gpu

SHAPES = [(4, 31), (4, 32), (8, 16), (8, 17), (1, 128), (1, 129), (2, 64), (2, 65), (8, 32), (1, 5)]


@pytest.mark.parametrize("G,w", SHAPES, ids=[f"g{g}_w{w}" for g, w in SHAPES])
def test_repair_layouts(G, w):
    from synth import f32_to_bf16_bits
    L = 700
    x = {n: a.copy() for n, a in gen(14, 0, 0, L, w=w, Hq=2 * G, Hkv=2).items()}
    four = f32_to_bf16_bits(np.full(128, 4.0, np.float32))
    x["q"][G, w // 2] = four      # a row of KV head 1 whose logit with key 100 is ~180 above its reference
    x["k"][1, 100] = four
    b = w + 40
    run_case([OP.SNAPKV, OP.H2O], [b, b], [[x], [x]], window=w, label=f"repair_g{G}_w{w}", status=4)
