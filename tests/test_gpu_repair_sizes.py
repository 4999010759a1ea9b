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


@pytest.mark.parametrize("keys,value", [((3500,), 4.0), ((100, 3500), 1.953125)], ids=["last_part", "over_all_parts"])
@pytest.mark.parametrize("force", ["0", "1"], ids=["pipelined", "window"])
def test_overflow_over_key_parts(keys, value, force, monkeypatch):
    """Four jobs of 32 slices: the window rows kernel cuts the keys into five parts of 832.  A row of fours
    with reference 0 overflows in the last part alone (a logit of 261 binary orders), or only in the sum over
    the parts: two keys of 2^127.52 each, in the first and the last one."""
    from synth import f32_to_bf16_bits
    monkeypatch.setenv("RKV_FORCE_WINDOW", force)
    L, w, G = 4096, 32, 4
    x = {n: a.copy() for n, a in gen(14, 0, 0, L, w=w, Hq=2 * G, Hkv=2).items()}
    x["q"][G, w // 2] = f32_to_bf16_bits(np.full(128, 4.0, np.float32))
    x["k"][1, [0, L - w + w // 2]] = 0
    for j in keys:
        x["k"][1, j] = f32_to_bf16_bits(np.full(128, value, np.float32))
    run_case([OP.SNAPKV, OP.H2O], [100, 100], [[x], [x]], window=w, label=f"parts_{keys}", status=4)
