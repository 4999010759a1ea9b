"""GPU parity of the window scoring kernels at the edges of their tiles: 64-key tiles in a ring of
four, 32-key subtiles, 128-key slices, four and eight row tiles, one to four row tiles per head,
padded rows, split keys; and of the calls that the pipelined kernel hands to them (many jobs of few
slices or with padded rows).  Against the oracle, at the bar of the other prefill tests."""
import pytest

from oracle import prefill as OP
from test_gpu_prefill import gen, run_case

pytestmark = pytest.mark.gpu

SHAPES = [
    # L, w, Hq, Hkv, pool
    (64, 32, 8, 2, 7),       # one tile, the window its second half
    (65, 8, 8, 2, 7),        # a one-key second tile
    (127, 32, 6, 2, 7),      # three heads per group
    (191, 32, 8, 2, 7),      # three tiles: an odd count
    (255, 31, 8, 2, 5),
    (256, 32, 8, 2, 7),      # the ring exactly full
    (257, 32, 8, 2, 7),      # its first reuse, one key
    (385, 33, 4, 2, 7),      # two row tiles per head, the second with one row
    (513, 64, 8, 2, 3),      # eight row tiles, two per head
    (642, 96, 4, 2, 7),      # three row tiles per head
    (900, 128, 2, 1, 7),     # four row tiles per head
    (1345, 32, 16, 2, 7),    # eight heads per group
    (1500, 65, 2, 2, 1),     # one head per group, no pooling
    (2300, 32, 8, 1, 13),    # split keys (several parts)
]


@pytest.mark.parametrize("L,w,hq,hkv,pool", SHAPES, ids=[f"L{s[0]}_w{s[1]}_{s[2]}x{s[3]}_p{s[4]}" for s in SHAPES])
def test_window_tile_edges(L, w, hq, hkv, pool, monkeypatch):
    monkeypatch.setenv("RKV_FORCE_WINDOW", "1")
    b = min(L - 1, w + 20)
    layers = [[gen(31, 0, l, L, w=w, Hq=hq, Hkv=hkv)] for l in range(2)]
    run_case([OP.SNAPKV, OP.H2O], [b, b], layers, window=w, pool_kernel=pool, label=f"tiles_L{L}_w{w}")


@pytest.mark.parametrize("L,w,hq,hkv", [(300, 32, 32, 8), (1100, 32, 32, 8), (300, 27, 16, 8), (700, 32, 8, 8)],
                         ids=["few_slices", "nine_slices", "padded_window", "padded_heads"])
def test_many_jobs_take_the_window_kernels(L, w, hq, hkv):
    """128 jobs, from which the window kernels take padded layouts and unpadded ones of up to five slices, or 160
    of up to eleven (few_slices, nine_slices)."""
    n = 20 if L == 1100 else 16
    layers = [[gen(32, 0, l, L, w=w, Hq=hq, Hkv=hkv)] for l in range(n)]
    run_case([OP.SNAPKV, OP.H2O] * (n // 2), [60] * n, layers, window=w, label=f"many_L{L}_w{w}")


@pytest.mark.parametrize("L,w,hq,rules", [(1700, 40, 8, [OP.H2O]), (1700, 27, 16, [OP.H2O]), (2100, 32, 8, [OP.SNAPKV, OP.H2O]),
                                          (2300, 27, 32, [OP.SNAPKV]), (800, 32, 32, [OP.SNAPKV, OP.H2O])],
                         ids=["two_tiles_h2o", "two_heads_h2o", "one_tile", "padded_window", "whole_tiles"])
def test_jobs_just_past_a_wave_stay_in_the_pipelined_kernel(L, w, hq, rules):
    """520 jobs, eight more than the window kernels have resident, of more slices than these are the faster ones for:
    the long-run form of the pipelined kernel, with padded rows and empty row tiles too."""
    import paper_2606_15157_amd as rkv
    layers = [[gen(34, s, l, L, w=w, Hq=hq, Hkv=8) for s in range(5)] for l in range(13)]
    rkv.profile_enable(rkv.STAGE_ZERO)   # the pipelined kernel's preparation; the window kernels have none
    try:
        run_case((rules * 13)[:13], [w + 40] * 13, layers, window=w, label=f"past_L{L}_w{w}")
        launches, _ = rkv.profile_read()
    finally:
        rkv.profile_enable(-1)
    assert launches == 1


@pytest.mark.parametrize("L,w,hq,hkv", [(3331, 27, 16, 8), (1024, 32, 32, 8)], ids=["padded", "few_slices"])
def test_window_kernels_are_as_exact_as_the_pipelined_one(L, w, hq, hkv):
    """The same layers in one call (160 jobs: the window kernels) and one by one (8 jobs: the pipelined kernel),
    against 64 bits: the first is no further off.  Both errors are means over 160 jobs of about 1e-7 each,
    so their ratio is known to about 2 %."""
    import paper_2606_15157_amd as rkv
    import torch
    from parity import bits_to_torch
    from test_gpu_causal_tiles import attention
    x = [gen(33, 0, l, L, w=w, Hq=hq, Hkv=hkv) for l in range(20)]
    q, k = ([bits_to_torch(y[n][None]) for y in x] for n in ("q", "k"))

    def scores(at):
        plan = rkv.Plan([rkv.SNAPKV] * len(at), [w + 100] * len(at), window=w, pool_kernel=7)
        out = rkv.evict_prefill(plan, [q[l] for l in at], [k[l] for l in at], [k[l] for l in at], score_out=True)
        return torch.cat(out["scores"])[..., :L - w].double()

    def pooled(a, b):
        sums = attention(a, b).sum(3)[..., :L - w]
        return torch.nn.functional.max_pool1d(sums.flatten(0, 2), 7, 1, 3).view(sums.shape).mean(2)

    want = torch.cat([pooled(a, b) for a, b in zip(q, k)])

    def error(got):
        return ((got - want).norm(dim=-1) / want.norm(dim=-1)).mean().item()

    window, pipelined = error(scores(range(20))), error(torch.cat([scores([l]) for l in range(20)]))
    assert window < 2e-7 and window <= 1.04 * pipelined, (window, pipelined)
