"""GPU parity of the kernels over causal logits (full-span H2O and the entropy profile) at the edges
of their tiles: 64-row tiles in a ring of four, 32-row subtiles, four and eight row tiles and one, two or
four key groups a workgroup (chosen by the number of jobs), inputs that are not 16-byte aligned, and a
row whose normaliser is not a number.  Against the same sums in 64 bits: 32-bit sums of at most a few
hundred rounded terms per lane, exponentials of logits that 32 bits hold to 1e-6."""
import math

import pytest

pytestmark = pytest.mark.gpu

RTOL = 1e-5


def gen(seed, *shape):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def shifted(x):
    """The same values 8 bytes into a buffer: contiguous, not 16-byte aligned."""
    import torch
    flat = torch.empty(x.numel() + 4, device=x.device, dtype=x.dtype)
    out = flat[4:].view(x.shape)
    out.copy_(x)
    assert out.data_ptr() % 16 == 8
    return out


def attention(q, k):
    """Causal softmax rows [B, Hkv, G, n, L] of q [B, Hq, n, d] (the last n positions), in 64 bits."""
    import torch
    b, hq, n, d = q.shape
    hkv, L = k.shape[1:3]
    z = torch.matmul(q.double().view(b, hkv, -1, d), k.double().transpose(2, 3).contiguous()).view(b, hkv, hq // hkv, n, L)
    t = torch.arange(L - n, L, device=q.device).unsqueeze(1)
    return torch.softmax((z / math.sqrt(d)).masked_fill(torch.arange(L, device=q.device) > t, -math.inf), dim=-1)


def full_span(q, k):
    """Scores of every key (all kept, so that every score is reported)."""
    import paper_2606_15157_amd as rkv
    import torch
    L = k.shape[2]
    out = rkv.evict_prefill(rkv.Plan([rkv.H2O_FULL], [L], window=1), [q], [k], [k], score_out=True)
    torch.cuda.synchronize()
    return out["scores"][0].double(), rkv.prefill_check(out["workspace"])


FULL = [
    # L, B, Hq, Hkv
    (1, 1, 4, 1), (31, 1, 4, 1), (64, 1, 2, 2), (65, 2, 4, 2), (127, 1, 8, 1), (193, 1, 8, 2), (256, 1, 16, 2),
    (257, 1, 1, 1), (321, 2, 2, 1), (640, 1, 8, 2),
    (129, 8, 32, 8), (129, 9, 32, 8), (300, 5, 32, 16), (200, 20, 32, 4),   # 64 to 160 blocks of 256 keys: four key groups
    (150, 160, 16, 8), (150, 35, 64, 8),    # 1280 and 280: one and four
    (300, 8, 8, 8), (300, 9, 8, 8),         # one head a group, 128 and 144: four and two
    (300, 16, 16, 8), (300, 17, 16, 8),     # two heads, 256 and 272: four and two
    (300, 20, 32, 8), (300, 21, 32, 8),     # four heads, 320 and 336: four and two
    (300, 41, 32, 4),                       # eight heads, 328: two
    (259, 48, 8, 8), (300, 64, 16, 8),      # 768 and 1024: one; four and eight row tiles
    (259, 48, 32, 8), (259, 96, 32, 4),     # 768: one, four and eight heads per group
    (700, 125, 12, 3),                      # 4125 blocks of query rows: job by job, 375 jobs in rounds of eight
]


@pytest.mark.parametrize("L,B,hq,hkv", FULL, ids=[f"L{s[0]}_b{s[1]}_{s[2]}x{s[3]}" for s in FULL])
def test_full_span_tile_edges(L, B, hq, hkv):
    import torch
    q, k = gen(41, B, hq, L, 128), gen(42, B, hkv, L, 128)
    got, status = full_span(q, k)
    assert status == 0
    torch.testing.assert_close(got, attention(q, k).sum(3).mean(2), rtol=RTOL, atol=0)


ENTROPY = [
    # L, n_q, B, Hq, Hkv
    (1, 1, 1, 4, 1), (64, 33, 1, 4, 1), (65, 65, 2, 2, 2), (127, 1, 1, 8, 1), (320, 129, 1, 4, 2), (513, 31, 1, 8, 2),
    (700, 257, 1, 1, 1), (641, 64, 1, 16, 2),
    (300, 300, 64, 16, 8), (260, 129, 128, 32, 8),   # eight row tiles, two and four heads per group
    (260, 129, 43, 12, 3),                           # the last half of the queries: job by job, 129 jobs
]


@pytest.mark.parametrize("L,n_q,B,hq,hkv", ENTROPY, ids=[f"L{s[0]}_q{s[1]}_b{s[2]}_{s[3]}x{s[4]}" for s in ENTROPY])
def test_entropy_tile_edges(L, n_q, B, hq, hkv):
    import paper_2606_15157_amd as rkv
    import torch
    q, k = gen(43, B, hq, n_q, 128), gen(44, B, hkv, L, 128)
    out = rkv.entropy_profile([q], [k])
    p = attention(q, k)
    ref = -torch.xlogy(p, p).sum(-1).view(1, B, hq, n_q)
    assert int(out["status"].item()) == 0
    # a row's entropy is a difference of terms of a few nats: 1e-5 of them absolutely
    torch.testing.assert_close(out["rows"].double(), ref, rtol=RTOL, atol=RTOL)
    torch.testing.assert_close(out["h"].double(), ref.mean(dim=(1, 2, 3)), rtol=RTOL, atol=RTOL)


def test_unaligned_inputs():
    """Streamed rows that are not 16-byte aligned take another way into LDS; the results are the same bits."""
    import paper_2606_15157_amd as rkv
    import torch
    L = 709
    q, k = gen(45, 1, 8, L, 128), gen(46, 1, 2, L, 128)
    a, b = rkv.entropy_profile([q], [k]), rkv.entropy_profile([shifted(q)], [shifted(k)])
    assert torch.equal(a["rows"], b["rows"]) and torch.equal(a["h"], b["h"])
    assert torch.equal(full_span(q, k)[0], full_span(shifted(q), shifted(k))[0])
    q = gen(45, 1, 2, L, 128)   # one head a group: an odd number of query tiles for every second key block
    assert torch.equal(full_span(q, k)[0], full_span(shifted(q), shifted(k))[0])


def test_unaligned_window_inputs(monkeypatch):
    import paper_2606_15157_amd as rkv
    import torch
    monkeypatch.setenv("RKV_FORCE_WINDOW", "1")
    L = 709
    q, k, v = gen(47, 1, 8, 32, 128), gen(48, 1, 2, L, 128), gen(49, 1, 2, L, 128)
    plan = rkv.Plan([rkv.SNAPKV], [200], window=32, pool_kernel=7)
    a, b = (rkv.evict_prefill(plan, [x], [y], [v], score_out=True) for x, y in ((q, k), (shifted(q), shifted(k))))
    assert torch.equal(a["scores"][0], b["scores"][0]) and torch.equal(a["idx"][0], b["idx"][0])


@pytest.mark.parametrize("which", ["queries", "keys"])
def test_unaligned_inputs_do_not_take_the_pipelined_kernel(which, monkeypatch):
    """One job of a short prompt, the pipelined kernel's, whose queries or keys are not 16-byte aligned: the
    window kernels' bits."""
    import paper_2606_15157_amd as rkv
    import torch
    L = 709
    q, k, v = gen(47, 1, 8, 32, 128), gen(48, 1, 2, L, 128), gen(49, 1, 2, L, 128)
    plan = rkv.Plan([rkv.SNAPKV, rkv.H2O], [200] * 2, window=32, pool_kernel=7)
    x, y = (shifted(q), k) if which == "queries" else (q, shifted(k))
    a = rkv.evict_prefill(plan, [q, x], [k, y], [v, v], score_out=True)   # the second layer's
    monkeypatch.setenv("RKV_FORCE_WINDOW", "1")
    b = rkv.evict_prefill(plan, [q, q], [k, k], [v, v], score_out=True)
    for l in range(2):
        assert torch.equal(a["scores"][l], b["scores"][l]) and torch.equal(a["idx"][l], b["idx"][l])


def test_full_span_row_that_is_not_a_number():
    """Query 100 of head 0 is NaN: keys up to 100 of its KV head get no score, the keys after it theirs."""
    import torch
    L, t = 300, 100
    q, k = gen(50, 1, 8, L, 128), gen(51, 1, 2, L, 128)
    q[0, 0, t] = math.nan
    got, status = full_span(q, k)
    assert status == 2
    ref = attention(q, k)
    ref[0, 0, 0, t, t + 1:] = 0
    ref = ref.sum(3).mean(2)
    assert got[0, 0, :t + 1].isnan().all()
    torch.testing.assert_close(got[0, 0, t + 1:], ref[0, 0, t + 1:], rtol=RTOL, atol=0)
    torch.testing.assert_close(got[0, 1], ref[0, 1], rtol=RTOL, atol=0)
