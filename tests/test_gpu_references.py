"""The row references of the scoring kernels (a row's logit with its own key or with key 0, whichever is
larger) are logits of the row: prompts on which a sum over other products of the same rows is far from it.
Queries have 4 added in the first four of every eight dimensions and key 0 has +4 in the first two of them,
-4 in the next two: the products cancel, while four times those of the first two dimensions are 2048, 261
binary orders above any exponential of the row, which would all vanish against it.  Compared with the same
sums in 64 bits: 32-bit sums of at most a few thousand terms, exponentials of logits that 32 bits hold to 1e-6."""
import pytest

from test_gpu_causal_tiles import attention, full_span, gen

pytestmark = pytest.mark.gpu

RTOL = 1e-5


def prompt(L, n_q, hq, hkv):
    import torch
    q, k = gen(71, 1, hq, n_q, 128).float(), gen(72, 1, hkv, L, 128).float()
    d = torch.arange(128, device="cuda") % 8
    q += 4.0 * (d < 4)
    k[:, :, 0] += 4.0 * (d < 2) - 4.0 * ((d >= 2) & (d < 4))
    return q.bfloat16(), k.bfloat16()


def test_full_span():
    import torch
    q, k = prompt(300, 300, 8, 2)
    got, status = full_span(q, k)
    assert status == 0
    torch.testing.assert_close(got, attention(q, k).sum(3).mean(2), rtol=RTOL, atol=0)


def test_entropy():
    import paper_2606_15157_amd as rkv
    import torch
    q, k = prompt(300, 129, 8, 2)
    out = rkv.entropy_profile([q], [k])
    p = attention(q, k)
    assert int(out["status"].item()) == 0
    torch.testing.assert_close(out["rows"].double(), -torch.xlogy(p, p).sum(-1).view(1, 1, 8, 129), rtol=RTOL, atol=RTOL)


@pytest.mark.parametrize("L,w", [(700, 32), (8300, 32), (700, 64)], ids=["four_tiles_short", "four_tiles", "eight_tiles"])
def test_window(L, w, monkeypatch):
    """The window kernels with 16x16x32 MFMA (prompts of up to 64 slices) and 32x32x16, four and eight row tiles."""
    import paper_2606_15157_amd as rkv
    import torch
    monkeypatch.setenv("RKV_FORCE_WINDOW", "1")
    q, k = prompt(L, w, 8, 2)
    out = rkv.evict_prefill(rkv.Plan([rkv.H2O], [L], window=w), [q], [k], [k], score_out=True)
    torch.cuda.synchronize()
    assert rkv.prefill_check(out["workspace"]) == 0
    torch.testing.assert_close(out["scores"][0].double(), attention(q, k).sum(3).mean(2), rtol=RTOL, atol=0)
