"""A decode step of H2O and TOVA layers at the sizes where its workgroup changes: 256 or 512 threads by
the number of workgroups and the LDS of the capacity, blocks of 64 or 128 entries, entries past the
prefetched 1024.  Against the same step in 64 bits (32-bit softmax rows of at most 2050 entries: 1e-5)."""
import math

import pytest

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, Hq, Hkv, C
    (1, 4, 1, 2), (1, 8, 2, 63), (1, 8, 2, 127), (1, 8, 2, 128), (1, 8, 1, 129), (2, 2, 2, 255), (1, 4, 2, 513),
    (1, 8, 2, 1023), (1, 8, 2, 1024), (1, 16, 2, 1025), (1, 8, 2, 2049),
    (65, 8, 2, 129), (65, 8, 2, 1025),        # more than 256 workgroups: 256 threads
    # eight heads a group: four workgroups a CU by LDS, 256 threads; three and 1200, 512; two and 520, 512; nine, 256
    (200, 16, 2, 1100), (300, 16, 2, 1400), (130, 16, 2, 2049), (200, 16, 2, 500),
    (260, 8, 2, 1800), (200, 8, 2, 1800),     # four heads: four and 1040, 512 threads; 800, 256
]


def threads(B, hq, hkv, C):
    """(threads, workgroups a CU by LDS, whether there are more than 256 workgroups) of the two-layer step below:
    the rule of the launch, kept alike with csrc/decode.hip."""
    grid, by_lds = 2 * B * hkv, 160 * 1024 // (4 * (hq // hkv + 1) * (C + 1))
    wide = C >= 128 if grid <= 256 else by_lds <= (3 if hq // hkv == 8 else 4) and grid > 256 * by_lds
    return 512 if wide else 256, min(by_lds, 6), grid > 256


def test_shapes_take_every_branch():
    got = {threads(*s) for s in SHAPES}
    assert {(t, many) for t, _, many in got} == {(256, False), (512, False), (256, True), (512, True)}
    assert {(512, 2, True), (512, 3, True), (512, 4, True), (256, 4, True), (256, 6, True)} <= got


@pytest.mark.parametrize("B,hq,hkv,C", SHAPES, ids=[f"b{s[0]}_{s[1]}x{s[2]}_c{s[3]}" for s in SHAPES])
def test_decode_step_sizes(B, hq, hkv, C):
    import paper_2606_15157_amd as rkv
    import torch
    rules, g, d, p = [rkv.H2O, rkv.TOVA], hq // hkv, 128, 5 * C + 7
    rng = torch.Generator(device="cuda").manual_seed(61)

    def gen(*shape):
        return torch.randn(shape, generator=rng, device="cuda", dtype=torch.bfloat16)

    state = {"k_cache": [gen(B, hkv, C, d) for _ in rules], "v_cache": [gen(B, hkv, C, d) for _ in rules], "pos": [], "acc": []}
    for r in rules:
        at = torch.rand((B, hkv, 5 * C), generator=rng, device="cuda").topk(C, dim=-1).indices
        state["pos"].append(at.sort(dim=-1).values.to(torch.int32))
        state["acc"].append(torch.rand((B, hkv, C), generator=rng, device="cuda") * 0.1 if r == rkv.H2O else None)
    q, k, v = ([gen(B, h, d) for _ in rules] for h in (hq, hkv, hkv))
    before = {key: [t.clone() if t is not None else None for t in ts] for key, ts in state.items()}
    victim = [torch.empty((B, hkv), dtype=torch.int32, device="cuda") for _ in rules]
    rkv.decode_step(rkv.Plan([rkv.FULL] * 2, [0] * 2, rules, [C] * 2), state, q, k, v, p, victim_out=victim)
    torch.cuda.synchronize()
    for l, r in enumerate(rules):
        keys = torch.cat([before["k_cache"][l], k[l].unsqueeze(2)], dim=2).double()
        z = torch.matmul(q[l].double().view(B, hkv, g, d), keys.transpose(2, 3).contiguous()) / math.sqrt(d)
        score = torch.softmax(z, dim=-1).mean(dim=2)
        if r == rkv.H2O:
            score[:, :, :C] += before["acc"][l]
        pos = torch.cat([before["pos"][l], torch.full((B, hkv, 1), p, dtype=torch.int32, device="cuda")], dim=2)
        held = score.masked_fill(pos > (p - C // 2 if r == rkv.H2O else p), math.inf)
        got = torch.where(victim[l] < 0, C, victim[l]).long().unsqueeze(-1)
        least = held.min(-1, keepdim=True).values
        if not torch.isinf(least).any():
            assert (held.gather(-1, got) <= least * (1 + 1e-5)).all(), "the victim is not a minimum"
        slots = torch.arange(C, device="cuda") == got          # no slot where the new token is dropped
        assert torch.equal(state["pos"][l], torch.where(slots, p, before["pos"][l]))
        for key, new in (("k_cache", k), ("v_cache", v)):
            assert torch.equal(state[key][l], torch.where(slots.unsqueeze(-1), new[l].unsqueeze(2), before[key][l]))
        if r == rkv.H2O:
            want = torch.where(slots, score[:, :, C:], score[:, :, :C])
            torch.testing.assert_close(state["acc"][l].double(), want, rtol=1e-5, atol=0)
