"""The attention task order covers every (batch, head, query block) row exactly
where the row count or the group count does not divide the order's phases: each
call equals, bit for bit, the calls on its (batch, KV head) groups one by one
(whose phases differ), into outputs filled with NaN beforehand."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
seer = pytest.importorskip("paper_2410_13276_amd")


# 1 and 2 blocks with odd group counts (phases rounded up over groups), block counts around 8, and K + V beyond
# the 32 MiB of a phase (261 and 523 blocks; 205, 261: half of the groups per phase; 611 at 7 heads a group: one
# launch per group); interleaved rows: 1, 9 and 10 blocks, 1021 and 523 with few heads a group
@pytest.mark.parametrize("B,Hq,Hkv,seq", [(1, 1, 1, 1), (9, 2, 1, 100), (3, 6, 3, 64), (5, 3, 3, 449), (1, 4, 2, 577),
                                          (2, 14, 2, 1001), (1, 16, 8, 16700), (1, 8, 8, 33409), (1, 4, 2, 65300),
                                          (1, 12, 12, 577), (3, 2, 2, 640), (2, 16, 4, 13100), (1, 16, 4, 16700),
                                          (1, 14, 2, 39050)])
def test_every_row_once(B, Hq, Hkv, seq):
    print(f"[task order] {B} {Hq}/{Hkv} {seq}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(seq)
    q, k, v = (torch.randn(B, h, seq, 128, generator=gen, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    nb, G = -(-seq // 64), Hq // Hkv
    i = torch.arange(nb, device="cuda")
    keep = torch.rand(B, Hq, nb, nb, generator=gen, device="cuda") < 4.0 / nb
    dense = ((keep | (i[None, :] == i[:, None])) & (i[None, :] <= i[:, None])).to(torch.uint8)
    mask = seer.mask_from_dense(dense, heads_kv=Hkv)
    o = torch.full_like(q, float("nan"))
    lse = torch.full((B, Hq, seq), float("nan"), device="cuda")
    seer.bsattn(q, k, v, mask, out=o, lse=lse)
    od = torch.full_like(q, float("nan"))
    if nb <= 300:
        seer.dense_attn(q, k, v, out=od)
    for b in range(B):
        for g in range(Hkv):
            hs = slice(g * G, g * G + G)
            qs, ks, vs = q[b:b + 1, hs], k[b:b + 1, g:g + 1], v[b:b + 1, g:g + 1]
            m = seer.BlockMask(count=mask.count[b:b + 1, hs].contiguous(), idx=mask.idx[b:b + 1, hs].contiguous())
            o1, l1 = seer.bsattn(qs, ks, vs, m, out=torch.empty_like(qs).contiguous(), want_lse=True)
            assert torch.equal(o[b:b + 1, hs].view(torch.int16), o1.view(torch.int16))
            assert torch.equal(lse[b:b + 1, hs], l1)
            if nb <= 300:
                od1, _ = seer.dense_attn(qs, ks, vs, out=torch.empty_like(qs).contiguous())
                assert torch.equal(od[b:b + 1, hs].view(torch.int16), od1.view(torch.int16))


# one group at a time (261 and 523 blocks, no multiple of the XCDs per group) and all groups at once (130 blocks)
@pytest.mark.parametrize("Hq,Hkv,seq", [(16, 8, 16700), (4, 2, 33409), (8, 8, 8320)])
def test_every_row_of_a_shared_mask_once(Hq, Hkv, seq):
    print(f"[task order] shared mask {Hq}/{Hkv} {seq}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(seq)
    q, k, v = (torch.randn(1, h, seq, 128, generator=gen, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    nb, G = -(-seq // 64), Hq // Hkv
    i = torch.arange(nb, device="cuda")
    keep = torch.rand(1, Hkv, nb, nb, generator=gen, device="cuda") < 4.0 / nb
    dense = ((keep | (i[None, :] == i[:, None])) & (i[None, :] <= i[:, None])).to(torch.uint8)
    mask = seer.mask_from_dense(dense, kv_shared=True)
    o = torch.full_like(q, float("nan"))
    seer.bsattn(q, k, v, mask, out=o)
    for g in range(Hkv):
        hs = slice(g * G, g * G + G)
        m = seer.BlockMask(count=mask.count[:, g:g + 1].contiguous(), idx=mask.idx[:, g:g + 1].contiguous(), kv_shared=True)
        qs = q[:, hs].contiguous()
        o1, _ = seer.bsattn(qs, k[:, g:g + 1], v[:, g:g + 1], m)
        assert torch.equal(o[:, hs].view(torch.int16), o1.view(torch.int16))


@pytest.mark.parametrize("Hq,Hkv,seq,launches", [(8, 8, 39050, 1), (8, 8, 40960, 1), (12, 4, 50001, 1), (14, 2, 39050, 2),
                                                 (28, 4, 65536, 4)])
def test_groups_of_few_rows_share_a_launch(Hq, Hkv, seq, launches):
    """One launch per KV group only from 4096 rows a group on."""
    q, k = (torch.empty(1, h, seq, 128, dtype=torch.bfloat16, device="cuda") for h in (Hq, Hkv))
    mask = seer.alloc_mask(1, Hq, seq)
    assert seer.attn_launches(q, k, k, mask) == launches
