"""The fp32 attention kernel's tile groups and key halves against the fp64 oracle:
row counts on both sides of each rule (256 and 768 rows), rows of fewer tiles than
groups, partial last tiles, empty rows,
lists that end early, with and without causality; the ground truth's map and the
dense outputs equal whatever the KV groups per launch.  Bar: 1e-4 max-abs (the
fp32 bar of the other tests; measured 5e-7)."""
import numpy as np
import pytest

import oracle
from helpers import ATOL_F32, lists_from_dense, small_inputs, stable_seed, to_device, upload_mask

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
seer = pytest.importorskip("paper_2410_13276_amd")


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,Hq,Hkv,S,D", [(1, 2, 1, 1, 64), (1, 2, 1, 130, 64), (1, 2, 1, 1000, 64), (1, 16, 4, 1024, 64),
                                          (1, 16, 4, 1025, 64), (1, 6, 2, 300, 64), (2, 24, 8, 1024, 64), (1, 49, 7, 1000, 64),
                                          (1, 2, 1, 65, 128), (1, 16, 4, 1024, 128), (1, 16, 4, 1030, 128),
                                          (1, 26, 2, 1900, 128)])
def test_f32_sparse_and_dense(B, Hq, Hkv, S, D, causal):
    print(f"[f32] {B} {Hq}/{Hkv} {S} {D} {causal}", flush=True)
    seed = stable_seed("f32", B, Hq, S, D, causal)
    _, q, k, v, _, _ = small_inputs(B, Hq, Hkv, S, D, "f32", seed=seed)
    nb = -(-S // 64)
    rng = np.random.default_rng(seed)
    m = (rng.random((B, Hq, nb, nb)) < 0.35).astype(np.uint8)
    m[:, 0, nb // 2] = 0  # an empty row
    if causal:
        m *= np.tril(np.ones((nb, nb), np.uint8))
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    cnt, idx = lists_from_dense(m)
    if causal and nb > 1:  # an entry past the diagonal ends the row, whatever follows
        cnt[0, 1, 0], idx[0, 1, 0, 0] = 2, 0
        idx[0, 1, 0, 1] = nb - 1
        m[0, 1, 0] = 0
        m[0, 1, 0, 0] = 1
    o, lse = seer.bsattn(qd, kd, vd, upload_mask(cnt, idx), causal=causal, want_lse=True, out=torch.full_like(qd, 9.0))
    O, L = oracle.attn(q, k, v, mask=m, causal=causal)
    ref, lref = O.reshape(B, Hq, nb * 64, D)[:, :, :S], L.reshape(B, Hq, nb * 64)[:, :, :S]
    assert float(np.abs(o.cpu().numpy() - np.nan_to_num(ref)).max()) <= ATOL_F32
    got = lse.cpu().numpy()
    fin = np.isfinite(lref)
    assert np.array_equal(fin, np.isfinite(got)) and bool((np.abs(got[fin] - lref[fin]) <= 1e-4).all())
    od, _ = seer.dense_attn(qd, kd, vd, causal=causal)
    O, _ = oracle.attn(q, k, v, causal=causal)
    assert float(np.abs(od.cpu().numpy() - O.reshape(B, Hq, nb * 64, D)[:, :, :S]).max()) <= ATOL_F32
    og, _, gt = seer.attn_gt(qd, kd, vd, causal=causal)
    ws = torch.empty(seer.attn_gt_workspace_bytes(qd, kd, vd, 1), dtype=torch.uint8, device="cuda")
    o1, _, gt1 = seer.attn_gt(qd, kd, vd, causal=causal, workspace=ws)  # one KV group per launch
    assert torch.equal(og, od) and torch.equal(o1, od) and torch.equal(gt1, gt)


def test_more_rows_than_one_launch_holds():
    """2^24 + 64 rows of one token (a launch holds fewer than 2^32 threads, 256 a row): O = V exactly."""
    B, Hq, D = (1 << 18) + 1, 64, 64
    print(f"[f32] {B} x {Hq} rows of one token", flush=True)
    q = torch.ones(1, 1, 1, D, device="cuda").expand(B, Hq, 1, D)
    k = torch.ones(B, 1, 1, D, device="cuda")
    v = torch.arange(B, dtype=torch.float32, device="cuda").view(B, 1, 1, 1).expand(B, 1, 1, D).contiguous()
    o = torch.full((B, Hq, 1, D), -1.0, device="cuda")
    seer.dense_attn(q, k, v, out=o)
    assert bool((o == v).all())
    mask = seer.BlockMask(count=torch.ones(B, Hq, 1, dtype=torch.int32, device="cuda"),
                          idx=torch.zeros(B, Hq, 1, 1, dtype=torch.uint16, device="cuda"))
    o.fill_(-1.0)
    seer.bsattn(q, k, v, mask, out=o)
    assert bool((o == v).all())


# 6 and 126 rows (a workgroup per query half), 378 (two tile groups), 1032 (one)
@pytest.mark.parametrize("B,S", [(3, 130), (9, 448), (27, 448), (86, 381)])
def test_scores_beyond_the_finite(B, S):
    """+inf and NaN scores make the rows that see them NaN; -inf scores and the type's lowest are weights like
    any other beside an ordinary one (a row of nothing but -inf is empty: O = 0, LSE = -inf), wherever in the tiles, key halves and tile
    groups they stand.  Against softmax in 64 bits."""
    print(f"[f32] non-finite scores {B} {S}", flush=True)
    D, low = 64, -3.0e38
    gen = torch.Generator().manual_seed(S)
    s = torch.randn(B, S, generator=gen) * 3
    inf = float("inf")
    kind = torch.arange(B) % 3
    s[kind == 0, S // 2] = inf          # rows from S // 2 on are NaN
    s[kind == 0, :40] = -inf            # rows before 40 are empty, a whole key half
    s[kind == 1, S // 3] = float("nan")
    s[kind == 1, 1:S // 4] = low        # (key 0 stays: a row's largest score has to be one that its own rounding times
    s[kind == 2, :] = -inf              # the scale, 2^-24 of it, does not swamp)
    s[kind == 2, S - 3] = 1.0           # the only key of the last rows
    q = torch.zeros(B, 1, S, D)
    q[..., 0] = 1.0
    k = torch.zeros(B, 1, S, D)
    k[:, 0, :, 0] = s
    v = torch.randn(B, 1, S, D, generator=gen)
    w = (s.double() / 8).view(B, 1, S).expand(B, S, S)
    w = w.masked_fill(~torch.ones(S, S, dtype=torch.bool).tril(), -inf)
    empty = (w == -inf).all(-1)
    p = torch.softmax(w, -1)
    ref = torch.where(empty.unsqueeze(-1), 0.0, p @ v[:, 0].double())
    # (a zero weight times a finite value: NaN comes from the scores alone)
    bad = torch.isnan(p).any(-1) & ~empty
    o, lse = seer.dense_attn(q.cuda(), k.cuda(), v.cuda(), want_lse=True)
    nb = -(-S // 64)
    full = torch.ones(B, 1, nb, nb, dtype=torch.uint8, device="cuda").tril()
    o2, _ = seer.bsattn(q.cuda(), k.cuda(), v.cuda(), seer.mask_from_dense(full))
    for out in (o[:, 0].cpu(), o2[:, 0].cpu()):
        assert torch.equal(torch.isnan(out).any(-1), bad) and bool(torch.isnan(out[bad]).all())
        assert float((out[~bad].double() - ref[~bad]).abs().max()) <= ATOL_F32
    got, want = lse[:, 0].cpu(), torch.logsumexp(w, -1)
    assert bool((got[empty] == -inf).all())
    fin = ~bad & ~empty
    assert bool(((got[fin] - want[fin]).abs() <= 1e-4 * want[fin].abs().clamp(min=1)).all())
