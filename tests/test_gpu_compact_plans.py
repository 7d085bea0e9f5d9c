"""Compaction against a plain gather where its plan changes: lists by value and uploaded (more
than 64), column slabs of a long list in few planes, odd budgets (none, one, all), per-head
lists, and the ids moved with the first list of each sequence."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _case(lens, hkv, L, d, paged, per_head, seed, budgets):
    from paper_2607_27600_amd import cc
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = np.random.default_rng(seed)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    n, P, cap = int(cu[-1]), 16, max(lens)
    if paged:
        pages = [(x + P - 1) // P for x in lens]
        perm = r.permutation(sum(pages))
        bt = np.zeros((len(lens), max(pages)), np.int32)
        at = 0
        for b, m in enumerate(pages):
            bt[b, :m] = perm[at:at + m]
            at += m
        shape = (L, sum(pages), hkv, P, d)
        table = torch.from_numpy(bt).cuda()
    else:
        shape = (len(lens), L, hkv, cap, d)
    k, v = (torch.randint(-30000, 30000, shape, generator=g, device="cuda", dtype=torch.int16).view(torch.bfloat16)
            for _ in range(2))
    if paged:
        view = lambda a, b: cc.kv_paged(a, b, table, n_layers=L, layer_stride=shape[1] * hkv * P * d,
                                        page_stride=hkv * P * d, head_stride=P * d, tok_stride=d, page_size=P)
    else:
        view = lambda a, b: cc.kv_contiguous(a, b, n_layers=L, seq_stride=L * hkv * cap * d,
                                             layer_stride=hkv * cap * d, head_stride=cap * d, tok_stride=d)
    ids, pos = (torch.randint(0, 1 << 30, (n,), generator=g, device="cuda", dtype=torch.int32) for _ in range(2))
    per = hkv if per_head else 1
    ks, lists = [], []
    for b, x in enumerate(lens):
        for h in range(per):
            kk = budgets(b, h, x)
            ks.append(kk)
            lists.append(np.sort(r.choice(x, kk, replace=False)).astype(np.int32))
    keep = torch.from_numpy(np.concatenate(lists) if sum(ks) else np.zeros(1, np.int32)).cuda()
    ek, ev, ei, ep = k.clone(), v.clone(), ids.clone(), pos.clone()
    for b in range(len(lens)):
        first = torch.from_numpy(lists[b * per].astype(np.int64)).cuda()
        for src, dst in ((ids, ei), (pos, ep)):
            dst[cu[b]:cu[b] + len(first)] = src[cu[b] + first]
        for h in range(hkv):
            idx = torch.from_numpy(lists[b * per + (h if per_head else 0)].astype(np.int64)).cuda()
            to = torch.arange(len(idx), device="cuda")
            for src, dst in ((k, ek), (v, ev)):
                if paged:
                    t = table[b].long()
                    dst[:, t[to // P], h, to % P] = src[:, t[idx // P], h, idx % P]
                else:
                    dst[b, :, h, :len(idx)] = src[b, :, h, idx]
    p = cc.problem(dtype="bf16", cu_seqlens=cu.tolist(), n_heads_q=hkv, n_heads_kv=hkv, head_dim=d, hidden=64,
                   vocab=8)
    return cc, p, view, (k, v, ids, pos), (ek, ev, ei, ep), keep, ks


@pytest.mark.parametrize("lens,hkv,L,d,paged,per_head,budget", [
    ((5000,), 1, 2, 128, False, False, "most"),        # slabs
    ((4001, 3000), 1, 1, 128, True, False, "most"),    # slabs, paged
    ((2500,), 2, 1, 64, True, True, "odd"),            # slabs of 64-wide heads, per-head lists
    (tuple(range(1, 71)), 2, 1, 64, False, False, "odd"),   # 70 lists: uploaded
    (tuple(range(20, 42)), 3, 2, 128, True, True, "odd"),   # 66 lists: uploaded
    ((300, 1, 77), 2, 3, 128, False, True, "odd"),
])
def test_in_place(lens, hkv, L, d, paged, per_head, budget):
    pick = {"most": lambda b, h, n: n - n // 5, "odd": lambda b, h, n: (0, 1, n, n // 2)[(b + h) % 4]}[budget]
    cc, p, view, (k, v, ids, pos), want, keep, ks = _case(lens, hkv, L, d, paged, per_head, 3, pick)
    cc.cc_compact_kv(p, view(k, v), keep, ks, int(per_head), token_ids=ids, pos_ids=pos)
    torch.cuda.synchronize()
    for got, ref in zip((k, v, ids, pos), want):
        assert torch.equal(got.view(torch.int16 if got.dtype == torch.bfloat16 else torch.int32),
                           ref.view(torch.int16 if ref.dtype == torch.bfloat16 else torch.int32))


@pytest.mark.parametrize("n,width", [(5000, 512), (3000, 8), (700, 3584)])
def test_rows_in_place(n, width):
    from paper_2607_27600_amd import cc
    rows = torch.randint(0, 30000, (n, width), device="cuda", dtype=torch.int16)
    kk = n - n // 3
    keep = torch.sort(torch.randperm(n, device="cuda")[:kk]).values.to(torch.int32)
    want = rows.clone()
    want[:kk] = rows[keep.long()]
    p = cc.problem(dtype="bf16", cu_seqlens=[0, n], n_heads_q=1, n_heads_kv=1, head_dim=64, hidden=64, vocab=8)
    cc.cc_compact_rows(p, rows, keep, [kk], 0)
    torch.cuda.synchronize()
    assert torch.equal(rows, want)


@pytest.mark.parametrize("budget", [1, 63, 64, 65, 448, 449, 512, 513])
@pytest.mark.parametrize("paged,hkv,L,d", [(False, 2, 33, 128), (True, 2, 30, 128), (False, 1, 2, 128), (True, 1, 3, 64)])
def test_short_lists_in_place(budget, paged, hkv, L, d):
    """Lists that pass through the registers at once and the first that do not (512 rows of 256 bytes
    are 8 a thread; few planes are cut into slabs), with a shorter list beside the longest."""
    pick = lambda b, h, n: min(n, budget)
    cc, p, view, (k, v, ids, pos), want, keep, ks = _case((600, 70), hkv, L, d, paged, False, budget, pick)
    cc.cc_compact_kv(p, view(k, v), keep, ks, 0, token_ids=ids, pos_ids=pos)
    torch.cuda.synchronize()
    for got, ref in zip((k, v, ids, pos), want):
        t = torch.int16 if got.dtype == torch.bfloat16 else torch.int32
        assert torch.equal(got.view(t), ref.view(t))
