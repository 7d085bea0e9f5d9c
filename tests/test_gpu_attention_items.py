"""Attention where its launch changes: work items found from up to 16 sequences by value and from
the uploaded table beyond, and two key groups a workgroup for launches of few items (up to 256, and up to 512 with long chains; one
tile, an odd and an even number of tiles, sequences with no key at all)."""
import numpy as np
import pytest

from synth import configs as C
from tests.test_gpu_attention import _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,hq,hkv,d,paged", [
    ((1, 64, 65, 129, 192, 193, 260), 4, 2, 128, False),
    ((1, 64, 65, 129, 192, 193, 260), 7, 1, 64, True),
    (tuple(range(3, 99, 6)), 2, 2, 128, True),             # 16 sequences, by value
    (tuple(range(99, 3, -6)) + (40,), 2, 2, 128, True),    # 17: the table
    ((700, 100, 701, 0, 1), 32, 8, 128, False),            # more than 256 items
    ((513,), 28, 4, 128, False),
    ((1800, 700, 0, 65, 1), 14, 2, 64, True),              # 284 items of up to 29 tiles: two groups
    ((1530, 1), 28, 4, 128, False),                        # 340 items of up to 24 tiles
])
@pytest.mark.parametrize("diag", ["strict", "inclusive"])
def test_bf16(lens, hq, hkv, d, paged, diag):
    cfg = C.shrink(C.C2, seq_lens=lens, n_heads_q=hq, n_heads_kv=hkv, head_dim=d, paged=paged, cache_layers=1,
                   keep=(0,) * len(lens))
    got, ref, _ = _run(cfg, diag)
    _check(got, ref, "bf16", f"{lens[:4]} {hq}/{hkv} d={d}")


def test_f32_many_sequences():
    for lens in (tuple(range(1, 33, 2)), tuple(range(1, 35, 2))):
        cfg = C.shrink(C.C1, seq_lens=lens, keep=(0,) * len(lens))
        got, ref, _ = _run(cfg)
        _check(got, ref, "f32")


@pytest.mark.parametrize("lens,hq,hkv,d", [((1711, 333, 1024, 97, 2047), 16, 4, 64), ((3000,), 8, 1, 128),
                                           ((700,) * 20, 28, 4, 128)])
def test_repeats_bit_for_bit(lens, hq, hkv, d):
    """A tile's buffer is refilled only when every wave has read it: launches of many items with the
    same inputs agree in every bit.  (Refilled after the first tile behind no barrier, a late wave
    could read keys of the third: one launch in hundreds.)"""
    import torch
    from paper_2607_27600_amd import cc
    n, P = sum(lens), 16
    g = torch.Generator(device="cuda").manual_seed(n)
    pages = [(x + P - 1) // P for x in lens]
    perm = torch.randperm(sum(pages), generator=g, device="cuda").int()
    table = torch.zeros((len(lens), max(pages)), dtype=torch.int32, device="cuda")
    cu = [0]
    for b, m in enumerate(pages):
        table[b, :m] = perm[sum(pages[:b]):sum(pages[:b]) + m]
        cu.append(cu[-1] + lens[b])
    k, v = (torch.randn((1, sum(pages), hkv, P, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    q = torch.randn((n, hq, d), generator=g, device="cuda", dtype=torch.bfloat16)
    kv = cc.kv_paged(k, v, table, n_layers=1, layer_stride=k.numel(), page_stride=hkv * P * d, head_stride=P * d,
                     tok_stride=d, page_size=P)
    p = cc.problem(dtype="bf16", cu_seqlens=cu, n_heads_q=hq, n_heads_kv=hkv, head_dim=d, hidden=1024, vocab=1024)
    first = cc.cc_attention_cc(p, q, kv, 0, torch.empty_like(q))
    again = [cc.cc_attention_cc(p, q, kv, 0, torch.empty_like(q)) for _ in range(100)]
    assert all(torch.equal(o, first) for o in again)
