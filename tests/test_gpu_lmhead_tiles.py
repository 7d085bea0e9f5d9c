"""The LM head over batches of different sizes: an entry's neighbours may change nothing."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _operands(N, D, vocab, seed, std=0.05):
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.randn((N, D), generator=g, device="cuda").to(torch.bfloat16)
    w = (std * torch.randn((vocab, D), generator=g, device="cuda")).to(torch.bfloat16)
    ids = torch.randint(0, vocab, (N,), generator=g, device="cuda", dtype=torch.int32)
    return u, w, ids


def _run(form, u, w, ids, cu=None):
    """Scores and log-sum-exps of the rows of u; codes and scales where the form has them."""
    from paper_2607_27600_amd import cc
    N, D = u.shape
    f32 = form == "f32"
    p = cc.problem(dtype="f32" if f32 else "bf16", cu_seqlens=cu or [0, N], n_heads_q=1, n_heads_kv=1, head_dim=128,
                   hidden=D, vocab=w.shape[0], lmhead_packed=form == "packed")
    s = torch.full((N,), float("nan"), device="cuda")
    lse = torch.full((N,), float("nan"), device="cuda")
    if form == "row":
        cc.cc_lmhead_score(p, u, w, ids, s, lse)
    elif form == "f32":
        cc.cc_lmhead_score(p, u.float(), w.float(), ids, s, lse)
    elif form == "packed":
        cc.cc_lmhead_score_packed(p, u, cc.cc_pack_lmhead(w), ids, s, lse)
    else:
        codes, scale = cc.cc_quantize_fp8("bf16", w, per_row=False)
        cc.cc_lmhead_score_fp8(p, u, codes, scale, ids, s, lse)
        return s, lse, codes, scale
    return s, lse


@pytest.mark.parametrize("form", ["row", "packed", "fp8", "f32"])
def test_an_entry_is_scored_the_same_in_any_batch(form):
    """Bit for bit: the tile width, the order of tiles and the combine's entries a workgroup follow
    the number of entries, the sums of an entry do not.  (157 vocabulary tiles of 256 rows, 625 of 64:
    several a group of the combine.)"""
    D, vocab = 256, 40000
    u, w, ids = _operands(3000, D, vocab, 5)
    _, full, *_ = _run(form, u, w, ids, cu=[0, 7, 1000, 3000])
    for n in (1, 5, 100, 200, 513, 2048, 2049):
        print(f"[lmhead tiles] {form} first {n} of 3000", flush=True)
        _, lse, *_ = _run(form, u[:n].contiguous(), w, ids[:n].contiguous())
        assert torch.equal(lse, full[:n]), (n, float((lse - full[:n]).abs().max()))
