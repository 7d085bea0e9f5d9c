"""The LM head at every tile width of its dispatch (64, 128, 192 and 256 entries), on row-major,
packed and E4M3 weights, with dense random operands: fewer k-tiles than a ring holds, as many, and
enough for every ring to wrap twice; a vocabulary edge; both orders of tiles.  (The width follows the
rounds of workgroups: a small vocabulary takes the narrowest, 157 vocabulary tiles take each in turn
from 1, 77, 129 and 220 entries on, 641 and 1500 three and six columns of the widest.)  And what an
entry's neighbours may change: nothing."""
import numpy as np
import pytest
import torch

from oracle import cc_oracle as O

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


def _e4m3(codes):
    return torch.as_tensor(codes).view(torch.float8_e4m3fn).double()


@pytest.mark.parametrize("k_tiles", [1, 3, 4, 11])
@pytest.mark.parametrize("V,N", [(700, n) for n in (1, 37, 64, 77, 300, 641)] +
                         [(40100, n) for n in (1, 37, 64, 77, 129, 220, 300, 641, 1500)])
@pytest.mark.parametrize("form", ["row", "packed", "fp8"])
def test_against_fp64(form, V, N, k_tiles):
    D = (128 if form == "fp8" else 64) * k_tiles
    print(f"[lmhead tiles] {form} {V} x {D} N={N}", flush=True)
    u, w, ids = _operands(N, D, V, N + D)
    s, lse, *q = _run(form, u, w, ids)
    if q:
        if V == 700:
            assert np.array_equal(q[0].cpu().numpy(), O.quantize_fp8(w.float().cpu().numpy(), per_row=False)[0])
        uc, us = O.quantize_fp8(u.float().cpu().numpy(), per_row=True)
        a = (_e4m3(uc) * torch.as_tensor(us).double()[:, None]).cuda()
        b = _e4m3(q[0].cpu()).cuda() * q[1].double()
    else:
        a, b = u.double(), w.double()
    z = a @ b.t().contiguous()
    ref = torch.logsumexp(z, 1).cpu()
    target = z[torch.arange(N, device="cuda"), ids.long()].cpu()
    # D fp32 additions of products that are exact (two roundings more for the scales of E4M3); then
    # exponentials, sums and the logarithm of the result, some ulps of it
    bound = (D + 2) * 2.0 ** -24 * (a.abs() @ b.abs().t().contiguous()).amax(1).cpu() + 2.0 ** -22 * ref.abs() + 4e-6
    err = (lse.cpu().double() - ref).abs()
    assert (err <= bound).all(), float((err / bound).max())
    got, want = s.cpu().double(), (ref - target).clamp(min=0)
    assert got[-1] == np.inf
    err = (got - want).abs()[:-1]
    assert (err <= 2 * bound[:-1]).all(), float((err / bound[:-1]).max())


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
