"""Contractions over rows of 2^22 columns and more, which the tiles address in 64 bits: rows 16 MB
apart, so that a tile of 256 of them spans more than 4 GB.  Operands are 0 and +-1, with what is not 0
at both ends of the rows and at random columns between: every sum is a small whole number, exact
in fp32."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS, N = 300, 70   # features or vocabulary, entries: edges of every tile


def _sparse(K, dtype, one, minus, seed):
    """x [N][K], w [ROWS][K] and the exact x w^T."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    at = torch.cat([torch.arange(64), torch.arange(K - 64, K), torch.randint(64, K - 64, (512,))]).unique().cuda()
    m = len(at)
    a = torch.randint(-1, 2, (N, m), generator=g, device="cuda")
    b = torch.randint(-1, 2, (ROWS, m), generator=g, device="cuda") * (torch.rand(ROWS, m, generator=g, device="cuda") < 0.1)
    x = torch.zeros((N, K), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((ROWS, K), dtype=dtype, device="cuda")
    x[:, at] = a.to(torch.bfloat16)
    w[:, at] = torch.where(b > 0, one, torch.where(b < 0, minus, 0)).to(dtype)
    return x, w, a.double() @ b.double().t().contiguous()


def test_linear():
    from paper_2607_27600_amd import cc
    for K in (1 << 22, 1 << 23):
        print(f"[wide] linear K={K}", flush=True)
        x, w, ref = _sparse(K, torch.bfloat16, 1, -1, K)
        y = torch.empty((N, ROWS), dtype=torch.bfloat16, device="cuda")
        cc.cc_linear("bf16", x, w, y)
        assert torch.equal(y, ref.to(torch.bfloat16))


@pytest.mark.parametrize("form", ["row", "packed", "fp8"])
def test_lmhead(form):
    from paper_2607_27600_amd import cc
    fp8 = form == "fp8"
    K = 1 << (24 if fp8 else 23)
    print(f"[wide] {form} K={K}", flush=True)
    x, w, z = _sparse(K, torch.uint8, 0x38, 0xb8, 3) if fp8 else _sparse(K, torch.bfloat16, 1, -1, 3)
    ids = torch.randint(0, ROWS, (N,), device="cuda", dtype=torch.int32)
    p = cc.problem(dtype="bf16", cu_seqlens=[0, N], n_heads_q=1, n_heads_kv=1, head_dim=128, hidden=K, vocab=ROWS,
                   lmhead_packed=form == "packed")
    s, lse = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
    if form == "row":
        cc.cc_lmhead_score(p, x, w, ids, s, lse)
    elif form == "packed":
        cc.cc_lmhead_score_packed(p, x, cc.cc_pack_lmhead(w), ids, s, lse)
    else:
        cc.cc_lmhead_score_fp8(p, x, w, torch.ones(1, device="cuda"), ids, s, lse)
    ref = torch.logsumexp(z, 1)
    # exact logits (E4M3: times 1 / 448 and back, two roundings), then exponentials and a logarithm
    bound = 2.0 ** -21 * (ref.abs() + z.abs().amax(1)) + 4e-6
    assert ((lse.double() - ref).abs() <= bound).all()
    want = (ref - z[torch.arange(N, device="cuda"), ids.long()]).clamp(min=0)
    assert ((s.double() - want).abs()[:-1] <= 2 * bound[:-1]).all() and torch.isinf(s[-1])
