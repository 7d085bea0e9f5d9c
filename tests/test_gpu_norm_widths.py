"""The norm and the start of a pass at the widths where their kernel changes (1024, 4096, 16384
columns), with and without a remainder, over a whole pass of one layer: alone, and adding up the
slices of a projection that is cut along K."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 960, 1024, 1088, 4096, 4160, 16384, 16448])
@pytest.mark.parametrize("n", [1, 2, 37])   # (the last entry has no score: one entry alone checks no norm)
def test_rows(D, n):
    """RMSNorm of a two-entry step against fp64: rows of bf16 activations through a layer whose
    projections are zero, so the last norm sees exactly the widened rows; the LM head is a slice of
    the identity, so a score is logsumexp(y) - y[id] of the normed row's first 64 columns."""
    from paper_2607_27600_amd import cc
    g = torch.Generator(device="cuda").manual_seed(D + n)
    V, F, hq, d = 64, 64, 1, 128
    rows = torch.randn((n, D), generator=g, device="cuda", dtype=torch.bfloat16)
    zeros = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    gain = torch.rand(D, generator=g, device="cuda").to(torch.bfloat16)
    w = dict(attn_norm=gain, mlp_norm=gain, wq=zeros(hq * d, D), wo=zeros(D, hq * d), w_gate=zeros(F, D),
             w_up=zeros(F, D), w_down=zeros(D, F))
    w_lm = zeros(V, D)
    w_lm[torch.arange(V), torch.arange(V)] = 1
    ids = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    k = torch.randn((1, 1, 1, n, d), generator=g, device="cuda", dtype=torch.bfloat16)
    kv = cc.kv_contiguous(k, k, n_layers=1, seq_stride=n * d, layer_stride=n * d, head_stride=n * d, tok_stride=d)
    p = cc.problem(dtype="bf16", cu_seqlens=[0, n], n_heads_q=hq, n_heads_kv=1, head_dim=d, hidden=D, vocab=V,
                   mode="last_layer_h", ffn=F, rope_theta=1e4, rms_eps=1e-5)
    scores = torch.empty(n, dtype=torch.float32, device="cuda")
    cc.cc_score(p, cc.inputs(kv=kv, token_ids=ids, w_lm=w_lm, layers=[w], final_norm=gain, h_last=rows), scores)
    x = rows.double().cpu().numpy()
    y = x / np.sqrt((x * x).mean(1, keepdims=True) + 1e-5) * gain.double().cpu().numpy()
    z = y[:, :V]
    lse = np.log(np.exp(z - z.max(1, keepdims=True)).sum(1)) + z.max(1)
    ref = np.maximum(lse - z[np.arange(n), ids.cpu().numpy()], 0.0)
    got = scores.double().cpu().numpy()
    assert np.isinf(got[-1])
    # a logit is a bf16-rounded y (half an ulp: 2^-9 of it), twice in a score
    bound = 2.0 ** -8 * np.abs(z).max(1) + 1e-5
    assert (np.abs(got[:-1] - ref[:-1]) <= bound[:-1]).all()


def _align(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("D,F", [(1088, 4096), (4160, 8192), (16448, 16384)])
def test_rows_after_a_sliced_projection(D, F):
    """W_down long enough to be cut along K: the norm adds its slices to the residual stream.  One call
    for every 64 columns, whose LM head is that slice of the identity, against fp64 (activations
    rounded to bf16 as the path rounds them)."""
    from paper_2607_27600_amd import cc
    n, V, hq, d = 3, 64, 1, 128
    print(f"[norm] D={D} F={F}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(D)
    normal = lambda *s, std=1.0: (torch.randn(s, generator=g, device="cuda") * std).to(torch.bfloat16)
    zeros = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    rows, gain = normal(n, D), torch.rand(D, generator=g, device="cuda").to(torch.bfloat16) + 0.5
    w = dict(attn_norm=gain, mlp_norm=gain, wq=zeros(hq * d, D), wo=zeros(D, hq * d), w_gate=normal(F, D, std=D ** -0.5),
             w_up=normal(F, D, std=D ** -0.5), w_down=normal(D, F, std=2 * F ** -0.5))
    k = zeros(1, 1, 1, n, d)
    kv = cc.kv_contiguous(k, k, n_layers=1, seq_stride=n * d, layer_stride=n * d, head_stride=n * d, tok_stride=d)
    p = cc.problem(dtype="bf16", cu_seqlens=[0, n], n_heads_q=hq, n_heads_kv=1, head_dim=d, hidden=D, vocab=V,
                   mode="last_layer_h", ffn=F, rope_theta=1e4, rms_eps=1e-5)
    # what the workspace holds beside the slices
    rest = (_align(16) + _align(n * d // 2 * 8) + _align(n * D * 4) + _align(n * D * 2) + 2 * _align(n * hq * d * 2) +
            _align(n * F * 2) + cc.cc_lmhead_workspace(p))
    assert cc.cc_score_workspace(p) - rest >= 2 * n * D * 4, "W_down is not cut: the case misses its point"

    def norm(h):
        return h / torch.sqrt((h * h).mean(1, keepdim=True) + 1e-5) * gain.double()

    def product(x, m):   # fp64, a block of weight rows at a time
        return torch.cat([x @ m[i:i + 2048].double().t().contiguous() for i in range(0, m.shape[0], 2048)], 1)

    h = rows.double()
    b = norm(h).to(torch.bfloat16).double()
    act = torch.nn.functional.silu(product(b, w["w_gate"])) * product(b, w["w_up"])
    mlp = product(act.to(torch.bfloat16).double(), w["w_down"])
    assert mlp.std() > 0.2
    y = norm(h + mlp)
    # a logit is a bf16-rounded y; the activations behind it may round to the next bf16 where fp32 and
    # fp64 sums straddle a tie (2^-8 of one, summed at random: 2^-8 of the product's scale and less)
    bound = 2.0 ** -8 * y.abs() + 2.0 ** -7 * y.square().mean(1, keepdim=True).sqrt()
    ids = torch.arange(n, dtype=torch.int32, device="cuda") * 31
    scores = torch.empty(n, dtype=torch.float32, device="cuda")
    for c in range(0, D, V):
        w_lm = zeros(V, D)
        w_lm[torch.arange(V), torch.arange(c, c + V)] = 1
        cc.cc_score(p, cc.inputs(kv=kv, token_ids=ids, w_lm=w_lm, layers=[w], final_norm=gain, h_last=rows), scores)
        z = y[:, c:c + V]
        ref = torch.logsumexp(z, 1) - z[torch.arange(n), ids.long()]
        assert torch.isinf(scores[-1])
        err = (scores.double() - ref.clamp(min=0)).abs()[:-1]
        assert (err <= 2 * bound[:, c:c + V].amax(1)[:-1]).all(), (c, err)
