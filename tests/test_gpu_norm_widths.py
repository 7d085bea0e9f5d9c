"""The norm and the start of a pass at the widths where their kernel changes (1024, 4096, 16384
columns), with and without a remainder, over a whole pass of one layer."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 960, 1024, 1088, 4096, 4160, 16384, 16448])
@pytest.mark.parametrize("n", [1, 37])
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
