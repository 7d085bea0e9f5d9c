"""GPU parity of the fp32 kernels at the edges of their tiles: attention (32-row blocks, 16-key
tiles dealt to four or eight waves), the projection and the LM head (64 x 64 to 32 x 32 tiles, 32
columns of K a step, element-wise loads where K or a pointer rules 16-byte ones out)."""
import numpy as np
import pytest
import torch

from oracle import cc_oracle as O
from synth import configs as C
from tests.gpu_util import F32_ATOL, assert_scores_close, dev, f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,hq,hkv,d,paged,diag", [
    ((1, 2, 15, 16, 17, 33), 4, 4, 64, False, "strict"),
    ((1, 31, 65, 130), 7, 1, 128, True, "strict"),
    ((97, 64), 8, 2, 64, True, "inclusive"),
    ((300,), 2, 1, 128, False, "inclusive"),
    ((127,), 4, 2, 64, False, "strict"),        # the longest item has 8 tiles: four waves
    ((128, 0, 1), 4, 2, 64, True, "strict"),    # from here eight, up to 256 items
    ((530, 129, 3), 7, 1, 64, False, "inclusive"),
    ((600, 580), 7, 1, 64, True, "strict"),     # 259 items: four
])
def test_attention(lens, hq, hkv, d, paged, diag):
    from tests.test_gpu_attention import _run
    cfg = C.shrink(C.C1, seq_lens=lens, n_heads_q=hq, n_heads_kv=hkv, head_dim=d, paged=paged,
                   keep=(1,) * len(lens))
    got, ref, _ = _run(cfg, diag)
    np.testing.assert_allclose(got, ref, rtol=0, atol=F32_ATOL)


def test_attention_infinite_value_reaches_only_rows_that_see_it():
    from paper_2607_27600_amd import cc
    n, j = 40, 21
    r = np.random.default_rng(5)
    q = r.standard_normal((n, 2, 64)).astype(np.float32)
    k, v = (r.standard_normal((1, n, 64)).astype(np.float32) for _ in range(2))
    v[0, j, 3] = np.inf
    kd, vd = dev(k), dev(v)
    kv = cc.kv_contiguous(kd, vd, n_layers=1, layer_stride=n * 64, head_stride=n * 64, tok_stride=64)
    p = cc.problem(dtype="f32", cu_seqlens=[0, n], n_heads_q=2, n_heads_kv=1, head_dim=64,
                   hidden=64, vocab=8)
    o = torch.empty((n, 2, 64), device="cuda")
    cc.cc_attention_cc(p, dev(q), kv, 0, o)
    torch.cuda.synchronize()
    v0 = v.copy()
    v0[0, j, 3] = 0.0
    ref = O.attention_cc(q, k, v0, "strict")
    got = f64(o)
    assert np.all(got[:j, :, 3] == np.inf)
    got[:j, :, 3] = ref[:j, :, 3]
    np.testing.assert_allclose(got, ref, rtol=0, atol=F32_ATOL)


@pytest.mark.parametrize("M,N,K,off", [(1, 1, 1, 0), (31, 33, 31, 0), (32, 32, 32, 0), (65, 63, 36, 0),
                                       (65, 63, 36, 1), (1030, 1025, 100, 0)])
def test_linear(M, N, K, off):
    from paper_2607_27600_amd import cc
    r = np.random.default_rng(6)
    x, w = (r.standard_normal((rows, K)).astype(np.float32) for rows in (M, N))
    xd = torch.empty(M * K + off, device="cuda")[off:].view(M, K)   # off = 1: 4-byte aligned rows
    xd.copy_(dev(x))
    y = torch.full((M, N), float("nan"), device="cuda")
    cc.cc_linear("f32", xd, dev(w), y)
    torch.cuda.synchronize()
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    # K products and K - 1 sums in fp32: at most K 2^-23 of the sum of their magnitudes
    bound = K * 2.0 ** -23 * (np.abs(x).astype(np.float64) @ np.abs(w).astype(np.float64).T)
    assert np.all(np.abs(f64(y) - ref) <= bound)


@pytest.mark.parametrize("N,D,V", [(1, 64, 1), (63, 33, 65), (64, 128, 64), (65, 100, 1000), (1030, 40, 1000)])
def test_lmhead(N, D, V):
    from paper_2607_27600_amd import cc
    r = np.random.default_rng(7)
    u = r.standard_normal((N, D)).astype(np.float32)
    w = (0.05 * r.standard_normal((V, D))).astype(np.float32)
    ids = r.integers(0, V, N).astype(np.int32)
    p = cc.problem(dtype="f32", cu_seqlens=[0, N], n_heads_q=1, n_heads_kv=1, head_dim=64, hidden=D,
                   vocab=V)
    scores, lse = (torch.empty(N, device="cuda") for _ in range(2))
    cc.cc_lmhead_score(p, dev(u), dev(w), dev(ids), scores, lse)
    torch.cuda.synchronize()
    s_ref, lse_ref, _ = O.surprise(u.astype(np.float64), w, ids)
    s_ref[-1] = np.inf
    assert_scores_close(scores.cpu().numpy(), s_ref, "f32", "lmhead f32")
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, rtol=0, atol=F32_ATOL)
