"""GPU parity of the projections at the shapes where a tile shape or a slice count of the plan
can go wrong: entries and features that are no multiple of any tile, few k-tiles, K cut into
unequal slices, and the fused residual + norm of a split and an unsplit projection."""
import numpy as np
import pytest
import torch

from oracle import cc_oracle as O
from synth import gen
from tests.gpu_util import dev, f64

pytestmark = pytest.mark.gpu


def _bf16(r, shape, std=1.0):
    return gen.f32_to_bf16_bits((std * r.standard_normal(shape)).astype(np.float32))


@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (63, 130, 64), (65, 96, 128), (257, 1001, 192),
                                   (129, 3584, 448), (700, 2050, 320), (2049, 260, 64), (5000, 1030, 128)])
def test_linear_bf16_edges(M, N, K):
    from paper_2607_27600_amd import cc
    r = np.random.default_rng(M + N)
    x, w = _bf16(r, (M, K)), _bf16(r, (N, K))
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    cc.cc_linear("bf16", dev(x), dev(w), y)
    torch.cuda.synchronize()
    a, b = O.f64(x), O.f64(w)
    ref = a @ b.T
    # one bf16 rounding (2^-8) and K fp32 sums of exact products (K 2^-23 of their magnitudes)
    bound = 2.0 ** -8 * np.abs(ref) + K * 2.0 ** -23 * (np.abs(a) @ np.abs(b).T)
    assert np.all(np.abs(f64(y) - ref) <= bound)


def test_linear_bf16_odd_output_address():
    from paper_2607_27600_amd import cc
    r = np.random.default_rng(3)
    x, w = _bf16(r, (70, 64)), _bf16(r, (132, 64))
    buf = torch.zeros(70 * 132 + 1, dtype=torch.bfloat16, device="cuda")
    cc.cc_linear("bf16", dev(x), dev(w), buf[1:].view(70, 132))
    y = torch.empty((70, 132), dtype=torch.bfloat16, device="cuda")
    cc.cc_linear("bf16", dev(x), dev(w), y)
    assert torch.equal(buf[1:].view(70, 132), y) and buf[0] == 0


@pytest.mark.parametrize("n,D,F,hq,hkv", [(40, 192, 2048, 2, 1), (200, 320, 4160, 3, 1), (333, 448, 960, 4, 2),
                                          (1100, 256, 1088, 2, 2)])
def test_full_layer_edges(n, D, F, hq, hkv):
    """One layer of the full pass: W_q with RoPE, W_o and W_down into the residual stream (K of
    W_down long against its output: cut into slices), gate/up."""
    from paper_2607_27600_amd import cc
    from synth import configs as C
    from tests.gpu_util import assert_scores_close
    from paper_2607_27600_amd.workload import Workload
    cfg = C.shrink(C.C4, seq_lens=(n,), n_heads_q=hq, n_heads_kv=hkv, hidden=D, ffn=F, vocab=700,
                   n_layers=2, cache_layers=2, keep=(1,), w_std=0.05)
    w = Workload(cfg, keep_host=True)
    scores = torch.full((n,), float("nan"), device="cuda")
    cc.cc_score(w.problem, w.inputs(), scores)
    torch.cuda.synchronize()
    h = w.host
    kvl = h["kv_layers"]
    ref = O.full_scores(h["ids"], lambda l: (kvl[l]["k"], kvl[l]["v"]), lambda l: h["layers"][l],
                        h["embed"], h["final_norm"], h["w_lm"], cfg.cu_seqlens, cfg.n_layers,
                        cfg.n_heads_q, cfg.head_dim, cfg.rope_theta, cfg.rms_eps)
    print(assert_scores_close(scores.cpu().numpy(), ref, "bf16", f"full n={n} D={D} F={F}"))
