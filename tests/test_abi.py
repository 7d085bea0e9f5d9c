"""Host-side checks of the C ABI: the library loads and exports every entry point the
header declares, the ctypes structures match the C layout, and argument validation
rejects bad problems before anything touches a GPU (workspace queries are host-only)."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "cc.h")


def _declared():
    txt = open(HEADER).read()
    return sorted(set(re.findall(r"^\s*(?:const\s+)?\w+\s*\*?\s*(cc_\w+)\s*\(", txt, re.M)))


def test_library_exports_every_declared_symbol():
    from paper_2607_27600_amd import cc
    names = _declared()
    assert len(names) >= 13
    out = subprocess.run(["nm", "-D", "--defined-only", cc.LIB_PATH], capture_output=True,
                         text=True, check=True).stdout
    exported = set(re.findall(r"\bT (cc_\w+)", out))
    assert set(names) <= exported, set(names) - exported
    assert set(names) == set(cc.EXPORTED)
    assert cc.cc_version().startswith("libcc gfx950")


def test_struct_layouts_match_header(tmp_path):
    from paper_2607_27600_amd import cc
    prog = tmp_path / "layout.c"
    fields = {
        "cc_kv": [f[0] for f in cc.c_kv._fields_],
        "cc_problem": [f[0] for f in cc.c_problem._fields_],
        "cc_inputs": [f[0] for f in cc.c_inputs._fields_],
        "cc_layer_weights": [f[0] for f in cc.c_layer_weights._fields_],
    }
    lines = ['#include <stdio.h>', '#include <stddef.h>', '#include "cc.h"', "int main(void){"]
    for s, fs in fields.items():
        lines.append(f'printf("{s} %zu\\n", sizeof({s}));')
        for f in fs:
            lines.append(f'printf("{s}.{f} %zu\\n", offsetof({s}, {f}));')
    lines.append("return 0;}")
    prog.write_text("\n".join(lines))
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-I", os.path.join(ROOT, "include"), str(prog), "-o", str(exe)],
                   check=True)
    got = dict(l.split() for l in subprocess.run([str(exe)], capture_output=True, text=True,
                                                 check=True).stdout.splitlines())
    classes = {"cc_kv": cc.c_kv, "cc_problem": cc.c_problem, "cc_inputs": cc.c_inputs,
               "cc_layer_weights": cc.c_layer_weights}
    for s, cls in classes.items():
        assert int(got[s]) == ctypes.sizeof(cls), s
        for f in fields[s]:
            assert int(got[f"{s}.{f}"]) == getattr(cls, f).offset, f"{s}.{f}"


def _prob(**kw):
    from paper_2607_27600_amd import cc
    cu = (ctypes.c_int32 * 3)(0, 100, 250)
    p = cc.c_problem()
    p.dtype, p.mode, p.diag, p.n_seqs = cc.CC_BF16, cc.CC_MODE_LAST_LAYER, cc.CC_DIAG_STRICT, 2
    p.cu_seqlens_h = ctypes.cast(cu, ctypes.POINTER(ctypes.c_int32))
    p.cu_seqlens_d = 0x1000          # never dereferenced by a workspace query
    p.n_heads_q, p.n_heads_kv, p.head_dim, p.hidden, p.vocab = 32, 8, 128, 4096, 128256
    for k, v in kw.items():
        setattr(p, k, v)
    return p, cu


def test_workspace_queries_and_validation():
    from paper_2607_27600_amd import cc
    lib = cc._lib
    n = ctypes.c_size_t(0)
    p, _keep = _prob()
    assert lib.cc_score_workspace(ctypes.byref(p), ctypes.byref(n)) == cc.CC_OK
    N = 250
    assert n.value >= N * 32 * 128 * 2 + N * 4096 * 2 + 501 * N * 8
    bad = [
        (dict(n_heads_q=30), cc.CC_ERR_SHAPE),
        (dict(head_dim=96), cc.CC_ERR_UNSUPPORTED),
        (dict(hidden=4000), cc.CC_ERR_UNSUPPORTED),
        (dict(dtype=7), cc.CC_ERR_DTYPE),
        (dict(diag=3), cc.CC_ERR_ARG),
        (dict(n_frozen=-1), cc.CC_ERR_ARG),
        (dict(softmax_scale=float("nan")), cc.CC_ERR_ARG),
        (dict(cu_seqlens_d=None), cc.CC_ERR_ARG),
        (dict(mode=cc.CC_MODE_FULL, n_layers=0), cc.CC_ERR_SHAPE),
    ]
    for kw, want in bad:
        q, _k = _prob(**kw)
        assert lib.cc_score_workspace(ctypes.byref(q), ctypes.byref(n)) == want, kw
    cu_bad = (ctypes.c_int32 * 3)(0, 100, 50)
    q, _k = _prob()
    q.cu_seqlens_h = ctypes.cast(cu_bad, ctypes.POINTER(ctypes.c_int32))
    assert lib.cc_score_workspace(ctypes.byref(q), ctypes.byref(n)) == cc.CC_ERR_SHAPE
    assert lib.cc_select_workspace(4, ctypes.byref(n)) == cc.CC_OK and n.value >= 4 * 24
    assert lib.cc_select_workspace(-1, ctypes.byref(n)) == cc.CC_ERR_ARG
    assert lib.cc_compact_workspace(ctypes.byref(p), 32, 1, ctypes.byref(n)) == cc.CC_OK
    assert lib.cc_compact_workspace(ctypes.byref(p), 32, 2, ctypes.byref(n)) == cc.CC_ERR_ARG


@pytest.mark.parametrize("mode", ["last_layer", "last_layer_fused", "last_layer_h", "full"])
@pytest.mark.parametrize("cu,D,F", [([0, 0], 64, 64), ([0, 0], 4096, 14336), ([0, 0, 0], 512, 64)])
def test_an_empty_cache_needs_no_workspace(mode, cu, D, F):
    """In a process of its own: a division by the number of tiles would end it."""
    prog = ("from paper_2607_27600_amd import cc\n"
            f"p = cc.problem(dtype='bf16', cu_seqlens={cu}, n_heads_q=2, n_heads_kv=1, head_dim=128, hidden={D},\n"
            f"               vocab=1024, device='cpu', mode='{mode}', n_layers=2, ffn={F}, rope_theta=1e4,\n"
            "               rms_eps=1e-5)\n"
            "print(cc.cc_score_workspace(p))\n")
    r = subprocess.run([sys.executable, "-c", prog], capture_output=True, text=True, cwd=ROOT)
    assert r.returncode == 0 and r.stdout.split()[-1] == "0", (r.returncode, r.stderr[-300:])


def test_calls_with_bad_arguments_enqueue_nothing():
    """Argument errors are reported before any HIP call (no GPU is needed to see them)."""
    from paper_2607_27600_amd import cc
    lib = cc._lib
    p, _keep = _prob()
    assert lib.cc_score(ctypes.byref(p), None, None, None, 0, None) == cc.CC_ERR_ARG
    kv = cc.c_kv()
    assert lib.cc_attention_cc(ctypes.byref(p), None, ctypes.byref(kv), 0, None, None, 0,
                               None) == cc.CC_ERR_ARG
    # a paged view whose page spans 4 GiB or more is refused (in-page offsets are 32-bit)
    kvp = cc.c_kv()
    kvp.layout, kvp.n_layers = cc.CC_KV_PAGED, 1
    kvp.k = kvp.v = 0x10000                       # 16-byte aligned, never dereferenced
    kvp.head_stride, kvp.tok_stride, kvp.page_size, kvp.max_pages = 16 * 128, 128, 16, 16
    kvp.block_table = 0x10000
    dummy16 = ctypes.c_void_p(0x10000)
    for page_stride, want in (((1 << 31), cc.CC_ERR_UNSUPPORTED), ((1 << 31) - 8, cc.CC_ERR_WORKSPACE)):
        kvp.page_stride = page_stride                # elements: x2 bytes reaches 2^32 or not
        assert lib.cc_attention_cc(ctypes.byref(p), dummy16, ctypes.byref(kvp), 0, dummy16, None, 0,
                                   None) == want
    st = (ctypes.c_int64 * 1)(0)
    ln = (ctypes.c_int32 * 1)(10)
    kk = (ctypes.c_int32 * 1)(11)                   # k > len
    assert lib.cc_select_keep(None, 1, st, ln, kk, None, None, 0, None) == cc.CC_ERR_SHAPE
    dummy = ctypes.c_void_p(0x1000)   # never dereferenced: the shape is rejected first
    assert lib.cc_linear(cc.CC_BF16, dummy, dummy, dummy, 4, 4, 100, None) == cc.CC_ERR_UNSUPPORTED
    assert lib.cc_linear(cc.CC_BF16, None, None, None, 4, 4, 64, None) == cc.CC_ERR_ARG
    assert lib.cc_linear(5, None, None, None, 4, 4, 64, None) == cc.CC_ERR_DTYPE
    for s in range(7):
        assert cc.cc_status_str(s)


def test_fused_and_fp8_entry_points_validate_on_the_host():
    """The W_o-fusion and FP8 entry points reject bad shapes, dtypes and alignments before
    anything is enqueued, and their workspace queries are host-only."""
    from paper_2607_27600_amd import cc
    lib = cc._lib
    n = ctypes.c_size_t(0)
    dummy = ctypes.c_void_p(0x1000)     # never dereferenced: every case fails first
    odd = ctypes.c_void_p(0x1002)
    # fused weight
    assert lib.cc_fuse_wo_lmhead_workspace(cc.CC_BF16, 4096, 4096, ctypes.byref(n)) == cc.CC_OK
    assert n.value >= 4096 * 4096 * 2
    assert lib.cc_fuse_wo_lmhead_workspace(9, 4096, 4096, ctypes.byref(n)) == cc.CC_ERR_DTYPE
    assert lib.cc_fuse_wo_lmhead(cc.CC_BF16, dummy, dummy, dummy, 100, 100, 128, dummy, 1 << 30,
                                 None) == cc.CC_ERR_UNSUPPORTED          # hidden % 64
    assert lib.cc_fuse_wo_lmhead(cc.CC_BF16, odd, dummy, dummy, 100, 128, 128, dummy, 1 << 30,
                                 None) == cc.CC_ERR_ARG                  # alignment
    assert lib.cc_fuse_wo_lmhead(cc.CC_BF16, dummy, dummy, dummy, 100, 128, 128, dummy, 16,
                                 None) == cc.CC_ERR_WORKSPACE
    assert lib.cc_fuse_wo_lmhead(cc.CC_BF16, None, dummy, dummy, 100, 128, 128, dummy, 1 << 30,
                                 None) == cc.CC_ERR_ARG
    # fused mode: a problem in that mode passes validation; W_o may be null, q may not
    p, _keep = _prob(mode=cc.CC_MODE_LAST_LAYER_FUSED)
    assert lib.cc_score_workspace(ctypes.byref(p), ctypes.byref(n)) == cc.CC_OK
    fused_ws = n.value
    q2, _k2 = _prob()
    assert lib.cc_score_workspace(ctypes.byref(q2), ctypes.byref(n)) == cc.CC_OK
    assert fused_ws < n.value               # no W_o output buffer in the fused layout
    q3, _k3 = _prob(mode=4)
    assert lib.cc_score_workspace(ctypes.byref(q3), ctypes.byref(n)) == cc.CC_ERR_ARG
    # quantization
    assert lib.cc_quantize_fp8_workspace(1000, ctypes.byref(n)) == cc.CC_OK and n.value >= 4004
    assert lib.cc_quantize_fp8_workspace(-1, ctypes.byref(n)) == cc.CC_ERR_ARG
    big = ctypes.c_size_t(1 << 30)
    assert lib.cc_quantize_fp8(cc.CC_BF16, dummy, 10, 6, 1, dummy, dummy, dummy, big,
                               None) == cc.CC_ERR_SHAPE                  # cols % 4
    assert lib.cc_quantize_fp8(cc.CC_BF16, dummy, 10, 8, 2, dummy, dummy, dummy, big,
                               None) == cc.CC_ERR_ARG                    # per_row flag
    assert lib.cc_quantize_fp8(cc.CC_F32, odd, 10, 8, 1, dummy, dummy, dummy, big,
                               None) == cc.CC_ERR_ARG                    # x alignment
    assert lib.cc_quantize_fp8(cc.CC_F32, dummy, 10, 8, 1, odd, dummy, dummy, big,
                               None) == cc.CC_ERR_ARG                    # codes alignment
    assert lib.cc_quantize_fp8(cc.CC_F32, dummy, 10, 8, 1, dummy, dummy, dummy, 8,
                               None) == cc.CC_ERR_WORKSPACE
    assert lib.cc_quantize_fp8(3, dummy, 10, 8, 1, dummy, dummy, dummy, big,
                               None) == cc.CC_ERR_DTYPE
    assert lib.cc_quantize_fp8(cc.CC_F32, dummy, 0, 8, 1, None, None, None, 0, None) == cc.CC_OK
    # FP8 LM head
    p, _keep = _prob()
    assert lib.cc_lmhead_fp8_workspace(ctypes.byref(p), ctypes.byref(n)) == cc.CC_OK
    assert n.value >= 250 * 4096 + 501 * 250 * 8
    q4, _k4 = _prob(hidden=4032)            # a multiple of 64, not of 128
    assert lib.cc_lmhead_score_fp8(ctypes.byref(q4), dummy, dummy, dummy, dummy, dummy, None,
                                   dummy, big, None) == cc.CC_ERR_UNSUPPORTED
    assert lib.cc_lmhead_score_fp8(ctypes.byref(p), dummy, odd, dummy, dummy, dummy, None,
                                   dummy, big, None) == cc.CC_ERR_ARG    # codes alignment
    assert lib.cc_lmhead_score_fp8(ctypes.byref(p), dummy, dummy, None, dummy, dummy, None,
                                   dummy, big, None) == cc.CC_ERR_ARG    # no scale
    assert lib.cc_lmhead_score_fp8(ctypes.byref(p), dummy, dummy, dummy, dummy, dummy, None,
                                   dummy, 64, None) == cc.CC_ERR_WORKSPACE


def test_packed_lmhead_entry_points_validate_on_the_host():
    """The packed LM head's queries are host-only, and its entry points reject bad shapes,
    dtypes, alignments, overlaps and missing packed weights before anything is enqueued."""
    from paper_2607_27600_amd import cc
    lib = cc._lib
    n = ctypes.c_size_t(0)
    dummy = ctypes.c_void_p(0x1000)
    odd = ctypes.c_void_p(0x1002)
    # packed size: rows rounded up to 256
    assert lib.cc_pack_lmhead_bytes(300, 64, ctypes.byref(n)) == cc.CC_OK
    assert n.value == 512 * 64 * 2
    assert lib.cc_pack_lmhead_bytes(256, 96, ctypes.byref(n)) == cc.CC_OK and n.value == 256 * 96 * 2
    assert lib.cc_pack_lmhead_bytes(0, 32, ctypes.byref(n)) == cc.CC_OK and n.value == 0
    assert lib.cc_pack_lmhead_bytes(10, 48, ctypes.byref(n)) == cc.CC_ERR_ARG     # cols % 32
    assert lib.cc_pack_lmhead_bytes(-1, 32, ctypes.byref(n)) == cc.CC_ERR_ARG
    big = ctypes.c_size_t(1 << 30)
    far = ctypes.c_void_p(0x10000000)
    assert lib.cc_pack_lmhead(dummy, 10, 32, odd, big, None) == cc.CC_ERR_ARG     # alignment
    assert lib.cc_pack_lmhead(None, 10, 32, far, big, None) == cc.CC_ERR_ARG
    assert lib.cc_pack_lmhead(dummy, 10, 32, far, 1024, None) == cc.CC_ERR_WORKSPACE
    assert lib.cc_pack_lmhead(dummy, 10, 32, ctypes.c_void_p(0x1100), big, None) == cc.CC_ERR_ARG  # overlap
    assert lib.cc_pack_lmhead(None, 0, 32, None, 0, None) == cc.CC_OK
    # problems: packed is bf16 only, a 0/1 flag, and adds the packed rows to the workspace
    p, _k = _prob(lmhead_packed=1)
    assert lib.cc_lmhead_workspace(ctypes.byref(p), ctypes.byref(n)) == cc.CC_OK
    packed_ws = n.value
    p0, _k0 = _prob()
    assert lib.cc_lmhead_workspace(ctypes.byref(p0), ctypes.byref(n)) == cc.CC_OK
    assert packed_ws - n.value >= 256 * 4096 * 2              # 250 rows -> one 256-row tile
    pf, _kf = _prob(lmhead_packed=1, dtype=cc.CC_F32)
    assert lib.cc_lmhead_workspace(ctypes.byref(pf), ctypes.byref(n)) == cc.CC_ERR_UNSUPPORTED
    p2, _k2 = _prob(lmhead_packed=2)
    assert lib.cc_score_workspace(ctypes.byref(p2), ctypes.byref(n)) == cc.CC_ERR_ARG
    # the packed sub-step needs a packed problem and weight; the row-major one refuses it
    ws = ctypes.c_void_p(0x100000)
    assert lib.cc_lmhead_score_packed(ctypes.byref(p0), dummy, dummy, dummy, dummy, None,
                                      ws, big, None) == cc.CC_ERR_ARG
    assert lib.cc_lmhead_score_packed(ctypes.byref(p), dummy, None, dummy, dummy, None,
                                      ws, big, None) == cc.CC_ERR_ARG
    assert lib.cc_lmhead_score_packed(ctypes.byref(p), dummy, odd, dummy, dummy, None,
                                      ws, big, None) == cc.CC_ERR_ARG
    assert lib.cc_lmhead_score(ctypes.byref(p), dummy, dummy, dummy, dummy, None, ws, big,
                               None) == cc.CC_ERR_ARG


def test_selection_takes_scalars_and_refuses_what_does_not_fit(monkeypatch):
    """Every form of the host lists reaches the library, whose host checks then refuse the budgets
    (k > length), or raises what numpy raises for it."""
    import numpy as np
    import torch
    from paper_2607_27600_amd import cc
    monkeypatch.setattr(cc, "_stream", lambda stream=None: None)
    t = torch.zeros(64)
    ws = torch.empty(4096, dtype=torch.uint8)

    def status(start, length, k):
        with pytest.raises(cc.CCError) as e:
            cc.cc_select_keep(t, start, length, k, t.int(), workspace=ws)
        return e.value.status

    for start, length, k in [([0], [5], [7]), ((0, 5), (5, 5), (1, 7)), (0, 5, 7), (np.int64(0), np.int32(5), 7),
                             ([np.int64(0)], [np.int32(5)], [np.int32(7)]), ([0.0], [5.0], [7.0]), ([0], [5], [True + 6]),
                             (np.zeros(1, np.int64), np.array([5], np.int32), np.array([7], np.int32)),
                             (range(2), [5] * 2, [7] * 2), ([0] * 100, [5] * 100, [7] * 100),
                             (torch.zeros(1, dtype=torch.int64), torch.tensor([5]), torch.tensor([7]))]:
        assert status(start, length, k) == cc.CC_ERR_SHAPE, (start, length, k)
    for bad in ([2 ** 64 + 1], [2 ** 70]):
        with pytest.raises(OverflowError):
            cc.cc_select_keep(t, [0], [5], bad, t.int(), workspace=ws)
    assert [list(cc._host_array(x, np.int64, cc._i64)[0][:2]) for x in ([3, 2 ** 40], np.array([3, 2 ** 40]))] == [[3, 2 ** 40]] * 2


def test_device_lengths_that_the_kernels_would_misread_are_refused():
    import torch
    from paper_2607_27600_amd import cc
    kw = dict(dtype="bf16", cu_seqlens=[0, 5, 9], n_heads_q=1, n_heads_kv=1, head_dim=64, hidden=64, vocab=64,
              device="cpu")
    cu = torch.tensor([0, 5, 9], dtype=torch.int32)
    assert cc.problem(cu_device=cu, **kw).cu_d is cu
    for bad in (cu.long(), cu[:2], cu.view(1, 3), torch.zeros(6, dtype=torch.int32)[::2]):
        with pytest.raises(ValueError):
            cc.problem(cu_device=bad, **kw)


@pytest.mark.parametrize("mode", ["last_layer", "last_layer_fused", "last_layer_h", "full"])
def test_workspace_holds_no_tables_that_nothing_writes(mode):
    """A packed weight adds nothing to a score's workspace (the entry rows are read as they are), and
    compaction needs its keep lists (32 bytes or fewer each), whatever the layers and slabs."""
    from paper_2607_27600_amd import cc
    n = ctypes.c_size_t()
    modes = {"last_layer": 0, "full": 1, "last_layer_h": 2, "last_layer_fused": 3}
    kw = dict(mode=modes[mode], n_layers=2, ffn=1024, rope_theta=1e4, rms_eps=1e-5)
    sizes = []
    for packed in (0, 1):
        p, _k = _prob(lmhead_packed=packed, **kw)
        assert cc._lib.cc_score_workspace(ctypes.byref(p), ctypes.byref(n)) == cc.CC_OK
        sizes.append(n.value)
    assert sizes[0] == sizes[1] > 0
    for per_head in (0, 1):
        lists = p.n_seqs * (p.n_heads_kv if per_head else 1)
        for layers in (1, 80):
            assert cc._lib.cc_compact_workspace(ctypes.byref(p), layers, per_head, ctypes.byref(n)) == cc.CC_OK
            assert 24 * lists <= n.value <= 32 * lists + 256
        assert cc._lib.cc_compact_rows_workspace(ctypes.byref(p), 1 << 20, per_head, ctypes.byref(n)) == cc.CC_OK
        assert 24 * p.n_seqs <= n.value <= 32 * p.n_seqs + 256
