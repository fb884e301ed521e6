"""The C ABI without a GPU: the library loads, exports every symbol the header
declares, the ctypes structs match the C layout, and every argument error is
reported by return code before anything touches the device."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2401_06706_amd import binding as M

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "mcsd.h")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(M.LIB_PATH):
        from paper_2401_06706_amd.build import build
        build(verbose=False)
    return M.lib()


def declared_functions():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(mcsd_[a-z_]+)\s*\(", src)))


def test_exports_every_declared_symbol(lib):
    names = declared_functions()
    assert set(M.EXPORTS) == set(names)
    for n in names:
        assert getattr(lib, n) is not None
    assert b"gfx950" in lib.mcsd_version()


def test_struct_layout_matches_header(tmp_path):
    """Compile a C program against the header and compare sizeof/offsetof with ctypes."""
    fields = {"mcsd_attn_desc": (M.AttnDesc, ["struct_size", "B", "d", "L_stride", "scale", "parent_per_seq", "root_row"]),
              "mcsd_attn_bufs": (M.AttnBufs, ["q", "prefix_len", "out", "workspace", "workspace_bytes"]),
              "mcsd_verify_desc": (M.VerifyDesc, ["V", "P", "variant", "gamma_max", "near_tie_eps", "parent_per_seq"]),
              "mcsd_verify_bufs": (M.VerifyBufs, ["target_logits", "temperature", "acc_child", "ratio",
                                                  "flags", "residual_out", "workspace_bytes"]),
              "mcsd_paged_kv": (M.PagedKV, ["page_size", "n_pages", "max_pages_per_seq", "block_table"]),
              "mcsd_draft_desc": (M.DraftDesc, ["B", "V", "P", "variant", "near_tie_eps", "parent_per_seq"]),
              "mcsd_draft_bufs": (M.DraftBufs, ["draft_logits", "q_row", "u_draw", "temperature", "cand_tok", "flags"]),
              "mcsd_commit_desc": (M.CommitDesc, ["B", "H_kv", "dtype", "L_stride", "gamma_max", "n_layers", "root_row"]),
              "mcsd_commit_bufs": (M.CommitBufs, ["k_prefix", "v_tree", "n_accepted", "out_tokens", "prefix_len",
                                                  "next_root", "flags"])}
    lines = ['#include <stdio.h>', '#include <stddef.h>', '#include "mcsd.h"', "int main(void){"]
    for cname, (_, fs) in fields.items():
        lines.append(f'printf("{cname} %zu\\n", sizeof({cname}));')
        for f in fs:
            lines.append(f'printf("{cname}.{f} %zu\\n", offsetof({cname}, {f}));')
    lines.append("return 0;}")
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "layout"
    subprocess.check_call(["gcc", "-std=c99", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                           str(src), "-o", str(exe)])
    got = dict(l.split() for l in subprocess.check_output([str(exe)], text=True).splitlines())
    for cname, (ct, fs) in fields.items():
        assert int(got[cname]) == C.sizeof(ct)
        for f in fs:
            assert int(got[f"{cname}.{f}"]) == getattr(ct, f).offset


def test_tree_validate(lib):
    M.mcsd_tree_validate(np.array([-1, -1, 0, 0, 1, 1], np.int32))
    for bad in ([0], [-1, 1], [-1, -2], [-1, 0, 5]):
        with pytest.raises(M.McsdError) as e:
            M.mcsd_tree_validate(np.array(bad, np.int32))
        assert e.value.code == -4
    with pytest.raises(M.McsdError) as e:
        M.mcsd_tree_validate(np.full(129, -1, np.int32))
    assert e.value.code == -4
    assert lib.mcsd_tree_validate(None, 3) == -1


def good_attn_desc(**kw):
    a = dict(B=2, N=6, H_q=4, H_kv=2, d=128, dtype=M.DTYPE_BF16, L_stride=4096, scale=0.088)
    a.update(kw)
    return M.attn_desc(**a)


def test_attn_workspace_and_descriptor_errors(lib):
    assert M.mcsd_attn_workspace_bytes(good_attn_desc()) % 256 == 0
    assert M.mcsd_attn_workspace_bytes(good_attn_desc()) > 0
    assert M.mcsd_attn_workspace_bytes(good_attn_desc(dtype=M.DTYPE_FP32, d=64)) == 0
    # shapes outside the d = 128 kernel bring no workspace and touch none, however long the cache
    for d in (8, 64, 96, 256):
        for kw in (dict(L_stride=16384, B=1), dict(L_stride=2000, B=8), dict(L_stride=0, B=300)):
            assert M.mcsd_attn_workspace_bytes(good_attn_desc(d=d, **kw)) == 0, (d, kw)
    bufs = M.AttnBufs(C.sizeof(M.AttnBufs), 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 1 << 40)
    cases = [(dict(N=0), -4), (dict(N=129), -4), (dict(H_q=5), -2), (dict(B=0), -2), (dict(d=130), -3),
             (dict(d=512), -3), (dict(dtype=7), -3), (dict(scale=float("nan")), -2), (dict(L_stride=-1), -2)]
    for kw, code in cases:
        d = good_attn_desc(**kw)
        assert M.mcsd_attn_workspace_bytes(d) == 0
        assert lib.mcsd_tree_attn(C.byref(d), C.byref(bufs), None) == code, kw
        assert len(lib.mcsd_last_error()) > 0
    d = good_attn_desc()
    d.struct_size = 12
    assert lib.mcsd_tree_attn(C.byref(d), C.byref(bufs), None) == -2
    d = good_attn_desc()
    assert lib.mcsd_tree_attn(None, C.byref(bufs), None) == -1
    assert lib.mcsd_tree_attn(C.byref(d), None, None) == -1
    # buffer errors: NULL tensor, missing / short / misaligned workspace, misaligned tensor
    need = M.mcsd_attn_workspace_bytes(d)
    b = M.AttnBufs(C.sizeof(M.AttnBufs), None, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, need)
    assert lib.mcsd_tree_attn(C.byref(d), C.byref(b), None) == -1
    b = M.AttnBufs(C.sizeof(M.AttnBufs), 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, None, 0)
    assert lib.mcsd_tree_attn(C.byref(d), C.byref(b), None) == -5
    b = M.AttnBufs(C.sizeof(M.AttnBufs), 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, need - 1)
    assert lib.mcsd_tree_attn(C.byref(d), C.byref(b), None) == -5
    b = M.AttnBufs(C.sizeof(M.AttnBufs), 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096 + 64, need)
    assert lib.mcsd_tree_attn(C.byref(d), C.byref(b), None) == -5
    b = M.AttnBufs(C.sizeof(M.AttnBufs), 4096 + 2, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, need)
    assert lib.mcsd_tree_attn(C.byref(d), C.byref(b), None) == -2
    b = M.AttnBufs(7, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, need)
    assert lib.mcsd_tree_attn(C.byref(d), C.byref(b), None) == -2


def good_verify_desc(**kw):
    a = dict(B=2, N=6, V=64, P=3, variant=0, gamma_max=2, near_tie_eps=1e-6)
    a.update(kw)
    return M.VerifyDesc(C.sizeof(M.VerifyDesc), a["B"], a["N"], a["V"], a["P"], a["variant"],
                        a["gamma_max"], a["near_tie_eps"])


def test_verify_descriptor_errors(lib):
    ptrs = [4096] * 16 + [None]
    bufs = M.VerifyBufs(C.sizeof(M.VerifyBufs), *ptrs, 0)
    assert M.mcsd_verify_workspace_bytes(good_verify_desc()) == 0
    cases = [(dict(N=0), -4), (dict(N=200), -4), (dict(V=0), -2), (dict(V=70000), -3), (dict(P=9), -2),
             (dict(variant=3), -3), (dict(gamma_max=0), -2), (dict(near_tie_eps=-1.0), -2),
             (dict(B=70000), -3), (dict(P=0), -2)]
    for kw, code in cases:
        d = good_verify_desc(**kw)
        assert lib.mcsd_verify_sample(C.byref(d), C.byref(bufs), None) == code, kw
    d = good_verify_desc()
    assert lib.mcsd_verify_sample(None, C.byref(bufs), None) == -1
    assert lib.mcsd_verify_sample(C.byref(d), None, None) == -1
    for i in (0, 3, 7, 8, 11, 14):        # required pointers
        p2 = list(ptrs); p2[i] = None
        b = M.VerifyBufs(C.sizeof(M.VerifyBufs), *p2, 0)
        assert lib.mcsd_verify_sample(C.byref(d), C.byref(b), None) == -1, i
    p2 = list(ptrs); p2[0] = 4100           # V % 4 == 0 rows are read with 16-byte loads
    b = M.VerifyBufs(C.sizeof(M.VerifyBufs), *p2, 0)
    assert lib.mcsd_verify_sample(C.byref(d), C.byref(b), None) == -2
    # verify_step validates both halves before enqueueing anything
    ad = good_attn_desc(N=0)
    ab = M.AttnBufs(C.sizeof(M.AttnBufs), 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 1 << 40)
    assert lib.mcsd_verify_step(C.byref(ad), C.byref(ab), C.byref(d), C.byref(bufs), None) == -4
    ad = good_attn_desc()
    dv = good_verify_desc(V=0)
    assert lib.mcsd_verify_step(C.byref(ad), C.byref(ab), C.byref(dv), C.byref(bufs), None) == -2


def test_binding_fails_loudly_without_library(monkeypatch, tmp_path):
    monkeypatch.setattr(M, "_lib", None)
    monkeypatch.setattr(M, "LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(FileNotFoundError):
        M.lib()


def test_draft_descriptor_errors(lib):
    def desc(**kw):
        a = dict(B=2, N=6, V=64, P=3, variant=0, near_tie_eps=1e-6)
        a.update(kw)
        return M.DraftDesc(C.sizeof(M.DraftDesc), a["B"], a["N"], a["V"], a["P"], a["variant"], a["near_tie_eps"])
    ptrs = [4096] * 7
    bufs = M.DraftBufs(C.sizeof(M.DraftBufs), *ptrs)
    cases = [(dict(N=0), -4), (dict(N=200), -4), (dict(V=0), -2), (dict(V=70000), -3), (dict(P=9), -2),
             (dict(variant=3), -3), (dict(near_tie_eps=-1.0), -2), (dict(B=70000), -3), (dict(P=0), -2)]
    for kw, code in cases:
        d = desc(**kw)
        assert lib.mcsd_draft_sample(C.byref(d), C.byref(bufs), None) == code, kw
        assert len(lib.mcsd_last_error()) > 0
    d = desc()
    assert lib.mcsd_draft_sample(None, C.byref(bufs), None) == -1
    assert lib.mcsd_draft_sample(C.byref(d), None, None) == -1
    for i in range(7):
        p2 = list(ptrs); p2[i] = None
        assert lib.mcsd_draft_sample(C.byref(d), C.byref(M.DraftBufs(C.sizeof(M.DraftBufs), *p2)), None) == -1, i
    assert lib.mcsd_draft_sample(C.byref(d), C.byref(M.DraftBufs(5, *ptrs)), None) == -2
    p2 = list(ptrs); p2[0] = 4096 + 4
    assert lib.mcsd_draft_sample(C.byref(d), C.byref(M.DraftBufs(C.sizeof(M.DraftBufs), *p2)), None) == -2


def test_tree_size_and_build_errors(lib):
    assert M.mcsd_tree_size((4, 2, 2, 1, 1)) == (60, 45)
    assert M.mcsd_tree_size((2, 2)) == (6, 3)
    assert M.mcsd_tree_size((128,)) == (128, 1)
    for bad, code in [((4, 4, 4, 2), -4), ((2, 0), -2), ((), -2), ((1,) * 17, -2)]:
        with pytest.raises(M.McsdError) as e:
            M.mcsd_tree_size(bad)
        assert e.value.code == code
    kc = np.array([2, 2], np.int32)
    kp = kc.ctypes.data_as(C.c_void_p)
    assert lib.mcsd_tree_size(None, 2, None, None) == -1
    assert lib.mcsd_tree_build(kp, 2, 1, None, None, 4096, 4096, None, 0, None) == -1      # NULL output
    assert lib.mcsd_tree_build(kp, 2, 1, None, 4096, 4096, 4096, 4096, 0, None) == -1      # position ids without prefix_len
    assert lib.mcsd_tree_build(kp, 2, 0, 4096, 4096, 4096, 4096, 4096, 0, None) == -2      # B = 0 with position ids
    assert lib.mcsd_tree_build(kp, 2, 1, 4096, 4096, 4096, 4096, 4096, 2, None) == -2      # root_row is 0 or 1


def test_commit_descriptor_errors(lib):
    def desc(**kw):
        a = dict(B=2, N=6, H_kv=2, d=128, dtype=M.DTYPE_BF16, L_stride=64, gamma_max=2, n_layers=1)
        a.update(kw)
        return M.CommitDesc(C.sizeof(M.CommitDesc), a["B"], a["N"], a["H_kv"], a["d"], a["dtype"], a["L_stride"],
                            a["gamma_max"], a["n_layers"])
    ptrs = [4096] * 10
    bufs = M.CommitBufs(C.sizeof(M.CommitBufs), *ptrs)
    cases = [(dict(N=0), -4), (dict(N=129), -4), (dict(B=0), -2), (dict(H_kv=0), -2), (dict(d=4), -2),
             (dict(dtype=5), -3), (dict(L_stride=0), -2), (dict(gamma_max=0), -2), (dict(n_layers=0), -2),
             (dict(B=70000), -3)]
    for kw, code in cases:
        d = desc(**kw)
        assert lib.mcsd_kv_commit(C.byref(d), C.byref(bufs), None) == code, kw
    d = desc()
    assert lib.mcsd_kv_commit(None, C.byref(bufs), None) == -1
    assert lib.mcsd_kv_commit(C.byref(d), None, None) == -1
    for i in range(10):
        p2 = list(ptrs); p2[i] = None
        assert lib.mcsd_kv_commit(C.byref(d), C.byref(M.CommitBufs(C.sizeof(M.CommitBufs), *p2)), None) == -1, i
    p2 = list(ptrs); p2[2] = 4096 + 8
    assert lib.mcsd_kv_commit(C.byref(d), C.byref(M.CommitBufs(C.sizeof(M.CommitBufs), *p2)), None) == -2
    # paged form: the same descriptor checks, then the paged descriptor
    pk = M.PagedKV(C.sizeof(M.PagedKV), 32, 10, 2, 4096)
    assert lib.mcsd_kv_commit_paged(C.byref(desc(N=0)), C.byref(bufs), C.byref(pk), None) == -4
    assert lib.mcsd_kv_commit_paged(C.byref(d), C.byref(bufs), None, None) == -1
    for kw, code in [(dict(page_size=40), -2), (dict(n_pages=0), -2), (dict(max_pages=1), -2), (dict(table=None), -1)]:
        a = dict(page_size=32, n_pages=10, max_pages=2, table=4096); a.update(kw)
        pk = M.PagedKV(C.sizeof(M.PagedKV), a["page_size"], a["n_pages"], a["max_pages"], a["table"])
        assert lib.mcsd_kv_commit_paged(C.byref(d), C.byref(bufs), C.byref(pk), None) == code, kw


def test_paged_descriptor_errors(lib):
    d = good_attn_desc()
    need = M.mcsd_attn_workspace_bytes(d)
    bufs = M.AttnBufs(C.sizeof(M.AttnBufs), 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, 4096, need)
    def paged(**kw):
        a = dict(page_size=64, n_pages=200, max_pages_per_seq=64, block_table=4096)
        a.update(kw)
        return M.PagedKV(C.sizeof(M.PagedKV), a["page_size"], a["n_pages"], a["max_pages_per_seq"], a["block_table"])
    cases = [(dict(page_size=48), -2), (dict(page_size=0), -2), (dict(n_pages=0), -2), (dict(max_pages_per_seq=0), -2),
             (dict(max_pages_per_seq=63), -2), (dict(block_table=None), -1)]
    for kw, code in cases:
        pk = paged(**kw)
        assert lib.mcsd_tree_attn_paged(C.byref(d), C.byref(bufs), C.byref(pk), None) == code, kw
    pk = paged()
    assert lib.mcsd_tree_attn_paged(C.byref(d), C.byref(bufs), None, None) == -1
    assert lib.mcsd_tree_attn_paged(C.byref(d), None, C.byref(pk), None) == -1
    pk.struct_size = 3
    assert lib.mcsd_tree_attn_paged(C.byref(d), C.byref(bufs), C.byref(pk), None) == -2


def test_static_scratch_entry_point_refuses_oversized_shapes_before_touching_the_device(lib):
    """mcsd_tree_attn_static holds MCSD_STATIC_SCRATCH_BYTES of scratch; a shape whose split partials
    need more is refused by return code (the pointers here are never dereferenced)."""
    hdr = open(HEADER).read()
    m = re.search(r"#define MCSD_STATIC_SCRATCH_BYTES \(\(size_t\)(\d+) << (\d+)\)", hdr)
    assert m and (int(m.group(1)) << int(m.group(2))) == M.STATIC_SCRATCH_BYTES
    d = M.attn_desc(16, 84, 64, 8, 128, M.DTYPE_BF16, 16384, 0.088)
    assert M.mcsd_attn_workspace_bytes(d) > M.STATIC_SCRATCH_BYTES
    b = M.AttnBufs(C.sizeof(M.AttnBufs), 256, 256, 256, 256, 256, 256, 256, 256, None, 0)
    assert lib.mcsd_tree_attn_static(C.byref(d), C.byref(b), None) == -5
    assert b"static buffer holds" in lib.mcsd_last_error()
    assert lib.mcsd_tree_attn_static(C.byref(d), None, None) == -1
    d.N = 0
    assert lib.mcsd_tree_attn_static(C.byref(d), C.byref(b), None) == -4
