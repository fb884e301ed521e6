"""Tree attention with fp32 storage or a head dimension other than 128 against the CPU oracle: head
dimensions around the paddings (64, 128, 256), row counts around the row tiles, prefixes around the
16- and 32-key tiles and long enough for many steps; the paged cache and a call without a workspace
give the same attention."""
import numpy as np
import pytest
import torch

from oracle import mcsd_oracle as O
from paper_2401_06706_amd import binding as M
from paper_2401_06706_amd import device as D
from paper_2401_06706_amd import workloads as W
from tests.parity import assert_attn_close

pytestmark = pytest.mark.gpu

# (dtype, d, B, H_q, H_kv, k-configuration, shortest and longest prefix)
CASES = [
    ("bf16", 8, 1, 1, 1, (1,), (0, 0)), ("bf16", 40, 2, 6, 2, (3, 2), (31, 33)), ("bf16", 64, 3, 4, 4, (4, 2, 2), (0, 900)),
    ("bf16", 64, 2, 8, 4, (4, 2, 2), (1, 700)), ("bf16", 64, 2, 16, 2, (4, 2, 2), (63, 2500)), ("bf16", 72, 1, 8, 2, (2, 2), (15, 17)),
    ("bf16", 96, 2, 4, 2, (4, 4, 2, 1), (5, 600)), ("bf16", 120, 1, 8, 1, (128,), (300, 300)), ("bf16", 136, 2, 2, 2, (4, 2, 2), (33, 400)),
    ("bf16", 200, 1, 4, 1, (4, 2, 2), (100, 1000)), ("bf16", 256, 2, 4, 2, (4, 2), (0, 1500)), ("bf16", 256, 1, 3, 3, (16, 2, 2), (64, 64)),
    ("fp32", 4, 1, 1, 1, (1,), (0, 0)), ("fp32", 8, 2, 6, 2, (3, 2), (15, 17)), ("fp32", 64, 3, 4, 2, (4, 2, 2), (0, 700)),
    ("fp32", 68, 1, 8, 1, (2, 2, 2, 2, 2, 2), (127, 129)), ("fp32", 128, 2, 4, 4, (4, 2, 2), (1, 1100)), ("fp32", 128, 5, 32, 32, (2, 2), (20, 90)),
    ("fp32", 132, 2, 2, 1, (16,), (16, 300)), ("fp32", 256, 1, 4, 4, (128,), (33, 33)), ("fp32", 256, 5, 32, 32, (4,), (0, 40)),
]


@pytest.mark.parametrize("dtype,d,B,H_q,H_kv,kconfig,prefix", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_against_oracle(dtype, d, B, H_q, H_kv, kconfig, prefix):
    w = W.Workload(name="t", index=70, B=B, H_q=H_q, H_kv=H_kv, d=d, dtype=dtype, prefix=prefix, kconfig=kconfig, V=8,
                   sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(d + H_q), L_stride=prefix[1] + 3)
    print(f"[any] {dtype} d={d} B={B} H={H_q}/{H_kv} N={ai.N} L={ai.prefix_len.tolist()}", flush=True)
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale,
                      O.FP32 if dtype == "fp32" else O.BF16, n_threads=16)
    call = D.make_attn_call(ai)
    M.mcsd_tree_attn(call.args)
    torch.cuda.synchronize()
    assert_attn_close(call.out_numpy(), ref, dtype, "contiguous")
    paged_call, paged, _ = D.make_paged_attn_call(call, ai, 32, seed=d)
    M.mcsd_tree_attn_paged(paged_call.args, paged)
    torch.cuda.synchronize()
    assert torch.equal(paged_call.out, call.out)
    # without a workspace the same attention
    t = call.tensors
    whole = torch.zeros_like(t["out"])
    M.mcsd_tree_attn(M.attn_args(t["q"], t["k_prefix"], t["v_prefix"], t["prefix_len"], t["k_tree"], t["v_tree"], t["parent"],
                                 whole, ai.scale))
    torch.cuda.synchronize()
    assert_attn_close(whole.to(torch.float32).cpu().numpy().astype(np.float64), ref, dtype, "no workspace")


@pytest.mark.parametrize("dtype,d,H_q,H_kv,prefix", [("bf16", 64, 32, 8, (200, 2000)), ("bf16", 96, 4, 2, (1500, 1500)), ("bf16", 256, 2, 1, (900, 1100)),
                                                     ("fp32", 128, 4, 4, (700, 700))])
def test_no_workspace_is_used_and_the_bits_depend_on_the_inputs_alone(dtype, d, H_q, H_kv, prefix):
    """A workspace that comes along is not written, of whatever size and alignment; the result has the same
    bits with it, without it, from the entry point that brings none, and from two streams at once that
    were handed the same pointer."""
    w = W.Workload(name="t", index=71, B=2, H_q=H_q, H_kv=H_kv, d=d, dtype=dtype, prefix=prefix, kconfig=(4, 2, 2), V=8, sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(d), L_stride=prefix[1] + 500)
    t = D.make_attn_call(ai).tensors
    ws = torch.full((64 << 20,), 77, dtype=torch.uint8, device="cuda:0")
    results = []
    def args(workspace=None):
        results.append(torch.zeros_like(t["out"]))
        return M.attn_args(t["q"], t["k_prefix"], t["v_prefix"], t["prefix_len"], t["k_tree"], t["v_tree"], t["parent"],
                           results[-1], ai.scale, workspace)
    for workspace in (None, ws, ws[:1000], ws[64:]):
        M.mcsd_tree_attn(args(workspace))
    M.mcsd_tree_attn_static(args())
    streams = [torch.cuda.Stream() for _ in range(2)]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for _ in range(4):
        for s in streams:
            a = args(ws)
            s.wait_stream(torch.cuda.current_stream())
            M.mcsd_tree_attn(a, stream=s)
    torch.cuda.synchronize()
    for r in results[1:]:
        assert torch.equal(r.view(torch.int16), results[0].view(torch.int16))
    assert (ws == 77).all()
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale,
                      O.FP32 if dtype == "fp32" else O.BF16, n_threads=16)
    assert_attn_close(results[0].to(torch.float32).cpu().numpy().astype(np.float64), ref, dtype, "no workspace")


# many units, so that every instantiation is met (the cases above are the small launches)
SPLITS = [
    (64, 16, 10, 2, (4, 2, 2)), (64, 13, 20, 1, (2, 2)), (64, 15, 10, 4, (4, 2, 2)), (64, 20, 20, 2, (4, 2, 2)), (40, 16, 32, 4, (4, 2, 2)),
    (72, 16, 10, 2, (4, 2, 2)), (128 - 8, 13, 20, 1, (2, 2)), (96, 15, 20, 2, (4, 2, 2)), (96, 12, 32, 4, (4, 2, 2)),
    (136, 2, 3, 1, (2, 2)), (200, 10, 10, 1, (2, 2)), (136, 10, 10, 1, (2, 2)), (256, 20, 10, 1, (2, 2)), (248, 13, 20, 1, (2, 2)), (256, 13, 10, 2, (4, 2, 2))]


@pytest.mark.parametrize("d,B,H_kv,G,kconfig", SPLITS)
def test_every_split_of_the_rows_and_columns(d, B, H_kv, G, kconfig):
    w = W.Workload(name="t", index=72, B=B, H_q=H_kv * G, H_kv=H_kv, d=d, dtype="bf16", prefix=(0, 70), kconfig=kconfig, V=8, sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(d + B), L_stride=300)
    call = D.make_attn_call(ai)
    M.mcsd_tree_attn(call.args)
    torch.cuda.synchronize()
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale, O.BF16, n_threads=16)
    assert_attn_close(call.out_numpy(), ref, "bf16", f"d={d} units={B * H_kv} rows={ai.N * G}")


@pytest.mark.parametrize("d,B,H_kv,G,kconfig", SPLITS)
def test_every_split_over_several_steps(d, B, H_kv, G, kconfig):
    """The same launches with lengths of up to three steps of the widest form (eight tiles of 32 keys), around its
    ends, in a cache with spare rows that hold NaN; through pages, which have no straight-line step, the same
    bits.  The oracle on every length, 1500 rows in all."""
    lengths = (600, 0, 70, 255, 256, 257, 300, 512, 513, 530)
    w = W.Workload(name="t", index=73, B=B, H_q=H_kv * G, H_kv=H_kv, d=d, dtype="bf16", prefix=(0, 600), kconfig=kconfig, V=8, sigma_q=1.0, variant=0)
    rng = np.random.default_rng(d + B)
    ai = W.gen_attn_inputs(w, rng, L_stride=640)
    ai.prefix_len[:] = [lengths[b % len(lengths)] for b in range(B)]
    call = D.make_attn_call(ai)
    for b in range(B):
        call.tensors["k_prefix"][b, :, int(ai.prefix_len[b]):] = float("nan")
        call.tensors["v_prefix"][b, :, int(ai.prefix_len[b]):] = float("nan")
    M.mcsd_tree_attn(call.args)
    torch.cuda.synchronize()
    n = 1500
    sel = np.stack([np.arange(n) % B, rng.integers(0, ai.N, n), rng.integers(0, ai.H_q, n)], 1).astype(np.int32)
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale, O.BF16, sel=sel, n_threads=16)
    got = call.out_numpy()
    assert np.isfinite(got).all()
    assert_attn_close(got[sel[:, 0], sel[:, 1], sel[:, 2]], ref, "bf16", f"d={d} units={B * H_kv} rows={ai.N * G}")
    for page in (32, 96):
        paged_call, paged, _ = D.make_paged_attn_call(call, ai, page, seed=d)
        M.mcsd_tree_attn_paged(paged_call.args, paged)
        torch.cuda.synchronize()
        assert torch.equal(paged_call.out, call.out)


@pytest.mark.parametrize("d", [8, 40, 64, 72, 88, 96, 104, 120, 128])
@pytest.mark.parametrize("H_kv,G", [(2, 1), (64, 4)], ids=["slices", "whole"])
def test_tiles_behind_the_first(d, H_kv, G):
    """Lengths around the steps of eight tiles, where a wavefront has one tile, or one more that comes while the first
    is computed: whole ones, ragged ones and the tree's; columns that end inside an operand. Contiguous and through pages."""
    lengths = np.array([257] if H_kv > 2 else [225, 255, 256, 257, 300, 511, 513, 780], np.int32)
    w = W.Workload(name="t", index=73, B=len(lengths), H_q=H_kv * G, H_kv=H_kv, d=d, dtype="bf16", prefix=(800, 800), kconfig=(4, 2, 2), V=8, sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(d + H_kv), L_stride=803)
    ai.prefix_len[:] = lengths
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale, O.BF16, n_threads=16)
    call = D.make_attn_call(ai)
    M.mcsd_tree_attn(call.args)
    torch.cuda.synchronize()
    assert_attn_close(call.out_numpy(), ref, "bf16", f"d={d}")
    paged_call, paged, _ = D.make_paged_attn_call(call, ai, 32, seed=d)
    M.mcsd_tree_attn_paged(paged_call.args, paged)
    torch.cuda.synchronize()
    assert torch.equal(paged_call.out, call.out)
