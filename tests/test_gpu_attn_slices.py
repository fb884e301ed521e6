"""Tree attention where requests go out ahead of the sequence length, and where the output columns are
sliced over workgroups: the rows of the cache past a sequence's length hold NaN, lengths lie around the
tiles and steps (16, 32, 128, 256 keys) and are shorter than the capacity, head dimensions end inside a slice."""
import numpy as np
import pytest
import torch

from oracle import mcsd_oracle as O
from paper_2401_06706_amd import binding as M
from paper_2401_06706_amd import device as D
from paper_2401_06706_amd import workloads as W
from tests.parity import assert_attn_close

pytestmark = pytest.mark.gpu

LENGTHS = (0, 1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 255, 256, 257, 300)


def run(dtype, d, H_q, H_kv, kconfig, lengths, capacity):
    w = W.Workload(name="t", index=72, B=len(lengths), H_q=H_q, H_kv=H_kv, d=d, dtype=dtype, prefix=(max(lengths), max(lengths)),
                   kconfig=kconfig, V=8, sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(d + H_q + capacity), L_stride=capacity)
    ai.prefix_len[:] = lengths
    print(f"[slices] {dtype} d={d} H={H_q}/{H_kv} N={ai.N} L={list(lengths)} capacity={capacity}", flush=True)
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale,
                      O.FP32 if dtype == "fp32" else O.BF16, n_threads=16)
    call = D.make_attn_call(ai)
    for b, n in enumerate(lengths):
        call.tensors["k_prefix"][b, :, n:] = float("nan")
        call.tensors["v_prefix"][b, :, n:] = float("nan")
    M.mcsd_tree_attn(call.args)
    torch.cuda.synchronize()
    assert_attn_close(call.out_numpy(), ref, dtype, f"{dtype} d={d}")
    # through pages: the same tiles, hence the same bits
    paged_call, paged, _ = D.make_paged_attn_call(call, ai, 96, seed=d)
    M.mcsd_tree_attn_paged(paged_call.args, paged)
    torch.cuda.synchronize()
    assert torch.equal(paged_call.out, call.out)


# bf16 at d = 128: 28 rows whole (capacity below the slices' range) and sliced, 56, 112 and 224 rows sliced,
# 112 rows in segments (capacity beyond it); the other head dimensions and fp32, whose last slice is ragged
@pytest.mark.parametrize("dtype,d,H_q,H_kv,kconfig,capacity", [
    ("bf16", 128, 2, 2, (4, 2, 2), 300), ("bf16", 128, 2, 2, (4, 2, 2), 640), ("bf16", 128, 8, 8, (4, 2, 2), 1000),
    ("bf16", 128, 2, 2, (8, 2, 1, 1), 301), ("bf16", 128, 4, 1, (4, 2, 2), 300), ("bf16", 128, 8, 1, (4, 2, 2), 1504),
    ("bf16", 128, 32, 8, (4, 2, 2), 320), ("bf16", 128, 16, 4, (4, 2, 2), 300), ("bf16", 128, 4, 1, (4, 2, 2), 4000), ("bf16", 64, 4, 2, (4, 2, 2), 300),
    ("bf16", 40, 2, 2, (4, 2, 2), 300), ("bf16", 24, 2, 2, (2, 2), 300), ("bf16", 96, 2, 2, (4, 2, 2), 301), ("bf16", 72, 8, 8, (4, 2, 2), 300),
    ("bf16", 120, 16, 16, (2, 2), 300), ("bf16", 200, 2, 2, (4, 2, 2), 300), ("fp32", 64, 2, 2, (4, 2, 2), 300), ("fp32", 36, 2, 2, (2, 2), 300),
    ("fp32", 128, 1, 1, (4, 2, 2), 303), ("fp32", 128, 16, 16, (4, 2, 2), 300), ("fp32", 100, 1, 1, (2, 2), 300), ("fp32", 228, 1, 1, (2, 2), 300),
])
def test_rows_past_the_length_are_not_used(dtype, d, H_q, H_kv, kconfig, capacity):
    for i in range(0, len(LENGTHS), 5):
        run(dtype, d, H_q, H_kv, kconfig, LENGTHS[i:i + 5], capacity)


def test_a_capacity_below_the_first_tiles():
    for dtype, d in (("bf16", 128), ("bf16", 64), ("fp32", 128)):
        for capacity in (1, 31, 96, 128):
            run(dtype, d, 2, 2, (4, 2, 2), (0, capacity // 2, capacity), capacity)


# The first tiles are asked for ahead of the lengths while they are 8 MiB or less in all: 4 sequences of these shapes
# are (at the line, where they lie on it), 16 are not.  Both forms walk the same tiles in the same order.
@pytest.mark.parametrize("kconfig,capacity,few", [((4, 2, 2), 300, 4), ((4, 2, 2, 1, 1), 300, 8)])
def test_first_tiles_ahead_of_the_lengths_or_not(kconfig, capacity, few):
    lengths = (20, 0, 1, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 257, 299, 300)
    w = W.Workload(name="t", index=74, B=16, H_q=32, H_kv=32, d=128, dtype="bf16", prefix=(300, 300), kconfig=kconfig, V=8, sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(few), L_stride=capacity)
    ai.prefix_len[:] = lengths
    call = D.make_attn_call(ai)
    t = call.tensors
    for b, n in enumerate(lengths):
        t["k_prefix"][b, :, n:] = float("nan")
        t["v_prefix"][b, :, n:] = float("nan")
    M.mcsd_tree_attn(call.args)
    outs = []
    for b in range(0, 16, few):
        part = {k: t[k][b:b + few] for k in ("q", "k_prefix", "v_prefix", "prefix_len", "k_tree", "v_tree")}
        outs.append(torch.zeros_like(part["q"]))
        M.mcsd_tree_attn(M.attn_args(part["q"], part["k_prefix"], part["v_prefix"], part["prefix_len"], part["k_tree"], part["v_tree"],
                                     t["parent"], outs[-1], ai.scale, t["workspace"]))
    torch.cuda.synchronize()
    assert torch.equal(torch.cat(outs).view(torch.int16), call.out.view(torch.int16))
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale, O.BF16, n_threads=16)
    assert_attn_close(call.out_numpy(), ref, "bf16", f"{kconfig} capacity={capacity}")


def writes_partials(call, run):
    """Whether the call `run` leaves something in its workspace: segments and a merge do, slices do not."""
    call.tensors["workspace"].fill_(77)
    run()
    torch.cuda.synchronize()
    return not bool((call.tensors["workspace"] == 77).all())


# Both sides of the lines between slices and segments, one sequence full and the others short (capacities in
# tiles of 32 keys, one or two of the tree: 65 + 1 and 66 + 1, 53 + 1 and 54 + 1, 48 + 2 and 49 + 2, ...)
@pytest.mark.parametrize("B,H_q,H_kv,kconfig,capacity,slices", [
    (4, 32, 8, (4, 2, 2), 2080, True), (4, 32, 8, (4, 2, 2), 2081, False), (2, 64, 8, (4, 2, 2), 2080, True), (3, 32, 8, (4, 2, 2), 1696, True), (3, 32, 8, (4, 2, 2), 1697, False),
    (8, 32, 8, (4, 2, 2), 1696, True), (8, 32, 8, (4, 2, 2), 1697, False), (4, 32, 32, (4, 2, 2, 1, 1), 2048, True),
    (4, 32, 32, (4, 2, 2, 1, 1), 2049, False), (2, 32, 32, (4, 2, 2, 1, 1), 1536, True), (2, 32, 32, (4, 2, 2, 1, 1), 1537, False),
    (1, 32, 32, (4, 2, 2, 1, 1), 1536, True), (1, 32, 32, (4, 2, 2, 1, 1), 1537, False)])
def test_lines_between_slices_and_segments(B, H_q, H_kv, kconfig, capacity, slices):
    w = W.Workload(name="t", index=76, B=B, H_q=H_q, H_kv=H_kv, d=128, dtype="bf16", prefix=(capacity, capacity), kconfig=kconfig, V=8, sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(capacity))
    ai.prefix_len[1:] = 100
    call = D.make_attn_call(ai)
    for b in range(1, B):
        call.tensors["k_prefix"][b, :, 100:] = float("nan")
        call.tensors["v_prefix"][b, :, 100:] = float("nan")
    assert writes_partials(call, lambda: M.mcsd_tree_attn(call.args)) != slices
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale, O.BF16, n_threads=16)
    assert_attn_close(call.out_numpy(), ref, "bf16", f"{B} x {H_q}/{H_kv} capacity={capacity}")


# The same for up to 32 rows per KV head: 49 + 1 tiles above 160 workgroups, 34 + 1 from 129 up to there
@pytest.mark.parametrize("B,H_q,H_kv,kconfig,capacity,slices", [
    (8, 32, 32, (4, 2, 2), 1568, True), (8, 32, 32, (4, 2, 2), 1569, False), (23, 28, 7, (2, 2), 1567, True), (23, 28, 7, (2, 2), 1600, False),
    (5, 32, 32, (4, 2, 2), 1088, True), (5, 32, 32, (4, 2, 2), 1089, False)])
def test_lines_of_up_to_32_rows(B, H_q, H_kv, kconfig, capacity, slices):
    test_lines_between_slices_and_segments(B, H_q, H_kv, kconfig, capacity, slices)


# (whole below ten tiles, slices from there on; both without partials)
@pytest.mark.parametrize("capacity", [224, 225, 256, 257, 383])
def test_the_lower_line_of_the_slices(capacity):
    run("bf16", 128, 32, 32, (4, 2, 2, 1, 1), (capacity, capacity - 33, 31), capacity)


# (28 rows: slices up to six tiles and from nine on, whole between; 60 rows of 60 nodes and 56 of 28 by more than 128 workgroups)
@pytest.mark.parametrize("B,H_q,H_kv,kconfig", [(2, 4, 4, (4, 2, 2)), (5, 16, 16, (4, 2, 2, 1, 1)), (17, 16, 8, (4, 2, 2))])
@pytest.mark.parametrize("capacity", [1, 33, 160, 161, 224, 225, 256, 257])
def test_the_lower_lines_for_few_rows(B, H_q, H_kv, kconfig, capacity):
    lengths = tuple(max(0, capacity - 37 * b) for b in range(B))
    run("bf16", 128, H_q, H_kv, kconfig, lengths, capacity)


# (257 to 512 workgroups of 32 rows: 64 rows in lockstep up to 16 tiles at d <= 64 and eight beyond, then 32 rows with tiles of their own)
@pytest.mark.parametrize("d,capacity", [(64, 480), (64, 481), (40, 700), (96, 224), (96, 225), (72, 300), (120, 520)])
@pytest.mark.parametrize("B,H_q,H_kv,kconfig", [(9, 32, 8, (4, 2, 2)), (13, 20, 10, (4, 2, 2)), (6, 80, 16, (2, 2, 2))])
def test_more_than_one_workgroup_of_32_rows_per_cu(d, capacity, B, H_q, H_kv, kconfig):
    lengths = tuple(max(0, capacity - 41 * b) for b in range(B))
    run("bf16", d, H_q, H_kv, kconfig, lengths, capacity)


@pytest.mark.parametrize("H_q,H_kv,bad", [(4, 4, {1: -5, 9: 2 ** 30}), (4, 4, {0: 2 ** 30, 20: -1}), (8, 2, {4: -(2 ** 31), 12: 2 ** 31 - 1}), (4, 4, {25: -5, 26: 2 ** 30})])
def test_table_entries_outside_the_pool_read_as_zero_keys(H_q, H_kv, bad):
    """Pages of 32 rows of one sequence of 600 keys in a cache of 864, in slices: page j is tile j, the first
    step of a workgroup is tiles 0 .. 7.  Entries of used pages outside the pool read as zero keys, those of pages past the
    length (the last case) as nothing."""
    w = W.Workload(name="t", index=75, B=1, H_q=H_q, H_kv=H_kv, d=128, dtype="bf16", prefix=(600, 600), kconfig=(4, 2, 2), V=8, sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(H_q), L_stride=864)
    tree = D.make_attn_call(ai)
    paged_call, paged, table = D.make_paged_attn_call(tree, ai, 32)
    entries = table.astype(np.int64)
    for j, e in bad.items():
        entries[0, j] = e
        ai.k_prefix[0, :, 32 * j:32 * j + 32] = 0
        ai.v_prefix[0, :, 32 * j:32 * j + 32] = 0
    paged_call.tensors["block_table"].copy_(torch.from_numpy(entries.astype(np.int32)))
    assert not writes_partials(paged_call, lambda: M.mcsd_tree_attn_paged(paged_call.args, paged))
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale, O.BF16, n_threads=4)
    assert_attn_close(paged_call.out_numpy(), ref, "bf16", f"{bad}")


@pytest.mark.parametrize("H_q,H_kv,capacity", [(32, 32, 512), (8, 1, 1500), (32, 8, 1000)])
def test_slices_give_the_same_bits_on_every_run(H_q, H_kv, capacity):
    """Scores that grow along the prefix raise the running maxima again and again (as in the test of the whole and
    segmented kernels): a result read before it has landed would move the raises around."""
    w = W.Workload(name="t", index=77, B=2, H_q=H_q, H_kv=H_kv, d=128, dtype="bf16", prefix=(capacity, capacity), kconfig=(4, 2, 2), V=8, sigma_q=1.0, variant=0)
    ai = W.gen_attn_inputs(w, np.random.default_rng(H_q))
    ramp = np.linspace(0.2, 3.0, capacity, dtype=np.float32)[None, None, :, None]
    ai.k_prefix = W.f32_to_bf16_bits(W.bf16_bits_to_f32(ai.k_prefix) * ramp)
    ref = O.tree_attn(ai.q, ai.k_prefix, ai.v_prefix, ai.prefix_len, ai.k_tree, ai.v_tree, ai.parent, ai.scale, O.BF16, n_threads=16)
    call = D.make_attn_call(ai)
    assert not writes_partials(call, lambda: M.mcsd_tree_attn(call.args))
    first = call.out.clone()
    assert_attn_close(call.out_numpy(), ref, "bf16", f"ramp {H_q}/{H_kv}")
    for rep in range(4):
        call.out.fill_(3.0)
        M.mcsd_tree_attn(call.args)
        torch.cuda.synchronize()
        assert torch.equal(call.out.view(torch.int16), first.view(torch.int16)), rep


# (the lines of make_attn_plan between whole and sliced launches without partials: one row per node and more than 128 workgroups of
# 32 rows, slices below ten tiles from 51 rows of the tree on, the root's among them; 28 rows, slices up to six tiles and from nine on)
@pytest.mark.parametrize("B,H,nodes,root,capacity,sliced", [
    (3, 32, 33, False, 96, False), (3, 32, 40, False, 31, False), (5, 16, 50, False, 96, False), (5, 16, 51, False, 96, True), (3, 32, 32, True, 96, False),
    (3, 32, 49, True, 96, False), (3, 32, 50, True, 96, True), (4, 32, 63, True, 1, True), (3, 32, 33, False, 256, True), (2, 16, 33, False, 96, True),
    (2, 16, 28, False, 160, True), (2, 16, 28, False, 161, False), (2, 16, 28, False, 224, False), (2, 16, 28, False, 225, True)])
def test_which_kernel_runs(B, H, nodes, root, capacity, sliced):
    """Seen by the bits: the plan override never slices, and the slices add up their keys in another order."""
    rng = np.random.default_rng(nodes + capacity)
    n, lengths = nodes + root, [max(1, capacity - 3 * b) for b in range(B)]
    bf16 = lambda *shape: W.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))
    q, k, v, kt, vt = bf16(B, n, H, 128), bf16(B, H, capacity, 128), bf16(B, H, capacity, 128), bf16(B, H, n, 128), bf16(B, H, n, 128)
    parent = np.array([-1] + [i // 2 for i in range(nodes - 1)], np.int32)
    dev = [torch.from_numpy(x.view(np.int16)).cuda().view(torch.bfloat16) for x in (q, k, v, kt, vt)]
    out = []
    for variant in (0, 2 if n > 32 else 1):
        o = torch.full_like(dev[0], 3.0)
        args = M.attn_args(dev[0], dev[1], dev[2], torch.tensor(lengths, dtype=torch.int32, device="cuda"), dev[3], dev[4], torch.from_numpy(parent).cuda(), o, 128 ** -0.5,
                           workspace=torch.empty(1 << 26, dtype=torch.uint8, device="cuda"))
        print(f"[which] B={B} H={H} nodes={nodes} root={root} capacity={capacity} variant={variant}", flush=True)
        M.mcsd_attn_plan_override(variant=variant)
        try:
            M.mcsd_tree_attn(args)
            torch.cuda.synchronize()
        finally:
            M.mcsd_attn_plan_override()
        out.append(o)
    assert torch.equal(out[0], out[1]) != sliced
    full = np.concatenate([[-1], parent + 1]).astype(np.int32) if root else parent
    sel = np.stack([np.arange(600) % B, rng.integers(0, n, 600), rng.integers(0, H, 600)], 1).astype(np.int32)
    ref = O.tree_attn(q, k, v, np.array(lengths, np.int32), kt, vt, full, 128 ** -0.5, O.BF16, sel=sel, n_threads=16)
    for o in out:
        got = o.float().cpu().numpy()
        assert_attn_close(got[sel[:, 0], sel[:, 1], sel[:, 2]], ref, "bf16", f"{nodes}")


# (65 to 96 and 129 to 160 rows by more than 256 workgroups of 64 rows and up to 512 of 32: 32 rows with tiles of their own at any capacity)
@pytest.mark.parametrize("d,capacity", [(96, 60), (72, 225), (120, 300)])
@pytest.mark.parametrize("B,H_q,H_kv,kconfig", [(13, 20, 10, (5, 2, 2)), (17, 20, 10, (5, 2, 2)), (10, 50, 10, (4, 2, 2))])
def test_more_than_one_workgroup_of_64_rows_per_cu(d, capacity, B, H_q, H_kv, kconfig):
    lengths = tuple(max(0, capacity - 19 * b) for b in range(B))
    run("bf16", d, H_q, H_kv, kconfig, lengths, capacity)
