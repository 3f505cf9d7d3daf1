"""Chunks that stage 1 holds in registers (at most 256 tokens at d = 128, 512 at d = 64), chunks that a whole call works on as
one, the cut of a task's rows over several workgroups, and stage 2 by the number of partial results and of rows, at the
sizes where they can go wrong.  Same tolerance as tests/test_gpu_parity.py, whose paths of fewer than 1024 tokens also get
the tight bound of two-term weights."""

import numpy as np
import pytest
import torch

from paper_2404_00242_amd import binding, workloads as wl

from .test_gpu_parity import check, reference, reference_abs_v, run_gpu

pytestmark = pytest.mark.gpu


def tree(root, branches, Hq, Hkv, d, seed):
    """a root of `root` tokens under branches of the given lengths, one query each (0: on a node without tokens)"""
    lens = np.asarray([root] + list(branches), dtype=np.int32)
    begin = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int32)
    parent = np.asarray([-1] + [0] * len(branches), dtype=np.int32)
    return wl.Tree(name=f"short_{root}", node_tok_begin=begin, node_tok_len=lens, node_parent=parent,
                   query_node=np.arange(1, len(lens), dtype=np.int32), ntok=int(lens.sum()), Hq=Hq, Hkv=Hkv, d=d, value_seed=seed)


# blocks per wave 1 and 2 (and 4 at d = 64), whole and broken last blocks, waves without a block, one token
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("root", [1, 31, 33, 96, 128, 129, 255, 256, 257, 300, 385, 512, 513])
def test_one_chunk_of_every_length(root, d):
    t = tree(root, [0, 3, 1, 2], 6, 2, d, seed=root)
    Q, K, V = wl.make_qkv(t)
    got, _ = run_gpu(t, Q, K, V, chunk_size=1024, out_dtype=torch.float32, mode="node")
    check(got, reference(t, Q, K, V), strict=False, abs_v=reference_abs_v(t, Q, K, V), two_term=True)


# 1 to 17 row tiles, the last one full, nearly full or with one row; KV heads that leave the chip empty (rows cut as
# finely as they go), nearly full, and over-full (not cut at all)
@pytest.mark.parametrize("nq,G", [(1, 1), (17, 1), (33, 1), (12, 4), (13, 5), (129, 1), (65, 4)])
@pytest.mark.parametrize("Hkv", [1, 8, 48])
def test_row_tiles_and_workgroup_cuts(nq, G, Hkv):
    if nq * G * Hkv > 4000:
        Hkv = 12
    t = tree(700, [(5 * i) % 7 for i in range(nq)], G * Hkv, Hkv, 128, seed=nq)
    Q, K, V = wl.make_qkv(t)
    for chunk in (96, 256, 640):
        got, _ = run_gpu(t, Q, K, V, chunk_size=chunk, out_dtype=torch.float32)
        check(got, reference(t, Q, K, V), strict=False, abs_v=reference_abs_v(t, Q, K, V), two_term=True)


# long paths (bf16 weights) through the same shapes; both splits
@pytest.mark.parametrize("mode", ["flatten", "balanced"])
@pytest.mark.parametrize("nq,Hq,Hkv,d", [(3, 8, 8, 128), (20, 32, 8, 128), (9, 24, 2, 64), (70, 8, 2, 64)])
def test_long_paths_in_short_chunks(nq, Hq, Hkv, d, mode):
    t = tree(1100, [(7 * i) % 90 for i in range(nq)], Hq, Hkv, d, seed=nq)
    Q, K, V = wl.make_qkv(t)
    for chunk in (128, 224, 256):
        got, _ = run_gpu(t, Q, K, V, chunk_size=chunk, out_dtype=torch.float32, mode=mode)
        check(got, reference(t, Q, K, V), strict=False)


# stage 2 by the number of partial results of a query: one wave, two, four, slot ids past the record, several passes
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("parts", [1, 16, 17, 29, 30, 32, 33, 61, 62, 125, 126, 257, 300])
def test_any_number_of_partial_results(parts, d):
    t = tree(32 * parts - 7, [0, 40], 6, 2, d, seed=parts)
    Q, K, V = wl.make_qkv(t)
    for out_dtype in (torch.float32, torch.bfloat16):
        got, _ = run_gpu(t, Q, K, V, chunk_size=32, out_dtype=out_dtype, mode="node_chunk")
        check(got, reference(t, Q, K, V), strict=False)


# plans of many short chunks: prefixes, several branches, wide next to narrow, short next to long paths; a whole call (which
# may work on several chunks as one, see test_stage2_after_a_whole_call) and the stages called apart give the same result
@pytest.mark.parametrize("mode,chunk", [("flatten", 128), ("flatten", 96), ("node_chunk", 64), ("balanced", 128), ("query", 160)])
@pytest.mark.parametrize("Hq,Hkv,d,root", [(32, 32, 128, 900), (24, 24, 64, 1500), (96, 24, 128, 2100)])
def test_joined_chunks(mode, chunk, Hq, Hkv, d, root):
    t = tree(root, [(37 * i) % 150 for i in range(14)], Hq, Hkv, d, seed=root)
    Q, K, V = wl.make_qkv(t)
    got, plan = run_gpu(t, Q, K, V, chunk_size=chunk, out_dtype=torch.float32, mode=mode)
    ref = reference(t, Q, K, V)
    check(got, ref, strict=False)
    dev = torch.device("cuda:0")
    q, k, v = Q.to(dev), K.to(dev), V.to(dev)
    o = torch.empty((t.nq, Hq, d), dtype=torch.float32, device=dev)
    lib, img, ws = binding.load_library(), plan.image(Hq, Hkv, dev), plan.workspace(Hq, Hkv, d, dev)
    ws.fill_(0xFF)  # NaN: every slot that stage 2 reads has to be written by stage 1
    st = torch.cuda.current_stream().cuda_stream
    assert lib.deft_stage1_partial_attention(plan.handle, img.data_ptr(), q.data_ptr(), k.data_ptr(), v.data_ptr(), Hq,
                                             Hkv, d, 0.0, ws.data_ptr(), ws.numel(), st) == 0
    assert lib.deft_stage2_global_reduction(plan.handle, img.data_ptr(), o.data_ptr(), Hq, Hkv, d, 0.0, 1, ws.data_ptr(),
                                            ws.numel(), st) == 0
    torch.cuda.synchronize()
    check(o.cpu().numpy().astype(np.float64), ref, strict=False)
    ws.fill_(0xFF)
    binding.deft_tree_attn_decode(plan, q, k, v, out=o, workspace=ws)
    torch.cuda.synchronize()
    check(o.cpu().numpy().astype(np.float64), ref, strict=False)


def stages(plan, q, k, v, ws, one=True, two=True, out_f32=1):
    """the two stages called apart on a workspace; returns stage 2's output"""
    nq, Hq, d = q.shape
    Hkv, dev = k.shape[1], q.device
    lib, img, st = binding.load_library(), plan.image(Hq, Hkv, dev), torch.cuda.current_stream().cuda_stream
    o = torch.empty((nq, Hq, d), dtype=torch.float32 if out_f32 else torch.bfloat16, device=dev)
    if one:
        assert lib.deft_stage1_partial_attention(plan.handle, img.data_ptr(), q.data_ptr(), k.data_ptr(), v.data_ptr(),
                                                 Hq, Hkv, d, 0.0, ws.data_ptr(), ws.numel(), st) == 0
    if two:
        assert lib.deft_stage2_global_reduction(plan.handle, img.data_ptr(), o.data_ptr(), Hq, Hkv, d, 0.0, out_f32,
                                                ws.data_ptr(), ws.numel(), st) == 0
    torch.cuda.synchronize()
    return o


def empty_slots(plan, ws, Hq, d):
    """(slot, head) pairs of a workspace that hold no token: m = -inf, l = 0"""
    rows = plan.view()["n_slots"] * Hq
    f = ws.view(torch.float32)
    m, l = f[rows * d: rows * (d + 1)], f[rows * (d + 1): rows * (d + 2)]
    return int(((m == -np.inf) & (l == 0)).sum())


JOINING = ("flatten", "balanced")


# Stage 2 may follow a whole call on its workspace (a second output type, say), whether or not the call worked on several
# chunks as one; the comparison strategies are run chunk by chunk.
@pytest.mark.parametrize("mode", ["flatten", "balanced", "node_chunk", "query"])
@pytest.mark.parametrize("Hq,Hkv,d", [(32, 32, 128), (40, 20, 64), (64, 16, 128)])
def test_stage2_after_a_whole_call(mode, Hq, Hkv, d):
    t = tree(2900, [(37 * i) % 150 for i in range(14)], Hq, Hkv, d, seed=Hq)
    Q, K, V = wl.make_qkv(t)
    q, k, v = (x.to("cuda:0") for x in (Q, K, V))
    _, plan = run_gpu(t, Q, K, V, chunk_size=64, out_dtype=torch.float32, mode=mode)
    ref, ws = reference(t, Q, K, V), plan.workspace(Hq, Hkv, d, q.device)
    ws.fill_(0xFF)  # NaN
    whole = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32, workspace=ws)
    after = stages(plan, q, k, v, ws, one=False)
    joined = empty_slots(plan, ws, Hq, d)
    check(whole.cpu().numpy().astype(np.float64), ref, strict=False)
    check(after.cpu().numpy().astype(np.float64), ref, strict=False)
    check(stages(plan, q, k, v, ws, one=False, out_f32=0).float().cpu().numpy().astype(np.float64), ref, strict=False)
    ws.fill_(0xFF)
    check(stages(plan, q, k, v, ws).cpu().numpy().astype(np.float64), ref, strict=False)
    assert empty_slots(plan, ws, Hq, d) == 0
    assert (joined > 0) == (mode in JOINING), joined


# Inf and NaN in V reach the queries that see them and, inside one chunk, its other queries (0 * Inf); a whole call must
# not carry them further than the two stages do chunk by chunk, and in the node and query plans, whose chunks hold nothing
# that some query of the group does not see, no further than the reference.
@pytest.mark.parametrize("mode,chunk", [("flatten", 64), ("balanced", 64), ("node_chunk", 64), ("node", 0), ("query", 96)])
@pytest.mark.parametrize("Hq,Hkv,d", [(32, 32, 128), (24, 24, 64)])
def test_infinities_of_a_sibling_stay_where_they_are(mode, chunk, Hq, Hkv, d):
    t = tree(2100, [20 + (37 * i) % 90 for i in range(24)], Hq, Hkv, d, seed=d)
    Q, K, V = wl.make_qkv(t)
    at = int(t.node_tok_begin[5]) + 3
    V[at, :, 7], V[at + 1, :, 9] = float("inf"), float("nan")
    q, k, v = (x.to("cuda:0") for x in (Q, K, V))
    got, plan = run_gpu(t, Q, K, V, chunk_size=chunk, out_dtype=torch.float32, mode=mode)
    ws = plan.workspace(Hq, Hkv, d, q.device)
    apart = stages(plan, q, k, v, ws).cpu().numpy()
    assert not np.isfinite(got[4]).all()  # the query of node 5
    assert (np.isfinite(got) >= np.isfinite(apart)).all()
    if mode not in JOINING:
        others = [j for j in range(t.nq) if j != 4]
        assert np.isfinite(got[others]).all()
        V[at, :, 7] = V[at + 1, :, 9] = 0
        check(got[others], reference(t, Q, K, V)[others], strict=False)


# stage 2 with one wave to a row (more than 2048 rows), with two and with four, slot ids in the record up to its last one
# and past it, in more than one batch of 64; every 40th query has `parts` partial results, the others one
@pytest.mark.parametrize("nq,Hq,Hkv,d", [(40, 24, 8, 128), (40, 48, 8, 64), (80, 40, 8, 128)])
@pytest.mark.parametrize("parts", [29, 30, 61, 65, 125, 126, 130])
def test_stage2_waves_by_rows(parts, nq, Hq, Hkv, d):
    lens = [32 * parts - 5 if i % 40 == 7 else 20 + i % 3 for i in range(nq)]
    t = wl._finish("waves", lens, [-1] * nq, list(range(nq)), Hq, Hkv, d, parts)
    Q, K, V = wl.make_qkv(t)
    got, plan = run_gpu(t, Q, K, V, chunk_size=32, out_dtype=torch.float32, mode="node_chunk")
    assert int(np.diff(plan.view()["q_part_ptr"]).max()) == parts
    check(got, reference(t, Q, K, V), strict=False)


# more rows than 256 threads each would leave within 32 bits of grid x block (2^24): 17 queries x 2^20 heads
def test_more_than_2_to_the_24_rows():
    lens, Hq, d, dev = [33 * 32] + [20] * 16, 1 << 20, 64, torch.device("cuda:0")
    begin = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int32)
    plan = binding.deft_plan(begin, lens, [-1] * 17, list(range(17)), sum(lens), 32, binding.SPLIT_MODES["node_chunk"])
    g = torch.Generator(device=dev).manual_seed(24)
    q = torch.empty((17, Hq, d), dtype=torch.bfloat16, device=dev).normal_(generator=g)
    k, v = (torch.empty((sum(lens), 1, d), dtype=torch.bfloat16, device=dev).normal_(generator=g) for _ in range(2))
    o = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32)
    torch.cuda.synchronize()
    heads = torch.tensor([0, 1, 127, 128, 65537, Hq - 1], device=dev)
    for j, n in enumerate(lens):
        kj, vj = (x[int(begin[j]): int(begin[j]) + n, 0].double() for x in (k, v))
        want = torch.softmax(q[j, heads].double() @ kj.T.contiguous() / d ** 0.5, dim=-1) @ vj
        check(o[j, heads].cpu().numpy().astype(np.float64), want.cpu().numpy(), strict=False)


# the cut of rows is the one for the head count of the upload, also if a size was asked for with another
def test_cut_does_not_depend_on_an_earlier_size_query():
    t = tree(4000, [256] * 20, 32, 8, 128, seed=1)
    Q, K, V = wl.make_qkv(t)
    q, k, v = (x.to("cuda:0") for x in (Q, K, V))
    outs = []
    for ask in (False, True):
        plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, 128)
        if ask:
            plan.device_bytes(4, 1)
        outs.append(binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32))
    torch.cuda.synchronize()
    assert torch.equal(*outs)  # another cut rounds the weights elsewhere


# joined chunks over scattered pages (of one token: a piece per token; of seven: pieces that end inside a block), through the
# call with a static workspace, and captured, with eager calls between the replays
@pytest.mark.parametrize("page_size", [1, 7, 16])
def test_joined_chunks_over_pages_static_and_captured(page_size):
    t = tree(2400, [(37 * i) % 150 for i in range(14)], 64, 16, 128, seed=page_size)
    Q, K, V = wl.make_qkv(t)
    pp, pg, npool, row_of = wl.to_paged(t, page_size, seed=3)
    q, k, v = Q.to("cuda:0"), *(wl.scatter_to_pool(x, row_of, npool * page_size, i).to("cuda:0") for i, x in ((1, K), (2, V)))
    plan = binding.deft_plan_paged(pp, pg, page_size, npool, t.node_tok_len, t.node_parent, t.query_node, 64)
    ref, ws = reference(t, Q, K, V), plan.workspace(t.Hq, t.Hkv, t.d, q.device)
    ws.fill_(0xFF)
    want = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32, workspace=ws)
    torch.cuda.synchronize()
    assert empty_slots(plan, ws, t.Hq, t.d) > 0
    check(want.cpu().numpy().astype(np.float64), ref, strict=False)
    check(stages(plan, q, k, v, ws, one=False).cpu().numpy().astype(np.float64), ref, strict=False)
    o, lib = torch.empty_like(want), binding.load_library()
    assert lib.deft_tree_attn_decode_static(plan.handle, plan.image(t.Hq, t.Hkv, q.device).data_ptr(), q.data_ptr(),
                                            k.data_ptr(), v.data_ptr(), o.data_ptr(), t.Hq, t.Hkv, t.d, 0.0, 1,
                                            torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(o, want)
    graph, got = torch.cuda.CUDAGraph(), torch.empty_like(want)
    with torch.cuda.graph(graph):
        binding.deft_tree_attn_decode(plan, q, k, v, out=got, workspace=ws)
    for scale in (1.0, 0.5, 2.0):
        q.copy_(Q * scale)
        got.zero_()
        ws.fill_(0xFF)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32))


# wide chunks of several pieces in a launch of one round and of more (tests/test_schedule.py counts their workgroups)
ONE_ROUND = [(128, 20, 32, 8), (128, 31, 32, 8), (64, 34, 32, 8)]
ROUNDS = [(128, 35, 32, 8), (128, 50, 32, 8), (128, 34, 64, 8), (64, 40, 32, 8)]


@pytest.mark.parametrize("d,leaves,Hq,Hkv", ONE_ROUND + ROUNDS)
def test_wide_chunks_of_several_pieces_in_a_launch_of_several_rounds(d, leaves, Hq, Hkv):
    # a chunk across the end of a shared node is wide and made of pieces, and resident whatever the launch
    t = wl._finish("rounds", [2977] + [150] * leaves, [-1] + [0] * leaves, list(range(1, leaves + 1)), Hq, Hkv, d, 17)
    Q, K, V = wl.make_qkv(t)
    plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, 128)
    got = binding.deft_tree_attn_decode(plan, Q.cuda(), K.cuda(), V.cuda(), out_dtype=torch.float32)
    check(got.cpu().numpy().astype(np.float64), reference(t, Q, K, V), strict=False)
