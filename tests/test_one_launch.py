"""Whole calls made in one launch: stage 2's workgroups wait for stage 1's inside the kernel, and leave rows that are late to
them.

The same call in two launches, which a workspace without room for the marks gives, is the reference: both sum the same
partial results in fp32, in another order, so outputs differ by a few units of 2^-24 of the attention of |V|."""

import ctypes

import numpy as np
import pytest
import torch

from paper_2404_00242_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


def base_bytes(plan, t):
    return plan.view()["n_slots"] * t.Hq * (t.d + 2) * 4 + 32


def prepared(t, chunk, flags=0):
    Q, K, V = (x.cuda() for x in wl.make_qkv(t))
    plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, chunk, flags)
    return plan, Q, K, V


def two_launches(plan, t, q, k, v):
    ws = torch.empty(base_bytes(plan, t), dtype=torch.uint8, device="cuda")
    return binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32, workspace=ws)


def close(a, b, v):
    # every output is a mean of V; two fp32 summations of n <= 512 terms differ by at most 2 n 2^-24 of the largest |V|
    assert (a - b).abs().max().item() <= 2 * 512 * 2.0**-24 * v.abs().max().item()


def star(root, leaves, length, Hq, Hkv, d, nq=None):
    lens, parents = [root] + [length] * leaves, [-1] + [0] * leaves
    return wl._finish("star", lens, parents, list(range(1, leaves + 1)) if leaves else [0] * (nq or 1), Hq, Hkv, d, 7)


TREES = [
    (star(1, 0, 0, 1, 1, 64), 32),           # one token, one row of output
    (star(40, 0, 0, 4, 4, 128), 32),         # two partials
    (star(29 * 32, 0, 0, 2, 2, 64), 32),     # 29 partials at d = 64, and one more: past what a wave has in flight
    (star(30 * 32, 0, 0, 2, 2, 64), 32),
    (star(16 * 32, 0, 0, 5, 5, 128), 32),    # one wave to a row up to 16 partials, four beyond
    (star(17 * 32, 0, 0, 5, 5, 128), 32),
    (star(70 * 32, 0, 0, 2, 1, 128), 32),    # more partials than a record holds
    (star(300 * 32, 0, 0, 3, 3, 64), 32),    # more than 64 for each of four waves
    (star(64, 3, 20, 7, 1, 128), 32),        # 7 heads: rows that do not fill tiles, waves without a row
    (star(700, 26, 9, 4, 4, 128), 128),      # two tiles
    (star(2000, 33, 40, 8, 2, 128), 512),    # streaming tasks of nine tiles, cut in two
    (star(1500, 20, 60, 16, 2, 64), 256),
    (star(300, 3, 400, 6, 2, 128), 2048),    # chunks of several pieces, both kinds of softmax weights
    (star(900, 6, 200, 8, 4, 128), 96),
    (star(96, 0, 0, 8, 2, 128, nq=17), 32),  # queries on the root alone
    (star(32 * 32, 0, 0, 4, 1, 128), 32),    # 32 and 33 partials at d = 128, 64 and 65 at d = 64: a batch and one more
    (star(33 * 32, 0, 0, 4, 1, 128), 32),
    (star(64 * 32, 0, 0, 4, 1, 64), 32),
    (star(65 * 32, 0, 0, 4, 1, 64), 32),
    (star(200, 7, 30, 4, 4, 128), 64),       # 28, 32, 36 and 64 rows: every wave of stage 2 has one, or some two
    (star(200, 8, 30, 4, 1, 128), 64),
    (star(200, 9, 30, 4, 2, 64), 64),
    (star(200, 16, 30, 4, 2, 128), 64),
]


def batches(t, plan):
    """what the rule for one launch goes by, next to the sizes of K and V: rows for 32 waves, partial results in flight"""
    parts = int(np.diff(plan.view()["q_part_ptr"]).max())
    return -(-t.nq * t.Hq // 32) * -(-parts // (32 if t.d == 128 else 64))


def test_trees_are_on_both_sides_of_the_rule():
    n = [batches(t, prepared(t, chunk)[0]) for t, chunk in TREES]
    assert sum(x == 1 for x in n) >= 8 and sum(x == 2 for x in n) >= 4 and sum(x > 2 for x in n) >= 4


@pytest.mark.parametrize("i", range(len(TREES)))
def test_equals_two_launches(i):
    t, chunk = TREES[i]
    plan, q, k, v = prepared(t, chunk)
    want = two_launches(plan, t, q, k, v)
    ws = torch.empty(plan.workspace_bytes(t.Hq, t.Hkv, t.d), dtype=torch.uint8, device="cuda")
    for fill in (0, 0xFF, 0x5A):  # whatever the workspace holds
        ws.fill_(fill)
        got = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32, workspace=ws)
        close(got, want, v)
        again = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32, workspace=ws)
        assert torch.equal(got, again)
    b16 = binding.deft_tree_attn_decode(plan, q, k, v, workspace=ws)
    assert torch.equal(b16, got.to(torch.bfloat16))
    # the partial results are there for a stage 2 called apart
    out = torch.empty_like(got)
    img = plan.image(t.Hq, t.Hkv, "cuda")
    rc = binding.load_library().deft_stage2_global_reduction(
        plan.handle, img.data_ptr(), out.data_ptr(), t.Hq, t.Hkv, t.d, 0.0, binding.DEFT_OUT_F32, ws.data_ptr(), ws.numel(),
        torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    close(out, want, v)


def test_queries_without_tokens_and_precise_weights():
    t = wl._finish("empty", [0, 70, 0, 33], [-1, -1, 1, 1], [0, 2, 3, 0], 4, 2, 128, 3)
    for flags in (0, binding.DEFT_PRECISE_WEIGHTS):
        plan, q, k, v = prepared(t, 32, flags)
        got = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32)
        close(got, two_launches(plan, t, q, k, v), v)
        assert not got[[0, 3]].any()


def test_workspace_shared_by_plans_of_other_layouts():
    a, b = star(640, 4, 33, 8, 2, 128), star(333, 11, 17, 4, 4, 64)
    plans = [prepared(t, 64) for t in (a, b)]
    ws = torch.empty(max(p.workspace_bytes(t.Hq, t.Hkv, t.d) for (p, *_), t in zip(plans, (a, b))), dtype=torch.uint8, device="cuda")
    want = [two_launches(p, t, q, k, v) for (p, q, k, v), t in zip(plans, (a, b))]
    for _ in range(4):
        for (p, q, k, v), w in zip(plans, want):
            close(binding.deft_tree_attn_decode(p, q, k, v, out_dtype=torch.float32, workspace=ws), w, v)


def test_two_streams_with_a_workspace_each():
    t = star(900, 4, 50, 8, 2, 128)
    plan, q, k, v = prepared(t, 64)
    want = two_launches(plan, t, q, k, v)
    plan.image(t.Hq, t.Hkv, "cuda")
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    spaces = [torch.empty(plan.workspace_bytes(t.Hq, t.Hkv, t.d), dtype=torch.uint8, device="cuda") for _ in streams]
    outs = [[torch.empty_like(want) for _ in range(20)] for _ in streams]
    for i in range(20):
        for st, ws, o in zip(streams, spaces, outs):
            binding.deft_tree_attn_decode(plan, q, k, v, out=o[i], workspace=ws, stream=st)
    torch.cuda.synchronize()
    for o in outs:
        for x in o:
            close(x, want, v)


def test_captured_calls_replayed_with_eager_calls_between():
    t = star(600, 4, 90, 8, 2, 128)
    plan, q, k, v = prepared(t, 64)
    ws = torch.empty(plan.workspace_bytes(t.Hq, t.Hkv, t.d), dtype=torch.uint8, device="cuda")
    out = torch.zeros((t.nq, t.Hq, t.d), dtype=torch.float32, device="cuda")
    binding.deft_tree_attn_decode(plan, q, k, v, out=out, workspace=ws)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        for _ in range(2):
            binding.deft_tree_attn_decode(plan, q, k, v, out=out, workspace=ws, stream=side)
    for i in range(4):
        q.normal_()  # new inputs: a replay that read the partial results of the one before would show
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        close(out, two_launches(plan, t, q, k, v), v)
        if i == 1:
            binding.deft_tree_attn_decode(plan, q, k, v, workspace=ws)


@pytest.mark.parametrize("dtype", [None, torch.float32])
def test_output_of_one_query_from_a_wider_tensor_has_plain_strides(dtype):
    t = star(200, 0, 0, 8, 2, 64)
    plan, q, k, v = prepared(t, 64)
    wide = torch.cat([q, q, q], 1)[:, : t.Hq]
    assert wide.is_contiguous() and wide.stride(0) == 3 * t.Hq * t.d
    got = binding.deft_tree_attn_decode(plan, wide, k, v, out_dtype=dtype)
    assert got.stride() == (t.Hq * t.d, t.d, 1)
    assert torch.equal(got, binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=dtype))


class Activation(torch.Tensor):
    pass


@pytest.mark.parametrize("dtype", [None, torch.float32])
def test_output_is_a_plain_tensor_whatever_q_is(dtype):
    t = star(200, 4, 30, 8, 2, 64)
    plan, q, k, v = prepared(t, 64)
    want = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=dtype)
    for x in (q.as_subclass(Activation), torch.nn.Parameter(q)):
        got = binding.deft_tree_attn_decode(plan, x, k, v, out_dtype=dtype)
        assert type(got) is torch.Tensor and not got.requires_grad and torch.equal(got, want)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("token", [0, 2047, 1000])
def test_infinite_value_in_any_partial_result(token, d):
    t = star(2048, 0, 0, 4, 4, d)  # whole blocks, a path long enough for single-term weights
    plan, q, k, v = prepared(t, 128)
    want = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32)
    v[token, :, 5] = float("inf")
    got = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32)
    assert (got[..., 5] == float("inf")).all()
    keep = [i for i in range(d) if i != 5]
    assert torch.equal(got[..., keep], want[..., keep])


@pytest.mark.parametrize("i", [0, 3, 8, 15])
def test_captured_call_takes_two_launches(i):
    # replays have no host work to save, and all of them would write one ticket into the marks
    t, chunk = TREES[i]
    assert batches(t, prepared(t, chunk)[0]) == 1
    plan, q, k, v = prepared(t, chunk)
    ws = torch.empty(plan.workspace_bytes(t.Hq, t.Hkv, t.d), dtype=torch.uint8, device="cuda")
    out = torch.zeros((t.nq, t.Hq, t.d), dtype=torch.float32, device="cuda")
    binding.deft_tree_attn_decode(plan, q, k, v, out=out, workspace=ws)
    torch.cuda.synchronize()
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g, stream=side):
        binding.deft_tree_attn_decode(plan, q, k, v, out=out, workspace=ws, stream=side)
    n = ctypes.c_size_t(0)
    assert binding.load_library().hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert n.value == 2
    g.instantiate()
    want = two_launches(plan, t, q, k, v)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


def call_with_polls(plan, t, q, k, v, out, ws, polls, stream=None):
    """the call with another limit to the wait inside the kernel (deft_internal.h)"""
    img = plan.image(t.Hq, t.Hkv, "cuda")
    st = (stream or torch.cuda.current_stream()).cuda_stream
    flags = binding.DEFT_OUT_F32 if out.dtype == torch.float32 else binding.DEFT_OUT_BF16
    p = ctypes.c_void_p
    assert binding.load_library().deft_decode_polls(
        plan.handle, p(img.data_ptr()), p(q.data_ptr()), p(k.data_ptr()), p(v.data_ptr()), p(out.data_ptr()), t.Hq, t.Hkv, t.d,
        ctypes.c_float(0.0), flags, p(ws.data_ptr()), ctypes.c_size_t(ws.numel()), p(st), polls) == 0


@pytest.mark.parametrize("i", [0, 1, 4, 5, 8, 12, 13, 16, 18, 20, 22])
def test_rows_that_are_late_are_merged_by_stage_1(i):
    t, chunk = TREES[i]
    plan, q, k, v = prepared(t, chunk)
    ws = torch.zeros(plan.workspace_bytes(t.Hq, t.Hkv, t.d), dtype=torch.uint8, device="cuda")
    want = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32, workspace=ws)
    for polls in (1, 1, 2, 3, 4, 6, 9, 14):  # from a wait that is given up at once to one that may just do
        out = torch.full_like(want, float("nan"))
        ws.zero_()
        call_with_polls(plan, t, q, k, v, out, ws, polls)
        assert torch.equal(out, want), polls


@pytest.mark.parametrize("t,chunk,one", [
    (star(256, 4, 32, 4, 4, 64), 0, True),
    (star(8191, 0, 0, 32, 8, 128), 256, True),       # 32 MiB of K and V, 32 partial results
    (star(10600, 0, 0, 32, 8, 128), 352, False),     # 41 MiB
    (star(4000, 0, 0, 16, 8, 128), 64, True),        # 63 partial results, 15.6 MiB
    (star(4100, 0, 0, 16, 8, 128), 96, False),       # 43, 16.02 MiB
    (star(4160, 0, 0, 8, 1, 128), 64, False),        # 65
    (star(8192, 0, 0, 8, 1, 64), 64, True),          # 128 at d = 64
    (star(1000, 8, 50, 4, 1, 128), 64, True),        # 32 rows of output, 18 partial results
    (star(1000, 11, 50, 3, 1, 128), 64, False),      # 33 rows
    (star(1000, 9, 50, 4, 4, 128), 64, False),       # 36 rows
    (star(2000, 9, 50, 4, 4, 64), 64, False),        # 34 partial results at d = 64
    (star(1500, 12, 50, 4, 4, 64), 64, True),        # 26
    (star(900, 1, 100, 64, 8, 128), 128, True),      # 64 rows, 9 partial results
    (star(200, 17, 20, 4, 4, 128), 64, False),       # 68 rows
])
def test_which_calls_take_one_launch(t, chunk, one):
    # one launch writes its ticket into the marks, two leave them as they were
    plan, q, k, v = prepared(t, chunk)
    rows = plan.view()["n_slots"] * t.Hq
    ws = torch.full((plan.workspace_bytes(t.Hq, t.Hkv, t.d),), 0xFF, dtype=torch.uint8, device="cuda")
    got = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32, workspace=ws)
    marks = ws[4 * (rows * t.d + (2 * rows + 3) // 4 * 4):][: 16 * rows].view(torch.int64).view(-1, 2)[:, 1]
    assert bool((marks != -1).any()) == one
    close(got, two_launches(plan, t, q, k, v), v)
