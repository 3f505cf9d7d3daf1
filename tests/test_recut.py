"""Wide chunks cut anew, one long task to a compute unit: the schedule on the host under the sanitizers
(tests/sanitize/recut_driver.cpp), which calls use it, and calls on both sides of its lines.  Same tolerance as
tests/test_gpu_parity.py."""

import os
import shutil

import numpy as np
import pytest
import torch

from paper_2404_00242_amd import binding, workloads as wl

from .test_sanitizers import ROOT, SAN, run
from .test_gpu_parity import reference_abs_v
from .test_short_chunks import check, empty_slots, reference, stages
from .test_upload_errors import fake, needs_gxx, run as run_faked  # noqa: F401


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_recut_sets_of_random_plans(tmp_path):
    exe = str(tmp_path / "recut_driver")
    csrc = os.path.join(ROOT, "paper_2404_00242_amd", "csrc")
    run(["g++", "-std=c++17", *SAN, "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "deft_plan.cpp"),
         os.path.join(ROOT, "tests", "sanitize", "recut_driver.cpp"), "-lpthread", "-o", exe])
    assert "recut sets checked" in run([exe])


# (root, leaves, Hq, Hkv, chunk): us a call as planned and cut anew.  A run more costs Hkv workgroups for every eight row tiles, and
# where that is many the launch would stop well short of the compute units, or a few long tasks would end it.
SLOWER = [(15589, [1] * 35, 64, 8, 768),  # 39.9, 46.8
          (15733, [1] * 34, 64, 8, 768),  # 39.9, 46.7
          (11083, [1] * 50, 64, 8, 768),  # 39.3, 44.4
          (8000, [1] * 64, 128, 16, 1024),  # 61.8, 67.2
          (6000, [1] * 130, 32, 32, 768),  # 50.7, 53.0
          (4096, [0] * 280, 64, 8, 256)]  # 93.6, 98.3
FASTER = [(12345, [1] * 26, 32, 8, 256),  # 25.0, 22.4
          (4000, [1] * 51, 32, 8, 160),  # 26.6, 22.2
          (9000, [1] * 81, 16, 16, 256),  # 34.0, 25.1
          (7853, [30] * 35, 64, 8, 384)]  # 44.6, 33.1


# (root, leaves, Hq, Hkv, d, chunk) of the calls below, those that are cut anew (with d = 128) in each split
CALLED = [(12345, [1] * 26, 32, 8, 128, 256), (4000, [1] * 51, 32, 8, 128, 160), (6017, [300] + [2, 1, 3] * 8, 28, 4, 128, 96),
          (5120, [0, 1, 2] * 11, 32, 4, 128, 128), (9000, [1] * 81, 16, 16, 128, 256), (9000, [1] * 81, 16, 16, 64, 256),
          (9040, [0, 1, 2] * 11, 32, 8, 128, 128), (12017, [300] + [2, 1, 3] * 8, 28, 4, 128, 96),
          (1000, [1] * 96, 64, 64, 128, 160)]
CUT = {(12345, "flatten"), (12345, "balanced"), (4000, "flatten"), (9000, "flatten"), (9000, "balanced"), (9040, "flatten"),
       (9040, "balanced"), (12017, "flatten"), (12017, "balanced")}


def flags_of(mode, G):
    return binding.SPLIT_MODES[mode] | (binding.rows_per_query(G) if mode == "balanced" else 0)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_cut_anew_only_where_the_launch_ends_earlier(tmp_path):
    exe = str(tmp_path / "star_driver")
    csrc = os.path.join(ROOT, "paper_2404_00242_amd", "csrc")
    run(["g++", "-std=c++17", *SAN, "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "deft_plan.cpp"),
         os.path.join(ROOT, "tests", "sanitize", "star_driver.cpp"), "-lpthread", "-o", exe])
    for cases, route in ((SLOWER, "as planned"), (FASTER, "cut anew")):
        for root, leaves, Hq, Hkv, chunk in cases:
            assert run([exe, *map(str, (Hq, Hkv, chunk, 0, root, *leaves))]).startswith(route), (root, len(leaves), Hq, Hkv)
    for root, leaves, Hq, Hkv, _, chunk in CALLED:
        for mode in ("flatten", "balanced"):
            route = "cut anew" if (root, mode) in CUT else "as planned"
            assert run([exe, *map(str, (Hq, Hkv, chunk, flags_of(mode, Hq // Hkv), root, *leaves))]).startswith(route), (root, mode)


CALLS = """
class Launches(ctypes.Structure):
    _fields_ = Fake._fields_ + [("grid", ctypes.c_int32 * 16), ("kernel", ctypes.c_void_p * 16)]
fake = Launches.in_dll(fake_lib, "fake")
def star(root, leaves, chunk):
    lens = np.array([root] + [1] * leaves, np.int32)
    begins = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int32)
    return binding.deft_plan(begins, lens, np.array([-1] + [0] * leaves, np.int32), np.arange(1, leaves + 1, dtype=np.int32),
                             int(lens.sum()), chunk)
def memory(n):
    b = np.zeros(n + 16, np.uint8)
    return b[-b.ctypes.data % 16:][:n]
def image_of(plan, Hq, Hkv):
    img = memory(plan.device_bytes(Hq, Hkv))
    assert lib.deft_plan_upload(plan.handle, Hq, Hkv, img.ctypes.data, img.size, STREAM) == 0
    return img
def launches(call):
    fake.launches = 0
    assert call() == 0
    return list(zip(fake.grid[:fake.launches], fake.kernel[:fake.launches]))
x = memory(4096)  # q, k, v and the output: nothing reads them here
def decode(plan, img, Hq, Hkv, d):
    ws = memory(plan.workspace_bytes(Hq, Hkv, d))
    return launches(lambda: lib.deft_tree_attn_decode(plan.handle, img.ctypes.data, *[x.ctypes.data] * 4, Hq, Hkv, d, 0.0, 1,
                                                      ws.ctypes.data, ws.size, STREAM))
"""


@needs_gxx
def test_cut_anew_only_for_the_kv_heads_it_was_made_for(fake):  # noqa: F811
    # 49 chunks of up to 256 tokens with seven row tiles each, or eight runs of 1568 for 32 KV heads
    run_faked(fake, CALLS + """
plan = star(12345, 26, 128)
img = image_of(plan, 128, 32)
assert decode(plan, img, 128, 32, 128)[0][0] < 512
assert decode(plan, img, 8, 2, 128)[0][0] >= 2 * 49
assert decode(plan, img, 128, 32, 128)[0][0] < 512
""")


@needs_gxx
def test_only_a_stage_2_that_may_find_empty_slots_looks_for_them(fake):  # noqa: F811
    # called apart after a whole call with d = 128 it may; with d = 64 or other KV heads nothing is cut anew (nor joined, in
    # chunks of 160)
    run_faked(fake, CALLS + """
plan = star(6500, 96, 160)
img = image_of(plan, 32, 32)
def stage2(Hq, Hkv, d):
    ws = memory(plan.workspace_bytes(Hq, Hkv, d))
    return launches(lambda: lib.deft_stage2_global_reduction(plan.handle, img.ctypes.data, x.ctypes.data, Hq, Hkv, d, 0.0, 1,
                                                             ws.ctypes.data, ws.size, STREAM))
assert decode(plan, img, 32, 32, 128)[0][0] != decode(plan, img, 32, 32, 64)[0][0]
for (Hq, Hkv, d), same in (((32, 32, 128), False), ((32, 32, 64), True), ((16, 16, 128), True)):
    assert (stage2(Hq, Hkv, d) == decode(plan, img, Hq, Hkv, d)[1:]) == same, (Hq, Hkv, d)
""")


def star(root, leaves, Hq, Hkv, d, seed):
    return wl._finish("recut", [root] + leaves, [-1] + [0] * len(leaves), list(range(1, len(leaves) + 1)), Hq, Hkv, d, seed)


# one-token leaves in the root's last chunk, in chunks of their own, a first leaf that fills it, and leaves without a token, whose
# queries see nothing of the rest; rows that fill no tile, several tasks to a run, roots that end inside a block; d = 64, which
# keeps the plan's chunks, as do two-term weights.  The stages called apart after a whole call find the slots
# that it left empty.
@pytest.mark.gpu
@pytest.mark.parametrize("root,leaves,Hq,Hkv,d,chunk", CALLED)
def test_recut_calls(root, leaves, Hq, Hkv, d, chunk):
    t = star(root, leaves, Hq, Hkv, d, root)
    Q, K, V = wl.make_qkv(t)
    ref = reference(t, Q, K, V)
    q, k, v = Q.cuda(), K.cuda(), V.cuda()
    lib = binding.load_library()
    short = dict(abs_v=reference_abs_v(t, Q, K, V), two_term=True) if root + max(leaves) < 1024 else {}
    for mode in ("flatten", "balanced"):
        plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, chunk,
                                 flags_of(mode, Hq // Hkv))
        got = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32)
        check(got.cpu().numpy().astype(np.float64), ref, strict=False, **short)
        ws, o = plan.workspace(Hq, Hkv, d, q.device), torch.empty_like(got)
        st = torch.cuda.current_stream().cuda_stream
        img = plan.image(Hq, Hkv, q.device)
        assert lib.deft_stage2_global_reduction(plan.handle, img.data_ptr(), o.data_ptr(), Hq, Hkv, d, 0.0, binding.DEFT_OUT_F32,
                                                ws.data_ptr(), ws.numel(), st) == 0
        check(o.cpu().numpy().astype(np.float64), ref, strict=False, **short)


# A call whose chunks are cut anew is as near to 64 bits as the plan's chunks are: nine row tiles that are held in registers stay
# there (streamed they are 1.27 times as far), and a long stream starts a new reference where each chunk would have begun (with one
# reference in the place of four to six it is 1.05 times as far).  The errors of two ways to sum the same 272 x 8 and more rows
# differ by about 1 % of themselves (100 trees: 0.995 times, 1.01 at most).
@pytest.mark.gpu
@pytest.mark.parametrize("root,leaves,Hq,Hkv,chunk", [(5000, 34, 32, 8, 256), (6400, 96, 32, 32, 160), (9600, 34, 32, 8, 160)])
def test_cut_anew_is_as_precise(root, leaves, Hq, Hkv, chunk):
    t = star(root, [1] * leaves, Hq, Hkv, 128, root)
    Q, K, V = wl.make_qkv(t)
    ref = reference(t, Q, K, V)
    q, k, v = Q.cuda(), K.cuda(), V.cuda()
    plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, chunk)
    whole = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32)
    apart = stages(plan, q, k, v, plan.workspace(Hq, Hkv, 128, q.device))
    err = [np.linalg.norm(o.cpu().numpy().astype(np.float64) - ref) for o in (whole, apart)]
    assert err[0] <= 1.025 * err[1], err


# two wide roots, of long and of short paths (bf16 weights, cut anew, and two-term weights in one launch), as they lie and over pages in order; through
# the call with a static workspace, and captured, with eager calls between the replays
@pytest.mark.gpu
@pytest.mark.parametrize("page", [0, 16])
def test_recut_mixed_weights_static_and_captured(page):
    Hq, Hkv = 32, 8
    t = wl._finish("mixed", [9000, 250] + [1] * 70, [-1, -1] + [0] * 40 + [1] * 30, list(range(2, 72)), Hq, Hkv, 128, 5)
    Q, K, V = wl.make_qkv(t)
    ref, q = reference(t, Q, K, V), Q.cuda()
    if page:
        pp, pg, npool, row_of = wl.to_paged(t, page, shuffle=False)
        k, v = (wl.scatter_to_pool(x, row_of, npool * page, i).cuda() for i, x in ((1, K), (2, V)))
        plan = binding.deft_plan_paged(pp, pg, page, npool, t.node_tok_len, t.node_parent, t.query_node, 128)
    else:
        k, v = K.cuda(), V.cuda()
        plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, 128)
    ws = plan.workspace(Hq, Hkv, 128, q.device)
    ws.fill_(0xFF)  # NaN: every slot that stage 2 reads has to be written by stage 1
    want = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32, workspace=ws)
    check(want.cpu().numpy().astype(np.float64), ref, strict=False)
    # runs of more than two of the plan's chunks, which joining does not make
    assert 2 * empty_slots(plan, ws, Hq, 128) > Hq * plan.view()["n_slots"]
    o, lib = torch.empty_like(want), binding.load_library()
    assert lib.deft_tree_attn_decode_static(plan.handle, plan.image(Hq, Hkv, q.device).data_ptr(), q.data_ptr(), k.data_ptr(),
                                            v.data_ptr(), o.data_ptr(), Hq, Hkv, 128, 0.0, 1, torch.cuda.current_stream().cuda_stream) == 0
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


# Inf and NaN in a leaf's V go no further than the two stages carry them chunk by chunk
@pytest.mark.gpu
def test_recut_infinities_of_a_leaf(root=4000, leaves=51, Hq=32, Hkv=8, chunk=160):
    t = star(root, [1] * leaves, Hq, Hkv, 128, 3)
    Q, K, V = wl.make_qkv(t)
    V[root + 4, :, 7], V[root + 20, :, 9] = float("inf"), float("nan")
    q, k, v = Q.cuda(), K.cuda(), V.cuda()
    plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, chunk)
    got = binding.deft_tree_attn_decode(plan, q, k, v, out_dtype=torch.float32).cpu().numpy()
    apart = stages(plan, q, k, v, plan.workspace(Hq, Hkv, 128, q.device)).cpu().numpy()
    assert not np.isfinite(got[4, :, 7]).any() and not np.isfinite(got[20, :, 9]).any()
    assert (np.isfinite(got) >= np.isfinite(apart)).all()


# New references on the way (RowState) where the scores fall, rise or jump by far more than one reference may go down: 98 bits over
# the root, and back and forth by 40 every 200 tokens.  A weight rounded to bf16 is off by at most 2^-9 of itself, in numerator and
# denominator: |err| <= 2^-8 attention(|V|), and 1e-5 for what is summed in fp32.
@pytest.mark.gpu
@pytest.mark.parametrize("course", ["falls", "rises", "jumps"])
def test_recut_scores_that_drift(course, root=4000, leaves=51, Hq=32, Hkv=8, chunk=160):
    t = star(root, [1] * leaves, Hq, Hkv, 128, 11)
    Q, K, V = wl.make_qkv(t)
    at = torch.arange(t.ntok) / root
    drift = {"falls": 3 - 6 * at, "rises": 6 * at - 3, "jumps": 2.5 * ((torch.arange(t.ntok) // 200) % 2)}[course]
    Q = (1 + Q.float() / 16).to(torch.bfloat16)
    K = (K.float() / 4 + drift[:, None, None]).to(torch.bfloat16)
    plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, chunk)
    got = binding.deft_tree_attn_decode(plan, Q.cuda(), K.cuda(), V.cuda(), out_dtype=torch.float32)
    err = np.abs(got.cpu().numpy().astype(np.float64) - reference(t, Q, K, V))
    assert (err <= 2.0 ** -8 * reference_abs_v(t, Q, K, V) + 1e-5).all()
