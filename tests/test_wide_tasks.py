"""Wide tasks: those of three row tiles, which stream where they are many.  Same tolerance as tests/test_gpu_parity.py."""

import numpy as np
import pytest
import torch

from paper_2404_00242_amd import binding, workloads as wl

from .test_short_chunks import check, reference


def star(root, leaves, Hq, Hkv, seed, d=128):
    lens = [root] + [1 + 2 * (i % 3) for i in range(leaves)]
    return wl._finish("wide", lens, [-1] + [0] * leaves, list(range(1, leaves + 1)), Hq, Hkv, d, seed)


# three-tile tasks that stream (more than 256) or are resident; tokens that fill no block and rows that fill no
# tile (heads x queries a multiple of 16 or not)
@pytest.mark.gpu
@pytest.mark.parametrize("root,leaves,Hq,Hkv", [(2048, 48, 16, 16), (2080, 45, 16, 16), (2049, 33, 17, 17), (4095, 41, 8, 8), (4224, 48, 8, 8)])
def test_three_tile_tasks(root, leaves, Hq, Hkv):
    t = star(root, leaves, Hq, Hkv, leaves)
    Q, K, V = wl.make_qkv(t)
    for chunk in (96, 128, 256):
        plan = binding.deft_plan(t.node_tok_begin, t.node_tok_len, t.node_parent, t.query_node, t.ntok, chunk)
        got = binding.deft_tree_attn_decode(plan, Q.cuda(), K.cuda(), V.cuda(), out_dtype=torch.float32)
        check(got.cpu().numpy().astype(np.float64), reference(t, Q, K, V), strict=False)
