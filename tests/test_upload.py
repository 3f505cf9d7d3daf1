"""Plan images as the device finds them: the kernel that fetches them from the staging slots, at sizes around what one of
its workgroups takes, and more uploads than there are slots."""

import numpy as np
import pytest
import torch

from paper_2404_00242_amd import binding

pytestmark = pytest.mark.gpu

GROUP = 16 * 1024  # bytes that one workgroup of the fetch takes
LEN, BEGIN0, SLOT_BASE = 8, 9, 7  # fields of a task's descriptor, which has 16 int32


def forest(n):
    """n trees of one node: every chunk is one node, has one task, and every array of the image grows with n"""
    lens = np.arange(1, n + 1, dtype=np.int32) % 31 + 1
    begins = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int32)
    return binding.deft_plan(begins, lens, np.full(n, -1, np.int32), np.arange(n, dtype=np.int32), int(lens.sum()), 32,
                             binding.DEFT_SPLIT_NODE), begins, lens


def check(plan, begins, lens, img):
    raw = img.cpu().numpy()
    n = len(lens)
    assert (raw[: 4 * n].view(np.int32) == begins).all()  # the image begins with the segments' first rows
    # per segment five arrays of 16-byte words, the query order, records and 64 bytes a task, which are the last
    pad = lambda x: (x + 15) // 16 * 16
    at = 6 * pad(4 * n)
    at = (at + 63) // 64 * 64 + 32 * 4 * n
    tasks = raw[at: at + 64 * n].view(np.int32).reshape(n, 16)
    assert sorted(tasks[:, LEN]) == sorted(lens) and sorted(tasks[:, BEGIN0]) == sorted(begins)
    assert sorted(tasks[:, SLOT_BASE]) == list(range(n))
    return at + 64 * n


@pytest.mark.parametrize("n", [1, 2, 3, 74, 75, 76, 148, 149, 150, 151, 152, 700, 2900])
def test_image_arrives_whole_and_nothing_behind_it(n):
    plan, begins, lens = forest(n)
    size = plan.device_bytes(4, 4)
    img = torch.full((size + 64,), 0xAB, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    assert binding.load_library().deft_plan_upload(plan.handle, 4, 4, img.data_ptr(), size, st) == 0
    end = check(plan, begins, lens, img)
    print(f"\n    image of {end} bytes, {end / GROUP:.2f} workgroups", flush=True)
    assert (img[end:] == 0xAB).all()


def test_image_in_pinned_host_memory():
    """memory that is not the stream's device's takes the copy command; the slots around it are reused as before"""
    st = torch.cuda.current_stream().cuda_stream
    for i in range(20):
        plan, begins, lens = forest(50 + i)
        size = plan.device_bytes(4, 4)
        img = torch.full((size + 64,), 0xAB, dtype=torch.uint8, device="cuda") if i % 2 else \
            torch.full((size + 64,), 0xAB, dtype=torch.uint8, pin_memory=True)
        assert binding.load_library().deft_plan_upload(plan.handle, 4, 4, img.data_ptr(), size, st) == 0
        torch.cuda.synchronize()
        end = check(plan, begins, lens, img)
        assert (img[end:] == 0xAB).all()


def test_more_uploads_than_slots_in_two_streams():
    plans = [forest(40 + 37 * i) for i in range(30)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    x = torch.randn(2048, 2048, device="cuda")
    torch.cuda.synchronize()
    imgs = []
    for i, (plan, begins, lens) in enumerate(plans):
        with torch.cuda.stream(streams[i % 2]):
            x @ x  # work in front of it
            img = torch.empty(plan.device_bytes(4, 4), dtype=torch.uint8, device="cuda")
            st = streams[i % 2].cuda_stream
            assert binding.load_library().deft_plan_upload(plan.handle, 4, 4, img.data_ptr(), img.numel(), st) == 0
            imgs.append(img)
    torch.cuda.synchronize()
    for (plan, begins, lens), img in zip(plans, imgs):
        check(plan, begins, lens, img)


@pytest.mark.parametrize("n", [1, 20, 33, 34, 300])  # images of one part and of several, and around a part's end
def test_captured_upload_replays_its_own_image(n):
    plan, begins, lens = forest(n)
    size = plan.device_bytes(4, 4)
    img = torch.full((size + 64,), 0xAB, dtype=torch.uint8, device="cuda")
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        assert binding.load_library().deft_plan_upload(plan.handle, 4, 4, img.data_ptr(), size, side.cuda_stream) == 0
    del plan
    st, other = torch.cuda.current_stream().cuda_stream, torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    for i in range(4):
        for j in range(9):  # every staging slot holds another plan's image by now
            p, b, l = forest(n + 1 + j)
            assert binding.load_library().deft_plan_upload(p.handle, 4, 4, other.data_ptr(), other.numel(), st) == 0
            check(p, b, l, other)
        img.fill_(0xAB)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        end = check(None, begins, lens, img)
        assert (img[end:] == 0xAB).all()
