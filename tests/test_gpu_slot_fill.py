"""Background slot fill (moe_load_expert) beside running forwards, then the map switch:
forwards before the switch are undisturbed, forwards after it match the oracle on the new placement."""
import numpy as np
import pytest

from workloads import MoEWorkload, relayout_maps

pytestmark = pytest.mark.gpu

MID = dict(hidden=512, inter=264, n_experts=32, top_k=4, n_slots=16, n_local=16,
           act_dtype="bf16", router_dtype="f32", gate="softmax", seed=31)


def test_fill_beside_forwards_then_switch():
    import torch
    from gpu_util import Case, tensor_to_host, check_routing, check_bookkeeping, check_output
    wl = MoEWorkload(name="fill", tokens=900, **MID)
    map_a, map_b = relayout_maps(wl)                     # phase A: experts 0..7 in slots 0..7; B adds 8..15 shuffled
    case = Case(wl, expert_map=map_a)
    dev = case.x_dev.device
    serve = torch.cuda.current_stream(dev)
    copy = torch.cuda.Stream(device=dev)
    before = case.run()
    # sources staged on the device (the landing buffers of a peer transfer)
    src = {e: (case.layer.upload(case.inp["w13_experts"][e]), case.layer.upload(case.inp["w2_experts"][e]))
           for e in range(8, 16)}
    torch.cuda.synchronize()
    alloc0 = torch.cuda.memory_stats()["allocation.all.allocated"]
    outs = []
    for e in range(8, 16):
        outs.append(case.layer.forward(case.x_dev, shared_range=wl.shared_range))           # serving goes on ...
        case.layer.load_expert_async(int(map_b[e]), src[e][0], src[e][1], copy, serve, copy_blocks=8)  # ... beside the fill
    outs.append(case.layer.forward(case.x_dev, shared_range=wl.shared_range))
    case.place(map_b, upload=False)                      # switch: waits (on the stream) for all eight fills
    after = case.layer.forward(case.x_dev, shared_range=wl.shared_range)
    torch.cuda.synchronize()
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == alloc0 + len(outs) + 1   # only the output tensors
    for o in outs:                                       # forwards under the old map never saw the fills
        np.testing.assert_array_equal(tensor_to_host(o), before)
    np.testing.assert_array_equal(tensor_to_host(case.layer.w13), case.w13_pool)             # the pool is the new placement's
    np.testing.assert_array_equal(tensor_to_host(case.layer.w2), case.w2_pool)
    v = case.layer.view(wl.tokens)
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, wl.tokens, wl.shared_range)
    check_output(case, tensor_to_host(after), ids)
    assert v["counts"][8:].sum() > 0                     # the new slots are in use


def test_fill_of_a_live_slot_and_same_stream_are_rejected():
    import torch
    from gpu_util import Case
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="fill_err", tokens=16, **MID)
    map_a, _ = relayout_maps(wl)
    case = Case(wl, expert_map=map_a)
    dev = case.x_dev.device
    copy = torch.cuda.Stream(device=dev)
    serve = torch.cuda.current_stream(dev)
    w13 = case.layer.upload(case.inp["w13_experts"][9])
    w2 = case.layer.upload(case.inp["w2_experts"][9])
    with pytest.raises(B.MoEError, match="active map"):
        case.layer.load_expert_async(3, w13, w2, copy, serve)           # slot 3 holds expert 3
    with pytest.raises(B.MoEError, match="differ"):
        case.layer.load_expert_async(12, w13, w2, serve, serve)
    with pytest.raises(B.MoEError, match="outside"):
        case.layer.load_expert_async(16, w13, w2, copy, serve)
    case.layer.load_expert_async(12, w13, w2, copy, serve)               # a free slot is fine
    torch.cuda.synchronize()


def test_copy_blocks_throttle_a_fill():
    """A workgroup of a throttled fill is 256 threads with one 16-byte piece on its way each: 4 KB per memory round trip,
    9 GB/s where that takes 430 ns.  One of them may not move 16 GB/s (250 ns); without a throttle a fill moves much more.
    Any number of workgroups copies whole slots, also where they divide unevenly."""
    import torch
    from gpu_util import Case
    wl = MoEWorkload(name="fill_rate", tokens=16, hidden=1024, inter=520, n_experts=8, top_k=2, n_slots=8, n_local=4,
                     act_dtype="bf16", router_dtype="f32", gate="softmax", seed=33)
    case = Case(wl)
    copy = torch.cuda.Stream()
    w13, w2 = (torch.randint(-2**15, 2**15, t.shape, dtype=torch.int16, device=t.device) for t in (case.layer.w13[0], case.layer.w2[0]))
    nbytes = 2 * (w13.numel() + w2.numel())
    rate = {}
    for blocks in (1, 0, 3, 1000):
        for _ in range(2):                                   # the second one is timed
            case.layer.w13[6].zero_(), case.layer.w2[6].zero_()
            torch.cuda.synchronize()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(copy)
            case.layer.load_expert_async(6, w13, w2, copy, copy_blocks=blocks)
            b.record(copy)
            torch.cuda.synchronize()
            rate[blocks] = nbytes / (a.elapsed_time(b) * 1e6)
            assert torch.equal(case.layer.w13[6], w13) and torch.equal(case.layer.w2[6], w2)
    assert rate[1] < 16 < rate[0], rate
