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
    (The source has to come from memory: out of an XCD's L2, where a fill before it has left it, a round trip takes 250 to 265 ns,
    15.2 to 16.2 GB/s, on the limit; a write of 512 MB, twice what the caches hold, puts it out of them: 8.8 to 9.3.)  Any number
    of workgroups copies whole slots, also where they divide unevenly."""
    import torch
    from gpu_util import Case
    wl = MoEWorkload(name="fill_rate", tokens=16, hidden=1024, inter=520, n_experts=8, top_k=2, n_slots=8, n_local=4,
                     act_dtype="bf16", router_dtype="f32", gate="softmax", seed=33)
    case = Case(wl)
    copy = torch.cuda.Stream()
    w13, w2 = (torch.randint(-2**15, 2**15, t.shape, dtype=torch.int16, device=t.device) for t in (case.layer.w13[0], case.layer.w2[0]))
    nbytes = 2 * (w13.numel() + w2.numel())
    rate, elsewhere = {}, torch.empty(1 << 27, dtype=torch.int32, device=w13.device)
    for blocks in (1, 0, 3, 1000):
        for _ in range(2):                                   # the second one is timed
            case.layer.w13[6].zero_(), case.layer.w2[6].zero_(), elsewhere.fill_(blocks)
            torch.cuda.synchronize()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(copy)
            case.layer.load_expert_async(6, w13, w2, copy, copy_blocks=blocks)
            b.record(copy)
            torch.cuda.synchronize()
            rate[blocks] = nbytes / (a.elapsed_time(b) * 1e6)
            assert torch.equal(case.layer.w13[6], w13) and torch.equal(case.layer.w2[6], w2)
    assert rate[1] < 16 < rate[0], rate


@pytest.mark.parametrize("copy_blocks", [0, 1])
def test_fills_on_two_copy_streams_and_refills(copy_blocks):
    """Fills alternate between two copy streams (a stream's event stands for its latest fill) while forwards run; the switch
    waits for all of them.  Then a second round of fills into the slots that this switch freed, the streams in the other order,
    so that the events of the first round are recorded again for other streams."""
    import torch
    from gpu_util import Case, tensor_to_host, check_routing, check_output
    wl = MoEWorkload(name="fill2", tokens=600, **dict(MID, n_experts=24, n_slots=24, n_local=24))
    order = np.random.Generator(np.random.PCG64(9)).permutation(24)
    def placement(experts_in):                               # {expert: slot}
        m = np.full(24, -1, np.int32)
        for e, s in experts_in.items():
            m[e] = s
        return m
    first = {e: int(order[e]) for e in range(8)}
    second = {e: int(order[e]) for e in range(8, 16)}       # into free slots, then the first ones leave
    third = {e: int(order[e - 16]) for e in range(16, 24)}  # into the slots the first ones left
    case = Case(wl, expert_map=placement(first))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    src = {e: (case.layer.upload(case.inp["w13_experts"][e]), case.layer.upload(case.inp["w2_experts"][e])) for e in range(8, 24)}
    torch.cuda.synchronize()
    for new, turn in ((second, 0), (third, 1)):
        for i, (e, s) in enumerate(new.items()):
            case.layer.forward(case.x_dev)
            case.layer.load_expert_async(s, src[e][0], src[e][1], streams[(i + turn) % 2], copy_blocks=copy_blocks)
        case.place(placement(new), upload=False)
        out = case.layer.forward(case.x_dev)
        torch.cuda.synchronize()
        for e, s in new.items():
            np.testing.assert_array_equal(tensor_to_host(case.layer.w13[s]), case.w13_pool[s])
            np.testing.assert_array_equal(tensor_to_host(case.layer.w2[s]), case.w2_pool[s])
        v = case.layer.view(wl.tokens)
        ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
        check_output(case, tensor_to_host(out), ids)


def test_fills_from_two_threads_on_their_own_streams_under_one_handle():
    """The handle of the per-thread stream (2) names another stream in every thread: the event recorded again for the second
    thread's short fill must still stand for the first thread's long one."""
    import threading
    import torch
    from gpu_util import Case, tensor_to_host
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="fill_threads", tokens=64, **dict(MID, hidden=1024, inter=1024, n_experts=8, n_slots=8, n_local=8))
    case = Case(wl, expert_map=np.array([0, 1, 2, 3, -1, -1, -1, -1], np.int32))
    src = {e: (case.layer.upload(case.inp["w13_experts"][e]), case.layer.upload(case.inp["w2_experts"][e])) for e in (4, 5)}
    serve = torch.cuda.current_stream()
    case.layer.forward(case.x_dev)
    torch.cuda.synchronize()
    done, errors = threading.Event(), []

    def fill(e, blocks, filled):
        try:
            torch.cuda.set_device(0)
            B.moe_load_expert(case.layer.handle, e, src[e][0].data_ptr(), src[e][1].data_ptr(), 2, serve.cuda_stream, blocks)
        except Exception as ex:   # noqa: BLE001 - reported by the test's thread
            errors.append(ex)
        filled.set()
        done.wait(60)             # the thread, and its stream, live until the fills are done
    threads = []
    for e, blocks in ((4, 1), (5, 0)):                       # 6.3 MB by one small workgroup (0.7 ms), then at full speed
        filled = threading.Event()
        threads.append(threading.Thread(target=fill, args=(e, blocks, filled)))
        threads[-1].start()
        assert filled.wait(60)
    case.place(np.array([0, 1, 2, 3, 4, 5, -1, -1], np.int32), upload=False)
    got13, got2 = case.layer.w13[4:6].clone(), case.layer.w2[4:6].clone()   # on the serving stream, behind the switch
    torch.cuda.synchronize()
    done.set()
    for t in threads:
        t.join()
    assert not errors, errors
    np.testing.assert_array_equal(tensor_to_host(got13), case.w13_pool[4:6])
    np.testing.assert_array_equal(tensor_to_host(got2), case.w2_pool[4:6])


@pytest.mark.parametrize("serve_default", [True, False])
def test_a_fill_waits_for_what_the_serving_stream_still_has(serve_default):
    """Fills in a row with and without work left on the serving stream, which also writes their sources: a fill that asks the stream
    first must see all of it, whether the layer or somebody else enqueued it."""
    import torch
    from gpu_util import Case, tensor_to_host
    wl = MoEWorkload(name="fill_wait", tokens=64, **dict(MID, hidden=1024, inter=1024, n_experts=8, n_slots=8, n_local=8))
    case = Case(wl, expert_map=np.array([0, 1, -1, -1, -1, -1, -1, -1], np.int32))
    src = {e: (case.layer.upload(case.inp["w13_experts"][e]), case.layer.upload(case.inp["w2_experts"][e])) for e in range(2, 8)}
    serve = torch.cuda.current_stream() if serve_default else torch.cuda.Stream()
    copy = torch.cuda.Stream()
    stage = [(torch.zeros_like(a), torch.zeros_like(b)) for a, b in src.values()]
    work = torch.randn(4096, 4096, device=case.x_dev.device)
    torch.cuda.synchronize()
    with torch.cuda.stream(serve):
        for i, (e, (a, b)) in enumerate(src.items()):
            if i != 3:                                       # one fill finds the stream as the one before it left it
                for _ in range(4):
                    work @ work                              # a while on the serving stream, then the source
            stage[i][0].copy_(a)
            stage[i][1].copy_(b)
            case.layer.load_expert_async(e, stage[i][0], stage[i][1], copy, serve)
            if i == 1:
                torch.cuda.synchronize()                     # everything done once in between; the next sources are behind it again
            if i == 2:
                case.layer.forward(case.x_dev)
        case.place(np.array([0, 1, 2, 3, 4, 5, 6, 7], np.int32), upload=False)
        got13, got2 = case.layer.w13.clone(), case.layer.w2.clone()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(tensor_to_host(got13), case.w13_pool)
    np.testing.assert_array_equal(tensor_to_host(got2), case.w2_pool)


@pytest.mark.parametrize("serve_default", [True, False])
def test_fills_behind_work_that_the_serving_stream_has_done(serve_default):
    """Sources written by the serving stream, which is idle again when the fills are issued: all but the first find it so and go without
    an event.  They copy what was written, round after round into the same source buffers."""
    import torch
    from gpu_util import Case, tensor_to_host
    wl = MoEWorkload(name="fill_idle", tokens=64, **dict(MID, hidden=1024, inter=1024, n_experts=8, n_slots=8, n_local=8))
    case = Case(wl, expert_map=np.array([0, 1, -1, -1, -1, -1, -1, -1], np.int32))
    src = {e: (case.layer.upload(case.inp["w13_experts"][e]), case.layer.upload(case.inp["w2_experts"][e])) for e in range(2, 8)}
    serve = torch.cuda.current_stream() if serve_default else torch.cuda.Stream()
    copy = torch.cuda.Stream()
    stage = [(torch.zeros_like(src[2][0]), torch.zeros_like(src[2][1])) for _ in range(3)]
    torch.cuda.synchronize()
    with torch.cuda.stream(serve):
        for first in (2, 5):
            for i, (s13, s2) in enumerate(stage):
                s13.copy_(src[first + i][0])
                s2.copy_(src[first + i][1])
            serve.synchronize()
            for i, (s13, s2) in enumerate(stage):            # nothing else on the serving stream from here on
                case.layer.load_expert_async(first + i, s13, s2, copy, serve)
            copy.synchronize()
        case.place(np.array([0, 1, 2, 3, 4, 5, 6, 7], np.int32), upload=False)
        got13, got2 = case.layer.w13.clone(), case.layer.w2.clone()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(tensor_to_host(got13), case.w13_pool)
    np.testing.assert_array_equal(tensor_to_host(got2), case.w2_pool)


def test_fills_beside_a_capture_leave_it_alone():
    """A graph capture of the serving thread's forward goes on while slots are filled on other streams."""
    import torch
    from gpu_util import Case, tensor_to_host
    wl = MoEWorkload(name="fill_cap", tokens=64, **dict(MID, n_experts=8, n_slots=8, n_local=8))
    case = Case(wl, expert_map=np.array([0, 1, 2, 3, -1, -1, -1, -1], np.int32))
    src = {e: (case.layer.upload(case.inp["w13_experts"][e]), case.layer.upload(case.inp["w2_experts"][e])) for e in range(4, 8)}
    before = case.run()
    copy, other, cap = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    out = torch.empty_like(case.x_dev)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=cap):
        case.layer.forward(case.x_dev, out=out, shared_range=wl.shared_range)
        for e in src:                                        # the second and later ones ask `other`, which is idle
            case.layer.load_expert_async(e, src[e][0], src[e][1], copy, other)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(tensor_to_host(out), before)
    case.place(np.arange(8, dtype=np.int32), upload=False)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(tensor_to_host(case.layer.w13), case.w13_pool)
    np.testing.assert_array_equal(tensor_to_host(case.layer.w2), case.w2_pool)
