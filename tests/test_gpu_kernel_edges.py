"""Expert kernels at the sizes where their dispatch changes: ring geometries of the large-tile kernels by the number
of token tiles and K-steps, and the few-token path with more slots than a wavefront has lanes."""
import numpy as np
import pytest

from workloads import MoEWorkload, block_expert_map

pytestmark = pytest.mark.gpu


def _kernels(case, tokens, shared_range=(0, 0), routed=False):
    """The kernels of a pass over the case's first tokens, names without template arguments."""
    import torch
    from gpu_util import kernels_of
    x, out, k = case.x_dev[:tokens], torch.empty_like(case.x_dev[:tokens]), case.layer.cfg.top_k
    if routed:
        ids, w = (torch.zeros((tokens, k), dtype=t, device=x.device) for t in (torch.int32, torch.float32))
        names = kernels_of(lambda s: case.layer.forward_routed(x, ids, w, out=out, shared_range=shared_range, stream=s))
    else:
        names = kernels_of(lambda s: case.layer.forward(x, out=out, shared_range=shared_range, stream=s))
    return [n.split("<")[0] for n in names]


def _expert_kernels(case, tokens, shared_range=(0, 0), routed=False):
    """The kernel of GEMM-1 in such a pass."""
    return next(n for n in _kernels(case, tokens, shared_range, routed) if "expert" in n)


@pytest.mark.parametrize("hidden,inter", [(64, 64), (128, 192), (192, 128), (320, 256), (512, 320)])
def test_large_tile_rings_at_every_token_tile_count(hidden, inter):
    """Slots with 1, 2, 3 ... 10 token tiles of 32 rows, full and with one row in the last, on contractions of 1 to 8
    K-steps (shorter and longer than every ring is deep): each token has one expert, so the counts are exact."""
    from gpu_util import Case
    from test_gpu_routed import _check
    counts = [1, 32, 33, 64, 65, 97, 128, 129, 160, 161, 193, 225, 256, 257, 288, 289, 320]
    tokens = sum(counts)
    wl = MoEWorkload(name="rings", tokens=tokens, hidden=hidden, inter=inter, n_experts=len(counts), top_k=1, n_slots=len(counts),
                     n_local=len(counts), act_dtype="bf16", router_dtype="f32", gate="softmax", seed=300 + hidden)
    g = np.random.Generator(np.random.PCG64(hidden))
    ids = g.permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)[:, None]
    case = Case(wl)
    _check(case, ids, g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32))
    rows = np.sort(case.layer.view(tokens)["tiles"][:, 2])
    np.testing.assert_array_equal(rows, np.sort(counts))      # the large-tile kernels ran: a tile per slot


@pytest.mark.parametrize("hidden,inter,rows,parts", [
    (64, 192, "few", (8, 8)), (320, 128, "few", (8, 8)), (448, 448, "few", (4, 8)), (4096, 64, "few", (8, 8)),       # 34 workgroups or so, half and quarter slices of 64 columns
    (64, 192, "many", (4, 4)), (448, 448, "many", (4, 4)),                                                           # more than 224 rows a slot
    (320, 512, "few", (4, 8)), (64, 1152, "few", (2, 8)), (2304, 64, "few", (8, 2)), (64, 2048, "few", (8, 8)),      # 68, 153 workgroups, a round and 16
    (64, 2944, "many", (2, 4)), (4096, 2048, "chunks", (4, 4)), (64, 192, "chunks", (8, 8))])                        # a round and 135; several tiles a slot
def test_last_round_of_the_large_tiles_in_parts(hidden, inter, rows, parts):
    """N-slices as two or four workgroups (wavefronts 4 x 2 and 8 x 1) and whole ones, at every number of token tiles, on short contractions, and the numbers of workgroups on both sides of the rule; a
    column slice that ends inside its first, second and third part."""
    from gpu_util import Case, kernels_of
    from test_gpu_routed import _check
    counts = {"few": [1, 32, 33, 64, 65, 97, 128, 129, 160, 161, 193, 225, 256, 257, 288, 289, 320],
              "many": [193, 224, 225, 239, 240, 241, 255, 256, 257, 272, 273, 288, 289, 304, 305, 319, 320], "chunks": [321, 350, 400, 410]}[rows]
    tokens = sum(counts)
    wl = MoEWorkload(name="parts", tokens=tokens, hidden=hidden, inter=inter, n_experts=len(counts), top_k=1, n_slots=len(counts),
                     n_local=len(counts), act_dtype="bf16", router_dtype="f32", gate="softmax", seed=360 + hidden)
    g = np.random.Generator(np.random.PCG64(hidden))
    ids = g.permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)[:, None]
    case = Case(wl)
    import torch
    dev_ids, w, out = torch.from_numpy(ids).to(case.x_dev.device), torch.ones((tokens, 1), device=case.x_dev.device), torch.empty_like(case.x_dev)
    names = [n for n in kernels_of(lambda s: case.layer.forward_routed(case.x_dev, dev_ids, w, out=out, stream=s)) if n.startswith("k_expert_gemm_mfma8") and ", 0, " in n]
    assert [int(n.rstrip(">").split(", ")[-1]) for n in names] == list(parts), names
    _check(case, ids, g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32))


@pytest.mark.parametrize("hidden,inter,more,big,parts", [(512, 256, 79, False, (8, 8)), (448, 448, 103, False, (4, 8)), (448, 448, 103, True, (4, 4)), (64, 128, 223, False, (8, 8))])
def test_a_split_last_round_has_the_bits_of_whole_slices(hidden, inter, more, big, parts):
    """17 experts' tokens alone, whose slices run as two or four workgroups each, and beside `more` other experts, whose launches have a whole round or most of one: the same bits in h and in the output."""
    import torch
    from gpu_util import kernels_of
    from paper_2510_02613_amd.layer import MoELayer
    counts = [193, 224, 225, 239, 240, 241, 255, 256, 257, 272, 273, 288, 289, 304, 305, 319, 320] if big else [1, 32, 33, 64, 65, 97, 128, 129, 160, 161, 193, 225, 256, 257, 288, 289, 320]
    experts, dev = len(counts) + more, torch.device("cuda:0")
    round_rows = torch.cuda.get_device_properties(dev).multi_processor_count // 8
    gen = torch.Generator(device=dev).manual_seed(380 + hidden)
    ids = torch.repeat_interleave(torch.arange(experts, device=dev), torch.tensor(counts + [64] * more, device=dev)).to(torch.int32)[:, None].contiguous()
    x = torch.randn(len(ids), hidden, generator=gen, device=dev).bfloat16().view(torch.int16)
    weights = [(torch.randn(experts, *s, generator=gen, device=dev) * 0.1).bfloat16().view(torch.int16) for s in ((2 * inter, hidden), (hidden, inter))]

    def run(n, tokens):
        layer = MoELayer(hidden=hidden, inter=inter, n_experts=n, top_k=1, n_slots=n, max_tokens=tokens, act_dtype="bf16", router_dtype="f32", gate="softmax",
                         router_w=np.zeros((n, hidden), np.float32))
        layer.w13.copy_(weights[0][:n])
        layer.w2.copy_(weights[1][:n])
        layer.set_expert_map(list(range(n)))
        w, out = torch.ones((tokens, 1), device=dev), torch.empty_like(x[:tokens])
        names = kernels_of(lambda s: layer.forward_routed(x[:tokens], ids[:tokens], w, out=out, stream=s))
        layer.forward_routed(x[:tokens], ids[:tokens], w, out=out)
        v = layer.view(tokens)
        return ([int(k.rstrip(">").split(", ")[-1]) for k in names if k.startswith("k_expert_gemm_mfma8") and ", 0, " in k], out.cpu().numpy(), v["h"][v["inv"][:, 0]], v["unit_hdr"][:, 0])
    own = sum(counts)
    split, out, h, rows = run(len(counts), own)
    whole, out_whole, h_whole, rows_whole = run(experts, len(ids))
    assert split == list(parts) and whole == [2, 2]
    for r, part in zip(rows, parts):
        assert 0 < r % round_rows * (part // 2) <= round_rows, rows       # the unit list has such a round
    np.testing.assert_array_equal(out, out_whole[:own])
    np.testing.assert_array_equal(h, h_whole[:own])


@pytest.mark.parametrize("hidden,inter", [(64, 192), (320, 128)])
def test_large_tiles_stage_by_8_rows_and_multiply_by_16(hidden, inter):
    """Slots of more than 128 rows that end just before, at and behind multiples of 8 and 16, in each half of a 32-row tile and
    with the last tile at either wavefront row."""
    from gpu_util import Case
    from test_gpu_routed import _check
    counts = [130, 136, 137, 143, 144, 145, 152, 153, 168, 176, 177, 184, 185, 208, 209, 239, 240, 241, 271, 272, 273, 280, 281, 303, 304, 305, 312, 313]
    tokens = sum(counts)
    wl = MoEWorkload(name="halves", tokens=tokens, hidden=hidden, inter=inter, n_experts=len(counts), top_k=1, n_slots=len(counts),
                     n_local=len(counts), act_dtype="bf16", router_dtype="f32", gate="softmax", seed=340 + hidden)
    g = np.random.Generator(np.random.PCG64(hidden))
    ids = g.permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)[:, None]
    case = Case(wl)
    _check(case, ids, g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32))
    np.testing.assert_array_equal(np.sort(case.layer.view(tokens)["tiles"][:, 2]), np.sort(counts))


@pytest.mark.parametrize("tokens", [1, 17, 64])
@pytest.mark.parametrize("local", [64, 65, 127, 130, 255, 256])
def test_few_tokens_many_slots_derive_their_tiles(tokens, local):
    """1 to 4 slots per lane in the few-token GEMM-1 that derives its tiles itself, and the first count past it: output and tables as in the pass
    with separate bookkeeping kernels, bit for bit, and within the oracle's bar."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="few_many", tokens=tokens, hidden=136, inter=72, n_experts=256, top_k=4, n_slots=local + 1, n_local=local,
                     act_dtype="bf16", router_dtype="bf16", gate="softmax", n_shared=1, shared_range=(0, min(tokens, 20)), seed=900 + local)
    g = np.random.Generator(np.random.PCG64(local))
    case = Case(wl, expert_map=block_expert_map(256, 0, local, g.permutation(local)))
    runs = []
    for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
        out = case.run(flags=flags)
        runs.append((out, case.layer.view(tokens)))
    ids, _, _ = check_routing(case, runs[0][1]["topk_ids"], runs[0][1]["topk_w"])
    check_bookkeeping(case, runs[0][1], tokens, wl.shared_range)
    check_output(case, runs[0][0], ids)
    np.testing.assert_array_equal(runs[0][0], runs[1][0])
    for key in ("counts", "offsets", "perm", "inv", "tiles", "h", "y"):
        np.testing.assert_array_equal(runs[0][1][key], runs[1][1][key])


@pytest.mark.parametrize("tokens", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("experts,gate,hidden,inter,shared,most", [(65, "softmax", 136, 72, 0, 4), (128, "softmax", 520, 64, 2, 4), (96, "softmax", 64, 1200, 0, 3),
                                                                   (100, "softmax", 4160, 24, 4, 4), (129, "softmax", 136, 72, 0, 0), (96, "sigmoid_group", 64, 200, 1, 0),
                                                                   (100, "softmax", 128, 512, 2, 4)])
def test_a_token_to_four_are_selected_in_gemm1(tokens, experts, gate, hidden, inter, shared, most):
    """The register and ring GEMM-1 that select the experts themselves (up to 4 tokens, 128 experts and 1760 workgroups, no groups) and the sizes past it: routing, tables and output as in
    the pass with separate selection and bookkeeping kernels, bit for bit, and through the entry that brings its placement along."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    from paper_2510_02613_amd import binding as B
    local = experts - 8
    grouped = dict(gate="sigmoid_group", n_group=4, topk_group=2, routed_scale=2.5) if gate == "sigmoid_group" else dict(gate="softmax")
    wl = MoEWorkload(name="select", tokens=tokens, hidden=hidden, inter=inter, n_experts=experts, top_k=7, n_slots=local + shared, n_local=local,
                     act_dtype="bf16", router_dtype="f32", n_shared=shared, shared_range=(0, min(tokens, 2) if shared else 0), seed=77 + experts, **grouped)
    g = np.random.Generator(np.random.PCG64(experts + tokens))
    case = Case(wl, expert_map=block_expert_map(experts, 0, local, g.permutation(local)))
    assert ("k_gate_select_hist" not in _kernels(case, tokens, wl.shared_range)) == (tokens <= most)
    assert _expert_kernels(case, tokens, wl.shared_range) == ("k_expert_ring" if inter == 512 and tokens >= 4 else "k_expert_decode")
    runs = []
    for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED, 0):
        case.layer.workspace[int(B.moe_workspace_view(case.layer.handle).topk_ids - case.layer.workspace.data_ptr()):].fill_(0xee)
        out = case.run(flags=flags)
        runs.append((out, case.layer.view(tokens)))
    ids, _, _ = check_routing(case, runs[0][1]["topk_ids"], runs[0][1]["topk_w"])
    check_bookkeeping(case, runs[0][1], tokens, wl.shared_range)
    check_output(case, runs[0][0], ids)
    for other in runs[1:]:
        np.testing.assert_array_equal(runs[0][0], other[0])
        for key in ("topk_ids", "topk_w", "counts", "offsets", "perm", "inv", "tiles", "h", "y"):
            np.testing.assert_array_equal(runs[0][1][key], other[1][key])
    x = case.x_dev[:tokens]
    out = case.layer.forward_static(x, shared_range=wl.shared_range)
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint16).ravel(), np.asarray(runs[0][0]).view(np.uint16).ravel())


@pytest.mark.parametrize("tokens", [3, 17, 40])
@pytest.mark.parametrize("hidden,inter,first,second", [(1280, 640, 0, 0), (1288, 640, 1, 0), (1272, 648, 0, 1), (4096, 648, 1, 1), (4104, 72, 2, 0), (264, 264, 0, 0)])
def test_register_kernels_at_the_ends_of_their_forms(tokens, hidden, inter, first, second):
    """Contractions on both sides of the lines between the forms (wavefronts per SIMD, chunks ahead) of the register kernels: the form, tables and output as with
    separate bookkeeping kernels, bit for bit, and within the oracle's bar."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing, kernels_of
    from paper_2510_02613_amd import binding as B
    # rows of 8 more than a multiple of 64 stay off the ring kernels; the others are too few tasks for them
    wl = MoEWorkload(name="forms", tokens=tokens, hidden=hidden, inter=inter, n_experts=80, top_k=4, n_slots=14, n_local=14,
                     act_dtype="bf16", router_dtype="bf16", gate="softmax", seed=500 + hidden)
    case = Case(wl, expert_map=block_expert_map(80, 0, 14, np.random.Generator(np.random.PCG64(hidden)).permutation(14)))
    x, spare, runs = case.x_dev[:tokens], case.x_dev[:tokens].clone(), []
    names = kernels_of(lambda s: case.layer.forward(x, out=spare, stream=s))
    forms = [n.split("<")[1].rstrip(">").split(", ")[2] for n in names if n.startswith("k_expert_decode")]
    assert forms == [str(first), str(second)]
    for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
        out = case.run(flags=flags)
        runs.append((out, case.layer.view(tokens)))
    ids, _, _ = check_routing(case, runs[0][1]["topk_ids"], runs[0][1]["topk_w"])
    check_bookkeeping(case, runs[0][1], tokens, (0, 0))
    check_output(case, runs[0][0], ids)
    np.testing.assert_array_equal(runs[0][0], runs[1][0])
    for key in ("counts", "offsets", "perm", "inv", "tiles", "h", "y"):
        np.testing.assert_array_equal(runs[0][1][key], runs[1][1][key])


@pytest.mark.parametrize("router,experts", [("bf16", 200), ("f32", 100)])
@pytest.mark.parametrize("hidden,tokens", [(64, 24460), (128, 24460), (192, 24460), (256, 24460), (320, 24460), (1024, 12300)])
def test_largest_gate_tilings_at_few_steps(hidden, tokens, router, experts):
    """The largest tilings of the direct-to-LDS gate logits kernel (128 tokens x 256 experts, 128 with an fp32 router; a ring of three stages) on contractions of 1 to 5
    K-steps, shorter and longer than the ring, and of 8 in each of two K ranges; the last token and expert tiles are ragged.  Routing of every token against the oracle."""
    from gpu_util import Case, check_routing, kernels_of
    wl = MoEWorkload(name="gate_ring", tokens=tokens, hidden=hidden, inter=8, n_experts=experts, top_k=3, n_slots=2, n_local=2,
                     act_dtype="bf16", router_dtype=router, gate="softmax", seed=40 + hidden)
    case = Case(wl)
    spare = case.x_dev.clone()
    names = kernels_of(lambda s: case.layer.forward(case.x_dev, out=spare, stream=s))
    assert any(n.startswith("k_gate_logits_dma") and n.rstrip(">").endswith(", 3, 8, 2") for n in names), names
    case.run()
    v = case.layer.view(tokens)
    check_routing(case, v["topk_ids"], v["topk_w"])


@pytest.mark.parametrize("router,experts,hidden,tokens,tiling", [
    ("f32", 64, 1024, 129, "2, 1, 6, 4, 1"), ("f32", 100, 1088, 600, "2, 1, 6, 4, 1"), ("bf16", 65, 512, 250, "2, 1, 6, 4, 1"),
    ("f32", 100, 1088, 2600, "4, 1, 4, 8, 1"), ("bf16", 200, 1088, 2600, "2, 2, 6, 8, 2"), ("bf16", 256, 2112, 4100, "2, 2, 6, 8, 2"),
    ("f32", 128, 1088, 12300, "4, 2, 3, 8, 2"), ("bf16", 200, 1152, 12300, "4, 4, 3, 8, 2"), ("bf16", 129, 1152, 24460, "4, 4, 3, 8, 2")])
def test_gate_tilings_by_rounds_of_the_chip(router, experts, hidden, tokens, tiling):
    """The tilings that the rule by rounds and K-steps takes, with splits of 4, of 8 and of more K-steps (which go to a sum every 8) and shares of unequal length.  Routing of every
    token against the oracle."""
    from gpu_util import Case, check_routing, kernels_of
    wl = MoEWorkload(name="gate_rounds", tokens=tokens, hidden=hidden, inter=8, n_experts=experts, top_k=3, n_slots=2, n_local=2,
                     act_dtype="bf16", router_dtype=router, gate="softmax", seed=60 + hidden + experts)
    case = Case(wl)
    spare = case.x_dev.clone()
    names = kernels_of(lambda s: case.layer.forward(case.x_dev, out=spare, stream=s))
    assert any(n.startswith("k_gate_logits_dma") and n.rstrip(">").endswith(", " + tiling) for n in names), names
    case.run()
    v = case.layer.view(tokens)
    check_routing(case, v["topk_ids"], v["topk_w"])


@pytest.mark.parametrize("router,experts,hidden,tokens,direct", [
    ("f32", 512, 8256, 1, False), ("f32", 512, 8256, 32, False), ("f32", 512, 8256, 33, True), ("f32", 384, 7168, 32, False), ("f32", 384, 7168, 33, True), ("f32", 256, 7168, 64, False),
    ("f32", 256, 7168, 65, True), ("f32", 128, 7168, 128, False), ("f32", 128, 7168, 129, True), ("f32", 256, 4096, 64, False), ("f32", 256, 4096, 65, True), ("f32", 256, 2048, 128, False),
    ("bf16", 1024, 8256, 16, False), ("bf16", 1024, 8256, 17, True), ("bf16", 256, 7168, 64, False), ("bf16", 256, 7168, 65, True)])
def test_gate_of_few_tokens_by_the_router_s_size(router, experts, hidden, tokens, direct):
    """The logits kernel on both sides of the lines on blocks of tokens, bytes of router and experts (direct: the one with direct copies to LDS).  Routing of every token against the oracle."""
    from gpu_util import Case, check_routing, kernels_of
    wl = MoEWorkload(name="gate_few", tokens=tokens, hidden=hidden, inter=8, n_experts=experts, top_k=3, n_slots=2, n_local=2,
                     act_dtype="bf16", router_dtype=router, gate="softmax", seed=70 + experts)
    case = Case(wl)
    spare = case.x_dev.clone()
    names = [n.split("<")[0] for n in kernels_of(lambda s: case.layer.forward(case.x_dev, out=spare, stream=s))]
    assert ("k_gate_logits_dma" in names) == direct == ("k_gate_logits" not in names), names
    case.run()
    v = case.layer.view(tokens)
    check_routing(case, v["topk_ids"], v["topk_w"])


@pytest.mark.parametrize("tokens", [1, 2, 15, 32, 47, 64, 90])
@pytest.mark.parametrize("hidden,inter", [(64, 64), (128, 448), (192, 64), (320, 128), (768, 1024)])
def test_decode_ring_kernels(tokens, hidden, inter):
    """The few-token kernels, the LDS-ring or the register ones as the dispatch chooses by the expected tasks: short and long
    contractions, output widths that end inside a task's 128 columns, shared rows; tables and output as in the pass with
    separate bookkeeping kernels, bit for bit.  (The ring kernels by themselves: the next test.)"""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    from paper_2510_02613_amd import binding as B
    # eleven assignments a token keep the smallest layer above what k_token_experts takes
    experts, k = (256, 10) if hidden * inter < 8192 else (96, 4)
    local = experts - 6
    wl = MoEWorkload(name="ring", tokens=tokens, hidden=hidden, inter=inter, n_experts=experts, top_k=k, n_slots=local + 3, n_local=local,
                     act_dtype="bf16", router_dtype="f32", gate="softmax", n_shared=1, shared_range=(0, min(tokens, 30)), seed=700 + tokens)
    case = Case(wl, expert_map=block_expert_map(experts, 0, local, np.random.Generator(np.random.PCG64(3)).permutation(local + 2)[:local]))
    assert _expert_kernels(case, tokens, wl.shared_range) in ("k_expert_decode", "k_expert_ring")
    runs = []
    for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
        out = case.run(flags=flags)
        runs.append((out, case.layer.view(tokens)))
    ids, _, _ = check_routing(case, runs[0][1]["topk_ids"], runs[0][1]["topk_w"])
    check_bookkeeping(case, runs[0][1], tokens, wl.shared_range)
    check_output(case, runs[0][0], ids)
    np.testing.assert_array_equal(runs[0][0], runs[1][0])
    for key in ("counts", "offsets", "perm", "inv", "tiles", "h", "y"):
        np.testing.assert_array_equal(runs[0][1][key], runs[1][1][key])


def _ring_cases():
    """(tokens, experts, k, hidden, inter) that the dispatch sends to the ring kernels: 160 tasks or more, not 240 .. 330."""
    out = []
    for hidden, inter, experts, k in [(64, 64, 256, 10), (128, 64, 256, 8), (64, 128, 256, 8), (192, 192, 96, 4), (256, 256, 96, 4),
                                      (320, 320, 96, 4), (768, 1024, 96, 4)]:
        for tokens in (17, 32, 47, 64, 90):
            tasks = ((experts - 2) * (1 - (1 - k / experts) ** tokens) + 1) * (inter // 64)
            if tokens * k <= 4 * experts and tasks >= 162 and not 238 <= tasks < 332:
                out.append((tokens, experts, k, hidden, inter))
    return out


@pytest.mark.parametrize("tokens,experts,k,hidden,inter", _ring_cases())
def test_ring_kernels_at_every_contraction_length(tokens, experts, k, hidden, inter):
    """Contractions of 1, 2, 3, 4, 5 and more K-steps in both GEMMs of the ring kernels (the ring is 4 deep), with and without
    self-derived tiles.  A bias sends every token to expert 5, whose rows are full tiles of 32.  Tables and output as with separate bookkeeping kernels, bit for bit, and within the oracle's bar."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    from paper_2510_02613_amd import binding as B
    from workloads import make_inputs
    wl = MoEWorkload(name="ring_k", tokens=tokens, hidden=hidden, inter=inter, n_experts=experts, top_k=k, n_slots=experts, n_local=experts - 2,
                     act_dtype="bf16", router_dtype="f32", gate="softmax", n_shared=1, shared_range=(0, min(tokens, 30)), seed=1200 + tokens)
    inp = make_inputs(wl)
    inp["logit_bias"] = np.zeros(experts, np.float32)
    inp["logit_bias"][5] = 8.0
    order = np.random.Generator(np.random.PCG64(3)).permutation(experts - 1)[:experts - 2]
    case = Case(wl, expert_map=block_expert_map(experts, 0, experts - 2, order), inputs=inp)
    assert _expert_kernels(case, tokens, wl.shared_range) == "k_expert_ring"
    runs = []
    for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
        out = case.run(flags=flags)
        runs.append((out, case.layer.view(tokens)))
    ids, _, _ = check_routing(case, runs[0][1]["topk_ids"], runs[0][1]["topk_w"])
    assert (ids == 5).any(1).all()
    tiles = runs[0][1]["tiles"]
    rows = tiles[tiles[:, 0] == case.expert_map[5]][:, 2]
    assert rows.sum() == tokens and len(rows) == -(-tokens // 32)
    check_bookkeeping(case, runs[0][1], tokens, wl.shared_range)
    check_output(case, runs[0][0], ids)
    np.testing.assert_array_equal(runs[0][0], runs[1][0])
    for key in ("counts", "offsets", "perm", "inv", "tiles", "h", "y"):
        np.testing.assert_array_equal(runs[0][1][key], runs[1][1][key])


def test_decode_ring_kernels_with_a_crowded_expert():
    """Every token takes the same expert: its 64 rows are two tiles of the ring kernels."""
    from gpu_util import Case
    from test_gpu_routed import _check
    wl = MoEWorkload(name="crowd", tokens=64, hidden=256, inter=512, n_experts=64, top_k=4, n_slots=64, n_local=64,
                     act_dtype="bf16", router_dtype="f32", gate="softmax", seed=77)
    g = np.random.Generator(np.random.PCG64(5))
    ids = np.stack([np.concatenate([[7], 8 + g.permutation(56)[:3]]) for _ in range(64)]).astype(np.int32)
    case = Case(wl)
    _check(case, ids, g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32))
    tiles = case.layer.view(64)["tiles"]
    assert (tiles[tiles[:, 0] == 7][:, 2] == 32).all() and (tiles[:, 0] == 7).sum() == 2


@pytest.mark.parametrize("tokens,tile", [(3, 16), (4, 32), (8, 16), (12, 32)])
def test_few_token_kernels_by_task_count(tokens, tile):
    """A layer of 64 experts, 768 wide: 135, 175, 310 and 414 expected tasks of the ring kernels, which take the second
    and the last.  Expert 9 has all assignments (ids may repeat), so the tile list tells the kernels apart."""
    from gpu_util import Case
    from test_gpu_routed import _check
    wl = MoEWorkload(name="tasks", tokens=tokens, hidden=192, inter=768, n_experts=64, top_k=4, n_slots=64, n_local=64,
                     act_dtype="bf16", router_dtype="f32", gate="softmax", seed=80 + tokens)
    g = np.random.Generator(np.random.PCG64(tokens))
    case = Case(wl)
    _check(case, np.full((tokens, 4), 9, np.int32), g.uniform(0.5, 1.5, size=(tokens, 4)).astype(np.float32))
    rows = case.layer.view(tokens)["tiles"][:, 2]
    assert rows.sum() == 4 * tokens and len(rows) == -(-4 * tokens // tile)


@pytest.mark.parametrize("hidden,tile", [(4096, 16), (4160, 32)])
def test_few_token_kernels_by_row_length(hidden, tile):
    """255 expected tasks, a little more than one per compute unit: the register kernels up to rows of 4096, the ring beyond."""
    from gpu_util import Case
    from test_gpu_routed import _check
    wl = MoEWorkload(name="rows", tokens=8, hidden=hidden, inter=2048, n_experts=8, top_k=4, n_slots=8, n_local=8,
                     act_dtype="bf16", router_dtype="f32", gate="softmax", seed=88)
    g = np.random.Generator(np.random.PCG64(8))
    case = Case(wl)
    _check(case, np.full((8, 4), 3, np.int32), g.uniform(0.5, 1.5, size=(8, 4)).astype(np.float32))
    rows = case.layer.view(8)["tiles"][:, 2]
    assert rows.sum() == 32 and len(rows) == 32 // tile


@pytest.mark.parametrize("tokens,tiles", [(200, 2), (255, 2), (256, 1)])
def test_small_layers_take_the_128_row_kernels(tokens, tiles):
    """16 slots of a small layer, three assignments per token: 768 assignments are 48 rows a slot, where the large-tile
    kernels start (320 rows a tile); one expert has 200 rows and more, two tiles of 128 below that line."""
    from gpu_util import Case
    from test_gpu_routed import _check
    wl = MoEWorkload(name="line", tokens=tokens, hidden=128, inter=192, n_experts=16, top_k=3, n_slots=16, n_local=16,
                     act_dtype="bf16", router_dtype="bf16", gate="softmax", seed=90 + tokens)
    g = np.random.Generator(np.random.PCG64(tokens))
    ids = np.stack([np.concatenate([[5], 6 + g.permutation(10)[:2]]) for _ in range(tokens)]).astype(np.int32)
    case = Case(wl)
    _check(case, ids, g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32))
    assert (case.layer.view(tokens)["tiles"][:, 0] == 5).sum() == tiles


@pytest.mark.parametrize("tokens", [1, 16, 33, 64, 65, 257, 700])
@pytest.mark.parametrize("hidden,inter,router", [(64, 8, "f32"), (1368, 8, "f32"), (8, 1368, "bf16"), (136, 72, "bf16"), (264, 136, "f32"), (1024, 1032, "f32"),
                                                 (4104, 136, "bf16")])
def test_f32_layer_tiles_and_contractions(tokens, hidden, inter, router):
    """fp32 layers on both sides of the self-derived tiles (64 tokens) and of every tile height (16, 32, 64 rows), outputs narrower than a
    task's columns (the 64 x 8 layer goes token by token up to 256 tokens), with contractions that leave wavefronts of a task without a chunk and long ones (several planes of partial logits), and both
    router types."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    wl = MoEWorkload(name="f32_edges", tokens=tokens, hidden=hidden, inter=inter, n_experts=24, top_k=3, n_slots=22, n_local=20,
                     act_dtype="f32", router_dtype=router, gate="sigmoid_group", n_group=4, topk_group=2, routed_scale=2.5,
                     n_shared=1, shared_range=(tokens // 3, tokens), seed=400 + tokens)
    case = Case(wl)
    small = hidden * inter < 1000 and tokens <= 256
    assert _expert_kernels(case, tokens, wl.shared_range) == ("k_token_experts" if small else "k_expert_f32" if tokens * 3 <= 32 * 24 else "k_expert_f32_tile")
    out = case.run()
    v = case.layer.view(tokens)
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, tokens, wl.shared_range)
    check_output(case, out, ids)


@pytest.mark.parametrize("tokens", [33, 64])
def test_f32_self_derived_tiles_of_32_rows(tokens):
    """Up to 64 tokens with 17 to 32 rows a slot: GEMM-1 derives tiles of 32 rows; the same bits as with separate bookkeeping."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="f32_32", tokens=tokens, hidden=136, inter=72, n_experts=8, top_k=5, n_slots=8, n_local=6, act_dtype="f32",
                     router_dtype="f32", gate="softmax", n_shared=1, shared_range=(0, tokens), seed=470)
    case = Case(wl)
    assert _expert_kernels(case, tokens, wl.shared_range) == "k_expert_f32"
    out = case.run()
    v = case.layer.view(tokens)
    assert 16 < v["tiles"][:, 2].max() <= 32
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, tokens, wl.shared_range)
    check_output(case, out, ids)
    np.testing.assert_array_equal(out, case.run(flags=B.MOE_FLAG_PERMUTE_UNFUSED))


@pytest.mark.parametrize("hidden,inter", [(64, 64), (128, 192), (192, 320), (256, 64), (704, 128)])
def test_ring_tiles_of_64_rows(hidden, inter):
    """Weight-streaming tasks of up to 64 token rows: one token tile and two, full and with one row in the last, 8-row pieces
    that exist and that do not, several chunks of a slot; contractions of 1 to 11 K-steps, output widths that end inside a task's
    128 columns.  The tile list (chunks of 64) shows that they ran."""
    from gpu_util import Case
    from test_gpu_routed import _check
    counts = [1, 8, 9, 31, 32, 33, 40, 41, 56, 57, 64, 65, 128, 129]
    tokens, S = sum(counts), len(counts) + 40
    wl = MoEWorkload(name="ring64", tokens=tokens, hidden=hidden, inter=inter, n_experts=64, top_k=1, n_slots=S,
                     n_local=len(counts), act_dtype="bf16", router_dtype="f32", gate="softmax", seed=1500 + hidden)
    g = np.random.Generator(np.random.PCG64(hidden + inter))
    ids = g.permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)[:, None]
    case = Case(wl)
    _check(case, ids, g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32))
    rows = case.layer.view(tokens)["tiles"][:, 2]
    assert rows.max() == 64 and len(rows) == sum((c + 63) // 64 for c in counts)


@pytest.mark.parametrize("tokens,hidden,inter", [(40, 320, 192), (300, 192, 320), (320, 64, 64)])
def test_ring_tiles_of_64_rows_behind_the_gate(tokens, hidden, inter):
    """The same kernels behind both bookkeeping paths of a gated pass, with shared rows, through the entry without a workspace and
    under replicas: tables and output within the oracle's bar and the same bits every way; more assignments per slot than the large-tile kernels
    take elsewhere."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing, kernels_of, tensor_to_host
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="ring64g", tokens=tokens, hidden=hidden, inter=inter, n_experts=64, top_k=4 if tokens > 40 else 8, n_slots=14 if tokens > 40 else 6,
                     n_local=9 if tokens > 40 else 4, act_dtype="bf16", router_dtype="bf16", gate="sigmoid_group", n_group=4, topk_group=2, routed_scale=2.5,
                     n_shared=1, shared_range=(tokens // 8, tokens), seed=1550 + tokens)
    case = Case(wl)
    sr = wl.shared_range
    buf = case.layer.forward(case.x_dev, shared_range=sr)
    names = kernels_of(lambda s: case.layer.forward(case.x_dev, out=buf, shared_range=sr, stream=s))
    assert names[-3:] == ["k_expert_ring<true, false, 2>", "k_expert_ring<false, false, 2>", "k_combine<unsigned short, 0>"], names
    assert tokens * (wl.top_k + 1) >= 48 * wl.n_slots
    out = case.run()
    v = case.layer.view(tokens)
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, tokens, sr)
    check_output(case, out, ids)
    np.testing.assert_array_equal(out, case.run(flags=B.MOE_FLAG_PERMUTE_UNFUSED))
    np.testing.assert_array_equal(out, tensor_to_host(case.layer.forward_static(case.x_dev, shared_range=sr)))
    spare = sorted(set(range(wl.n_slots)) - set(case.expert_map.tolist()) - set(case.shared_slots.tolist()))
    copies = [[int(s)] if s >= 0 else [] for s in case.expert_map]
    for s, e in zip(spare, np.flatnonzero(case.expert_map >= 0)):
        case.layer.w13[s], case.layer.w2[s] = case.layer.w13[copies[e][0]], case.layer.w2[copies[e][0]]
        copies[e].append(int(s))
    case.layer.set_expert_replicas(copies, case.shared_slots.tolist())
    assert max(len(c) for c in copies) == 2
    np.testing.assert_array_equal(out, case.run())


@pytest.mark.parametrize("hidden,inter,experts,k,local,tokens,kernel", [
    (2048, 768, 64, 4, 16, 320, "k_expert_ring"), (2048, 768, 64, 4, 16, 321, "k_expert_gemm_mfma8"),            # 20 rows a slot
    (2048, 768, 128, 8, 84, 145, "k_expert_ring"),                                                               # 793 MB in use
    (2048, 768, 128, 8, 85, 144, "k_expert_ring"), (2048, 768, 128, 8, 85, 145, "k_expert_gemm_mfma8"),          # 802 MB: 9 rows a slot
    (1984, 768, 128, 8, 32, 100, "k_expert_ring"), (1984, 768, 128, 8, 33, 100, "k_expert_gemm_mfma"),           # shorter rows: 293 and 302 MB
    (2048, 768, 128, 8, 33, 100, "k_expert_ring"),
    (4096, 128, 128, 8, 33, 100, "k_expert_ring"), (4160, 128, 128, 8, 33, 100, "k_expert_gemm_mfma")])
def test_ring_tiles_of_64_rows_at_the_limits(hidden, inter, experts, k, local, tokens, kernel):
    """Both sides of every limit of the rule that sends a pass to them.  (Nothing runs: the weights are whatever the memory holds.)"""
    import types
    import torch
    from paper_2510_02613_amd.layer import MoELayer
    layer = MoELayer(hidden=hidden, inter=inter, n_experts=experts, top_k=k, n_slots=local, max_tokens=tokens, act_dtype="bf16", router_dtype="f32",
                     gate="softmax", router_w=np.zeros((experts, hidden), np.float32))
    layer.set_expert_map(list(range(local)) + [-1] * (experts - local))
    x = torch.empty(tokens, hidden, dtype=torch.int16, device="cuda:0")
    assert _expert_kernels(types.SimpleNamespace(layer=layer, x_dev=x), tokens) == kernel


@pytest.mark.parametrize("tokens,shared,kernel", [(320, 320, "k_expert_ring"), (321, 321, "k_expert_gemm_mfma8"), (1280, 320, "k_expert_ring"),
                                                  (1280, 321, "k_expert_gemm_mfma8"), (1281, 320, "k_expert_gemm_mfma8")])
def test_ring_tiles_of_64_rows_up_to_320_shared_rows(tokens, shared, kernel):
    """Top-1 of 64 experts: 20 assignments a slot are 1280 tokens, but a shared expert's weights are read once per 64 of its rows."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    wl = MoEWorkload(name="few_shared", tokens=tokens, hidden=128, inter=192, n_experts=64, top_k=1, n_slots=9, n_local=8, act_dtype="bf16",
                     router_dtype="f32", gate="softmax", n_shared=1, shared_range=(tokens - shared, tokens), seed=1580)
    case = Case(wl)
    assert _expert_kernels(case, tokens, wl.shared_range) == kernel
    out = case.run()
    v = case.layer.view(tokens)
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, tokens, wl.shared_range)
    check_output(case, out, ids)


@pytest.mark.parametrize("tokens,experts,k,local,routed,kernel", [
    (858, 64, 1, 8, True, "k_expert_ring"), (859, 64, 1, 8, True, "k_expert_gemm_mfma8"),       # 352 tasks of up to 64 rows, 528 on 8 slots
    (1163, 64, 1, 7, True, "k_expert_ring"), (1164, 64, 1, 7, True, "k_expert_gemm_mfma8"),     # 462 on 7 slots, 616
    (959, 64, 1, 20, True, "k_expert_ring"), (960, 64, 1, 20, True, "k_expert_gemm_mfma8"),     # not large: 440; large
    (622, 256, 8, 48, True, "k_expert_ring"), (623, 256, 8, 48, True, "k_expert_gemm_mfma8"),   # 24 rows a slot
    (96, 64, 1, 3, True, "k_expert_decode"), (97, 64, 1, 3, True, "k_expert_ring"),             # 528 tasks of 16 rows, 792
    (112, 64, 1, 7, True, "k_expert_decode"), (113, 64, 1, 7, True, "k_expert_ring"),           # 16 rows a slot
    (256, 64, 1, 2, True, "k_expert_ring"), (1024, 256, 1, 2, True, "k_expert_ring"),
    (1280, 64, 1, 8, False, "k_expert_ring"), (1280, 64, 1, 4, True, "k_expert_ring"), (1280, 64, 1, 64, True, "k_expert_ring")])
def test_routed_passes_count_the_rows_that_arrive(tokens, experts, k, local, routed, kernel):
    """Experts 1408 wide (22 tasks of the ring kernels a tile, 88 of the register ones): tokens that arrive routed have an expert here, so that
    few local ones expect many rows each, where a gated pass of as many tokens has T k / E.  Both sides of every limit."""
    from gpu_util import Case
    from test_gpu_routed import _check
    wl = MoEWorkload(name="arrive", tokens=tokens, hidden=64, inter=1408, n_experts=experts, top_k=k, n_slots=local, n_local=local, act_dtype="bf16",
                     router_dtype="f32", gate="softmax", seed=1590)
    case = Case(wl)
    assert _expert_kernels(case, tokens, routed=routed) == kernel
    if not routed:
        return
    g = np.random.Generator(np.random.PCG64(tokens))
    ids = np.concatenate([g.integers(0, local, size=(tokens, 1)), g.integers(0, experts, size=(tokens, k - 1))], 1).astype(np.int32)
    _check(case, ids, g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32))
    most = case.layer.view(tokens)["tiles"][:, 2].max()
    assert most <= {"k_expert_ring": 64, "k_expert_decode": 16}.get(kernel, 320) and (tokens < 32 * local or most > 32 or kernel == "k_expert_decode")


@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("tokens", [1, 16, 17, 64, 65, 256, 257])
@pytest.mark.parametrize("hidden,inter", [(8, 8), (64, 40), (200, 24), (24, 136), (136, 40), (136, 48), (1024, 8)])
def test_small_layers_token_by_token(act, tokens, hidden, inter):
    """Small layers whose experts run in one launch behind the bookkeeping (up to 256 tokens and 256 KB of weights per token; the
    first sizes past either go the common way): rows shorter and longer than 16 lanes' loads, one and several rounds of weight rows,
    shared rows, tokens without local experts.  Output, h, y and tables as with separate bookkeeping, bit for bit, and within the
    oracle's bar."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="token", tokens=tokens, hidden=hidden, inter=inter, n_experts=24, top_k=3, n_slots=22, n_local=12,
                     act_dtype=act, router_dtype="f32", gate="sigmoid_group", n_group=4, topk_group=2, routed_scale=2.5,
                     n_shared=1, shared_range=(tokens // 3, tokens // 3 + min(30, tokens - tokens // 3)), seed=1600 + tokens)
    case = Case(wl)
    small = tokens <= 256 and 3 * 4 * hidden * inter * (4 if act == "f32" else 2) <= 256 * 1024
    assert (_expert_kernels(case, tokens, wl.shared_range) == "k_token_experts") == small
    runs = []
    for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
        out = case.run(flags=flags)
        runs.append((out, case.layer.view(tokens)))
    ids, _, _ = check_routing(case, runs[0][1]["topk_ids"], runs[0][1]["topk_w"])
    check_bookkeeping(case, runs[0][1], tokens, wl.shared_range)
    check_output(case, runs[0][0], ids)
    np.testing.assert_array_equal(runs[0][0], runs[1][0])
    for key in ("counts", "offsets", "perm", "inv", "tiles", "h", "y"):
        np.testing.assert_array_equal(runs[0][1][key], runs[1][1][key])


@pytest.mark.parametrize("act,router", [("f32", "f32"), ("f32", "bf16"), ("bf16", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("tokens,experts,k,gate,hidden,inter,one", [
    (1, 8, 2, "softmax", 8, 8, True), (16, 64, 4, "sigmoid_group", 512, 8, True), (16, 40, 3, "softmax", 136, 24, True),
    (17, 32, 4, "softmax", 136, 24, True), (17, 33, 4, "softmax", 136, 24, False), (32, 17, 3, "sigmoid", 512, 8, True),
    (32, 16, 3, "sigmoid_group", 64, 40, False), (33, 16, 3, "sigmoid", 136, 24, True), (64, 16, 3, "softmax", 512, 8, True), (50, 16, 15, "softmax", 64, 16, True),
    (33, 16, 16, "softmax", 64, 16, False), (33, 17, 3, "softmax", 136, 24, False), (64, 9, 2, "softmax", 40, 64, True), (65, 16, 3, "softmax", 64, 40, False)])
def test_small_layers_gate_and_experts_in_one_launch(act, router, tokens, experts, k, gate, hidden, inter, one):
    """Few tokens of a small layer in one launch, the gate too: token tiles of 16, 32 and 64 tokens with 64, 32 and 16 lanes selecting a token, and the
    first sizes past each; shares of the contraction, equal scores, a selection bias, copies of an expert, experts elsewhere, a shared one on part of the batch.  Ids, weights, tables,
    h, y and output as with separate kernels, bit for bit, on a workspace poisoned before every pass; also with the placement as an argument.  (Many experts a token on rows of 64, not of 8:
    the oracle's bar is relative to a row's largest value, and sixteen terms rounded to bf16 can cancel to a quarter of one in all of eight values: 33 tokens, 8 x 40, row error 1.16e-2 in the separate kernels too.)"""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing, tensor_to_host
    from paper_2510_02613_amd import binding as B
    kw = dict(n_group=4, topk_group=2, routed_scale=2.5) if gate == "sigmoid_group" else {}
    wl = MoEWorkload(name="one", tokens=tokens, hidden=hidden, inter=inter, n_experts=experts, top_k=k, n_slots=experts + 4, n_local=experts - 2,
                     act_dtype=act, router_dtype=router, gate="softmax" if gate == "softmax" else "sigmoid_group", n_shared=1,
                     shared_range=(tokens // 3, tokens // 3 + (tokens + 1) // 2), seed=1900 + tokens + experts, **kw)
    case = Case(wl, select_bias=(np.arange(experts) * 5 % experts // 3 * 0.004).astype(np.float32))
    names = _kernels(case, tokens, wl.shared_range)
    read = ((32 if tokens <= 32 else 64) * (4 if act == "f32" else 2) + experts * (4 if router == "f32" else 2)) * hidden   # by every workgroup
    assert (names == ["k_token_experts"]) == (one and (tokens <= 16 or read <= 96 * 1024))
    scratch = B.moe_workspace_view(case.layer.handle).topk_ids - case.layer.workspace.data_ptr()
    keys = ("topk_ids", "topk_w", "counts", "offsets", "perm", "inv", "tiles", "h", "y")

    def both():
        runs = []
        for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
            case.layer.workspace[scratch:].fill_(0xff)
            runs.append((case.run(flags=flags), case.layer.view(tokens)))
        np.testing.assert_array_equal(runs[0][0], runs[1][0])
        for key in keys:
            np.testing.assert_array_equal(runs[0][1][key], runs[1][1][key])
        return runs[0]
    out, v = both()
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, tokens, wl.shared_range)
    check_output(case, out, ids)
    np.testing.assert_array_equal(out, tensor_to_host(case.layer.forward_static(case.x_dev, shared_range=wl.shared_range)))
    slots = case.shared_slots
    spare = [s for s in range(wl.n_slots) if s not in set(int(m) for m in case.expert_map) | set(int(s) for s in slots)][:2]
    for s in spare:
        case.layer.load_slot(s, case.w13_pool[case.expert_map[1]], case.w2_pool[case.expert_map[1]])
    case.layer.set_expert_replicas([[int(m)] + (spare if e == 1 else []) if m >= 0 else [] for e, m in enumerate(case.expert_map)], slots)
    both()
    case.layer.set_expert_map(case.expert_map, slots)
    case.layer.router_w.zero_()                    # equal scores everywhere: the bias decides, in threes, then the lower expert
    both()
    case.layer.router_w.view(experts, hidden)[experts // 2, hidden - 1] = 0x7fc0 if router == "bf16" else float("nan")   # an expert (softmax: every one) scores NaN
    both()


_ON_X = [   # act, tokens, experts, k, hidden, inter, flags, kernels of the pass with out on x
    ("f32", 1, 8, 2, 128, 56, 0, ["k_gate_small", "k_token_experts"]), ("f32", 16, 64, 4, 512, 8, 0, ["k_gate_small", "k_token_experts"]),
    ("f32", 64, 8, 2, 128, 56, 0, ["k_gate_small", "k_token_experts"]), ("bf16", 1, 8, 2, 128, 64, 0, ["k_gate_small", "k_token_experts"]),
    ("bf16", 32, 17, 3, 136, 24, 0, ["k_gate_small", "k_token_experts"]), ("bf16", 50, 16, 3, 136, 24, 0, ["k_gate_small", "k_token_experts"]),
    ("f32", 200, 8, 2, 128, 56, 0, "k_token_experts"), ("bf16", 256, 8, 2, 128, 64, 0, "k_token_experts"),
    ("f32", 20, 40, 4, 264, 264, 0, "k_expert_f32"), ("f32", 600, 40, 4, 264, 264, 0, "k_expert_f32_tile"),
    ("bf16", 1, 72, 4, 576, 512, 0, "k_expert_decode"), ("bf16", 7, 72, 4, 584, 520, 0, "k_expert_decode"),
    ("bf16", 4, 96, 8, 576, 512, 0, "k_expert_ring"), ("bf16", 47, 96, 4, 320, 320, 0, "k_expert_ring"), ("bf16", 300, 96, 4, 320, 320, 0, "k_expert_ring"),
    ("bf16", 700, 16, 4, 136, 200, 0, "k_expert_gemm_mfma"), ("bf16", 900, 16, 4, 64, 192, 0, "k_expert_gemm_mfma8"),
    ("bf16", 64, 16, 4, 136, 200, 2, "k_expert_gemm_generic"), ("bf16", 64, 16, 4, 136, 200, 1, "k_identity_experts")]


@pytest.mark.parametrize("act,tokens,experts,k,hidden,inter,flags,kernels", _ON_X)
def test_output_on_the_input(act, tokens, experts, k, hidden, inter, flags, kernels):
    """out = x with every family of expert kernels: output, ids, weights, tables, h and y as with a buffer of its own, bit for bit.  Small layers then have their gate in a launch of its own, in front of
    the one that writes out."""
    from gpu_util import Case, kernels_of
    wl = MoEWorkload(name="on_x", tokens=tokens, hidden=hidden, inter=inter, n_experts=experts, top_k=k, n_slots=experts, n_local=experts - 2,
                     act_dtype=act, router_dtype="f32", gate="softmax", n_shared=1, shared_range=(tokens // 3, tokens // 3 + (tokens + 2) // 4), seed=2100 + tokens)
    case = Case(wl)
    sr, x = wl.shared_range, case.x_dev

    def forward(inp, out, stream=None):
        return case.layer.forward(inp, out=out, shared_range=sr, flags=flags, stream=stream)
    names = [n.split("<")[0] for n in kernels_of(lambda s: forward(x, x, s))]
    assert names == kernels if isinstance(kernels, list) else kernels in names, names
    keys = ("topk_ids", "topk_w", "counts", "offsets", "perm", "inv", "tiles", "h", "y")
    want, v = forward(x, x.clone()), case.layer.view(tokens)
    own = x.clone()
    forward(own, own)
    w = case.layer.view(tokens)
    np.testing.assert_array_equal(own.cpu().numpy(), want.cpu().numpy())
    for key in keys:
        np.testing.assert_array_equal(v[key], w[key])
    if flags == 0 and tokens <= 64:
        own = x.clone()
        case.layer.forward_static(own, out=own, shared_range=sr)
        np.testing.assert_array_equal(own.cpu().numpy(), want.cpu().numpy())


@pytest.mark.parametrize("routed", [False, True])
@pytest.mark.parametrize("act,tokens,experts,k,hidden,inter", [("f32", 2, 8, 2, 128, 56), ("f32", 64, 8, 2, 128, 56), ("bf16", 50, 16, 3, 136, 24), ("f32", 200, 8, 2, 128, 56),
                                                               ("bf16", 256, 8, 2, 128, 64), ("bf16", 4, 96, 8, 576, 512), ("bf16", 300, 96, 4, 320, 320)])
def test_output_that_meets_the_input(act, tokens, experts, k, hidden, inter, routed):
    """out a few rows, or less than one, before or behind x: other kernels than token by token, and the output that a buffer of its own has, to the oracle's bar (bit for bit where the kernels are the same)."""
    import torch
    from gpu_util import TOL, Case, kernels_of, rel_err, tensor_to_host, to_f64
    wl = MoEWorkload(name="meets", tokens=tokens, hidden=hidden, inter=inter, n_experts=experts, top_k=k, n_slots=experts, n_local=experts - 2,
                     act_dtype=act, router_dtype="f32", gate="softmax", n_shared=1, shared_range=(0, tokens // 2), seed=2200 + tokens)
    case = Case(wl)
    sr, x = wl.shared_range, case.x_dev
    v = case.layer.forward(x, shared_range=sr) is not None and case.layer.view(tokens)
    ids, w = (torch.from_numpy(np.ascontiguousarray(v[key])).to(x.device) for key in ("topk_ids", "topk_w"))

    def forward(inp, out, stream=None):
        if routed:
            return case.layer.forward_routed(inp, ids, w, out=out, shared_range=sr, stream=stream)
        return case.layer.forward(inp, out=out, shared_range=sr, stream=stream)
    want = tensor_to_host(forward(x, x.clone()))
    same = "k_token_experts" not in [n.split("<")[0] for n in kernels_of(lambda s: forward(x, x.clone(), s))]
    for shift in (8, hidden, 3 * hidden):                       # elements between the two
        for ahead in (False, True):
            both = torch.empty(tokens * hidden + shift, dtype=x.dtype, device=x.device)
            lo, hi = both[:tokens * hidden].view(tokens, hidden), both[shift:].view(tokens, hidden)
            inp, out = (hi, lo) if ahead else (lo, hi)
            if shift < tokens * hidden:
                names = [n.split("<")[0] for n in kernels_of(lambda s: forward(inp, out, s))]
                assert "k_token_experts" not in names, names
            inp.copy_(x)
            got = tensor_to_host(forward(inp, out))
            if same:
                np.testing.assert_array_equal(got, want)
            assert rel_err(to_f64(got), to_f64(want)) <= TOL[act]


@pytest.mark.parametrize("tokens,experts,k,local,shared", [(33, 256, 4, 60, 1), (64, 256, 4, 63, 1), (65, 96, 3, 63, 2), (65, 256, 8, 254, 0), (128, 256, 8, 200, 0), (256, 64, 4, 61, 1), (257, 64, 4, 20, 4),
                                                           (511, 256, 4, 255, 1), (513, 256, 4, 256, 1), (1024, 256, 4, 129, 1), (1025, 256, 4, 129, 1)])
def test_ring_kernels_derive_the_tiles_of_many_tokens(tokens, experts, k, local, shared):
    """The ring's GEMM-1 that derives its tiles for up to 1024 tokens and 256 slots, at the ends of blocks of 16 tokens, of the 16 blocks of a load, of a slot per lane, of a workgroup's share
    of the tables, and the first sizes past it: several tiles a slot, experts elsewhere, a slot without rows, copies of an expert.  Tables, h, y and output as with separate bookkeeping kernels, bit for bit, on a
    workspace poisoned before every pass."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="many", tokens=tokens, hidden=128, inter=128, n_experts=experts, top_k=k, n_slots=local + shared, n_local=local - 2,
                     act_dtype="bf16", router_dtype="bf16", gate="softmax", n_shared=shared, shared_range=(0, min(tokens, 300) if shared else 0), seed=2000 + tokens + local)
    case = Case(wl, expert_map=block_expert_map(experts, 0, local - 2, np.random.Generator(np.random.PCG64(local)).permutation(local)[:local - 2]))
    names = _kernels(case, tokens, wl.shared_range)
    assert "k_expert_ring" in names and ("k_scan_place" in names) == (tokens > 1024 or local + shared > 256), names
    scratch = B.moe_workspace_view(case.layer.handle).topk_ids - case.layer.workspace.data_ptr()

    def both():
        runs = []
        for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
            case.layer.workspace[scratch:].fill_(0xff)
            runs.append((case.run(flags=flags), case.layer.view(tokens)))
        np.testing.assert_array_equal(runs[0][0], runs[1][0])
        for key in ("topk_ids", "topk_w", "counts", "offsets", "perm", "inv", "tiles", "h", "y"):
            np.testing.assert_array_equal(runs[0][1][key], runs[1][1][key])
        return runs[0]
    out, v = both()
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, tokens, wl.shared_range)
    check_output(case, out, ids)
    taken = set(int(m) for m in case.expert_map) | set(int(s) for s in case.shared_slots)
    spare = [s for s in range(wl.n_slots) if s not in taken][:2]
    case.layer.set_expert_replicas([[int(m)] + (spare if e == 1 else []) if m >= 0 else [] for e, m in enumerate(case.expert_map)], case.shared_slots if shared else None)
    both()
    case.layer.set_expert_map(case.expert_map, case.shared_slots if shared else None)
    case.layer.router_w.zero_()                    # equal scores: every token takes the first k experts, slots with all of them
    both()


@pytest.mark.parametrize("tokens,experts,k,routed,flags,tiles", [
    (300, 64, 4, False, 0, "2"), (300, 64, 4, True, 0, "2, TileList"), (300, 64, 4, False, 8, "2, TileList"), (1024, 256, 4, False, 0, "2, TileList"), (1025, 256, 4, False, 0, "2, TileList"),
    (90, 96, 4, False, 0, "1"), (90, 96, 4, True, 0, "1, TileList"), (47, 96, 4, True, 0, "1, TileList"), (47, 96, 4, False, 8, "1, TileList")])
def test_ring_kernels_that_read_the_tile_list(tokens, experts, k, routed, flags, tiles):
    """Which instance of the ring's GEMM-1 a pass launches: the one that reads the list behind every pass with a bookkeeping kernel.  (Nothing runs.)"""
    import types
    import torch
    from gpu_util import kernels_of
    from paper_2510_02613_amd.layer import MoELayer
    layer = MoELayer(hidden=320, inter=320, n_experts=experts, top_k=k, n_slots=experts, max_tokens=tokens, act_dtype="bf16", router_dtype="f32",
                     gate="softmax", router_w=np.zeros((experts, 320), np.float32))
    layer.set_expert_map(list(range(experts)))
    x = torch.empty(tokens, 320, dtype=torch.int16, device="cuda:0")
    ids, w = (torch.zeros((tokens, k), dtype=t, device=x.device) for t in (torch.int32, torch.float32))
    out = torch.empty_like(x)
    names = kernels_of(lambda s: layer.forward_routed(x, ids, w, out=out, flags=flags, stream=s) if routed else layer.forward(x, out=out, flags=flags, stream=s))
    assert f"k_expert_ring<true, false, {tiles}>" in names, names
    assert any(n.split("<")[0] in ("k_scan_place", "k_hist_place", "k_slot_place", "k_permute_one_block") for n in names) == ("TileList" in tiles), names


@pytest.mark.parametrize("tokens,slots,hidden,inter,derives", [
    (1024, 256, 1024, 64, True), (1024, 256, 960, 64, True), (700, 256, 960, 128, False), (256, 256, 320, 256, True), (257, 256, 320, 256, False),
    (512, 256, 128, 128, True), (513, 256, 128, 128, False), (512, 256, 256, 256, False), (1024, 128, 320, 192, True), (1024, 128, 320, 256, False), (1024, 64, 320, 320, True)])
def test_ring_kernels_derive_tiles_where_that_is_cheap(tokens, slots, hidden, inter, derives):
    """GEMM-1 on both sides of the line on its workgroups times what each adds up, short rows and long ones: the pass's launches, and the same bits as with the separate bookkeeping kernels."""
    from gpu_util import Case, kernels_of
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="cheap", tokens=tokens, hidden=hidden, inter=inter, n_experts=256, top_k=4, n_slots=slots, n_local=slots, act_dtype="bf16", router_dtype="bf16", gate="softmax", seed=2300 + tokens)
    case = Case(wl)
    out = case.x_dev.clone()
    names = kernels_of(lambda s: case.layer.forward(case.x_dev, out=out, stream=s))
    first = next(n for n in names if n.startswith("k_expert_ring<true"))
    assert ("TileList" not in first) == derives == (not any(n.startswith("k_scan_place") for n in names)), names
    out, v = case.run(), case.layer.view(tokens)
    np.testing.assert_array_equal(case.run(flags=B.MOE_FLAG_PERMUTE_UNFUSED), out)
    w = case.layer.view(tokens)
    for key in ("counts", "offsets", "perm", "inv", "tiles", "h", "y"):
        np.testing.assert_array_equal(v[key], w[key])


@pytest.mark.parametrize("tokens", [1, 2, 3])
@pytest.mark.parametrize("hidden,inter", [(136, 512), (72, 520), (64, 1024), (104, 1544), (4096, 72), (4104, 72)])
def test_second_gemm_and_combine_of_a_token_or_two(tokens, hidden, inter):
    """One launch for GEMM-2 and combine (one token; two on rows of up to 4096): contractions of one to four pieces of 512 with and
    without a remainder, more local experts than the workgroup has wavefronts, experts on other ranks, a shared one.  Output, h, y and
    tables as with separate bookkeeping, bit for bit, and within the oracle's bar."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="two", tokens=tokens, hidden=hidden, inter=inter, n_experts=40, top_k=13, n_slots=40, n_local=36,
                     act_dtype="bf16", router_dtype="f32", gate="softmax", n_shared=1, shared_range=(0, 1), seed=1700 + hidden)
    case = Case(wl)
    assert ("k_gemm2_combine" in _kernels(case, tokens, wl.shared_range)) == (tokens == 1 or (tokens == 2 and hidden <= 4096))
    runs = []
    for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
        out = case.run(flags=flags)
        runs.append((out, case.layer.view(tokens)))
    ids, _, _ = check_routing(case, runs[0][1]["topk_ids"], runs[0][1]["topk_w"])
    check_bookkeeping(case, runs[0][1], tokens, wl.shared_range)
    check_output(case, runs[0][0], ids)
    np.testing.assert_array_equal(runs[0][0], runs[1][0])
    for key in ("counts", "offsets", "perm", "inv", "tiles", "h", "y"):
        np.testing.assert_array_equal(runs[0][1][key], runs[1][1][key])


@pytest.mark.parametrize("hidden,inter", [(8, 8), (16, 24), (40, 264), (264, 40), (96, 136)])
def test_f32_tiles_of_64_rows(hidden, inter):
    """The fp32 kernel for larger groups: chunks of 64 rows and what is left of every number of 16-row groups, on contractions
    below, at and past a K-step of 32 and with every remainder of its four parts."""
    from gpu_util import Case
    from test_gpu_routed import _check
    counts = [1, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 80, 129]
    tokens = sum(counts)
    wl = MoEWorkload(name="f32_64", tokens=tokens, hidden=hidden, inter=inter, n_experts=len(counts), top_k=1, n_slots=len(counts),
                     n_local=len(counts), act_dtype="f32", router_dtype="f32", gate="softmax", seed=500 + hidden)
    g = np.random.Generator(np.random.PCG64(inter))
    ids = g.permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)[:, None]
    case = Case(wl)
    _check(case, ids, g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32))
    assert case.layer.view(tokens)["tiles"][:, 2].max() == 64


@pytest.mark.parametrize("act,router", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "bf16"), ("f32", "f32")])
@pytest.mark.parametrize("experts,hidden,tokens", [(4, 64, 1), (16, 512, 16), (17, 480, 17), (48, 136, 33), (64, 512, 64), (65, 512, 17), (64, 520, 17), (511, 64, 17), (512, 64, 17)])
def test_small_router_gate(act, router, experts, hidden, tokens):
    """Routers that are multiplied and selected from in one kernel (up to 64 experts, 512 wide) and the first sizes past
    it: 1 to 4 tiles of 16 experts, shares of the contraction with and without a remainder, one and several blocks of 16
    tokens; the pass that brings its placement along (512 table entries fit the argument) gives the same output."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing, tensor_to_host
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="gate", tokens=tokens, hidden=hidden, inter=64, n_experts=experts, top_k=2, n_slots=experts + 1, n_local=experts,
                     act_dtype=act, router_dtype=router, gate="softmax", n_shared=1, shared_range=(0, tokens), seed=500 + experts)
    case = Case(wl)
    out = case.run()
    v = case.layer.view(tokens)
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, tokens, wl.shared_range)
    check_output(case, out, ids)
    np.testing.assert_array_equal(out, case.run(flags=B.MOE_FLAG_PERMUTE_UNFUSED))
    np.testing.assert_array_equal(out, tensor_to_host(case.layer.forward_static(case.x_dev, shared_range=wl.shared_range)))


@pytest.mark.parametrize("experts,groups,kept", [(64, 4, 2), (128, 2, 1), (256, 8, 4), (256, 16, 4), (96, 4, 2), (512, 16, 8)])
def test_group_scores_leave_nan_experts_out(experts, groups, kept):
    """A NaN among the selection scores of a group (a NaN bias) counts neither as one of its two best nor in the place of
    one, whichever way the group's lanes are reduced (rows of 16, 32 and 64 lanes, or through LDS); the NaN expert itself
    sorts before every number when its group is kept."""
    from gpu_util import Case
    tokens, k = 200, 6
    wl = MoEWorkload(name="nan", tokens=tokens, hidden=128, inter=64, n_experts=experts, top_k=k, n_slots=experts, n_local=experts,
                     act_dtype="bf16", router_dtype="f32", gate="sigmoid_group", n_group=groups, topk_group=kept, seed=600 + experts)
    per = experts // groups
    nan_at = np.arange(groups // 2) * 2 * per + np.arange(groups // 2) * 7 % per   # one in every second group
    bias = np.zeros(experts, np.float32)
    bias[nan_at] = np.nan
    case = Case(wl, select_bias=bias)
    case.run()
    ids = case.layer.view(tokens)["topk_ids"]
    case.select_bias = None                                  # the scores without the bias, from the oracle
    c = case.oracle_route()[3].astype(np.float64)
    c[:, nan_at] = np.nan
    checked = 0
    for t in range(tokens):
        known = np.where(np.isnan(c[t]), -np.inf, c[t])
        best = np.sort(known.reshape(groups, per), axis=1)[:, ::-1]
        score = best[:, 0] + best[:, 1]
        order = np.sort(score)[::-1]
        rank = np.argsort(-score, kind="stable")[:kept]
        # scores are sigmoids: 2 and more stand for NaN (lower expert first, as all NaN are alike), -1 for dropped
        c_kept = np.where(np.isin(np.arange(experts) // per, rank), np.where(np.isnan(c[t]), 3.0 - np.arange(experts) / 1024, c[t]), -1.0)
        want = np.argsort(-c_kept, kind="stable")
        gaps = -np.diff(c_kept[want[:k + 1]])
        if order[kept - 1] - order[kept] > 2e-5 and (gaps >= 1e-5).all():
            np.testing.assert_array_equal(ids[t], want[:k], err_msg=f"token {t}")
            checked += 1
    assert checked > tokens // 2


@pytest.mark.parametrize("experts,k,groups,kept", [(257, 32, 1, 1), (320, 8, 1, 1), (320, 8, 10, 4), (384, 8, 6, 3), (512, 32, 8, 2), (513, 8, 1, 1)])
@pytest.mark.parametrize("tokens,hidden", [(1, 64), (33, 2048), (2100, 64)])
def test_selection_of_more_than_256_experts(experts, k, groups, kept, tokens, hidden):
    """Five to eight scores a lane, all kept in registers (and the first size past it), with one and with several planes of
    partial logits, in both forms of the selection kernel (2048 tokens) and in the one without ranking."""
    from gpu_util import Case, check_routing
    from paper_2510_02613_amd import binding as B
    wl = MoEWorkload(name="many", tokens=tokens, hidden=hidden, inter=64, n_experts=experts, top_k=k, n_slots=experts, n_local=8,
                     act_dtype="bf16", router_dtype="bf16", gate="softmax" if groups == 1 else "sigmoid_group", n_group=groups, topk_group=kept,
                     seed=1000 + experts)
    case = Case(wl)
    for flags in (0, B.MOE_FLAG_PERMUTE_UNFUSED):
        case.run(flags=flags)
        v = case.layer.view(tokens)
        check_routing(case, v["topk_ids"], v["topk_w"])


def test_kernel_choice_counts_the_slots_in_use():
    """A layer of 80 slots, 503 MB of weights, 7.5 assignments a slot: the large-tile kernels (320-row tiles) while all slots
    are in use, the 128 x 128 ones with 60 of them (377 MB); free slots hold no weights that a pass reads."""
    from gpu_util import Case
    from test_gpu_routed import _check
    wl = MoEWorkload(name="in_use", tokens=300, hidden=1024, inter=1024, n_experts=80, top_k=2, n_slots=80, n_local=80,
                     act_dtype="bf16", router_dtype="bf16", gate="softmax", seed=95)
    g = np.random.Generator(np.random.PCG64(4))
    ids = np.stack([np.concatenate([[5 if t < 250 else 6], 7 + g.permutation(73)[:1]]) for t in range(300)]).astype(np.int32)
    wts = g.uniform(0.5, 1.5, size=ids.shape).astype(np.float32)
    case = Case(wl)
    for used, tiles in ((80, 1), (60, 2), (80, 1)):
        case.expert_map = np.where(np.arange(80) < used, np.arange(80), -1).astype(np.int32)
        case.layer.set_expert_map(case.expert_map)
        _check(case, ids, wts)
        assert (case.layer.view(300)["tiles"][:, 0] == 5).sum() == tiles


@pytest.mark.parametrize("router,tokens", [("bf16", 8192), ("bf16", 18310), ("bf16", 18311), ("f32", 4577), ("f32", 4578), ("f32", 8193)])
def test_small_router_gate_of_many_tokens(router, tokens):
    """64 experts on rows of 512: both sides of where the separate logits kernel takes over from the one-kernel gate."""
    from gpu_util import Case, check_bookkeeping, check_output, check_routing
    wl = MoEWorkload(name="gate_many", tokens=tokens, hidden=512, inter=8, n_experts=64, top_k=2, n_slots=64, n_local=64,
                     act_dtype="bf16", router_dtype=router, gate="softmax", seed=78)
    case = Case(wl)
    out = case.run()
    v = case.layer.view(tokens)
    ids, _, _ = check_routing(case, v["topk_ids"], v["topk_w"])
    check_bookkeeping(case, v, tokens, wl.shared_range)
    check_output(case, out, ids)


def test_f32_grid_past_the_launch_limit():
    """16384 tokens on 1024 experts of 131072 columns: 2048 possible tiles of 8192 tasks of 256 threads are 2^32 threads, one
    more than a launch takes in one dimension.  W2 has one column per output, spread over the tasks, so that the reference
    needs only those columns of h."""
    import torch
    from paper_2510_02613_amd.layer import MoELayer
    T, E, H, I = 16384, 1024, 8, 131072
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(3)
    layer = MoELayer(hidden=H, inter=I, n_experts=E, top_k=1, n_slots=E, max_tokens=T, act_dtype="f32", router_dtype="f32",
                     gate="softmax", n_group=1, topk_group=1, renormalize=True, routed_scale=1.0, n_shared=0,
                     router_w=np.zeros((E, H), np.float32), device=dev)
    layer.w13.normal_(0.0, 0.5, generator=gen)
    layer.w2.zero_()
    cols = torch.linspace(0, I - 1, H, device=dev).round().long()
    layer.w2[:, torch.arange(H, device=dev), cols] = 1.0
    layer.set_expert_map(list(range(E)))
    x = torch.randn(T, H, generator=gen, device=dev)
    ids = torch.randperm(T, generator=gen, device=dev).to(torch.int32)[:, None] % E
    out = layer.forward_routed(x, ids, torch.ones(T, 1, device=dev))
    e = ids[:, 0].long()
    gate, up = ((layer.w13[e[:, None], c[None, :]].double() * x.double()[:, None, :]).sum(2) for c in (cols, cols + I))
    want = torch.nn.functional.silu(gate) * up
    assert float((out.double() - want).norm() / want.norm()) < 1e-6      # eight products and a hardware exp, each 2^-23


def test_f32_tiles_of_64_rows_past_one_row_of_the_grid():
    """33 rows a slot on 490 experts of 278528 columns: 8.5 million tasks of k_expert_f32_tile, more than the 2^23 of one row of the
    grid; every XCD's run of tasks ends in the second.  W2 as in the test above."""
    import torch
    from gpu_util import kernels_of
    from paper_2510_02613_amd.layer import MoELayer
    T, E, H, I = 16384, 490, 8, 278528
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(4)
    layer = MoELayer(hidden=H, inter=I, n_experts=E, top_k=1, n_slots=E, max_tokens=T, act_dtype="f32", router_dtype="f32",
                     gate="softmax", router_w=np.zeros((E, H), np.float32), device=dev)
    layer.w13.normal_(0.0, 0.5, generator=gen)
    layer.w2.zero_()
    cols = torch.linspace(0, I - 1, H, device=dev).round().long()
    layer.w2[:, torch.arange(H, device=dev), cols] = 1.0
    layer.set_expert_map(list(range(E)))
    x = torch.randn(T, H, generator=gen, device=dev)
    ids = torch.randperm(T, generator=gen, device=dev).to(torch.int32)[:, None] % E
    w = torch.ones(T, 1, device=dev)
    out = torch.empty_like(x)
    assert "k_expert_f32_tile<true, true>" in kernels_of(lambda s: layer.forward_routed(x, ids, w, out=out, stream=s))
    layer.forward_routed(x, ids, w, out=out)
    e = ids[:, 0].long()
    gate, up = ((layer.w13[e[:, None], c[None, :]].double() * x.double()[:, None, :]).sum(2) for c in (cols, cols + I))
    want = torch.nn.functional.silu(gate) * up
    assert float((out.double() - want).norm() / want.norm()) < 1e-6      # as above


@pytest.mark.parametrize("tokens,k,slots", [(128, 8, 16), (129, 8, 16), (1000, 4, 1500), (8192, 8, 40), (8193, 8, 40)])
def test_routed_bookkeeping_by_blocks(tokens, k, slots):
    """1024 assignments (one workgroup does it all), one more, more slots than a workgroup has threads, 65536 assignments (64
    blocks, the last that are scanned and placed in one launch) and 8 more; ids repeat within a token."""
    from gpu_util import Case
    from test_gpu_routed import _check, _routing
    wl = MoEWorkload(name="blocks", tokens=tokens, hidden=64, inter=8, n_experts=min(slots, 1024), top_k=k, n_slots=slots, n_local=min(slots, 1024),
                     act_dtype="bf16", router_dtype="bf16", gate="softmax", seed=1400)
    case = Case(wl)
    ids, wts = _routing(wl, tokens)
    _check(case, ids, wts)
    v = case.layer.view(tokens)
    flat = ids.reshape(-1)
    rows = np.where((flat >= 0) & (flat < wl.n_experts), 0, -1)
    slot = np.where(rows == 0, case.expert_map[np.clip(flat, 0, wl.n_experts - 1)], slots)
    order = np.argsort(slot, kind="stable")[:int((rows == 0).sum())]      # rows: by slot, then token and selection position
    want = np.full(len(flat), -1)
    want[order] = np.arange(len(order))
    np.testing.assert_array_equal(v["inv"].reshape(-1), want)
    np.testing.assert_array_equal(v["perm"][:len(order)], order // k)


@pytest.mark.parametrize("slots", [40, 1800])
@pytest.mark.parametrize("hidden,inter", [(2048, 64), (64, 2048)])
def test_large_tiles_on_long_rows_do_not_follow_the_slots(hidden, inter, slots):
    """Contractions of 2048, whose units of 129 to 320 rows may start anywhere in K: the same bits whichever slots the experts sit in,
    with a tile list that is ordered by size (40 slots) and with one that can get too long for that and stays in slot order (1800)."""
    import torch
    from paper_2510_02613_amd.layer import MoELayer
    E, k = 24, 8
    tokens = 48 * slots // k
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(hidden + slots)
    g = np.random.Generator(np.random.PCG64(slots))
    layer = MoELayer(hidden=hidden, inter=inter, n_experts=E, top_k=k, n_slots=slots, max_tokens=tokens, act_dtype="bf16", router_dtype="f32",
                     gate="softmax", router_w=np.zeros((E, hidden), np.float32), device=dev)
    counts = np.array([129, 160, 161, 192, 200, 224, 225, 256, 257, 288, 289, 320, 400, 1] + [140 + 16 * i for i in range(10)])
    if counts.sum() > tokens * k:                            # the small list: as many experts as the batch has assignments for
        counts[np.cumsum(counts) > tokens * k] = 0
    ids = np.full(tokens * k, -1, np.int32)
    ids[g.permutation(tokens * k)[:counts.sum()]] = g.permutation(np.repeat(np.arange(E), counts))
    ids = torch.from_numpy(ids.reshape(tokens, k)).to(dev)
    wts = torch.rand(tokens, k, generator=gen, device=dev) + 0.5
    x = torch.randn(tokens, hidden, generator=gen, device=dev).bfloat16().view(torch.int16)
    w13 = (torch.randn(E, 2 * inter, hidden, generator=gen, device=dev) * 0.05).bfloat16().view(torch.int16)
    w2 = (torch.randn(E, hidden, inter, generator=gen, device=dev) * 0.05).bfloat16().view(torch.int16)
    outs = []
    for order in (np.arange(E), slots - 1 - np.arange(E), g.permutation(slots)[:E]):
        at = torch.from_numpy(order.copy()).to(dev)
        layer.w13[at], layer.w2[at] = w13, w2
        layer.set_expert_map(order.tolist())
        outs.append(layer.forward_routed(x, ids, wts))
        tiles = layer.view(tokens)["tiles"]
        assert sorted(tiles[tiles[:, 3] == 1][:, 2]) == sorted(c for c in counts if 0 < c <= 320)   # the large-tile kernels ran
    assert outs[0].view(torch.bfloat16).float().abs().max() > 0
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


def test_split_last_round_does_not_follow_the_slots_of_a_long_list():
    """A contraction of 4096 on 300 tiles, a full round and 44 of another, under a list that can get too long to be ordered and stays in slot
    order: which tiles are the last ones follows from the slots, so none is shared out over K -- the same bits whichever slots the experts sit in."""
    import torch
    from paper_2510_02613_amd.layer import MoELayer
    E, k, slots, hidden, inter = 300, 8, 1800, 4096, 64
    tokens = 48 * slots // k
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(21)
    g = np.random.Generator(np.random.PCG64(21))
    layer = MoELayer(hidden=hidden, inter=inter, n_experts=E, top_k=k, n_slots=slots, max_tokens=tokens, act_dtype="bf16", router_dtype="f32",
                     gate="softmax", router_w=np.zeros((E, hidden), np.float32), device=dev)
    counts = g.integers(129, 321, size=E)
    ids = np.full(tokens * k, -1, np.int32)
    ids[g.permutation(tokens * k)[:counts.sum()]] = g.permutation(np.repeat(np.arange(E), counts))
    ids = torch.from_numpy(ids.reshape(tokens, k)).to(dev)
    wts = torch.rand(tokens, k, generator=gen, device=dev) + 0.5
    x = torch.randn(tokens, hidden, generator=gen, device=dev).bfloat16().view(torch.int16)
    w13 = (torch.randn(E, 2 * inter, hidden, generator=gen, device=dev) * 0.05).bfloat16().view(torch.int16)
    w2 = (torch.randn(E, hidden, inter, generator=gen, device=dev) * 0.05).bfloat16().view(torch.int16)
    outs = []
    for order in (np.arange(E), slots - 1 - np.arange(E)):
        at = torch.from_numpy(order.copy()).to(dev)
        layer.w13[at], layer.w2[at] = w13, w2
        layer.set_expert_map(order.tolist())
        outs.append(layer.forward_routed(x, ids, wts))
        assert len(layer.view(tokens)["tiles"]) == E                                     # the large-tile kernels ran
    assert torch.equal(outs[0], outs[1])
