"""Extend attention through the runner where its plan differs from the plain
one: key walks cut into parts, 128-row items, the page-wise store, and calls
that queue up behind each other. Against the fp64 oracle at
|gpu - ref| <= 2e-3 + 1e-2 |ref| and, in the 2-norm, at 2^-11 of out (each weight
is rounded to fp16, at most 2^-11 of itself) and 2^-14 of lse (fp32 sums of
scores up to about 2^6); stores bit for bit."""
import ctypes
import threading

import numpy as np
import pytest
import torch

from paper_2601_12784_amd import binding as B
from paper_2601_12784_amd.workloads import bf16_bits, build_extend
from test_gpu_extend import assert_close, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


CASES = {
    # few rows after long prefixes: 128-row items, walks cut into many parts; a diagonal that starts inside a part
    "long_walks": ([5000, 33, 2050], [3, 1, 40]),
    # parts in which the first rows of a block see no key at all
    "diagonal": ([1500], [1500]),
    # 384-row items cut, one sequence with no new tokens
    "large_cut": ([3000, 2900, 40, 3100], [260, 200, 0, 300]),
    # parts that end in a ragged page, with a block of one token
    "ragged": ([1999, 2001, 1985], [129, 56, 1]),
}


@pytest.mark.parametrize("store", [False, True])
@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("shape", [(28, 4, 128), (16, 1, 128), (3, 3, 64), (8, 2, 64)], ids=lambda s: "x".join(map(str, s)))
def test_runner_plan_matches_oracle(shape, case, store):
    hq, hkv, d = shape
    lens, qls = CASES[case]
    print(f"extend runner {case} {shape} store={store}", flush=True)
    eb = build_extend(lens, qls, hq, hkv, d, seed=41 + len(case) + hq, k_mult=2.0)
    k0, v0 = bf16_bits(eb.batch.k_pool).copy(), bf16_bits(eb.batch.v_pool).copy()
    kp = vp = None
    if store:   # the new tokens' slots hold NaN until the store writes them
        pages, slots = eb.slots()
        kh, vh = k0.copy(), v0.copy()
        kh[pages, :, :, slots, :] = 0x7FC0
        vh[pages, :, :, slots] = 0x7FC0
        kp, vp = (torch.from_numpy(x.view(np.int16)).view(torch.bfloat16) for x in (kh, vh))
    out, lse, k1, v1, _ = run_gpu(eb, store=store, k_pool=kp, v_pool=vp)
    assert np.array_equal(bf16_bits(k1), k0) and np.array_equal(bf16_bits(v1), v0)
    ref = run_oracle(eb)
    assert_close(out, lse, ref, f"{case} {shape}")
    rel, far = np.linalg.norm(out - ref[0]) / np.linalg.norm(ref[0]), np.abs(lse - ref[1]).max()
    print(f"  rel {rel:.2e}, lse {far:.2e}", flush=True)
    assert rel < 2.0 ** -11 and far < 2.0 ** -14


CUT = {   # lens, q_lens, heads; rows per item of the runner's plan
    "large": ([2600, 700], [300, 700], (28, 4, 128), 384),
    "resumed": ([8000] * 4, [256] * 4, (28, 4, 128), 384),
    "prompt": ([1000], [1000], (28, 4, 128), 128),
    "one_token": ([12774, 40, 9000], [1, 3, 2], (8, 8, 64), 128),
    "large_64": ([6000] * 6, [300] * 6, (32, 2, 64), 384),
}


@pytest.mark.parametrize("case", sorted(CUT))
def test_cut_walks_agree_with_whole_ones(case):
    """The same call through sf_extend_attn (whole 384-row items). A part takes
    its rows' softmax reference from the walk's first step, so both plans round
    the same weights to fp16 and the results differ by fp32 rounding alone: the
    merge's weights by the rounding of lse (below 32 in log2 units: 2^-20 ln 2
    each), the sums by a few 2^-24 per square root of the steps."""
    lens, qls, (hq, hkv, d), rows = CUT[case]
    print(f"extend cut and whole: {case}", flush=True)
    eb = build_extend(lens, qls, hq, hkv, d, seed=5)
    b = eb.batch
    desc = B.make_desc(len(lens), hq, hkv, d, b.block_table.shape[1], b.num_pages, b.scale)
    counts = np.zeros(5, np.int32)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    B.lib().sf_debug_extend_plan(desc, b.seq_lens.ctypes.data, eb.q_lens.ctypes.data, cus, 0, None, 0, counts.ctypes.data)
    assert counts[0] == rows and counts[2] > 0   # the runner cuts walks here
    out, lse, *_ = run_gpu(eb)
    info, work = B.sf_extend_attn_plan(desc, b.seq_lens, eb.q_lens)
    o2 = torch.empty(out.shape, dtype=torch.float32, device="cuda")
    l2 = torch.empty(lse.shape, dtype=torch.float32, device="cuda")
    B.sf_extend_attn(desc, info, None, torch.from_numpy(work).cuda(), eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(),
                     torch.from_numpy(b.block_table).cuda(), o2, l2)
    torch.cuda.synchronize()
    rel = float((o2.cpu() - torch.from_numpy(out)).norm() / o2.cpu().norm())
    far = float(np.abs(l2.cpu().numpy() - lse).max())
    print(f"  rel {rel:.2e}, lse {far:.2e}", flush=True)
    assert rel < 2.0 ** -17 and far < 2.0 ** -17


def test_queued_calls_with_growing_and_shrinking_plans():
    """Calls queue up without a wait between them, on two streams in turn, with
    plans that outgrow the lent memory and shrink again; each result is the
    call's own, bit for bit."""
    ebs = [build_extend(lens, qls, 28, 4, 128, seed=60 + i) for i, (lens, qls) in enumerate(
        [([300], [20]), ([4000, 4100], [64, 100]), ([90, 17], [90, 1]), ([6000], [700]), ([500], [500])])]
    data = []
    for eb in ebs:
        b = eb.batch
        data.append((eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(),
                     b.seq_lens, eb.q_lens, b.scale))
    want = []
    for x in data:
        want.append(B.ExtendAttention(28, 4, 128)(*x))
        torch.cuda.synchronize()
    call = B.ExtendAttention(28, 4, 128)
    side = torch.cuda.Stream()
    outs = []
    for i in range(60):
        x = data[(i * 7 + i // 9) % len(data)]
        out = torch.empty_like(want[(i * 7 + i // 9) % len(data)])
        torch.cuda.synchronize() if i % 20 == 19 else None
        outs.append(call(*x, out=out, stream=side if i // 10 % 2 else None))
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        assert torch.equal(out, want[(i * 7 + i // 9) % len(data)]), f"call {i}"


def test_captured_stream_is_left_to_the_plain_entry_point():
    """sf_runner_extend refuses a capturing stream before it launches or records
    anything, so the capture goes on."""
    call = B.ExtendAttention(8, 2, 64)
    eb = build_extend([60], [60], 8, 2, 64, seed=2)
    b = eb.batch
    args = (eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda())
    out = torch.empty((60, 8, 64), dtype=torch.float32, device="cuda")
    call(*args, b.seq_lens, eb.q_lens, b.scale, out=out)
    torch.cuda.synchronize()
    desc = B.make_desc(1, 8, 2, 64, b.block_table.shape[1], b.num_pages, b.scale)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        st = call._L.sf_runner_extend(call._runner, desc, b.seq_lens.ctypes.data, eb.q_lens.ctypes.data,
                                      *(t.data_ptr() for t in args[:1]), None, None, *(t.data_ptr() for t in args[1:]),
                                      out.data_ptr(), None, call._memory, torch.cuda.current_stream().cuda_stream,
                                      B.sf_extend_info())
        out.add_(1.0)
    before = out.clone()
    graph.replay()
    torch.cuda.synchronize()
    assert st == B.UNSUPPORTED and torch.equal(out, before + 1.0)


@pytest.mark.parametrize("lens,qls", [([60], [60]), ([3000, 700, 40], [300, 700, 1])])
def test_call_after_a_warm_one_is_captured(lens, qls):
    """A captured call allocates no pinned memory after an eager one over the same
    batch, and its graph keeps its own work list: replays with other eager calls
    of the object between them all give the eager result of the whole items."""
    eb, other = build_extend(lens, qls, 28, 4, 128, seed=4), build_extend([9000], [700], 28, 4, 128, seed=9)
    b, c = eb.batch, other.batch
    args = (eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens, eb.q_lens,
            b.scale)
    args2 = (other.q.cuda(), c.k_pool.cuda(), c.v_pool.cuda(), torch.from_numpy(c.block_table).cuda(), c.seq_lens,
             other.q_lens, c.scale)
    out = torch.zeros((int(sum(qls)), 28, 128), dtype=torch.float32, device="cuda")
    desc = B.make_desc(len(lens), 28, 4, 128, b.block_table.shape[1], b.num_pages, b.scale)
    info, work = B.sf_extend_attn_plan(desc, b.seq_lens, eb.q_lens)
    want = torch.zeros_like(out)
    B.sf_extend_attn(desc, info, None, torch.from_numpy(work).cuda(), *args[:4], want)
    call = B.ExtendAttention(28, 4, 128)
    call(*args, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(*args, out=out)
    first = None
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        again = call(*args2)   # outgrows the lent memory
        torch.cuda.synchronize()
        first = again if first is None else first
        assert torch.equal(again, first)


def _hip():
    """The HIP runtime that this process has loaded."""
    with open("/proc/self/maps") as f:
        path = next(x.split()[-1] for x in f if "libamdhip64" in x)
    return ctypes.CDLL(path)


def test_streams_that_end_between_calls():
    """An object's calls on streams that their owner destroys afterwards: nothing
    of an earlier call is recorded on its stream later, neither when the next
    call comes on another stream, nor when a slot is used again, nor when the
    lent memory grows."""
    hip = _hip()
    small, large = build_extend([300], [20], 28, 4, 128, seed=31), build_extend([6000], [700], 28, 4, 128, seed=32)
    args = []
    for eb in (small, large):
        b = eb.batch
        args.append((eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens,
                     eb.q_lens, b.scale))
    want = [B.ExtendAttention(28, 4, 128)(*x) for x in args]
    torch.cuda.synchronize()
    call = B.ExtendAttention(28, 4, 128)
    for i, (which, calls) in enumerate([(0, 1), (0, 40), (1, 1), (0, 2), (1, 9)]):
        h = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(h)) == 0
        outs = [torch.empty_like(want[which]) for _ in range(calls)]
        torch.cuda.synchronize()
        for out in outs:
            call(*args[which], out=out, stream=h.value)
        assert hip.hipStreamSynchronize(h) == 0 and hip.hipStreamDestroy(h) == 0
        for out in outs:
            assert torch.equal(out, want[which]), f"stream {i}"
    assert torch.equal(call(*args[0]), want[0])
    torch.cuda.synchronize()


def test_graphs_of_one_object_keep_their_own_lists():
    """Two graphs of different batches captured from one object, with a growing
    eager call between the captures and eager calls between the replays: each
    replay reads the work list of its own capture. A batch captured again shares
    its list."""
    ebs = [build_extend(lens, qls, 28, 4, 128, seed=50 + i) for i, (lens, qls) in enumerate(
        [([300, 90], [300, 20]), ([2000, 40, 700], [64, 40, 700]), ([9000], [900])])]
    args, want = [], []
    for eb in ebs:
        b = eb.batch
        args.append((eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens,
                     eb.q_lens, b.scale))
        desc = B.make_desc(b.num_seqs, 28, 4, 128, b.block_table.shape[1], b.num_pages, b.scale)
        info, work = B.sf_extend_attn_plan(desc, b.seq_lens, eb.q_lens)
        want.append(torch.zeros((eb.num_rows, 28, 128), dtype=torch.float32, device="cuda"))
        B.sf_extend_attn(desc, info, None, torch.from_numpy(work).cuda(), *args[-1][:4], want[-1])
    outs = [torch.zeros_like(w) for w in want[:2]]
    call = B.ExtendAttention(28, 4, 128)
    graphs = []
    for i in range(2):
        call(*args[i])
        torch.cuda.synchronize()
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[i]):
            call(*args[i], out=outs[i])
            call(*args[i], out=outs[i])
        call(*args[2])   # outgrows the lent memory
        torch.cuda.synchronize()
    assert len(call._captured) == 2
    for r in range(4):
        i = r % 2
        for o in outs:
            o.zero_()
        graphs[i].replay()
        call(*args[2 - r % 3])
        torch.cuda.synchronize()
        assert torch.equal(outs[i], want[i]) and not outs[1 - i].any(), f"replay {r}"


@pytest.mark.parametrize("side", [False, True])
def test_no_device_memory_for_a_cut_plan(side):
    """Where torch may not reserve the partial results of a cut plan, the call
    takes the whole items' plan; a later call with memory cuts again."""
    eb = build_extend([8000] * 4, [256] * 4, 28, 4, 128, seed=12)
    b = eb.batch
    args = (eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens, eb.q_lens,
            b.scale)
    desc = B.make_desc(4, 28, 4, 128, b.block_table.shape[1], b.num_pages, b.scale)
    info, work = B.sf_extend_attn_plan(desc, b.seq_lens, eb.q_lens)
    whole, out = (torch.zeros((eb.num_rows, 28, 128), dtype=torch.float32, device="cuda") for _ in range(2))
    B.sf_extend_attn(desc, info, None, torch.from_numpy(work).cuda(), *args[:4], whole)
    stream = torch.cuda.Stream() if side else None
    call = B.ExtendAttention(28, 4, 128)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    room = torch.cuda.memory_reserved() + (8 << 20)   # the plan asks for about 50 MB
    torch.cuda.set_per_process_memory_fraction(room / torch.cuda.get_device_properties(0).total_memory)
    try:
        call(*args, out=out, stream=stream)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(out, whole) and call.last_info.num_items == info.num_items
    out.zero_()
    torch.cuda.synchronize()
    call(*args, out=out, stream=stream)
    torch.cuda.synchronize()
    assert float((out - whole).norm() / whole.norm()) < 2.0 ** -17 and not torch.equal(out, whole)


def test_objects_share_scratch_over_threads_and_streams():
    """Two objects per thread in three threads, two of them on one stream and one
    on its own, all with cut plans at once: partial results are shared by the
    objects of a thread and stream, and by nobody else."""
    ebs = [build_extend(lens, qls, 28, 4, 128, seed=80 + i) for i, (lens, qls) in enumerate(
        [([8000] * 4, [256] * 4), ([3000, 2900], [260, 200]), ([1000], [1000])])]
    data, want = [], []
    for eb in ebs:
        b = eb.batch
        data.append((eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens,
                     eb.q_lens, b.scale))
        want.append(B.ExtendAttention(28, 4, 128)(*data[-1]))
    torch.cuda.synchronize()
    wrong = []

    def work(n, stream):
        with torch.cuda.stream(stream):
            calls = [B.ExtendAttention(28, 4, 128) for _ in range(2)]
            outs = [(i, calls[i % 2](*data[(n + i) % 3])) for i in range(24)]
            stream.synchronize()
            wrong.extend((n, i) for i, out in outs if not torch.equal(out, want[(n + i) % 3]))

    shared = torch.cuda.Stream()
    threads = [threading.Thread(target=work, args=(n, s)) for n, s in enumerate([shared, shared, torch.cuda.Stream()])]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong and not B._scratch._blocks


@pytest.mark.parametrize("lens,earlier", [([60], False), ([1000], True)])
def test_a_new_objects_first_call_plans_once(lens, earlier):
    """A short call fits what a new object lends, and a longer one the block that
    an object still alive has left."""
    eb = build_extend(lens, lens, 28, 4, 128, seed=3)
    b = eb.batch
    args = (eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens, eb.q_lens,
            b.scale)
    alive = B.ExtendAttention(28, 4, 128)
    if earlier:
        want = alive(*args)
    asked = []
    call = B.ExtendAttention(28, 4, 128)
    call._grow = lambda stream: asked.append(stream) or B.ExtendAttention._grow(call, stream)
    out = call(*args)
    torch.cuda.synchronize()
    assert not asked and (not earlier or torch.equal(out, want))


def test_object_dropped_during_a_capture():
    """Dropping an object waits for its calls, which a capture does not allow:
    its runner goes with the next object instead."""
    eb = build_extend([60], [60], 8, 2, 64, seed=2)
    b = eb.batch
    args = (eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens, eb.q_lens,
            b.scale)
    call, other = (B.ExtendAttention(8, 2, 64) for _ in range(2))
    want = call(*args)
    other(*args)
    out = torch.zeros_like(want)
    torch.cuda.synchronize()
    other(*args)   # not waited for
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        del other
        call(*args, out=out)
    assert len(B._scratch._dead) == 1
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, want) and torch.equal(B.ExtendAttention(8, 2, 64)(*args), want) and not B._scratch._dead


def test_memory_taken_for_another_stream_is_waited_for():
    """What an object lends is ordered on the current stream: before a first call
    on another one, and before one that grows it, the current stream is waited for."""
    side, waited = torch.cuda.Stream(), []
    for lens, qls in (([60], [60]), ([8000] * 4, [256] * 4)):
        eb = build_extend(lens, qls, 28, 4, 128, seed=3)
        b = eb.batch
        args = (eb.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens, eb.q_lens,
                b.scale)
        want = B.ExtendAttention(28, 4, 128)(*args)
        torch.cuda.synchronize()
        call = B.ExtendAttention(28, 4, 128)
        lend = call._lend
        call._lend = lambda slot, device, stream: (waited.append(stream), lend(slot, device, stream))
        out = torch.empty_like(want)
        torch.cuda.synchronize()
        call(*args, out=out, stream=side)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    assert len(waited) == 3 and all(s is side for s in waited)
