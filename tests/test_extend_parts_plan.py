"""The plan sf_runner_extend makes, on the CPU: every key step of every block of
new tokens in exactly one part, slots and merges that fit together, every page
of new tokens stored once; and argument checks that need no device."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2601_12784_amd import binding as B


def plan(lens, qls, hq, hkv, d, cus, store):
    L = B.lib()
    lens, qls = np.asarray(lens, np.int32), np.asarray(qls, np.int32)
    desc = B.make_desc(lens.size, hq, hkv, d, max(1, int(-(-lens.max() // 16))), 1 << 20, 0.1)
    counts = np.zeros(5, np.int32)
    args = (ctypes.byref(desc), lens.ctypes.data, qls.ctypes.data, cus, int(store))
    st = L.sf_debug_extend_plan(*args, None, 0, counts.ctypes.data)
    assert st == (3 if counts[1] else 0)
    work = np.full((int(counts[1:4].sum()) + 1, 8), -7, np.int32)
    assert L.sf_debug_extend_plan(*args, work.ctypes.data, work.nbytes - 32, counts.ctypes.data) == 0
    assert np.all(work[-1] == -7)
    rows, parts, merges, stores, slots = counts.tolist()
    return rows, slots, work[:parts], work[parts:parts + merges], work[parts + merges:-1]


CASES = [([1000], [1000], 28, 4, 128), ([8000, 8100, 8200, 8300], [256] * 4, 28, 4, 128), ([40, 16, 1, 0], [0, 9, 1, 0], 7, 7, 64),
         ([16384], [64], 28, 4, 128), ([3000] * 8, [700] * 8, 40, 8, 128), ([12774] * 8, [3] * 8, 8, 8, 64),
         ([100_000], [1], 16, 1, 128), ([0], [0], 4, 1, 64)]
CASES += [(L.tolist(), np.minimum(L, rng.integers(0, 900, L.size)).tolist(), hkv * g, hkv, d)
          for rng in [np.random.default_rng(4)] for _ in range(24)
          for L, hkv, g, d in [(rng.integers(1, 9000, rng.integers(1, 9)), int(rng.integers(1, 9)), int(rng.integers(1, 17)),
                                int(rng.choice([64, 128])))]]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("cus", [0, 8])
def test_plan_covers_every_step_once(case, cus):
    lens, qls, hq, hkv, d = CASES[case]
    g = hq // hkv
    rows, slots, parts, merges, stores = plan(lens, qls, hq, hkv, d, cus, True)
    assert rows in (128, 384) and np.all(np.diff(parts[:, 6] - parts[:, 2]) <= 0)
    cu = np.concatenate([[0], np.cumsum(qls)])
    walks = {}
    for seq, kvh, b, nt, first, qrow, e, slot in parts.tolist():
        prefix = lens[seq] - qls[seq]
        assert 1 <= nt <= rows // g and first - prefix == qrow - cu[seq] and 0 <= b < e
        walks.setdefault((seq, kvh, first, nt, qrow), []).append((b, e, slot))
    used = []
    for (seq, kvh, first, nt, qrow), ps in walks.items():
        ps.sort()
        assert ps[0][0] == 0 and ps[-1][1] == -(-(first + nt) // 32)
        assert all(x[1] == y[0] for x, y in zip(ps, ps[1:]))
        if len(ps) == 1:
            assert ps[0][2] == 0
        else:
            assert [s for _, _, s in ps] == list(range(ps[0][2], ps[0][2] + len(ps)))
            used.append([ps[0][2] - 1, len(ps), nt, qrow, kvh, 0, 0, 0])
    assert sorted(used) == sorted(merges.tolist()) and slots == sum(u[1] for u in used)
    assert sorted(s for u in used for s in range(u[0], u[0] + u[1])) == list(range(slots))
    # every (new token, KV head) in one block
    seen = np.zeros((int(cu[-1]), hkv), int)
    for (seq, kvh, first, nt, qrow) in walks:
        seen[qrow:qrow + nt, kvh] += 1
    assert np.all(seen == 1)
    # every page that new tokens land in, once
    want = {(s, p) for s in range(len(lens)) if qls[s] for p in range((lens[s] - qls[s]) // 16, -(-lens[s] // 16))}
    got = [(s, p) for s, p0, n, *_ in stores.tolist() for p in range(p0, p0 + n)]
    assert len(got) == len(set(got)) and set(got) == want
    for s, p0, n, first, end, qrow, *_ in stores.tolist():
        assert (first, end, qrow) == (lens[s] - qls[s], lens[s], cu[s])
    assert plan(lens, qls, hq, hkv, d, cus, False)[4].size == 0


@pytest.mark.parametrize("length", [2**31 - 1, 2**31 - 20, 2**31 - 33])
def test_longest_lengths(length):
    """Lengths whose rounding up to a step or a page passes 31 bits."""
    L, lens, qls, counts = B.lib(), np.array([length], np.int32), np.array([5], np.int32), np.zeros(5, np.int32)
    desc = B.make_desc(1, 4, 1, 64, 1 << 27, 8, 0.1)
    args = (ctypes.byref(desc), lens.ctypes.data, qls.ctypes.data, 256, 1)
    assert L.sf_debug_extend_plan(*args, None, 0, counts.ctypes.data) == 3
    work = np.zeros((int(counts[1:4].sum()), 8), np.int32)
    assert L.sf_debug_extend_plan(*args, work.ctypes.data, work.nbytes, counts.ctypes.data) == 0
    parts, store = work[: counts[1]], work[counts[1] + counts[2]:]
    order = np.argsort(parts[:, 2])
    assert parts[order[0], 2] == 0 and parts[order[-1], 6] == -(-length // 32)
    assert np.array_equal(parts[order[:-1], 6], parts[order[1:], 2]) and np.all(parts[:, 6] > parts[:, 2])
    assert store[:, 1].min() == (length - 5) // 16 and store[:, 1].max() + 1 == -(-length // 16)


def test_plan_rejects_what_the_plain_plan_rejects():
    L = B.lib()
    counts = np.zeros(5, np.int32)
    for lens, qls in (([10], [11]), ([10], [-1]), ([40], [3])):
        a, b = np.array(lens, np.int32), np.array(qls, np.int32)
        desc = B.make_desc(1, 4, 1, 64, 2, 8, 0.1)        # stride 2: at most 32 tokens
        assert L.sf_debug_extend_plan(ctypes.byref(desc), a.ctypes.data, b.ctypes.data, 0, 1, None, 0, counts.ctypes.data) == 1


def test_runner_extend_rejects_missing_arguments():
    assert ctypes.sizeof(B.sf_runner_memory) == 56
    lens = np.array([4], np.int32)
    desc = B.make_desc(1, 4, 1, 64, 1, 1, 0.1)
    assert B.lib().sf_runner_extend(None, ctypes.byref(desc), lens.ctypes.data, lens.ctypes.data, None, None, None, None,
                                    None, None, None, None, ctypes.byref(B.sf_runner_memory()), None,
                                    ctypes.byref(B.sf_extend_info())) == 1


def test_captured_calls_keep_their_lists():
    """A captured call's list is its own: equal lists are shared, others take
    further room, and without room the error says what to do."""
    call = B.ExtendAttention(4, 1, 64)
    call._spare = [torch.zeros(160, dtype=torch.uint8), 0, torch.zeros(192, dtype=torch.uint8), 32, 160]
    a, b = np.arange(16, dtype=np.int32), np.arange(24, dtype=np.int32)
    ha, da = call._captured_list(a)
    hb, db = call._captured_list(b)
    assert np.array_equal(ha.numpy(), a) and np.array_equal(hb.numpy(), b) and da.numel() == 16 and db.numel() == 24
    assert da.data_ptr() + 64 == db.data_ptr()
    assert call._captured_list(a.copy())[0] is ha and call._spare[4] == 0
    call._room = lambda nbytes: (_ for _ in ()).throw(RuntimeError("capturing"))
    with pytest.raises(RuntimeError, match="eager call"):
        call._captured_list(np.zeros(8, np.int32))
    assert np.array_equal(ha.numpy(), a) and len(call._captured) == 2


def test_shared_scratch_is_bounded_and_alternates():
    pool = B._SharedScratch()
    cpu = torch.device("cpu")
    key = lambda stream, thread=0: (thread, cpu, stream)   # noqa: E731
    pool.join()
    pool.join()
    pool.grow(key(1), 1024)
    a, v = pool.get(key(1)), pool.version
    pool.grow(key(1), 512)
    assert pool.get(key(1)) is a and pool.get(key(2)) is None and pool.get(key(1, thread=7)) is None and pool.version != v
    first, second = a.next(), a.next()
    assert {first, second} == {a.memory.data_ptr(), a.memory.data_ptr() + 1024} and a.next() == first
    assert a.nbytes == 1024 and a.memory.numel() == 2048
    for stream in (2, 3, 4):
        pool.grow(key(stream), 256)
    assert pool.get(key(1)) is a          # used last: stream 2 goes first
    pool.grow(key(5), 256)
    assert pool.get(key(2)) is None and pool.get(key(1)) is a and len(pool._blocks) == pool.BLOCKS
    pool.leave()
    assert pool.get(key(1)) is a
    v = pool.version
    pool.leave()
    assert not pool._blocks and pool.version != v
