"""The plan of a runner's step on the CPU: every page of every (sequence, KV head)
pair in exactly one segment, rows that fit together as the kernels read them,
and sf_decode_attn_plan's own plan wherever the caller chose the slices or the
batch has many pages per worker."""
import ctypes
import time

import numpy as np
import pytest

from paper_2601_12784_amd import binding as B


SHARED = 16


def runner_plan(lens, hq, hkv, d, kind=0, **opts):
    lens = np.asarray(lens, np.int32)
    desc = B.make_desc(lens.size, hq, hkv, d, max(1, int(-(-lens.max() // 16))), 1 << 20, 0.1)
    info, o, L = B.sf_plan_info(), B.make_opts(**opts), B.lib()
    args = (ctypes.byref(desc), lens.ctypes.data, ctypes.byref(o), kind)
    assert L.sf_runner_plan(*args, None, 0, ctypes.byref(info)) == 0
    work = np.full(info.work_bytes // 4 + 8, -7, np.int32)
    assert L.sf_runner_plan(*args, work.ctypes.data, info.work_bytes - 4, ctypes.byref(info)) == 3
    assert L.sf_runner_plan(*args, work.ctypes.data, info.work_bytes, ctypes.byref(info)) == 0
    assert np.all(work[-8:] == -7)
    return desc, info, work[:-8].reshape(-1, 8)


def spread(n, lo, hi):
    """n lengths from lo to hi, evenly."""
    return np.linspace(lo, hi, n).astype(np.int32)


# (kind, head_dim, waves per workgroup, lens, heads): a plan of shared groups of every size that the kernels are built
# for, with whole pairs and with cut ones (groups of 8 leave none to cut)
SHARED_CASES = [
    (0, 64, 2, spread(2, 10, 100), (3, 3)), (0, 64, 2, spread(4, 183, 1831), (3, 3)),
    (0, 64, 4, spread(1, 161, 179), (3, 3)), (0, 64, 4, spread(2, 90, 903), (3, 3)), (0, 64, 8, spread(1, 453, 504), (3, 3)),
    (0, 128, 2, spread(1, 81, 162), (8, 2)), (0, 128, 2, spread(17, 62, 629), (8, 2)),
    (0, 128, 4, spread(1, 129, 129), (8, 2)), (0, 128, 4, spread(1, 786, 874), (8, 2)), (0, 128, 8, spread(1, 323, 359), (8, 2)),
    (1, 64, 2, spread(1, 129, 129), (3, 3)), (1, 64, 2, spread(5, 109, 1093), (3, 3)),
    (1, 64, 4, spread(1, 225, 225), (3, 3)), (1, 64, 4, spread(2, 119, 1191), (3, 3)), (1, 64, 8, spread(1, 584, 584), (3, 3)),
    (1, 128, 2, spread(1, 99, 111), (8, 2)), (1, 128, 2, spread(12, 90, 901), (8, 2)),
    (1, 128, 4, spread(1, 163, 326), (8, 2)), (1, 128, 4, spread(1, 898, 898), (8, 2)), (1, 128, 8, spread(1, 450, 450), (8, 2)),
    (2, 64, 2, spread(2, 10, 100), (3, 3)), (2, 64, 2, spread(9, 16, 167), (8, 8)),
    (2, 64, 4, spread(1, 161, 179), (3, 3)), (2, 64, 4, spread(1, 258, 2580), (3, 3)), (2, 64, 8, spread(80, 1147, 1147), (3, 3)),
    (2, 128, 2, spread(1, 81, 162), (8, 2)), (2, 128, 2, spread(2, 19, 193), (8, 2)),
    (2, 128, 4, spread(1, 129, 129), (8, 2)), (2, 128, 4, spread(1, 193, 1932), (8, 2)), (2, 128, 8, spread(87, 460, 512), (8, 2)),
    # the widest groups of query heads, many sequences
    (0, 128, 8, np.arange(100, 600, 8, dtype=np.int32), (28, 4)), (1, 64, 8, spread(27, 657, 807), (8, 8)),
    (2, 64, 8, spread(255, 1911, 2013), (4, 1)), (0, 64, 4, spread(239, 226, 418), (4, 1)), (0, 128, 4, spread(1, 1000, 1000), (16, 1)),
]


@pytest.mark.parametrize("case", range(len(SHARED_CASES)))
def test_shared_cases_share(case):
    kind, d, group, lens, (hq, hkv) = SHARED_CASES[case]
    assert runner_plan(lens, hq, hkv, d, kind)[1].workers_per_group == SHARED + group


CASES = [([17, 64, 130, 300], 4, 1, 64), ([32768], 28, 4, 128), ([1000], 28, 4, 128), ([1, 0, 16, 17, 0, 33], 8, 8, 128),
         ([5] * 300, 28, 4, 128), ([600] * 64, 40, 8, 128), ([1] + [0] * 40, 16, 1, 64)]
# lengths that are whole multiples of the segments that a search may try, and one long pair among many
CASES += [([16 * 24 * (i % 9 + 1) for i in range(150)], 4, 1, 64), ([16 * 7] * 600 + [16 * 2100], 16, 1, 128),
          ([655360 - 16 * 200] + [16] * 100, 16, 1, 128)]
CASES += [(rng.integers(0, int(hi), int(n)).tolist(), hkv * g, hkv, d)
          for rng in [np.random.default_rng(8)] for _ in range(30)
          for hi, n, hkv, g, d in [(rng.choice([40, 300, 5000]), rng.integers(1, 400), int(rng.integers(1, 9)),
                                    int(rng.integers(1, 17)), int(rng.choice([64, 128])))]]


@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_plan_covers_every_page_once(case, kind):
    lens, hq, hkv, d = CASES[case]
    desc, info, rows = runner_plan(lens, hq, hkv, d, kind)
    w, n = info.num_workers, info.num_work
    table, items, comb = rows[:w], rows[w:w + n], rows[w + n:]
    assert comb.shape[0] == info.num_combine
    shared = info.workers_per_group > SHARED
    if shared:
        # workgroups of g8 workers: item i is cut into the table rows i g8 .. i g8 + g8 - 1
        g8 = info.workers_per_group - SHARED
        assert g8 in (2, 4, 8) and w == n * g8
        assert np.array_equal(table[:, 0], np.arange(w) // g8) and np.all(table[:, 1] == 1)
        cut = table.reshape(n, g8, 8)
        for col, of in ((2, 0), (3, 1), (6, 4), (7, 5)):
            assert np.all(cut[:, :, col] == items[:, None, of])
        assert np.array_equal(cut[:, 0, 4], items[:, 2]) and np.array_equal(cut[:, -1, 5], items[:, 3])
        assert np.array_equal(cut[:, :-1, 5], cut[:, 1:, 4])
        size = cut[:, :, 5] - cut[:, :, 4]
        assert np.all(size.max(1) - size.min(1) <= 1) and size.max() <= info.chunk_pages
    else:
        assert info.workers_per_group in (1, 2, 4, 8)
        # the table walks the items in order, and holds each worker's first
        assert table[0, 0] == 0 and np.array_equal(table[:-1, 0] + table[:-1, 1], table[1:, 0])
        assert table[-1, 0] + table[-1, 1] == n and np.all(table[:, 1] >= 1)
        assert np.array_equal(table[:, 2:], items[table[:, 0], :6])
    segs = {}
    for seq, kvh, b, e, length, slot, cidx, k in items.tolist():
        assert length == lens[seq]
        segs.setdefault((seq, kvh), []).append((b, e, slot, cidx, k))
    assert len(segs) == len(lens) * hkv
    slots = []
    for (seq, kvh), ss in segs.items():
        ss.sort()
        npg = -(-lens[seq] // 16)
        assert ss[0][0] == 0 and ss[-1][1] == npg and all(x[1] == y[0] for x, y in zip(ss, ss[1:]))
        assert all(s[4] == len(ss) for s in ss) and (shared or max(e - b for b, e, *_ in ss) <= info.chunk_pages)
        if len(ss) == 1:
            assert ss[0][2:4] == (-1, -1)
        else:
            c = comb[ss[0][3]].tolist()
            assert c[:5] == [seq, kvh, ss[0][2], len(ss), lens[seq]] and all(s[3] == ss[0][3] for s in ss)
            assert [s[2] for s in ss] == list(range(ss[0][2], ss[0][2] + len(ss)))
            slots += [s[2] for s in ss]
    assert sorted(slots) == list(range(info.num_partials))
    g = hq // hkv
    al = lambda x: -(-x // 256) * 256   # noqa: E731
    assert info.workspace_bytes == (al(info.num_partials * g * d * 4) + al(info.num_partials * g * 4) if slots else 0)


@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("case", ["lognormal", "two_long", "many", "heads"])
def test_search_costs_little_next_to_the_slices(case, kind):
    """The search for a cut is on the critical path of every step: skewed batches
    with few KV heads, where it counts most, take no more than four times the
    plan of equal slices (1 to 2.2 times measured; 4 to 12 times when every
    candidate was a pass with a division per sequence). Least of 30 runs each."""
    rng = np.random.default_rng(0)
    ln = lambda n, m: np.clip(np.exp(np.log(m) + rng.standard_normal(n)), max(1, m // 8), 16 * m)   # noqa: E731
    lens, hq, hkv, d = {"lognormal": (ln(512, 500), 16, 1, 128), "two_long": (np.r_[rng.integers(1, 200, 510), 30000, 30000], 16, 1, 128),
                        "many": (ln(1000, 200), 16, 1, 128), "heads": (ln(128, 500), 14, 2, 64)}[case]
    lens = lens.astype(np.int32)
    desc = B.make_desc(lens.size, hq, hkv, d, int(lens.max() // 16 + 1), 1 << 20, 0.1)
    info, L, work = B.sf_plan_info(), B.lib(), np.empty(1 << 18, np.int32)
    opts, slices = B.make_opts(), B.make_opts(workers_per_cu=8 if kind == 1 else 0)
    best = [1.0, 1.0]
    for _ in range(30):
        t = time.perf_counter()
        assert L.sf_decode_attn_plan(ctypes.byref(desc), lens.ctypes.data, ctypes.byref(slices), work.ctypes.data, work.nbytes,
                                     ctypes.byref(info)) == 0
        u = time.perf_counter()
        assert L.sf_runner_plan(ctypes.byref(desc), lens.ctypes.data, ctypes.byref(opts), kind, work.ctypes.data, work.nbytes,
                                ctypes.byref(info)) == 0
        best = [min(best[0], u - t), min(best[1], time.perf_counter() - u)]
    print(f"{case} {kind}: slices {best[0] * 1e6:.1f} us, runner {best[1] * 1e6:.1f} us")
    assert best[1] < 4 * best[0]


@pytest.mark.parametrize("opts", [dict(chunk_pages=3), dict(workers_per_cu=4), dict(min_chunk_pages=8),
                                  dict(xcd_parity_skew=20), dict(num_cus=8)])
def test_the_callers_slices_stand(opts):
    lens = np.random.default_rng(1).integers(1, 3000, 24).astype(np.int32)
    desc, info, rows = runner_plan(lens, 28, 4, 128, **opts)
    want, work = B.sf_decode_attn_plan(desc, lens, B.make_opts(**opts))
    assert bytes(info) == bytes(want) and np.array_equal(rows.reshape(-1), work[: want.work_bytes // 4])


def test_short_batches_give_every_worker_one_segment():
    for lens, hq, hkv, d in CASES[:7]:
        if any(lens) and 0 not in lens:
            _, info, rows = runner_plan(lens, hq, hkv, d)
            assert np.all(rows[: info.num_workers, 1] == 1), lens


def test_runner_plan_rejects_what_the_plan_rejects():
    L = B.lib()
    info, lens = B.sf_plan_info(), np.array([40], np.int32)
    for desc in (B.make_desc(1, 4, 1, 64, 2, 8, 0.1), B.make_desc(1, 4, 1, 64, 4, 0, 0.1), B.make_desc(1, 4, 1, 96, 4, 8, 0.1)):
        assert L.sf_runner_plan(ctypes.byref(desc), lens.ctypes.data, None, 0, None, 0, ctypes.byref(info)) == \
            L.sf_decode_attn_plan(ctypes.byref(desc), lens.ctypes.data, None, None, 0, ctypes.byref(info)) != 0


def test_shared_groups_are_the_runners_alone():
    """sf_decode_attn refuses a plan of shared groups before any device call."""
    desc, info, rows = runner_plan([600] * 64, 28, 4, 128)
    assert info.workers_per_group > SHARED
    fake = 1 << 20
    assert B.lib().sf_decode_attn(ctypes.byref(desc), ctypes.byref(info), None, fake, fake, fake, fake, fake, fake, None, fake,
                                  1 << 30, None) == 4


def reserved(full, hq, hkv, d, kind, seqs, **opts):
    """Bytes (device, slot) that a reserve for the batch `full`, planned as a step of `kind`, sees to."""
    desc, info, _ = runner_plan(full, hq, hkv, d, kind, **opts)
    return room_for(desc, info.workspace_bytes, info.work_bytes, seqs, -1, **opts)


def room_for(desc, workspace, work, seqs, pages, **opts):
    got = np.zeros(2, np.uint64)
    assert B.lib().sf_debug_runner_reserve(ctypes.byref(desc), ctypes.byref(B.make_opts(**opts)), workspace, work, seqs, pages,
                                           got.ctypes.data) == 0
    return got.tolist()


def taken(lens, hq, hkv, d, kind, **opts):
    """Bytes (device, slot) that a step takes, at most."""
    _, info, rows = runner_plan(lens, hq, hkv, d, kind, **opts)
    append = kind == 2
    pages = (len(lens) * 4 + 31) // 32 * 32 if append else 0
    items = rows[info.num_workers: info.num_workers + info.num_work]
    single = int((items[:, 5] < 0).sum()) if append else 0
    al = lambda x: -(-x // 256) * 256   # noqa: E731
    return [al(info.workspace_bytes) + (info.num_combine + single) * 32 + pages,
            info.work_bytes + (info.num_work * 32 if append else 0) + pages]


def test_smaller_batches_and_other_kinds_fit_what_a_large_one_reserves():
    """Over all kinds of the reserve and of the step, for batches of the same
    sequences and for fewer and shorter ones; with batches that are planned as
    whole pairs for one kind and as slices with many partial results for another
    or for a part of them."""
    rng = np.random.default_rng(3)
    trials = [(int(rng.choice([1, 3, 17, 64, 140, 200, 520, 1030])), int(rng.choice([1, 2, 4, 8])),
               int(rng.choice([40, 600, 4000, 20000]))) for _ in range(150)] + [(200, 4, 600)] * 60
    for trial, (n, hkv, top) in enumerate(trials):
        full = rng.integers(1, top, n)
        opts = {} if trial % 4 else [dict(workers_per_cu=int(rng.integers(1, 9))), dict(chunk_pages=int(rng.integers(1, 200))),
                                     dict(min_chunk_pages=int(rng.integers(1, 40))), dict(xcd_parity_skew=30)][trial // 4 % 4]
        # by the lengths, and by the plan of any kind (a forced slice size has no bound without the lengths)
        room = np.array([room_for(B.make_desc(0, 4 * hkv, hkv, 128, 1, 0, 1.0), 0, 0, n, int((-(-full // 16)).sum()) * hkv, **opts)])
        if "chunk_pages" not in opts:
            room = np.vstack([room, [reserved(full, 4 * hkv, hkv, 128, kind, n, **opts) for kind in range(3)]])
        room = room.min(0)
        for part in range(4):
            lens = full
            if part:
                lens = np.minimum(full, rng.integers(0, full.max() + 1, n) if rng.random() < .5 else rng.integers(1, full.max() + 1))
                lens = rng.permutation(lens)[: int(rng.integers(max(1, n * (part - 1) // 3), n + 1))]
            if lens.max() == 0:
                continue
            for kind in range(3):
                assert np.all(np.array(taken(lens, 4 * hkv, hkv, 128, kind, **opts)) <= room), (trial, part, kind, lens.tolist())


def test_reserve_is_bounded_for_any_options():
    """Worker counts beyond any batch's need do not become memory."""
    desc = B.make_desc(0, 28, 4, 128, 1, 0, 1.0)
    for opts in (dict(workers_per_cu=2**20), dict(num_cus=2**30), dict(num_cus=2**30, workers_per_cu=2**30), dict(chunk_pages=1)):
        assert room_for(desc, 1000, 4096, 64, -1, **opts) == [1024 + 4096 + 256, 12288]
    # four short sequences of one KV head: a page of pinned memory per slot or two
    assert room_for(B.make_desc(0, 4, 1, 64, 1, 0, 1.0), 0, 0, 4, 38)[1] <= 16384
