"""The plan of a runner's step on the CPU: every page of every (sequence, KV head)
pair in exactly one segment, rows that fit together as the kernels read them,
and sf_decode_attn_plan's own plan wherever the caller chose the slices or the
batch has many pages per worker."""
import ctypes

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


CASES = [([17, 64, 130, 300], 4, 1, 64), ([32768], 28, 4, 128), ([1000], 28, 4, 128), ([1, 0, 16, 17, 0, 33], 8, 8, 128),
         ([5] * 300, 28, 4, 128), ([600] * 64, 40, 8, 128), ([1] + [0] * 40, 16, 1, 64)]
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


def test_smaller_batches_fit_what_a_large_one_reserves():
    """sf_runner_reserve's floor, re-derived: segments of pairs take at most 4 per
    CU (8 where the pairs alone are more than 4 per CU) and 8 workers per CU,
    whatever the batch; its four times the reserved rows covers every batch that
    the reserved one shrinks to."""
    rng = np.random.default_rng(3)
    cus = 256
    for trial in range(200):
        hkv = int(rng.choice([1, 2, 4, 8]))
        n = int(rng.choice([1, 3, 17, 64, 140, 200, 520, 1030]))
        full = rng.integers(1, int(rng.choice([40, 600, 4000, 20000])), n)
        _, large, _ = runner_plan(full, 4 * hkv, hkv, 128)
        for _ in range(4):
            lens = np.minimum(full, rng.integers(0, full.max() + 1, n) if rng.random() < .5 else rng.integers(1, full.max() + 1))
            lens = rng.permutation(lens)[: int(rng.integers(1, n + 1))]
            _, info, _ = runner_plan(lens, 4 * hkv, hkv, 128)
            segments = 8 * cus if n * hkv > 4 * cus else 4 * cus
            rows = 8 * cus + segments + min(n * hkv, segments // 2)
            assert info.work_bytes <= max(large.work_bytes, min(rows * 32, 4 * large.work_bytes)), (trial, lens)
            assert info.num_partials <= max(large.num_partials, segments), (trial, lens)
