"""Decode steps of batches with few pages per worker, where a workgroup's waves
share a segment and merge in LDS, at the edges of that plan: segments of fewer
pages than waves, empty and one-token sequences, cut and whole pairs, with and
without lse; and at every group size for head_dim 64 and 128, plain, fp8 and
appending steps, each with a plan that is asserted to be of that size. Against
the fp64 oracle at |gpu - ref| <= 2e-3 + 1e-2 |ref|, and in the 2-norm at 2^-16:
the softmax weights carry 16 bits or more (each is off by 2^-17 of itself at
most), their sums 24, so out is off by less than 2^-16 of its norm wherever the
values of a sum do not cancel beyond their root mean square. lse: 2^-15, its
scores being fp32 sums of up to 128 products."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_12784_amd import binding as B
from paper_2601_12784_amd.workloads import PAGE, bf16_bits, build_batch, make_decode_loop, random_fp8_cache
from test_gpu_append import assert_close, run_loop
from test_runner_plan import SHARED, SHARED_CASES, runner_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


def assert_near(out, lse, ref, what):
    rel = np.linalg.norm(np.asarray(out, np.float64) - ref[0]) / np.linalg.norm(ref[0])
    fin = np.isfinite(ref[1])
    far = np.abs(np.asarray(lse, np.float64)[fin] - ref[1][fin]).max(initial=0.0)
    print(f"  {what}: rel {rel:.2e}, lse {far:.2e}", flush=True)
    assert rel < 2.0 ** -16 and far < 2.0 ** -15, what


CASES = {   # lens, heads: the waves per workgroup the plan takes are printed
    "few_pages": ([1, 16, 17, 130, 33], (4, 1, 64)),
    "empty": ([0, 300, 0, 1, 0], (28, 4, 128)),
    "one": ([1000], (28, 4, 128)),
    "whole_63": (list(range(100, 600, 8)), (28, 4, 128)),
    "whole_40": (list(range(20, 300, 7)), (40, 8, 128)),
    "whole_100": (list(range(60, 260, 2)), (28, 4, 128)),
    "whole_200": (list(range(1, 201)), (8, 8, 64)),
    "cut": ([9000, 17, 15000], (16, 1, 128)),
}


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_short_batch(case, fp8):
    lens, (hq, hkv, d) = CASES[case]
    b = build_batch(lens, hq, hkv, d, 300 + len(lens))
    kw, k, v = {}, b.k_pool, b.v_pool
    if fp8:
        c = random_fp8_cache(b, seed=7)
        kw, k, v = dict(fp8=(c.k_scale.cuda(), c.v_scale.cuda())), c.k8, c.v8
        ref = oracle.decode_attn_fp8(bf16_bits(b.q), c.k8.numpy(), c.v8.numpy(), c.k_scale.numpy(), c.v_scale.numpy(),
                                     b.block_table, b.seq_lens, b.scale)
    else:
        ref = oracle.decode_attn(bf16_bits(b.q), bf16_bits(b.k_pool), bf16_bits(b.v_pool), b.block_table, b.seq_lens, b.scale)
    runner = B.DecodeAttention(hq, hkv, d)
    args = (b.q.cuda(), k.cuda(), v.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens, b.scale)
    lse = torch.full((b.num_seqs, hq), float("nan"), device="cuda")
    out = runner(*args, lse=lse, **kw)
    i = runner.last_info
    print(f"short {case} fp8={fp8}: {i.num_workers} waves in groups of {i.workers_per_group}, {i.num_combine} cut", flush=True)
    bare = runner(*args, **kw)
    torch.cuda.synchronize()
    assert i.workers_per_group in (1, 2, 4, 8)
    assert_close(out.cpu().numpy(), ref[0], "out")
    assert_close(lse.cpu().numpy(), ref[1], "lse")
    assert_near(out.cpu().numpy(), lse.cpu().numpy(), ref, case)
    assert torch.equal(out, bare)


@pytest.mark.parametrize("case", range(len(SHARED_CASES)))
def test_every_shared_group_size(case):
    kind, d, group, lens, (hq, hkv) = SHARED_CASES[case]
    print(f"shared case {case}: kind {kind}, d={d}, groups of {group}, {hq}/{hkv} heads, {len(lens)} sequences", flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert runner_plan(lens, hq, hkv, d, kind, num_cus=cus)[1].workers_per_group == SHARED + group
    b = build_batch(lens, hq, hkv, d, 500 + case)
    kp, vp = bf16_bits(b.k_pool).copy(), bf16_bits(b.v_pool).copy()
    k, v, table, kw = b.k_pool, b.v_pool, b.block_table, {}
    if kind == 1:
        c = random_fp8_cache(b, seed=7)
        k, v, kw = c.k8, c.v8, dict(fp8=(c.k_scale.cuda(), c.v_scale.cuda()))
        ref = oracle.decode_attn_fp8(bf16_bits(b.q), c.k8.numpy(), c.v8.numpy(), c.k_scale.numpy(), c.v_scale.numpy(),
                                     table, b.seq_lens, b.scale)
    else:
        ref = oracle.decode_attn(bf16_bits(b.q), kp, vp, table, b.seq_lens, b.scale)
    if kind == 2:   # the newest token comes with the step: its slot holds NaN, and a page it opens is not in the table
        at, slot, rows = (b.seq_lens - 1) // PAGE, (b.seq_lens - 1) % PAGE, np.arange(len(lens))
        pages = table[rows, at]
        kn = kp[pages, :, :, slot, :].reshape(len(lens), hkv, d)
        vn = vp[pages, :, :, slot].reshape(len(lens), hkv, d)
        kh, vh, table = kp.copy(), vp.copy(), table.copy()
        kh[pages, :, :, slot, :] = 0x7FC0
        vh[pages, :, :, slot] = 0x7FC0
        fresh = np.where(slot == 0, pages, -1).astype(np.int32)
        table[rows[slot == 0], at[slot == 0]] = -1
        k, v, kn, vn = (torch.from_numpy(x.view(np.int16)).view(torch.bfloat16) for x in (kh, vh, kn, vn))
        kw = dict(append=(kn.cuda(), vn.cuda(), fresh))
    runner = B.DecodeAttention(hq, hkv, d)
    k, v, bt = k.cuda(), v.cuda(), torch.from_numpy(table).cuda()
    lse = torch.full((len(lens), hq), float("nan"), device="cuda")
    out = runner(b.q.cuda(), k, v, bt, b.seq_lens, b.scale, lse=lse, **kw)
    torch.cuda.synchronize()
    assert runner.last_info.workers_per_group == group
    assert_close(out.cpu().numpy(), ref[0], "out")
    assert_close(lse.cpu().numpy(), ref[1], "lse")
    assert_near(out.cpu().numpy(), lse.cpu().numpy(), ref, f"case {case}")
    if kind == 2:
        assert np.array_equal(bf16_bits(k.cpu()), kp) and np.array_equal(bf16_bits(v.cpu()), vp)
        assert np.array_equal(bt.cpu().numpy(), b.block_table)


@pytest.mark.parametrize("case", ["few_pages", "one", "whole_40", "whole_200", "cut"])
def test_short_appending_loop(case):
    lens, (hq, hkv, d) = CASES[case]
    print(f"short append {case}", flush=True)
    run = make_decode_loop(lens=lens, steps=18, cap_extra_max=18, seed=310, num_q_heads=hq, num_kv_heads=hkv, head_dim=d)
    run_loop(run, check_steps={0, 1, 2, 9, 16, 17})
