"""Decode steps of batches with few pages per worker, where a workgroup's waves
share a segment and merge in LDS, at the edges of that plan: segments of fewer
pages than waves, empty and one-token sequences, cut and whole pairs, every
group size, head_dim 64 and 128, plain, fp8 and appending steps, with and
without lse. Against the fp64 oracle at |gpu - ref| <= 2e-3 + 1e-2 |ref|."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_12784_amd import binding as B
from paper_2601_12784_amd.workloads import bf16_bits, build_batch, make_decode_loop, random_fp8_cache
from test_gpu_append import assert_close, run_loop

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


CASES = {   # lens, heads: the waves per workgroup the plan takes are printed
    "few_pages": ([1, 16, 17, 130, 33], (4, 1, 64)),
    "empty": ([0, 300, 0, 1, 0], (28, 4, 128)),
    "one": ([1000], (28, 4, 128)),
    "whole_8": (list(range(100, 600, 8)), (28, 4, 128)),
    "whole_4": (list(range(20, 300, 7)), (40, 8, 128)),
    "whole_2": (list(range(60, 260, 2)), (28, 4, 128)),
    "whole_1": (list(range(1, 201)), (8, 8, 64)),
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
    assert torch.equal(out, bare)


@pytest.mark.parametrize("case", ["few_pages", "one", "whole_4", "whole_1", "cut"])
def test_short_appending_loop(case):
    lens, (hq, hkv, d) = CASES[case]
    print(f"short append {case}", flush=True)
    run = make_decode_loop(lens=lens, steps=18, cap_extra_max=18, seed=310, num_q_heads=hq, num_kv_heads=hkv, head_dim=d)
    run_loop(run, check_steps={0, 1, 2, 9, 16, 17})
