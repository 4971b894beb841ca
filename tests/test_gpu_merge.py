"""The merge of pairs cut into many segments (one workgroup per pair and head),
at segment counts around its threshold (4 per pair) and its slices (8 at
head_dim 128, 16 at 64), against the fp64 oracle: |gpu - ref| <= 2e-3 + 1e-2 |ref|
for out and lse, and in the 2-norm at the precision of the weights and sums
(test_gpu_short_batches.py); pools and block tables bit for bit.

One-page slices (chunk_pages = 1) make a sequence of n pages n segments. The
appending steps pass through a step whose newest token opens a page: its
segment holds no cached token at all, alone in its slice."""
import pytest
import torch

import oracle
from paper_2601_12784_amd import binding as B
from paper_2601_12784_amd.workloads import PAGE, bf16_bits, build_batch, make_decode_loop
from test_gpu_append import assert_close, run_loop
from test_gpu_short_batches import assert_near

pytestmark = pytest.mark.gpu
SHAPES = [(28, 4, 128), (4, 1, 64), (16, 1, 128), (3, 3, 64)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("segments", [3, 4, 7, 8, 9, 17, 65])
@pytest.mark.parametrize("shape", SHAPES)
def test_merge_of_many_segments(shape, segments):
    hq, hkv, d = shape
    print(f"merge {shape} segments={segments}", flush=True)
    b = build_batch([PAGE * segments - 3, 1, PAGE * segments], hq, hkv, d, 70 + segments)
    runner = B.DecodeAttention(hq, hkv, d)
    lse = torch.empty((3, hq), dtype=torch.float32, device="cuda")
    out = runner(b.q.cuda(), b.k_pool.cuda(), b.v_pool.cuda(), torch.from_numpy(b.block_table).cuda(), b.seq_lens,
                 b.scale, lse=lse, chunk_pages=1)
    torch.cuda.synchronize()
    assert runner.last_info.num_combine == 2 * hkv and runner.last_info.num_partials == 2 * hkv * segments
    ref_o, ref_l = oracle.decode_attn(bf16_bits(b.q), bf16_bits(b.k_pool), bf16_bits(b.v_pool), b.block_table,
                                      b.seq_lens, b.scale)
    assert_close(out.cpu().numpy(), ref_o, "out")
    assert_close(lse.cpu().numpy(), ref_l, "lse")
    assert_near(out.cpu().numpy(), lse.cpu().numpy(), (ref_o, ref_l), f"{shape} {segments}")


@pytest.mark.parametrize("segments", [4, 8, 17])
@pytest.mark.parametrize("shape", SHAPES)
def test_appending_merge_of_many_segments(shape, segments):
    hq, hkv, d = shape
    print(f"appending merge {shape} segments={segments}", flush=True)
    run = make_decode_loop(lens=[PAGE * segments - 1, 3, PAGE * segments], steps=4, cap_extra_max=8, seed=80 + segments,
                           num_q_heads=hq, num_kv_heads=hkv, head_dim=d)
    run_loop(run, check_steps={0, 1, 2, 3}, chunk_pages=1)
