"""Step 1b where a thread has one item (a chunk of 8 positions by a batch of 8 channels), none, or a few, against the oracle."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, B.SPARQ_FLAG_TILED_K])
@pytest.mark.parametrize("d_h,dtype", [(64, "bf16"), (128, "f16"), (256, "bf16")])
@pytest.mark.parametrize("r", [1, 8, 9])
@pytest.mark.parametrize("chunks", [0, 1, 63, 65, 511, 512, 513, 575, 577, 1025])
def test_one_item_per_thread(d_h, dtype, r, chunks, flags):
    """A workgroup of 512 threads per head, row-major keys with helpers beside it (four units; without: test_gpu_eight_waves.py); the second
    sequence is shorter and ends inside a wave's chunks."""
    w = W.Workload("items", 2, 2, 2, d_h, chunks * 8 + 5, r, 20, dtype, seed=1200 + chunks)
    print("[case]", d_h, dtype, r, chunks, flags, flush=True)
    lens = torch.tensor([w.S, max(1, w.S - 8 * 37)], dtype=torch.int32)
    b = Hn.build_cache(w, seq_lens=lens, v_offset=True, flags=flags)
    q = W.draw_queries(w, b.K_src, b.seq_lens, q_scale=0.05)[0].contiguous()
    print(Hn.compare_decode(b, q, flags=flags), flush=True)


@pytest.mark.parametrize("r,S", [(32, 16384), (25, 15011), (64, 16384), (16, 36001)])
def test_one_item_per_thread_of_a_group(r, S):
    """Digit-bucket plan: two or four thread groups share a chunk's channels."""
    w = W.Workload("items", 1, 4, 4, 128, S, r, 300, "f16", seed=1300 + r)
    print("[case]", r, S, flush=True)
    b = Hn.build_cache(w, v_offset=True)
    q = W.draw_queries(w, b.K_src, b.seq_lens, q_scale=0.05)[0].contiguous()
    assert "digit-bucket" in B.sparq_decode_plan(b.cache.shape)
    print(Hn.compare_decode(b, q), flush=True)
