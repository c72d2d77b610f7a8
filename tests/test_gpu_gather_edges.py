"""Step 2b at the edges of the groups of rows that a lane weights together, against the oracle."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_h,dtype", [(64, "f16"), (128, "bf16"), (256, "f16")])
@pytest.mark.parametrize("h,h_kv,flags", [(2, 2, 0), (4, 2, B.SPARQ_FLAG_GQA_SHARED), (4, 1, B.SPARQ_FLAG_GQA_SHARED)])
@pytest.mark.parametrize("groups,more", [(0, 1), (0, 3), (1, -1), (1, 0), (1, 1), (2, -1), (2, 1), (3, 0)])
def test_rows_that_do_not_fill_a_group(d_h, dtype, h, h_kv, flags, groups, more):
    """k rows: a workgroup takes 64 rows of 64 channels (32 of 128, 16 of 256) per load, four loads (two with a group's heads)
    at a time."""
    k = groups * (8 * 64 * 8 // d_h) * (2 if flags else 4) + more
    w = W.Workload("rows", 2, h, h_kv, d_h, 900, 16, k, dtype, seed=950 + k)
    print("[case]", d_h, dtype, h, h_kv, flags, k, flush=True)
    b = Hn.build_cache(w, seq_lens=torch.tensor([900, 861], dtype=torch.int32), S_max=960, v_offset=True, flags=flags)
    q = W.draw_queries(w, b.K_src, b.seq_lens, q_scale=0.05)[0].contiguous()
    print(Hn.compare_decode(b, q, flags=flags), flush=True)
