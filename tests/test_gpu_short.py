"""Many units with short caches (workgroups of four waves): the newest rows in two rounds, edges of the selection's forms, the step."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Bn,h,h_kv,d_h,S_max,r,k,dtype,dup,window,flags", [
    (129, 4, 4, 128, 64, 16, 64, "f16", 0, 0, 0), (65, 8, 2, 64, 192, 9, 33, "bf16", 0, 0, 0), (43, 12, 12, 256, 128, 40, 20, "bf16", 0, 9, 0),
    (27, 20, 20, 128, 1088, 32, 100, "bf16", 900, 0, B.SPARQ_FLAG_RAGGED_BATCH), (18, 29, 29, 64, 1472, 8, 1200, "f16", 0, 0, 0),
    (260, 2, 1, 128, 256, 64, 1, "f16", 200, 1, B.SPARQ_FLAG_RAGGED_BATCH), (33, 16, 16, 256, 320, 24, 64, "f16", 0, 0, 0),
    (250, 3, 3, 128, 256, 64, 1, "f16", 200, 1, B.SPARQ_FLAG_RAGGED_BATCH), (256, 3, 3, 64, 128, 9, 30, "bf16", 0, 0, B.SPARQ_FLAG_RAGGED_BATCH),
    (257, 2, 2, 64, 128, 9, 30, "bf16", 0, 0, B.SPARQ_FLAG_RAGGED_BATCH),
    # where a lane's keys double, become bit masks, a thread has more than two chunks; the longest that four fit a CU's LDS
    (9, 58, 2, 64, 1024, 8, 113, "f16", 0, 0, 0), (9, 58, 1, 128, 1088, 16, 200, "bf16", 700, 13, 0), (9, 58, 1, 64, 2048, 8, 227, "bf16", 0, 0, 0),
    (9, 58, 2, 128, 2112, 16, 300, "f16", 1900, 37, 0), (9, 58, 1, 64, 4096, 8, 455, "f16", 0, 0, 0), (9, 58, 1, 64, 4160, 16, 500, "bf16", 3900, 5, 0),
    (9, 58, 2, 128, 4160, 9, 400, "f16", 0, 0, 0), (9, 58, 1, 64, 5504, 8, 900, "f16", 0, 0, 0), (9, 58, 1, 128, 4928, 16, 300, "bf16", 0, 21, 0),
    (9, 58, 1, 256, 3776, 8, 250, "bf16", 2500, 0, 0)])
def test_decode_and_step(Bn, h, h_kv, d_h, S_max, r, k, dtype, dup, window, flags):
    S = S_max - 1
    w = W.Workload("short", Bn, h, h_kv, d_h, S, r, k, dtype, seed=2100 + Bn)
    lens = (S - torch.arange(Bn, dtype=torch.int32) * 5 % S)                  # every length mod 8
    assert set((lens % 8).tolist()) == set(range(8))
    assert B.sparq_decode_plan(B.make_shape(Bn, h, h_kv, S_max, d_h, r, k, w.torch_dtype, flags, window)).endswith("workgroups of four waves")
    print("[case]", Bn, h, h_kv, d_h, S_max, r, k, dtype, dup, window, flags, flush=True)
    b = Hn.build_cache(w, seq_lens=lens, S_max=S_max, v_offset=True, dup_rows=dup)
    q = W.draw_queries(w, b.K_src, lens, q_scale=0.05)[0].contiguous()
    Hn.compare_decode(b, q, local_window=window, flags=flags)
    kn, vn = W.draw_kv(W.scaled(w, seed=w.seed + 1), "cuda", n_rows=1, v_offset=True)
    rows = torch.arange(S + 1, device="cuda")
    at = (rows[None] == lens.cuda()[:, None])[:, None, :, None]               # row S_b of each sequence
    grow = lambda src, new: torch.where(at, new, torch.nn.functional.pad(src, (0, 0, 0, S + 1 - src.shape[2])))
    grown = Hn.Built(w, b.cache, grow(b.K_src, kn), grow(b.V_src, vn), lens + 1, None)
    Hn.compare_decode(grown, q, local_window=window, flags=flags, step_rows=(kn[:, :, 0].contiguous(), vn[:, :, 0].contiguous()))
