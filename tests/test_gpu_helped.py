"""Few units, whose idle CUs fetch for them: every place of a unit on the XCDs, selections that are touched in part, the plan's line."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn


def decode_and_step(w, lens, dup, window):
    b = Hn.build_cache(w, seq_lens=lens, S_max=W.round_up(w.S + 1, 64), v_offset=True, dup_rows=dup)
    assert B.sparq_decode_plan(b.cache.shape).endswith("idle CUs fetch")
    q = W.draw_queries(w, b.K_src, lens, q_scale=0.05)[0].contiguous()
    Hn.compare_decode(b, q, local_window=window)
    kn, vn = W.draw_kv(W.scaled(w, seed=w.seed + 1), "cuda", n_rows=1, v_offset=True)
    rows = torch.arange(max(int(lens.max()) + 1, 1), device="cuda")
    at = (rows[None] == lens.cuda()[:, None])[:, None, :, None]               # row S_b of each sequence
    grow = lambda src, new: torch.where(at, new, torch.nn.functional.pad(src, (0, 0, 0, rows.numel() - src.shape[2])))
    grown = Hn.Built(w, b.cache, grow(b.K_src, kn), grow(b.V_src, vn), lens + 1, None)
    Hn.compare_decode(grown, q, local_window=window, step_rows=(kn[:, :, 0].contiguous(), vn[:, :, 0].contiguous()))


@pytest.mark.gpu
@pytest.mark.parametrize("Bn,h,h_kv,d_h,S,r,k,dtype,dup,window", [
    (1, 1, 1, 128, 2001, 1, 1, "f16", 0, 0), (7, 1, 1, 64, 1100, 9, 1100, "bf16", 0, 0), (3, 3, 1, 256, 1031, 24, 100, "bf16", 0, 40),
    (17, 1, 1, 128, 4097, 8, 64, "f16", 4000, 0), (4, 8, 2, 128, 1500, 64, 300, "bf16", 1200, 7), (3, 11, 11, 64, 1090, 16, 1, "f16", 0, 1),
    (1, 64, 64, 64, 1025, 64, 33, "f16", 0, 0), (4, 20, 5, 256, 1030, 12, 700, "f16", 900, 0), (27, 3, 3, 128, 1026, 32, 90, "bf16", 0, 0),
    (32, 4, 4, 64, 1041, 17, 120, "f16", 1000, 0),
    # short caches: fewer chunks than helpers, fewer positions than a helper's stride
    (1, 1, 1, 128, 17, 1, 3, "f16", 0, 0), (3, 1, 1, 64, 63, 9, 40, "bf16", 50, 2), (16, 8, 4, 256, 130, 40, 25, "f16", 0, 0), (5, 5, 5, 128, 420, 8, 100, "bf16", 300, 0),
    # long ones of few rows, which the digit-bucket plan serves with more
    (1, 20, 5, 64, 12301, 8, 100, "f16", 0, 0), (2, 16, 4, 128, 16385, 16, 300, "bf16", 9000, 0), (1, 64, 2, 64, 28600, 8, 400, "f16", 0, 7),
    (3, 6, 2, 256, 14001, 8, 200, "bf16", 0, 0), (1, 36, 4, 64, 33001, 8, 300, "f16", 20000, 0)])
def test_decode_and_step(Bn, h, h_kv, d_h, S, r, k, dtype, dup, window):
    w = W.Workload("helped", Bn, h, h_kv, d_h, S, r, k, dtype, seed=1900 + Bn)
    lens = (S - torch.arange(Bn, dtype=torch.int32) * 13 % max(S // 2, 1))          # the last rows of every kind: mod 8, tails
    if Bn > 2:
        lens[1] = 5
    print("[case]", Bn, h, h_kv, d_h, S, r, k, dtype, dup, window, flush=True)
    decode_and_step(w, lens, dup, window)


def test_workspace_does_not_depend_on_what_a_call_selects():
    """Between the digit-bucket plan and helped units r and k decide: a workspace sized with one pair serves the others."""
    plans = set()
    for units in (17, 32, 64):
        for S_max in (12288, 16384, 30016):
            sizes = set()
            for r, k in ((8, 64), (16, 256), (32, 512), (64, 2048)):
                sh = B.make_shape(1, units, units, S_max, 128, r, k, torch.float16)
                sizes.add(B.sparq_workspace_bytes(sh))
                plans.add(B.sparq_decode_plan(sh).split(" ")[0])
            assert len(sizes) == 1, (units, S_max, sizes)
    assert plans == {"bk_scores", "sparq_decode_fused"}
