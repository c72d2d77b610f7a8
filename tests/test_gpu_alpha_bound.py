"""alpha is a share: never above 1, and exactly 1 where every position is selected, under every plan."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu

SH, K1, TK = B.SPARQ_FLAG_GQA_SHARED, B.SPARQ_FLAG_SINGLE_K, B.SPARQ_FLAG_TILED_K


@pytest.mark.parametrize("Bn,h,h_kv,d_h,S_max,plan,flags", [
    (4, 4, 2, 128, 2048, "sparq_decode_fused", 0), (4, 4, 2, 64, 2048, "sparq_decode_fused", TK), (4, 4, 2, 64, 2048, "stored once", K1),
    (4, 4, 2, 128, 16384, "digit-bucket", 0), (4, 4, 2, 128, 36032, "digit-bucket", 0), (5, 32, 32, 64, 36032, "two-level", 0),
    (4, 4, 2, 128, 2048, "one workgroup per KV head", SH), (4, 4, 1, 64, 2048, "one workgroup per KV head", SH),
    (4, 4, 2, 128, 16384, "grouped-query rule on the digit-bucket", SH), (5, 32, 8, 64, 20480, "several workgroups per KV head", SH),
    # 120 units of 5 spans: the digit-bucket plan's merges in a launch of their own
    (5, 24, 12, 64, 40960, "digit-bucket", 0), (5, 24, 12, 64, 40960, "grouped-query rule on the digit-bucket", SH)])
def test_alpha_is_a_share(Bn, h, h_kv, d_h, S_max, plan, flags):
    k = 1201
    w = W.Workload("share", Bn, h, h_kv, d_h, k + 2, 24, k, "f16", seed=1500 + d_h)
    lens = torch.tensor([k, k - 1, 37, k + 1, k + 2][:Bn], dtype=torch.int32)
    b = Hn.build_cache(w, seq_lens=lens, S_max=S_max, v_offset=True, flags=flags & (K1 | TK))
    print("[case]", plan, Bn, h, h_kv, d_h, flags, flush=True)
    for scale in (1.0, 0.05, 0.005):
        q = W.draw_queries(w, b.K_src, lens, q_scale=scale)[0].contiguous()
        for more in (0, B.SPARQ_FLAG_TAU_SQRT_DH):
            c = b.cache.with_params(w.r, w.k, flags | more)
            assert plan in B.sparq_decode_plan(c.shape)
            alpha = c.decode(q, aux=True)[1].cpu()
            print(scale, more, (alpha - 1).abs().max().item(), flush=True)
            assert (alpha[:3] == 1).all(), (alpha[:3] - 1).abs().max()
            assert (alpha[3:] <= 1).all() and (alpha[3:] > 0).all()
