"""The digit-bucket plan at the edges of its spans: the unit's last workgroup merges, also when spans are empty, and
leaves its counters as it found them; the launches' own splits of a span's channel rows."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,h_kv,group", [(4, 2, False), (3, 3, False), (4, 1, True), (4, 2, True)])
@pytest.mark.parametrize("s_max,lens,r", [
    (16384, (16383, 1, 1025), 32),        # spans of 1024: all, one and two of them have positions
    (16384, (7, 16377, 8192), 9),         # two batches of channel rows
    (40960, (40959, 2047, 20000), 40),    # longer spans, five batches
])
def test_last_workgroup_of_a_unit(h, h_kv, group, s_max, lens, r):
    w = W.Workload("last", 3, h, h_kv, 64, s_max, r, 300, "bf16", seed=860 + r + h)
    print("[case]", h, h_kv, group, s_max, lens, r, flush=True)
    flags = B.SPARQ_FLAG_GQA_SHARED if group else 0
    seq = torch.tensor(lens, dtype=torch.int32)
    b = Hn.build_cache(w, seq_lens=seq, S_max=s_max, v_offset=True)
    b.cache.with_params(w.r, w.k, flags)
    assert "digit-bucket" in B.sparq_decode_plan(b.cache.shape)
    for scale in (1.0, 0.02):
        q = W.draw_queries(w, b.K_src, b.seq_lens, q_scale=scale)[0].contiguous()
        print(Hn.compare_decode(b, q, flags=flags), flush=True)     # twice, and compared bit for bit
    new_k, new_v = W.draw_kv(W.scaled(w, seed=w.seed + 1), "cuda", n_rows=1, v_offset=True)
    k1, v1 = new_k[:, :, 0].contiguous(), new_v[:, :, 0].contiguous()
    K_all, V_all = (torch.cat([x, y], dim=2) for x, y in ((b.K_src, new_k), (b.V_src, new_v)))
    for i, s in enumerate(lens):
        K_all[i, :, s], V_all[i, :, s] = k1[i], v1[i]
    after = Hn.Built(w, b.cache, K_all, V_all, seq + 1, None)
    print(Hn.compare_decode(after, q, flags=flags, step_rows=(k1, v1)), flush=True)
    assert b.cache.workspace[256:16384].count_nonzero() == 0
