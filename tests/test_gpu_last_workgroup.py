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


@pytest.mark.parametrize("group", [False, True])
def test_units_merged_by_a_launch_of_their_own(group):
    """120 units of 5 spans: more workgroups than run at once."""
    test_last_workgroup_of_a_unit(40, 20, group, 40960, (40959, 2047, 20000), 20)


@pytest.mark.parametrize("h,h_kv,flags", [(4, 2, 0), (4, 1, B.SPARQ_FLAG_GQA_SHARED), (4, 2, B.SPARQ_FLAG_GQA_SHARED)])
def test_a_unit_is_counted_from_zero(h, h_kv, flags):
    """What an earlier call left in the counters (sparq_decode_noalloc's buffer cannot be initialised again) changes nothing."""
    w = W.Workload("count", 3, h, h_kv, 64, 16384, 24, 200, "f16", seed=870 + h_kv)
    b = Hn.build_cache(w, seq_lens=torch.tensor([16384, 900, 5000], dtype=torch.int32), S_max=16384, v_offset=True)
    b.cache.with_params(w.r, w.k, flags)
    assert "digit-bucket" in B.sparq_decode_plan(b.cache.shape)
    q = W.draw_queries(w, b.K_src, b.seq_lens, q_scale=0.03)[0].contiguous()
    want = [x.clone() for x in b.cache.decode(q, aux=True)]
    counters = b.cache.workspace[256:256 + 4 * w.B * h].view(torch.int32)
    for left in (1, 15, -2, 1 << 20):
        counters.fill_(left)
        got = b.cache.decode(q, aux=True)
        assert all(torch.equal(x, y) for x, y in zip(want, got)), left
        assert counters.count_nonzero() == 0
    assert b.cache.error_flags() == 0


@pytest.mark.parametrize("name,kw,flags,lens", [
    # one workgroup per KV head under the grouped-query rule: the appended row alone, inside, completing a group of 8, at the bound
    ("group_one_workgroup", dict(H=8, H_kv=2, d_h=64, r=12, k=40), B.SPARQ_FLAG_GQA_SHARED, (0, 6, 7, 703, 704)),
    ("group_of_two_wide", dict(H=4, H_kv=2, d_h=256, r=40, k=900), B.SPARQ_FLAG_GQA_SHARED, (1, 15, 511, 703, 704)),
    # two spans of 8192 and more, many heads: an appended row that is a span of its own
    ("two_level", dict(H=26, H_kv=26, d_h=64, r=8, k=60), 0, (8191, 8192, 40959, 7, 36000)),
])
def test_steps_with_the_append_built_in(name, kw, flags, lens):
    """Nine steps equal nine appends and decodes; a sequence at its bound is left alone and reported."""
    s_max = 704 if max(lens) <= 704 else 40960
    w = W.Workload(name, len(lens), S=s_max, dtype="f16", seed=880 + max(lens), **kw)
    seq = torch.tensor(lens, dtype=torch.int32)
    a, f = (Hn.build_cache(w, seq_lens=seq, S_max=s_max, v_offset=True) for _ in range(2))
    for c in (a, f):
        c.cache.with_params(w.r, w.k, flags)
    kn, vn = W.draw_kv(W.scaled(w, seed=w.seed + 1), "cuda", n_rows=9, v_offset=True)
    for t in range(9):
        k_t, v_t = kn[:, :, t].contiguous(), vn[:, :, t].contiguous()
        q = W.draw_queries(w, a.K_src, a.cache.seq_lens.cpu().clamp(max=a.K_src.shape[2]), q_scale=0.03, stream=t)[0].contiguous()
        if t % 3 == 1:                      # the new row is the best match of the first KV head
            q[:, :w.g] = (k_t[:, :1].float() * 0.05).to(q.dtype)
        a.cache.append(k_t, v_t)
        one, two = a.cache.decode(q, aux=True), f.cache.step(k_t, v_t, q, aux=True)
        fa, ff = a.cache.error_flags(), f.cache.error_flags()
        assert fa == ff and fa in (0, B.SPARQ_ERR_APPEND_FULL), (fa, ff)
        assert torch.equal(a.cache.seq_lens, f.cache.seq_lens) and torch.equal(a.cache.v_mean, f.cache.v_mean)
        assert torch.equal(one[2], two[2]) and torch.equal(one[3], two[3])
        assert (one[1] - two[1]).abs().max().item() <= 1e-6
        # the same rows summed in another order, rounded to 16 bits: one unit in the last place
        assert ((one[0].float() - two[0].float()).abs() <= 2.0 ** -10 * one[0].float().abs() + 1e-6).all()
        for b, n in enumerate(a.cache.seq_lens.cpu().tolist()):
            assert torch.equal(a.cache.K[b, :, :n], f.cache.K[b, :, :n]) and torch.equal(a.cache.V[b, :, :n], f.cache.V[b, :, :n])
            assert torch.equal(a.cache.Kt[b, :, :, :n & ~7], f.cache.Kt[b, :, :, :n & ~7])
