"""dense_decode over several workgroups per KV head: edges of its row groups and splits, every bundle of query heads."""
import pytest
import torch

from oracle import sparq_oracle as O
from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W
from paper_2312_04985_amd.cache import DecodeCache

import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_h,g,dtype", [(64, 8, "f16"), (64, 1, "bf16"), (128, 8, "bf16"), (128, 4, "f16"), (128, 3, "bf16"),
                                         (256, 8, "bf16"), (256, 4, "f16"), (256, 2, "bf16"),
                                         # bundles that are not full: one of 6 or 7, 5 + 5, 6 + 5, two of 3, 3 + 2
                                         (128, 6, "f16"), (64, 7, "bf16"), (128, 10, "bf16"), (64, 11, "f16"), (256, 6, "f16"), (256, 5, "bf16")])
@pytest.mark.parametrize("b,h_kv,lens", [
    (4, 1, (1, 15, 16, 17)),                # below and above one tile of 16 rows
    (4, 2, (0, 255, 256, 321)),             # an empty sequence; one split, one row into the next
    (1, 1, (8192 + 5,)),                    # one unit over many splits
    (9, 1, (2500, 1, 2049, 0, 640, 576, 577, 1024, 2560)),   # more units than 8: other splits, some of them empty
])
def test_dense_decode_edges(d_h, g, dtype, b, h_kv, lens):
    w = W.Workload("dense", b, g * h_kv, h_kv, d_h, max(lens), 8, 8, dtype, seed=700 + d_h + g + b)
    print("[case]", d_h, g, dtype, b, h_kv, lens, flush=True)
    seq = torch.tensor(lens, dtype=torch.int32)
    c = Hn.build_cache(w, seq_lens=seq, v_offset=True)
    for scale in (1.0, 0.03):               # one row takes all the weight; many share it (the maximum keeps rising)
        q = W.draw_queries(w, c.K_src, seq, q_scale=scale)[0].contiguous()
        for _ in range(2):                  # the second call finds the counters as the first one left them
            out = c.cache.dense(q)
        K, V = Hn.host_cache_codes(c, c.cache.S_max)
        ref = O.dense_decode(K, V, W.to_codes(q), seq.numpy(), dtype=w.dtype_code)
        Hn.check_output(out.float().cpu().numpy(), ref, w.dtype_code)
    assert c.cache.error_flags() == 0


@pytest.mark.parametrize("rows", [200, 3000])      # one workgroup, several
def test_dense_decode_without_a_denominator(rows):
    """A key that is not a number gives the heads that share it zeros, and no one else."""
    w = W.Workload("nan", 2, 4, 2, 128, rows, 8, 8, "f16", seed=790)
    c = Hn.build_cache(w, v_offset=True)
    q = W.draw_queries(w, c.K_src, c.seq_lens, q_scale=0.03)[0].contiguous()
    good = c.cache.dense(q)
    c.cache.K[1, 0, rows // 2, 5] = float("nan")
    out = c.cache.dense(q)
    assert (out[1, :2] == 0).all()
    assert torch.equal(out[0], good[0]) and torch.equal(out[1, 2:], good[1, 2:])


@pytest.mark.parametrize("d_h,g,dtype", [(256, 1, "f16"), (128, 4, "bf16")])
def test_dense_decode_rows_beyond_4_gib_of_a_head(d_h, g, dtype):
    """The rows that count lie more than 2^32 bytes behind the head's first one; all others are zeros."""
    first, n = (1 << 32) // (2 * d_h), 300
    S = first + n
    w = W.Workload("far", 1, g, 1, d_h, S, 8, 8, dtype, seed=795)
    c = DecodeCache(1, g, 1, W.round_up(S, 64), d_h, 8, 8, w.torch_dtype, flags=B.SPARQ_FLAG_SINGLE_K)   # (no second copy of K)
    gen = torch.Generator().manual_seed(795)
    K, V, q = (torch.randn(x, generator=gen).to(w.torch_dtype) for x in ((n, d_h), (n, d_h), (g, d_h)))
    q[:, 0] = 16.0                          # a common part of every score, so that the 2^24 zeros do not take the weight
    K[:, 0] = 2.0 * d_h ** 0.5
    c.K[0, 0, first:S], c.V[0, 0, first:S], c.seq_lens[0] = K.cuda(), V.cuda(), S
    out = c.dense(q.cuda()[None].contiguous())
    score = q.double() @ K.double().T / d_h ** 0.5
    e = torch.exp(score - score.max(1, keepdim=True).values)
    y = (e @ V.double()) / (e.sum(1, keepdim=True) + first * torch.exp(-score.max(1, keepdim=True).values))
    Hn.check_output(out[0].float().cpu().numpy(), y.numpy(), w.dtype_code)
