"""The one-launch step of many units, its append in the decoding workgroups and in workgroups of its own: against append + decode, bit for bit."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu

TK = B.SPARQ_FLAG_TILED_K


SHORT, APART, ONE = "workgroups of four waves", "append of a step apart", "one launch)"


@pytest.mark.parametrize("Bn,h,h_kv,d_h,S_max,r,k,dtype,flags,build", [
    (103, 10, 10, 128, 128, 12, 20, "f16", 0, SHORT), (103, 10, 5, 64, 128, 12, 20, "bf16", 0, SHORT), (205, 5, 1, 256, 128, 12, 20, "f16", 0, SHORT),
    (41, 25, 25, 256, 128, 12, 20, "bf16", 0, SHORT), (1025, 1, 1, 64, 128, 12, 20, "f16", TK, APART), (103, 10, 5, 128, 128, 12, 20, "bf16", TK, APART),
    (103, 10, 10, 128, 128, 12, 20, "f16", B.SPARQ_FLAG_RAGGED_BATCH, SHORT), (205, 6, 6, 64, 128, 12, 20, "bf16", B.SPARQ_FLAG_RAGGED_BATCH, SHORT),
    (400, 3, 3, 128, 64, 12, 20, "f16", B.SPARQ_FLAG_RAGGED_BATCH, SHORT),
    # what a unit reads binds the call: workgroups of eight waves, the append in its own beyond 512 KV heads
    (103, 10, 10, 128, 704, 12, 704, "f16", 0, APART), (41, 26, 26, 256, 448, 64, 448, "bf16", 0, APART), (1025, 1, 1, 64, 1408, 12, 1408, "bf16", 0, APART),
    (103, 10, 5, 128, 704, 12, 704, "bf16", 0, APART), (103, 10, 10, 64, 1408, 9, 1408, "f16", B.SPARQ_FLAG_RAGGED_BATCH, APART),
    (260, 4, 4, 64, 1408, 9, 1400, "bf16", B.SPARQ_FLAG_RAGGED_BATCH, APART), (103, 20, 4, 128, 704, 12, 704, "f16", 0, ONE), (103, 10, 10, 64, 16320, 9, 300, "f16", 0, "waves read apart, " + APART)])
def test_step_equals_append_then_decode(Bn, h, h_kv, d_h, S_max, r, k, dtype, flags, build):
    w = W.Workload("many units", Bn, h, h_kv, d_h, S_max, r, k, dtype, seed=1700 + d_h)
    lens = (torch.arange(Bn, dtype=torch.int32) * 7) % (S_max + 1)      # every length mod 8, empty and full sequences
    lens[:3] = torch.tensor([0, S_max, S_max - 1])
    print("[case]", Bn, h, h_kv, d_h, S_max, r, k, dtype, flags, build, flush=True)
    assert B.sparq_decode_plan(B.make_shape(Bn, h, h_kv, S_max, d_h, r, k, w.torch_dtype, flags)).endswith(build)
    one, two = (Hn.build_cache(w, seq_lens=lens, S_max=S_max, v_offset=True, flags=flags) for _ in range(2))
    q = W.draw_queries(w, one.K_src, lens.clamp(min=1), q_scale=0.05)[0].contiguous()
    for step in range(3):
        kn, vn = W.draw_kv(W.scaled(w, seed=w.seed + 1 + step), "cuda", n_rows=1, v_offset=True)
        kn, vn = kn[:, :, 0].contiguous(), vn[:, :, 0].contiguous()
        out, alpha, idx, chan = one.cache.step(kn, vn, q, aux=True)
        two.cache.append(kn, vn)
        want = two.cache.decode(q, aux=True)
        # the order of the sums differs where the row comes from the inputs: 2 units of the 16-bit output, fp32 sums of alpha
        assert torch.equal(one.cache.seq_lens, two.cache.seq_lens)
        assert torch.equal(one.cache.v_mean, two.cache.v_mean)
        assert torch.equal(idx, want[2]) and torch.equal(chan, want[3])
        assert (alpha - want[1]).abs().max().item() <= Hn.ALPHA_TOL
        unit = 2.0 ** (-10 if dtype == "f16" else -7)
        diff = (out.float() - want[0].float()).abs()
        assert (diff <= 2 * unit * want[0].float().abs().clamp(min=unit)).all(), diff.max()
        for a, b in ((one.cache.key_rows(), two.cache.key_rows()), (one.cache.V, two.cache.V)):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        if not flags & TK:
            live = torch.arange(S_max, device="cuda") < (one.cache.seq_lens & ~7)[:, None]
            for a, b in ((one.cache.Kt, two.cache.Kt),):
                assert torch.equal(a.view(torch.int16)[live[:, None, None].expand_as(a)], b.view(torch.int16)[live[:, None, None].expand_as(b)])
        assert one.cache.error_flags() & 1 == 1 and two.cache.error_flags() & 1 == 1      # full sequences are reported
