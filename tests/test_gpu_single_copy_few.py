"""A key cache stored once, few units with long caches: the digit-bucket plan on key rows, and the workspace it falls back for."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu

K1 = B.SPARQ_FLAG_SINGLE_K


@pytest.mark.parametrize("Bn,h,h_kv,d_h,S_max,r,k,dtype,dup,window,more", [
    (1, 1, 1, 128, 4096, 16, 200, "f16", 0, 0, 0), (6, 4, 2, 64, 8256, 9, 1500, "bf16", 0, 33, 0), (3, 4, 4, 256, 5056, 40, 64, "bf16", 0, 0, 0),
    (5, 3, 1, 128, 12352, 32, 700, "f16", 9000, 0, 0), (2, 16, 4, 128, 6016, 128, 5900, "f16", 0, 0, B.SPARQ_FLAG_TAU_SQRT_DH),
    (3, 8, 8, 64, 6208, 8, 1, "f16", 4000, 1, B.SPARQ_FLAG_NO_REALLOC)])
def test_decode_and_step(Bn, h, h_kv, d_h, S_max, r, k, dtype, dup, window, more):
    S = S_max - 1
    w = W.Workload("single few", Bn, h, h_kv, d_h, S, r, k, dtype, seed=2300 + S_max)
    lens = torch.tensor([S, 3, 1025, S // 2, 2048, 1024][:Bn], dtype=torch.int32)
    print("[case]", Bn, h, h_kv, d_h, S_max, r, k, dtype, dup, window, more, flush=True)
    b = Hn.build_cache(w, seq_lens=lens, S_max=S_max, v_offset=True, dup_rows=dup, flags=K1)
    q = W.draw_queries(w, b.K_src, lens, q_scale=0.05)[0].contiguous()
    assert "digit-bucket" in B.sparq_decode_plan(b.cache.shape)
    Hn.compare_decode(b, q, flags=K1 | more, local_window=window)
    # a workspace that was sized for less runs one workgroup per unit: the same selection, the same sums but for their order
    c = b.cache
    out, alpha, idx, chan = c.decode(q, aux=True)
    full = c.workspace
    c.workspace = full[:B.sparq_workspace_bytes(c.shape) - 256]
    other = c.decode(q, aux=True)
    c.workspace = full
    assert torch.equal(idx, other[2]) and torch.equal(chan, other[3]) and (alpha - other[1]).abs().max().item() <= Hn.ALPHA_TOL
    assert (out.float() - other[0].float()).abs().max().item() <= 2 * 2.0 ** (-10 if dtype == "f16" else -7) * max(1.0, out.float().abs().max().item())
    kn, vn = W.draw_kv(W.scaled(w, seed=w.seed + 1), "cuda", n_rows=1, v_offset=True)
    rows = torch.arange(S + 1, device="cuda")
    at = (rows[None] == lens.cuda()[:, None])[:, None, :, None]               # row S_b of each sequence
    grow = lambda src, new: torch.where(at, new, torch.nn.functional.pad(src, (0, 0, 0, S + 1 - src.shape[2])))
    grown = Hn.Built(w, c, grow(b.K_src, kn), grow(b.V_src, vn), lens + 1, None)
    Hn.compare_decode(grown, q, flags=K1 | more, local_window=window, step_rows=(kn[:, :, 0].contiguous(), vn[:, :, 0].contiguous()))


@pytest.mark.parametrize("Bn,h,h_kv,d_h,S_max,r,k,dtype,dup,window", [
    (129, 4, 4, 128, 64, 16, 64, "f16", 0, 0), (65, 8, 2, 64, 192, 9, 33, "bf16", 0, 0), (43, 12, 12, 256, 128, 40, 20, "bf16", 0, 9),
    (27, 20, 4, 128, 576, 32, 100, "bf16", 400, 0), (9, 58, 2, 64, 1088, 8, 200, "f16", 0, 0), (9, 58, 1, 64, 2048, 16, 228, "bf16", 1500, 13),
    (9, 58, 1, 64, 2112, 9, 230, "f16", 0, 0), (9, 58, 1, 64, 2496, 8, 39, "bf16", 2000, 0), (9, 58, 1, 128, 1216, 16, 30, "f16", 0, 5)])
def test_many_units_with_short_caches(Bn, h, h_kv, d_h, S_max, r, k, dtype, dup, window):
    """Workgroups of four waves."""
    sh = B.make_shape(Bn, h, h_kv, S_max, d_h, r, k, {"f16": torch.float16, "bf16": torch.bfloat16}[dtype], K1, window)
    assert B.sparq_decode_plan(sh).endswith("workgroups of four waves")
    w = W.Workload("single short", Bn, h, h_kv, d_h, S_max, r, k, dtype, seed=2400 + S_max)
    lens = S_max - torch.arange(Bn, dtype=torch.int32) * 5 % S_max
    print("[case]", Bn, h, h_kv, d_h, S_max, r, k, dtype, dup, window, flush=True)
    b = Hn.build_cache(w, seq_lens=lens, S_max=S_max, v_offset=True, dup_rows=dup, flags=K1)
    q = W.draw_queries(w, b.K_src, lens, q_scale=0.05)[0].contiguous()
    Hn.compare_decode(b, q, flags=K1, local_window=window)
