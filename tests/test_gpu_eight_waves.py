"""Workgroups of eight waves without helpers (more than 128 units) beyond 1024 positions: the stream's and the selection's edges,
duplicated keys, the window, ragged order, capture, and waves that read apart."""
import pytest
import torch

from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu

RAGGED = B.SPARQ_FLAG_RAGGED_BATCH
ONE, RUNS = "one launch)", "waves read apart"


def decode_and_step(w, lens, S_max, build, *, dup=0, window=0, flags=0, scale=0.05):
    print("[case]", w, lens.tolist()[:8], S_max, build, dup, window, flags, flush=True)
    b = Hn.build_cache(w, seq_lens=lens, S_max=S_max, v_offset=True, dup_rows=dup)
    sh = B.make_shape(w.B, w.H, w.H_kv, S_max, w.d_h, w.r, w.k, w.torch_dtype, flags, window)
    assert w.B * w.H > 128 and B.sparq_decode_plan(sh).endswith(build), B.sparq_decode_plan(sh)
    q = W.draw_queries(w, b.K_src, lens, q_scale=scale)[0].contiguous()
    Hn.compare_decode(b, q, local_window=window, flags=flags)
    kn, vn = W.draw_kv(W.scaled(w, seed=w.seed + 1), "cuda", n_rows=1, v_offset=True)
    rows = torch.arange(int(lens.max()) + 1, device="cuda")
    at = (rows[None] == lens.cuda()[:, None])[:, None, :, None]               # row S_b of each sequence
    grow = lambda src, new: torch.where(at, new, torch.nn.functional.pad(src, (0, 0, 0, rows.numel() - src.shape[2])))
    grown = Hn.Built(w, b.cache, grow(b.K_src, kn), grow(b.V_src, vn), lens + 1, None)
    Hn.compare_decode(grown, q, local_window=window, flags=flags, step_rows=(kn[:, :, 0].contiguous(), vn[:, :, 0].contiguous()))


@pytest.mark.parametrize("d_h,dtype,r", [(64, "bf16", 9), (128, "f16", 1), (256, "bf16", 8)])
@pytest.mark.parametrize("chunks", [1, 63, 129, 511, 512, 513, 577, 1025, 1600])
def test_stream_edges(d_h, dtype, r, chunks):
    w = W.Workload("items", 3, 44, 2, d_h, chunks * 8 + 5, r, 20, dtype, seed=2500 + chunks)
    lens = torch.tensor([w.S, max(1, w.S - 8 * 37), max(1, w.S // 2)], dtype=torch.int32)
    decode_and_step(w, lens, W.round_up(w.S + 1, 64), ONE)


@pytest.mark.parametrize("S", [2047, 2049, 4095, 4100, 8200, 15900])
@pytest.mark.parametrize("window,dup", [(0, 0), (13, 0), (37, 1900)])
def test_selection_edges(S, window, dup):
    w = W.Workload("edges", 2, 66, 2, 64, S, 8, max(1, S // 9), "f16" if S % 2 else "bf16", planted=(1, 2), seed=2600 + S + window)
    decode_and_step(w, torch.tensor([S, S - S // 7], dtype=torch.int32), W.round_up(S + 1, 64), ONE, dup=dup, window=window, scale=0.03 if window else 1.0)


@pytest.mark.parametrize("Bn,h,h_kv,d_h,S_max,r,dtype", [
    (5, 27, 1, 64, 16320, 9, "f16"), (5, 27, 3, 128, 16448, 32, "bf16"), (5, 26, 1, 256, 16320, 40, "f16"), (5, 28, 2, 64, 32832, 16, "bf16"), (5, 26, 2, 64, 32640, 8, "f16")])
def test_waves_that_read_apart(Bn, h, h_kv, d_h, S_max, r, dtype):
    """Runs of 64 chunks: whole and not, one more for the first waves, none more; sequences too short for runs beside them."""
    w = W.Workload("apart", Bn, h, h_kv, d_h, S_max - 1, r, 500, dtype, seed=2700 + S_max)
    for chunks in ((1024, 1025, 1087, 1089, 1151), (S_max // 8 - 1, 1536, 1537, 1599, 3)):
        lens = torch.tensor([8 * c + 3 + i for i, c in enumerate(chunks)], dtype=torch.int32)
        decode_and_step(w, lens, S_max, RUNS, dup=9000 if chunks[0] == 1024 else 0, window=0 if chunks[0] == 1024 else 21)


@pytest.mark.parametrize("Bn,h,d_h,S_max,dtype", [(130, 1, 64, 1984, "f16"), (33, 4, 128, 1216, "bf16"), (260, 1, 64, 1088, "bf16")])
def test_ragged_order(Bn, h, d_h, S_max, dtype):
    """The longest sequences start first (H = H_kv); equal lengths and one-row sequences among them."""
    w = W.Workload("ragged", Bn, h, h, d_h, S_max - 1, 12, 90, dtype, seed=2800 + Bn)
    lens = 1 + (torch.arange(Bn, dtype=torch.int32) // 2 * 389) % (S_max - 2)
    decode_and_step(w, lens, S_max, ONE, flags=RAGGED)


@pytest.mark.parametrize("Bn,h,h_kv,S_max,k,build", [(3, 44, 2, 1536, 100, ONE), (5, 27, 1, 16320, 300, RUNS), (9, 60, 4, 576, 60, "workgroups of four waves"),
                                                     (41, 26, 26, 704, 700, "append of a step apart")])
def test_replayed_steps_match_eager_steps(Bn, h, h_kv, S_max, k, build):
    w = W.Workload("replay", Bn, h, h_kv, 128, S_max - 21, 12, k, "f16", seed=2900 + Bn)
    sides = [Hn.build_cache(w, S_max=S_max, v_offset=True, poison=None) for _ in range(2)]
    assert B.sparq_decode_plan(sides[0].cache.shape).endswith(build)
    kn, vn = W.draw_kv(W.scaled(w, seed=w.seed + 1), "cuda", n_rows=8, v_offset=True)
    qs = W.draw_queries(w, sides[0].K_src, sides[0].seq_lens, n=8, q_scale=0.02)
    ins = [[t[:, :, 0].contiguous() for t in (kn, vn)] + [qs[0].clone()] for _ in range(2)]
    out = [torch.empty_like(qs[0]) for _ in range(2)]

    def load(t):
        for i in range(2):
            for dst, src in zip(ins[i], (kn[:, :, t + i], vn[:, :, t + i], qs[t + i])):
                dst.copy_(src)

    load(0)
    for side in sides:                          # eagerly first: this makes the second pair of lengths and means
        for i in range(2):
            side.cache.step(*ins[i], out=out[i])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for i in range(2):
            sides[0].cache.step(*ins[i], out=out[i])
    for t in (2, 4, 6):
        load(t)
        graph.replay()
        torch.cuda.synchronize()
        for i in range(2):
            assert torch.equal(out[i].view(torch.int16), sides[1].cache.step(*ins[i]).view(torch.int16)), (t, i)
        assert torch.equal(sides[0].cache.v_mean, sides[1].cache.v_mean) and torch.equal(sides[0].cache.seq_lens, sides[1].cache.seq_lens)
    assert sides[0].cache.error_flags() == 0 and sides[1].cache.error_flags() == 0
