"""Bulk appends over several workgroups per KV head, at the edges of their tiles, against the definition."""
import numpy as np
import pytest
import torch

from oracle import sparq_oracle as O
from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W
from paper_2312_04985_amd.cache import DecodeCache

pytestmark = pytest.mark.gpu

# The mean before the call was rounded to fp32 and so is the one after it (2^-24 of a value each); sums are fp64.
# Means here are below 4 in magnitude: 2 * 4 * 2^-24 = 4.8e-7.
MEAN_TOL = 6e-7


@pytest.mark.parametrize("d_h,dtype", [(64, "f16"), (128, "bf16"), (256, "f16")])
@pytest.mark.parametrize("start,rows,scratch", [
    ((0, 0, 0), (2, 1, 2), None),                 # a start that is aligned, less than one group of 8
    ((0, 0, 0), (256, 64, 255), None),            # whole tiles, one short of it
    ((5, 63, 64), (260, 130, 257), None),         # starts inside a group, at the end of a line, at one
    ((7, 0, 450), (513, 0, 64), None),            # nothing for one sequence, the buffer's last row for another
    ((120, 1, 300), (300, 480, 513), None),       # one sequence would pass the end: left as it is
    ((61, 3, 0), (510, 499, 257), 65536),         # the smallest workspace: fewer partial sums fit
    ((7, 64, 0), (16, 9, 1), None),               # a short append where there are many KV heads (120): rows of a full group and beside it
    ((63, 560, 13), (64, 17, 3), None),           # ... for d_h 64 up to 64 rows; one sequence would pass the end
])
@pytest.mark.parametrize("h_kv", [2, 120])         # one launch; more than 192 workgroups: a second launch for means and lengths
def test_bulk_append_over_several_workgroups(d_h, dtype, start, rows, scratch, h_kv, s_max=576):
    n_b = 3
    w = W.Workload("bulk", n_b, h_kv, h_kv, d_h, s_max, 16, 32, dtype, seed=900 + d_h + rows[0])
    print("[case]", d_h, dtype, start, rows, scratch, flush=True)
    old_k, old_v = W.draw_kv(w, "cuda", n_rows=max(max(start), 1), v_offset=True)
    c = DecodeCache(n_b, h_kv, h_kv, s_max, d_h, 16, 32, w.torch_dtype, poison=6.0e4)
    for t in range(max(start)):                   # one row at a time: the kernel under test builds nothing here
        n = torch.tensor([int(t < s) for s in start], dtype=torch.int32, device="cuda")
        c.append(old_k[:, :, t].contiguous(), old_v[:, :, t].contiguous(), n)
    before = [x.clone() for x in (c.K, c.Kt, c.V)]
    want = O.mean_value(W.to_codes(c.V), np.array(start, dtype=np.int32), dtype=w.dtype_code)
    assert all(s == 0 or np.abs(c.v_mean[b].cpu().numpy() - want[b]).max() <= 1e-4 for b, s in enumerate(start))
    mean0 = c.v_mean.double().cpu()
    if scratch:
        c.workspace = torch.zeros(scratch + n_b * h_kv * 2 * (d_h + 2) * 4, dtype=torch.uint8, device="cuda")
    new_k, new_v = W.draw_kv(W.scaled(w, seed=w.seed + 1), "cuda", n_rows=max(rows), v_offset=True)
    c.append(new_k, new_v, torch.tensor(rows, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    flags = c.error_flags()
    assert flags == (B.SPARQ_ERR_APPEND_FULL if any(s + n > s_max for s, n in zip(start, rows)) else 0)
    for b, (s, n) in enumerate(zip(start, rows)):
        if n == 0 or s + n > s_max:
            n = 0
        e = s + n
        assert int(c.seq_lens[b]) == e
        K, V = before[0][b].clone(), before[2][b].clone()
        K[:, s:e], V[:, s:e] = new_k[b, :, :n], new_v[b, :, :n]
        assert torch.equal(c.K[b], K) and torch.equal(c.V[b], V)      # nothing else is written
        fl = e & ~7
        assert torch.equal(c.Kt[b, :, :, :fl], K[:, :fl].transpose(1, 2))
        last = -(-e // 8) * 8                                         # the columns of an unfinished group are unspecified
        assert torch.equal(c.Kt[b, :, :, last:], before[1][b, :, :, last:])
        if n:
            mean = (mean0[b] * s + V[:, s:e].double().sum(1).cpu()) / e if s else V[:, :e].double().mean(1).cpu()
            assert (c.v_mean[b].double().cpu() - mean).abs().max().item() <= MEAN_TOL
        else:
            assert torch.equal(c.v_mean[b].double().cpu(), mean0[b])
    assert c.workspace[256:16384].count_nonzero() == 0               # the counters are left as they were


@pytest.mark.parametrize("d_h,dtype", [(64, "bf16"), (128, "f16"), (256, "bf16")])
@pytest.mark.parametrize("start,rows", [((0, 7, 8), (64, 64, 64)), ((61, 0, 127), (33, 0, 49))])
def test_short_append_for_many_heads(d_h, dtype, start, rows):
    """768 KV heads and up to 64 rows: one workgroup per KV head, whatever d_h."""
    test_bulk_append_over_several_workgroups(d_h, dtype, start, rows, None, 256, s_max=192)


@pytest.mark.parametrize("d_h,dtype", [(64, "f16"), (128, "bf16"), (256, "f16")])
@pytest.mark.parametrize("h_kv,tiles", [(1, 16), (1, 17), (1, 65), (1, 96),         # one launch: up to 192 workgroups
                                        (7, 16), (7, 17), (7, 64), (7, 65), (7, 128)])
def test_many_partial_sums_per_head(d_h, dtype, h_kv, tiles):
    """Around the numbers of partial sums that one round of loads takes; the second sequence leaves most workgroups without rows."""
    rows = tiles * (16384 // d_h) - 63                    # append_split: that many tiles of 16384 / d_h positions
    print("[case]", d_h, dtype, h_kv, tiles, rows, flush=True)
    w = W.Workload("sums", 2, h_kv, h_kv, d_h, W.round_up(rows + 64, 64), 16, 32, dtype, seed=930 + d_h + tiles)
    c = DecodeCache(2, h_kv, h_kv, w.S, d_h, 16, 32, w.torch_dtype)
    k, v = W.draw_kv(w, "cuda", n_rows=rows, v_offset=True)
    done = torch.zeros(2, dtype=torch.long)
    for counts in ((5, 3), (rows, 70)):
        c.append(k, v, torch.tensor(counts, dtype=torch.int32, device="cuda"))
        for b, n in enumerate(counts):
            s, e = int(done[b]), int(done[b]) + n
            assert torch.equal(c.K[b, :, s:e], k[b, :, :n]) and torch.equal(c.V[b, :, s:e], v[b, :, :n])
            mean = c.V[b, :, :e].double().mean(1)
            assert (c.v_mean[b].double() - mean).abs().max().item() <= MEAN_TOL
            done[b] = e
    assert c.seq_lens.cpu().tolist() == done.tolist() and c.error_flags() == 0
    assert c.workspace[256:16384].count_nonzero() == 0
