"""Approximate logits at the ends of what fp32 holds, and logits that are no numbers."""
import pytest
import torch

from oracle import sparq_oracle as O
from paper_2312_04985_amd import binding as B
from paper_2312_04985_amd import workloads as W
from paper_2312_04985_amd.cache import DecodeCache

import harness as Hn

pytestmark = pytest.mark.gpu


def filled(b, h, h_kv, S, k, flags, dtype):
    """A cache whose first channel is 1 in every key row; everything else is drawn."""
    c = DecodeCache(b, h, h_kv, W.round_up(S, 64), 64, 8, k, dtype, flags=flags)
    gen = torch.Generator(device="cuda").manual_seed(840 + S)
    for x in (c.K, c.V):
        x[:, :, :S].normal_(generator=gen)
    c.K[:, :, :S, 0] = 1.0
    c.v_mean.copy_(c.V[:, :, :S].double().mean(2))
    c.seq_lens.fill_(S)
    return c


@pytest.mark.parametrize("b,h,h_kv,S,k,flags,plan", [
    (2, 2, 2, 701, 100, 0, "sparq_decode_fused"),
    (2, 4, 2, 701, 100, B.SPARQ_FLAG_GQA_SHARED, "sparq_decode_shared"),
    (2, 4, 1, 16381, 900, B.SPARQ_FLAG_GQA_SHARED, "gs_logits + bk_group_scores"),
    (20, 8, 2, 16381, 900, B.SPARQ_FLAG_GQA_SHARED, "gs_logits + gs_select"),
    (1, 2, 2, 32005, 900, 0, "bk_scores"),
    (65, 2, 2, 40957, 900, 0, "long_scores"),
])
def test_all_logits_near_the_lowest_finite_value(b, h, h_kv, S, k, flags, plan):
    """Every position has the logit numerator -1.9 * 2^127: the lowest k positions are taken and alpha is their share."""
    print("[case]", plan, flush=True)
    c = filled(b, h, h_kv, S, k, flags, torch.bfloat16)
    assert B.sparq_decode_plan(c.shape).startswith(plan)
    c.K[:, :, :S, 0] = -1.8984375 * 2.0 ** 64
    c.Kt.copy_(c.K.transpose(2, 3))
    q = torch.zeros((b, h, 64), dtype=torch.bfloat16, device="cuda")
    q[:, :, 0] = 2.0 ** 63
    out, alpha, idx, _ = c.decode(q, aux=True)
    assert c.error_flags() == 0
    assert (idx == torch.arange(k, device="cuda")).all()
    # sums of up to 40 957 ones in fp32, in a tree or over 64-bit lanes' shares: whole numbers below 2^24, exact
    assert (alpha - k / S).abs().max().item() <= 1e-6
    top, mean = c.V[:, :, :k].double().mean(2), c.V[:, :, :S].double().mean(2)
    y = (k / S * top + (1 - k / S) * mean).repeat_interleave(h // h_kv, dim=1)
    Hn.check_output(out.float().cpu().numpy(), y.cpu().numpy(), O.BF16)


@pytest.mark.parametrize("S,k", [(300, 300), (701, 40), (17000, 17000)])
def test_a_key_that_is_no_number_leaves_no_alpha(S, k):
    """alpha of the heads that read it is not a number, also where everything is selected; the others' is as without it."""
    c = filled(2, 2, 2, S, k, 0, torch.float16)
    c.Kt.copy_(c.K.transpose(2, 3))
    q = torch.randn((2, 2, 64), device="cuda", generator=torch.Generator(device="cuda").manual_seed(841)).half() * 0.1
    q[:, :, 0] = 1.0                        # channel 0 is among the chosen ones
    good = c.decode(q, aux=True)[1].clone()
    c.K[1, 0, S // 2, 0] = c.Kt[1, 0, 0, S // 2] = float("nan")
    alpha = c.decode(q, aux=True)[1]
    assert torch.isnan(alpha[1, 0])
    keep = torch.tensor([[True, True], [False, True]], device="cuda")
    assert torch.equal(alpha[keep], good[keep]) and (k < S or (alpha[keep] == 1).all())
