"""Plans keep a sequence in one piece - fp32 up to the final rounding - where they can: partial rows of key splits are bf16."""
import pytest

import paper_2509_15235_amd as vs


def _plan(B, T, Hq, Hkv, d, longest):
    cap = longest + T
    desc = vs.AttnDesc(B=B, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=vs.VS_BF16, softmax_scale=d ** -0.5, max_prefix_len=longest, capacity=cap,
                       stride_seq=Hkv * cap * d, stride_head=cap * d, stride_tok=d)
    rc, plan = vs.vs_attention_plan(desc)
    assert rc == 0
    return plan


@pytest.mark.parametrize("B,T,Hq,Hkv,longest", [(64, 17, 8, 1, 2100), (64, 17, 8, 1, 4096), (64, 17, 8, 1, 7025), (64, 29, 8, 1, 2100),
                                                (64, 29, 8, 1, 7025), (64, 17, 16, 1, 7794), (64, 48, 8, 2, 7794), (36, 18, 8, 1, 3650)])
def test_many_sequences_of_few_heads_keep_their_shares(B, T, Hq, Hkv, longest):
    """More than four row blocks: 64 shares, with which most sequences of a batch are one piece, and no splits of each."""
    plan = _plan(B, T, Hq, Hkv, 128, longest)
    assert (plan.schedule, plan.num_splits) == (vs.VS_SCHED_BALANCED, 64)
