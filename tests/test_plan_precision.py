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


@pytest.mark.parametrize("B,T,Hq,Hkv,d,longest,schedule,keys", [
    (9, 33, 28, 4, 128, 653, vs.VS_SCHED_PIPELINED, 256), (12, 25, 28, 4, 64, 424, vs.VS_SCHED_PIPELINED, 256),
    (6, 25, 28, 4, 128, 1061, vs.VS_SCHED_PIPELINED, 256), (23, 30, 8, 1, 128, 944, vs.VS_SCHED_PIPELINED, 256),
    (2, 36, 32, 8, 64, 548, vs.VS_SCHED_RESIDENT, 192), (12, 17, 8, 1, 128, 797, vs.VS_SCHED_RESIDENT, 256),
])
def test_short_sequences_of_a_batch_stay_in_one_piece(B, T, Hq, Hkv, d, longest, schedule, keys):
    """The kernels would be faster with shorter splits, but sequences of up to `keys` keys are whole in these."""
    plan = _plan(B, T, Hq, Hkv, d, longest)
    assert plan.schedule == schedule and plan.keys_per_split >= keys


@pytest.mark.parametrize("B,T,Hq,Hkv,longest", [(24, 25, 28, 4, 490), (10, 64, 28, 4, 203), (22, 35, 28, 4, 615)])
def test_whole_sequences_where_they_are_faster(B, T, Hq, Hkv, longest):
    plan = _plan(B, T, Hq, Hkv, 128, longest)
    assert (plan.schedule, plan.num_splits) == (vs.VS_SCHED_PIPELINED, 1)
