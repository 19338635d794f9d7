"""Launches that load K and V as data that is read once (large ones whose tiles one workgroup alone reads): own tiles of one and two row
blocks, four waves of the pipelined kernel on whole sequences and on balanced shares; and the same launches on paged caches, which load them
as any other data. Against fp64 sums of some (sequence, KV head) units; what the caches hold behind a sequence's last key is NaN."""
import ctypes

import pytest

import paper_2509_15235_amd as vs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,Hq,Hkv,d,longest,paged,schedule,waves", [
    (8, 3, 32, 32, 128, 330, 0, vs.VS_SCHED_LOOP, 8), (16, 2, 32, 32, 128, 200, 1, vs.VS_SCHED_LOOP, 4),
    (16, 5, 16, 16, 64, 700, 0, vs.VS_SCHED_LOOP, 8), (32, 4, 16, 16, 64, 400, 1, vs.VS_SCHED_LOOP, 4),
    (4, 60, 32, 32, 128, 2100, 0, vs.VS_SCHED_LOOP, 8), (4, 60, 32, 32, 128, 2100, 1, vs.VS_SCHED_LOOP, 8),
    (16, 60, 32, 32, 128, 1900, 0, vs.VS_SCHED_PIPELINED, 4), (16, 60, 32, 32, 128, 1900, 1, vs.VS_SCHED_PIPELINED, 4),
    (32, 60, 16, 16, 64, 3900, 0, vs.VS_SCHED_PIPELINED, 4), (32, 60, 16, 16, 64, 3900, 1, vs.VS_SCHED_PIPELINED, 4),
    (12, 60, 32, 32, 128, 2730, 0, vs.VS_SCHED_BALANCED, 4), (12, 60, 32, 32, 128, 2730, 1, vs.VS_SCHED_BALANCED, 4),
])
def test_against_fp64(B, T, Hq, Hkv, d, longest, paged, schedule, waves):
    import torch
    import gpu_util as gu
    gen = torch.Generator(device="cuda").manual_seed(3100 + longest)
    rand = lambda *n: torch.randn(*n, device="cuda", generator=gen, dtype=torch.bfloat16)
    block = 16
    blocks = -(-(longest + T) // block)
    lens = [longest - 37 * b % (longest // 3) for b in range(B)]
    q = rand(B, T, Hq, d)
    kv = [rand(B * blocks, Hkv, block, d) if paged else rand(B, Hkv, longest + T, d) for _ in range(2)]
    table = torch.randperm(B * blocks, device="cuda", generator=gen).int().view(B, blocks)
    for x in kv:
        for b, n in enumerate(lens):
            if paged:
                x[table[b, -(-(n + T) // block):].long()] = float("nan")
                x[table[b, (n + T - 1) // block].long(), :, (n + T - 1) % block + 1:] = float("nan")
            else:
                x[b, :, n + T:] = float("nan")
    parent = torch.tensor([[-1] + [(7 * i + b) % i for i in range(1, T)] for b in range(B)], device="cuda", dtype=torch.int32)
    desc = vs.AttnDesc(B=B, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=vs.VS_BF16, softmax_scale=d ** -0.5, max_prefix_len=longest, stride_tok=d)
    if paged:
        desc.paged, desc.block_size, desc.max_blocks, desc.num_blocks = 1, block, blocks, B * blocks
        desc.stride_block, desc.stride_head, desc.block_table = Hkv * block * d, block * d, table.data_ptr()
    else:
        desc.capacity, desc.stride_seq, desc.stride_head = longest + T, Hkv * (longest + T) * d, (longest + T) * d
    rc, plan = vs.vs_attention_plan(desc)
    assert rc == 0 and plan.schedule == schedule and plan.waves_per_group == waves and plan.row_groups == 1
    assert vs.lib().vs_internal_reads_once(ctypes.byref(desc), 1) == (0 if paged else 1)
    need = vs.vs_attention_workspace_bytes(desc)
    ws = torch.empty(max(need, 256), device="cuda", dtype=torch.uint8).random_(0, 256)
    out = torch.full((B, T, Hq, d), float("nan"), device="cuda", dtype=torch.bfloat16)
    status = torch.full((B,), -99, device="cuda", dtype=torch.int32)
    lens_dev = torch.tensor(lens, device="cuda", dtype=torch.int32)
    assert vs.vs_tree_verify_attention(desc, q, kv[0], kv[1], lens_dev, parent, None, out, status, ws, need, gu.stream_ptr()) == 0
    torch.cuda.synchronize()
    assert (status == 0).all() and not out.isnan().any()
    group = Hq // Hkv
    for b, h in {(0, 0), (B - 1, Hkv - 1), (B // 2, Hkv // 3)}:
        n = lens[b] + T
        k, v = (x[table[b].long(), h].reshape(-1, d)[:n].double() if paged else x[b, h, :n].double() for x in kv)
        see = torch.zeros(T, T, dtype=torch.bool)
        for i in range(T):
            j = i
            while j >= 0:
                see[i, j] = True
                j = int(parent[b, j])
        qs = q[b, :, h * group:(h + 1) * group].reshape(T * group, d).double()
        s = qs @ k.T.contiguous() * d ** -0.5
        s[:, n - T:].masked_fill_(~see.repeat_interleave(group, 0).cuda(), float("-inf"))
        ref = (s.softmax(-1) @ v).cpu().numpy()
        gu.check_close(out[b, :, h * group:(h + 1) * group].reshape(T * group, d).float().cpu().numpy().astype("float64"), ref, 1.2e-2, 6e-3)
