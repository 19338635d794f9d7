"""Work that users of this library have it do, as cases that can be timed and compared.

A case is one of these passes, each through the library's public calls on one stream:

  step       one verification step of a speculative decoder: ancestor masks, attention of every
             decoder layer, acceptance (greedy, or stochastic at a temperature), commit of the
             accepted path into every layer's K/V cache
  attention  the verification attention of one layer, for callers who interleave it with the rest
             of a layer
  compress   the vision adaptor's attention: a few queries over the embeddings of each image
  accept     acceptance alone (greedy, or stochastic at a temperature) over a batch's logits
  draft      construction of a draft tree: the expansions level by level and the final selection

Values are N(0, 1) rounded once to the storage type. Trees are random with a depth of at most six
and at most four children per node. Acceptance logits are peaked rows in which the draft tokens
are likely ones. Every buffer that a program would keep from step to step (outputs, workspaces,
descriptors) is made in prepare().
"""
import math

import numpy as np
import torch

import paper_2509_15235_amd as vs

MAX_DEPTH, MAX_CHILDREN = 6, 4


def _case(name, kind, **sizes):
    return dict(name=name, kind=kind, **sizes)


def listed():
    return [
        # the smallest step: a toy model in fp32 (8 nodes over 64 tokens), where launches are everything
        _case("step tiny fp32", "step", dtype="f32", B=1, T=8, Hq=4, Hkv=1, d=64, lo=64, hi=64, paged=0, layers=1,
              V=1000, temperature=0.0),
        # interactive use: one sequence with one image, 28 layers of a grouped-query model, greedy
        _case("step one sequence gqa", "step", dtype="bf16", B=1, T=60, Hq=28, Hkv=4, d=128, lo=1696, hi=1696, paged=0,
              layers=28, V=152064, temperature=0.0),
        # a small server: four sequences of a multi-head model with a large image each, sampling
        _case("step four sequences mha", "step", dtype="bf16", B=4, T=60, Hq=32, Hkv=32, d=128, lo=2880, hi=3392,
              paged=0, layers=32, V=32000, temperature=1.0),
        # one layer of one sequence with four images in its context
        _case("attention long context", "attention", dtype="bf16", B=1, T=60, Hq=28, Hkv=4, d=128, lo=6684, hi=6684,
              paged=0, block=16, mask=1),
        # one layer of a serving batch: sequences of very different lengths over a paged cache
        _case("attention ragged paged", "attention", dtype="bf16", B=16, T=60, Hq=28, Hkv=4, d=128, lo=1024, hi=8192,
              paged=1, block=16, mask=1),
        # one layer of a full server: the same with 64 sequences
        _case("attention large batch", "attention", dtype="bf16", B=64, T=60, Hq=28, Hkv=4, d=128, lo=1024, hi=8192,
              paged=1, block=16, mask=1),
        # 64-channel heads, the 31-node tree of a depth-3 top-8 draft, ragged contiguous caches
        _case("attention small heads", "attention", dtype="bf16", B=8, T=31, Hq=32, Hkv=8, d=64, lo=257, hi=2047,
              paged=0, block=16, mask=0),
        # fp32 storage beyond the toy size: checking a bf16 deployment, or a model kept in fp32
        _case("attention fp32", "attention", dtype="f32", B=2, T=31, Hq=8, Hkv=2, d=128, lo=333, hi=600, paged=0,
              block=16, mask=1),
        # four images of one request through the vision adaptor, 16 learnable queries
        _case("compress four images", "compress", dtype="bf16", B=4, T=16, Hq=28, Hkv=4, d=128, lo=1000, hi=1296),
        # greedy acceptance of a serving batch at a large vocabulary
        _case("accept batch greedy", "accept", B=16, T=60, V=152064, temperature=0.0),
        # sampling at a vocabulary whose rows are not 16-byte aligned
        _case("accept batch sampling", "accept", B=4, T=31, V=32003, temperature=0.8),
        # the draft side of a step: depth 3, 8 nodes per expansion, 30 draft tokens
        _case("draft tree", "draft", B=2, V=152064, K=8, depth=3, N=30),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.499)))))))


def _vocab(rng, lo, hi):
    v = _log(rng, lo, hi)
    return v if rng.random() < 0.4 else max(64, v // 64 * 64)


HEADS = [(28, 4, 128), (28, 4, 128), (32, 32, 128), (8, 2, 128), (8, 1, 128), (32, 8, 64), (16, 16, 64)]


def draw(rng):
    kind = rng.choice(["attention"] * 4 + ["step", "step", "compress", "accept", "accept", "draft"])
    if kind == "draft":
        depth, K = rng.randint(2, 5), rng.randint(4, 16)
        M = K + (depth - 1) * K * K
        return dict(kind=kind, B=_log(rng, 1, 8), V=_vocab(rng, 8000, 152064), K=K, depth=depth,
                    N=min(63, M, rng.randint(16, 63)))
    if kind == "accept":
        V, T = _vocab(rng, 1000, 152064), _log(rng, 2, 64)
        return dict(kind=kind, B=_log(rng, 1, max(1, min(32, 145_000_000 // (T * V)))), T=T, V=V,
                    temperature=rng.choice([0.0, 0.0, 0.7, 1.0]))
    Hq, Hkv, d = rng.choice(HEADS)
    c = dict(kind=kind, dtype="bf16", Hq=Hq, Hkv=Hkv, d=d)
    if kind == "compress":
        hi = _log(rng, 64, 2880)
        c.update(B=_log(rng, 1, 16), T=_log(rng, 1, 64), lo=max(1, hi * rng.choice([2, 3, 4]) // 4), hi=hi)
        return c
    if rng.random() < 0.15:  # fp32: the small sizes
        c.update(dtype="f32", Hq=Hq // Hkv * min(2, Hkv), Hkv=min(2, Hkv))
        hi = _log(rng, 48, 800)
        T = _log(rng, 2, 40)
        B = _log(rng, 1, min(4, max(1, 100 // T)))
    elif kind == "step":
        hi = _log(rng, 256, 4096)
        B, T = _log(rng, 1, 8), _log(rng, 4, 64)
    else:
        hi = _log(rng, 128, 8192)
        B, T = _log(rng, 1, max(1, min(64, 1_500_000_000 // (hi * Hkv * d * 4)))), _log(rng, 1, 64)
    c.update(B=B, T=T, lo=max(16, hi // rng.choice([1, 2, 8])), hi=hi, paged=rng.choice([0, 1]))
    if kind == "attention":
        c.update(block=rng.choice([16, 16, 64]), mask=rng.choice([0, 1, 1]))
        return c
    most = min(5e9 / (B * hi * c["Hkv"] * d * 4), 4e11 / (4.0 * d * c["Hq"] * B * T * hi), 32)
    if c["dtype"] == "f32":
        most = min(4, 9e5 / (B * T * c["Hq"] * hi))
    c.update(layers=_log(rng, 1, max(1, int(most))), V=_vocab(rng, 1000, 152064),
             temperature=rng.choice([0.0, 0.0, 1.0]))
    return c


# ------------------------------------------------------------------------------- inputs


def _tree(r, T):
    """parent[] of a random tree in level order."""
    parent, depth, room = [-1], [0], [0]
    kids = [0]
    for i in range(1, T):
        if i <= MAX_DEPTH:
            p = i - 1  # a spine that reaches the depth
        else:
            p = room[r.integers(len(room))]
        parent.append(p)
        depth.append(depth[p] + 1)
        kids.append(0)
        kids[p] += 1
        if kids[p] >= MAX_CHILDREN:
            room.remove(p)
        if depth[i] < MAX_DEPTH:
            room.append(i)
    order = sorted(range(T), key=lambda i: depth[i])
    at = {old: new for new, old in enumerate(order)}
    return np.array([-1 if parent[i] < 0 else at[parent[i]] for i in order], dtype=np.int32)


def _trees(r, B, T):
    return np.stack([_tree(r, T) for _ in range(B)])


def _i32(*shape):
    return torch.zeros(shape, device="cuda", dtype=torch.int32)


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), device="cuda", dtype=torch.uint8)


def _check(rc):
    if rc != 0:
        raise vs.VSError(rc, "libvispec_verify")


class _Attention:
    """Queries, caches and descriptor of `layers` layers that share trees and lengths."""

    def __init__(self, c, r, g, layers, tree=True):
        B, T, Hq, Hkv, d = c["B"], c["T"], c["Hq"], c["Hkv"], c["d"]
        f32 = c["dtype"] == "f32"
        dt = torch.float32 if f32 else torch.bfloat16
        self.B, self.T, self.layers = B, T, layers
        lens = r.integers(c["lo"], c["hi"] + 1, size=B).astype(np.int32)
        slots = lens.astype(np.int64) + (T if tree else 0)
        desc = vs.AttnDesc(B=B, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=vs.VS_F32 if f32 else vs.VS_BF16,
                           softmax_scale=1.0 / math.sqrt(d), max_prefix_len=int(lens.max()))
        kv = vs.KVDesc(B=B, T=T, Hkv=Hkv, d=d, dtype=desc.dtype, num_layers=layers)
        if c.get("paged"):
            bs = c.get("block", 16)
            nblk = (slots + bs - 1) // bs
            most = (c["hi"] + T + bs - 1) // bs + 1
            pool = B * most
            table = np.zeros((B, most), dtype=np.int32)
            ids, at = r.permutation(pool).astype(np.int32), 0
            for b in range(B):
                table[b, :nblk[b]] = ids[at:at + nblk[b]]
                at += int(nblk[b])
            self.table = _dev(table)
            shape = (layers, pool, Hkv, bs, d)
            for x in (desc, kv):
                x.paged, x.block_size, x.max_blocks, x.num_blocks = 1, bs, table.shape[1], pool
                x.stride_block, x.stride_head, x.stride_tok = Hkv * bs * d, bs * d, d
                x.block_table = self.table.data_ptr()
        else:
            cap = c["hi"] + T + 4
            shape = (layers, B, Hkv, cap, d)
            for x in (desc, kv):
                x.capacity, x.stride_seq, x.stride_head, x.stride_tok = cap, Hkv * cap * d, cap * d, d
        kv.stride_layer = int(np.prod(shape[1:]))
        self.desc, self.kv = desc, kv
        self.k = torch.randn(shape, generator=g, device="cuda", dtype=dt)
        self.v = torch.randn(shape, generator=g, device="cuda", dtype=dt)
        self.q = torch.randn((layers, B, T, Hq, d), generator=g, device="cuda", dtype=dt)
        self.out = torch.zeros_like(self.q)
        # one layer's tensors, as a model's layers hold them
        self.per_layer = [(self.q[i], self.k[i], self.v[i], self.out[i]) for i in range(layers)]
        self.lens = _dev(lens)
        self.status = _i32(B)
        size = vs.vs_attention_workspace_bytes if tree else vs.vs_compress_attention_workspace_bytes
        self.ws_bytes = size(desc)
        self.ws = _workspace(self.ws_bytes)


class _Accept:
    """Logits, draft tokens and results of one acceptance call."""

    def __init__(self, c, r, g, parent_host, parent):
        B, T, V = c["B"], c["T"], c["V"]
        self.B, self.T, self.V, self.temperature, self.parent = B, T, V, c["temperature"], parent
        tokens = r.integers(0, V, size=(B, T)).astype(np.int32)
        self.tokens = _dev(tokens)
        # rows N(0, 3^2); a draft token's logit sits near the row's log-sum-exp, so that it is often the
        # argmax and often accepted by a draw
        self.logits = torch.randn((B, T, V), generator=g, device="cuda").mul_(3.0)
        if T > 1:
            b = np.repeat(np.arange(B), T - 1)
            level = np.log(V) + 4.5 + 1.5 * r.standard_normal(B * (T - 1))
            self.logits[_dev(b), _dev(parent_host[:, 1:].reshape(-1).astype(np.int64)),
                        _dev(tokens[:, 1:].reshape(-1).astype(np.int64))] = _dev(level.astype(np.float32))
        self.length, self.path, self.bonus, self.argmax, self.status = _i32(B), _i32(B, T), _i32(B), _i32(B, T), _i32(B)
        if self.temperature > 0:
            self.u_accept = torch.rand((B, T), generator=g, device="cuda")
            self.u_bonus = torch.rand((B,), generator=g, device="cuda")
            self.ws_bytes = vs.vs_accept_sample_workspace_bytes(B, T, V)
        else:
            self.ws_bytes = vs.vs_accept_workspace_bytes(B, T, V)
        self.ws = _workspace(self.ws_bytes)

    def run(self, stream):
        if self.temperature > 0:
            _check(vs.vs_tree_accept_sample(self.logits, self.V, self.V, self.temperature, self.tokens, self.parent,
                                            self.u_accept, self.u_bonus, self.B, self.T, self.length, self.path,
                                            self.bonus, self.status, self.ws, self.ws_bytes, stream))
            return [self.length, self.path, self.bonus, self.status]
        _check(vs.vs_tree_accept(self.logits, self.V, self.V, self.tokens, self.parent, self.B, self.T, self.length,
                                 self.path, self.bonus, self.argmax, self.status, self.ws, self.ws_bytes, stream))
        return [self.length, self.path, self.bonus, self.argmax, self.status]


class _Masks:
    def __init__(self, r, B, T):
        self.B, self.T = B, T
        self.host = _trees(r, B, T)
        self.parent = _dev(self.host)
        self.mask = torch.zeros((B, T), device="cuda", dtype=torch.int64)
        self.depth, self.status = _i32(B, T), _i32(B)

    def run(self, stream):
        _check(vs.vs_tree_mask_build(self.parent, self.B, self.T, self.mask, self.depth, self.status, stream))


class Step:
    def __init__(self, c, r, g):
        self.trees = _Masks(r, c["B"], c["T"])
        self.att = _Attention(c, r, g, c["layers"])
        self.accept = _Accept(c, r, g, self.trees.host, self.trees.parent)
        self.new_lens, self.commit_status = _i32(c["B"]), _i32(c["B"])

    def run(self, stream):
        a, t = self.att, self.trees
        t.run(stream)
        for q, k, v, out in a.per_layer:
            _check(vs.vs_tree_verify_attention(a.desc, q, k, v, a.lens, t.parent, t.mask, out, a.status, a.ws,
                                               a.ws_bytes, stream))
        got = self.accept.run(stream)
        _check(vs.vs_tree_kv_commit(a.kv, a.k, a.v, a.lens, self.accept.path, self.accept.length, self.new_lens,
                                    self.commit_status, stream))
        return [a.out, a.status, t.mask, t.depth] + got + [a.k, a.v, self.new_lens, self.commit_status]


class Attention:
    def __init__(self, c, r, g):
        self.trees = _Masks(r, c["B"], c["T"])
        self.att = _Attention(c, r, g, 1)
        self.mask = None
        if c["mask"]:
            self.trees.run(torch.cuda.current_stream().cuda_stream)
            self.mask = self.trees.mask

    def run(self, stream):
        a = self.att
        q, k, v, out = a.per_layer[0]
        _check(vs.vs_tree_verify_attention(a.desc, q, k, v, a.lens, self.trees.parent, self.mask, out, a.status, a.ws,
                                           a.ws_bytes, stream))
        return [out, a.status]


class Compress:
    def __init__(self, c, r, g):
        self.att = _Attention(c, r, g, 1, tree=False)

    def run(self, stream):
        a = self.att
        q, k, v, out = a.per_layer[0]
        _check(vs.vs_compress_attention(a.desc, q, k, v, a.lens, out, a.status, a.ws, a.ws_bytes, stream))
        return [out, a.status]


class Accept:
    def __init__(self, c, r, g):
        host = _trees(r, c["B"], c["T"])
        self.accept = _Accept(c, r, g, host, _dev(host))

    def run(self, stream):
        return self.accept.run(stream)


class Draft:
    def __init__(self, c, r, g):
        B, V, K, D, N = (c[x] for x in ("B", "V", "K", "depth", "N"))
        self.c = c
        self.cap = K + (D - 1) * K * K
        # the draft model's logits at each level's frontier: a handful of tokens hold most of a row
        self.logits = [torch.randn((B, 1 if lv == 0 else K, V), generator=g, device="cuda").mul_(3.0) for lv in range(D)]
        self.tok, self.par = _i32(B, self.cap), _i32(B, self.cap)
        self.score = torch.zeros((B, self.cap), device="cuda")
        self.front = [_i32(B, K) for _ in range(D)]
        self.cum = [torch.zeros((B, K), device="cuda") for _ in range(D)]
        self.root = _dev(r.integers(0, V, size=B).astype(np.int32))
        self.parent, self.tokens, self.cand = _i32(B, N + 1), _i32(B, N + 1), _i32(B, N + 1)
        self.num, self.status = _i32(B), _i32(B)
        self.ws_bytes = vs.vs_draft_expand_workspace_bytes(B, K, V, K)
        self.ws = _workspace(self.ws_bytes)

    def run(self, stream):
        B, V, K, D, N = (self.c[x] for x in ("B", "V", "K", "depth", "N"))
        cum = front = None
        base = 0
        for lv in range(D):
            F = 1 if lv == 0 else K
            _check(vs.vs_draft_expand(self.logits[lv], V, V, cum, front, B, F, K, base, self.cap, self.tok, self.score,
                                      self.par, self.front[lv], self.cum[lv], self.ws, self.ws_bytes, stream))
            cum, front = self.cum[lv], self.front[lv]
            base += F * K
        _check(vs.vs_draft_tree_build(self.tok, self.score, self.par, B, base, self.cap, N, self.root, self.parent,
                                      self.tokens, self.cand, self.num, self.status, stream))
        return [self.tok, self.score, self.par, self.front[-1], self.cum[-1], self.parent, self.tokens, self.cand,
                self.num, self.status]


KINDS = {"step": Step, "attention": Attention, "compress": Compress, "accept": Accept, "draft": Draft}


def prepare(case, seed):
    r = np.random.default_rng(seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return KINDS[case["kind"]](case, r, g)


def run(state):
    return state.run(torch.cuda.current_stream().cuda_stream)


# ------------------------------------------------------------------------------- work, tolerance


def _attention_work(c, tree):
    eb = 4 if c["dtype"] == "f32" else 2
    keys = (c["lo"] + c["hi"]) / 2  # mean length
    own = min(MAX_DEPTH, c["T"] - 1) / 2 + 1 if tree else 0  # ancestors and self, about
    flops = 4.0 * c["d"] * c["Hq"] * c["B"] * c["T"] * (keys + own)
    rows = 2.0 * c["B"] * c["Hkv"] * (keys + (c["T"] if tree else 0))
    return {"bytes": (rows + 2.0 * c["B"] * c["T"] * c["Hq"]) * c["d"] * eb, "flops": flops}


def _accept_work(c):
    return {"bytes": 4.0 * c["B"] * c["T"] * (c["V"] + 4), "flops": (1.0 if c["temperature"] == 0 else 4.0) * c["B"] * c["T"] * c["V"]}


def work(case):
    c = case
    if c["kind"] == "accept":
        return _accept_work(c)
    if c["kind"] == "draft":
        rows = c["B"] * (1 + (c["depth"] - 1) * c["K"])
        return {"bytes": 4.0 * rows * c["V"], "flops": 4.0 * rows * c["V"]}
    a = _attention_work(c, c["kind"] != "compress")
    if c["kind"] != "step":
        return a
    p = _accept_work(c)
    eb = 4 if c["dtype"] == "f32" else 2
    moved = 4.0 * c["layers"] * c["B"] * c["Hkv"] * c["d"] * eb * 2  # two accepted rows, K and V, read and written
    return {"bytes": c["layers"] * a["bytes"] + p["bytes"] + moved, "flops": c["layers"] * a["flops"] + p["flops"]}


def tolerance(case):
    c = case
    # a uniform within 1e-5 of its threshold may fall on either side; so may two scores at a cut
    near = 0.01 if c["kind"] == "draft" or c.get("temperature", 0.0) > 0 else 0.0
    if c["kind"] == "accept":
        return {"rel": 0.0, "differ": near} if near else "exact"
    if c["kind"] == "draft" or c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": near}
    # bf16: the output is rounded to 2^-9, and so is every probability before the second product
    return {"rel": 1e-2, "max": 0.1, "differ": near}
