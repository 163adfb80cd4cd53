"""The calls whose speed this library is kept by, with inputs, exact results and the bytes each cannot do without.

A case is one call (or one exchange round) of sparsified SGD with error feedback as a training program makes it through
``paper_2009_09271_amd``: a worker's fused step, W workers' steps in one batch, the aggregate of W messages, or the
batch followed by the aggregate applied to the parameters.  Layouts are one flat vector or the parameter tensors of
the networks this repository measures (ResNet-18, ResNet-50, BERT-base; drawn cases vary their width and depth), as one
segment ("flat" scope) or one segment per tensor ("layer" scope).
"""

import math

import numpy as np
import torch

import paper_2009_09271_amd as E

DEV = "cuda"
MOMENTUM, DECAY = 0.9, 1e-6  # the paper's momentum; its weight decay of 1e-4 times a learning rate of 0.01


def listed():
    return [
        # one bucket of a bucketed backward pass: launches and latency count
        _case("topk_bucket", "topk", net="vector", size=100003, density=0.01),
        # a small model's whole gradient
        _case("randk_flat_1m", "randk", net="vector", size=1 << 20, density=0.01),
        # the paper's own setting: ResNet-18, layer-wise, 1 %
        _case("topk_resnet18_layer", "topk", net="resnet18", size=64, scope="layer", density=0.01),
        # a whole exchange round of 8 workers simulated on one GPU, up to the new parameters
        _case("round_randk_resnet18", "randk_round", net="resnet18", size=64, scope="layer", density=0.01, W=8),
        # the headline workload: 16 workers' steps on ResNet-50, global scope, 0.1 %
        _case("topk_batch_resnet50", "topk_batch", net="resnet50", size=64, density=0.001, W=16),
        # what every rank does with the 16 gathered messages: top-k's crowd into the layers of large gradients
        _case("agg_topk_resnet50", "agg_topk", net="resnet50", size=64, density=0.001, W=16),
        # the paper's cheapest scheme on a mixed-precision gradient
        _case("randblock_resnet50_bf16", "randblock", net="resnet50", size=64, scope="layer", density=0.001, block=4096, dtype="bf16"),
        # a transformer trained in mixed precision, layer-wise
        _case("topk_bert_layer_bf16", "topk", net="bert", size=768, depth=12, scope="layer", density=0.01, dtype="bf16"),
        # a mild compression: many values are sent
        _case("topk_bert_flat_10pct", "topk", net="bert", size=768, depth=12, density=0.1),
        # 16 gathered messages of the transformer, in both message formats
        _case("agg_randk_bert_layer", "agg_randk", net="bert", size=768, depth=12, scope="layer", density=0.01, W=16),
        _case("agg_block_bert_layer", "agg_block", net="bert", size=768, depth=12, scope="layer", density=0.01, block=4096, W=16),
        # the largest model that one GPU's worker steps through in one call
        _case("randk_flat_1g_bf16", "randk", net="vector", size=1000000000, density=0.01, dtype="bf16"),
    ]


def _case(name, op, net, size, depth=0, scope="flat", density=0.01, block=1, dtype="f32", W=1):
    c = {"name": name} if name else {}
    c.update(op=op, net=net, size=size, depth=depth, scope=scope, density=density, block=block, dtype=dtype, W=W)
    return c


def draw(rng):
    """A case of the listed kinds: any of their calls, networks of other widths and depths, other densities and workers."""
    op = rng.choice(["topk", "topk", "randk", "randk", "randblock", "topk_batch", "randk_round", "agg_topk", "agg_randk", "agg_block"])
    many = op not in ("topk", "randk", "randblock")
    net = rng.choice(["vector", "resnet18", "resnet50", "bert"])
    depth = 0
    if net == "vector":
        size = int(round(math.exp(rng.uniform(math.log(1 << 16), math.log((1 << 26) if many else (1 << 29))))))
    elif net == "bert":
        size, depth = 16 * rng.randint(8, 48), rng.randint(2, 12)
    else:
        size = rng.randint(16, 72)
    c = _case("", op, net, size, depth,
              scope="flat" if net == "vector" else rng.choice(["flat", "layer"]),
              density=round(math.exp(rng.uniform(math.log(0.001), math.log(0.1))), 6),
              block=1 << rng.randint(0, 16) if op in ("randblock", "agg_block") else 1,
              dtype=rng.choice(["f32", "bf16"]) if not op.startswith("agg") else "f32")
    if many:
        c["W"] = max(2, min(rng.randint(2, 16), 400000000 // sum(n for n, _, _ in _tensors(c))))
    return c


# ---- layouts ---------------------------------------------------------------------------------------------------------
def _tensors(case):
    """(elements, fan-in, columns of an embedding table or 0) of every parameter tensor, in flattening order."""
    net, w = case["net"], case["size"]
    out = []

    def mat(rows, cols, table=False):
        out.append((rows * cols, cols, cols if table else 0))

    def vec(n, times=1):
        for _ in range(times):
            out.append((n, out[-1][1], 0))

    if net == "vector":
        return [(w, 1, 0)]
    if net == "bert":
        mat(30522, w, True)
        mat(512, w)
        mat(2, w)
        vec(w, 2)
        for _ in range(case["depth"]):
            for rows, cols, norm in ((w, w, 0), (w, w, 0), (w, w, 0), (w, w, 2), (4 * w, w, 0), (w, 4 * w, 2)):
                mat(rows, cols)
                vec(rows, 1 + norm)
        mat(w, w)
        vec(w)
        return out
    deep = net == "resnet50"
    mat(w, 3 * 49)
    vec(w, 2)
    cin = w
    for planes, blocks in zip((w, 2 * w, 4 * w, 8 * w), (3, 4, 6, 3) if deep else (2, 2, 2, 2)):
        cout = 4 * planes if deep else planes
        for b in range(blocks):
            convs = ((planes, cin), (planes, 9 * planes), (cout, planes)) if deep else ((planes, 9 * cin), (planes, 9 * planes))
            for rows, cols in convs:
                mat(rows, cols)
                vec(rows, 2)
            if b == 0 and cin != cout:
                mat(cout, cin)
                vec(cout, 2)
            cin = cout
    mat(1000, cin)
    vec(1000)
    return out


def _offsets(case):
    sizes = [n for n, _, _ in _tensors(case)]
    offs = [0] + np.cumsum(np.asarray(sizes, dtype=np.int64)).tolist()
    return offs if case["scope"] == "layer" else [0, offs[-1]]


def _ks(case, offs):
    """k per segment: round half up of density times the segment's length, from 1 to that length."""
    return [min(max(int(math.floor(case["density"] * (b - a) + 0.5)), 1), b - a) for a, b in zip(offs, offs[1:])]


# ---- inputs ----------------------------------------------------------------------------------------------------------
class _Draws:
    """Gradients of one model: heavy-tailed values of a scale of its own per tensor, and rows of the embedding table that
    no batch touches (90 % of them) exactly zero."""

    def __init__(self, case, seed):
        self.gen = torch.Generator(DEV)
        self.gen.manual_seed(int(seed))
        self.tensors = _tensors(case)
        rng = np.random.default_rng([int(seed), 999])
        self.scale = [0.01 if len(self.tensors) == 1 else 10.0 ** rng.uniform(-1.5, 0.0) / math.sqrt(fan) for _, fan, _ in self.tensors]
        self.zero = [torch.from_numpy(rng.random(n // cols) < 0.9).to(DEV) if cols else None for n, _, cols in self.tensors]

    def gradient(self, dtype=torch.float32):
        d = sum(n for n, _, _ in self.tensors)
        g = torch.empty(d, dtype=dtype, device=DEV)
        at = 0
        for (n, _, cols), s, zero in zip(self.tensors, self.scale, self.zero):
            for a in range(0, n, 1 << 26):
                m = min(1 << 26, n - a)
                x = torch.randn(m, generator=self.gen, device=DEV)
                x.mul_(torch.empty(m, device=DEV).exponential_(1.0, generator=self.gen).mul_(2.0).sqrt_()).mul_(s)  # Laplace
                g[at + a:at + a + m] = x.to(dtype)
            if zero is not None:
                g[at:at + n].view(-1, cols)[zero] = 0.0
            at += n
        return g


def _grads(case, draws):
    """The gradients of four steps: two draws and their negations, so that the residual neither grows nor dies out over
    many steps (a training run's gradients are mostly noise around a small mean)."""
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    a, b = draws.gradient(dtype), draws.gradient(dtype)
    return [a, b, -a, -b]


def _seed_of(seed, w):
    return (int(seed) << 16) | w


def prepare(case, seed):
    op, W = case["op"], case["W"]
    offs = _offsets(case)
    lay = E.Layout(offs[-1], offs, case["density"], case["block"]).bind(DEV)
    draws = _Draws(case, seed)
    K, d, L = lay.K, lay.d, lay.n_seg
    s = {"op": op, "lay": lay, "W": W, "step": 0}
    if op.startswith("agg"):
        s["idx"], s["val"] = _messages(case, draws, offs)
        s["out"] = torch.empty(d, dtype=torch.float32, device=DEV)
        s["ws"] = lay.workspace(E.EF_OP_AGG_SPARSE, W, DEV) if op != "agg_block" else None
        return s
    rows = [_grads(case, draws) for _ in range(W)]
    s["g"] = [[r[t] for r in rows] for t in range(4)]
    s["e"] = [draws.gradient() for _ in range(W)]
    s["seeds"] = [_seed_of(seed, w) for w in range(W)]
    s["idx"] = torch.empty((W, L if op == "randblock" else K), dtype=torch.int32, device=DEV)
    s["val"] = torch.empty((W, K), dtype=torch.float32, device=DEV)
    if op in ("topk", "randk"):
        s["ws"] = lay.workspace(E.EF_OP_TOPK if op == "topk" else E.EF_OP_RANDK, 1, DEV)
    elif op in ("topk_batch", "randk_round"):
        s["ws"], s["stride"] = E.batch_workspace(lay, E.EF_OP_TOPK if op == "topk_batch" else E.EF_OP_RANDK, W, DEV)
    if op == "randk_round":
        s["x"], s["m"] = draws.gradient().mul_(10.0), draws.gradient()
        s["agg_ws"] = lay.workspace(E.EF_OP_AGG_SPARSE, W, DEV)
    return s


def _messages(case, draws, offs):
    """W messages as an allGather delivers them."""
    ks = _ks(case, offs)
    idx, val = [], []
    for _ in range(case["W"]):
        acc = draws.gradient()
        if case["op"] == "agg_block":
            sizes = np.diff(offs).tolist()
            blocks = [(bl, -(-n // bl)) for n, bl in ((n, case["block"] if n > case["block"] else 1) for n in sizes)]
            u = torch.rand(len(ks), generator=draws.gen, device=DEV, dtype=torch.float64).cpu().tolist()
            starts = [min(int(x * nb), nb - 1) * bl for x, (bl, nb) in zip(u, blocks)]
            pick = [(torch.arange(st, st + k, device=DEV) % n) + o for st, k, n, o in zip(starts, ks, sizes, offs)]
            idx.append(torch.tensor(starts, dtype=torch.int32, device=DEV))
            val.append(acc[torch.cat(pick)])
            continue
        key = acc.abs() if case["op"] == "agg_topk" else torch.rand(acc.numel(), generator=draws.gen, device=DEV)
        pick = torch.cat([torch.topk(key[o:e], k, sorted=False).indices.sort().values + o for o, e, k in zip(offs, offs[1:], ks)])
        idx.append(pick.to(torch.int32))
        val.append(acc[pick])
    return torch.stack(idx), torch.stack(val)


# ---- one pass --------------------------------------------------------------------------------------------------------
def run(s):
    op, lay, W = s["op"], s["lay"], s["W"]
    if op.startswith("agg"):
        E.decompress_aggregate(lay, E.EF_MSG_BLOCK if op == "agg_block" else E.EF_MSG_SPARSE, W, s["idx"], s["val"], s["out"], s["ws"])
        return {"out": s["out"]}
    t = s["step"]
    s["step"] = t + 1
    g, e = s["g"][t % 4], s["e"]
    out = {"e": e, "idx": s["idx"], "val": s["val"]}
    if op == "topk":
        E.ef_step_topk(lay, g[0], e[0], s["idx"][0], s["val"][0], s["ws"])
    elif op == "randk":
        E.ef_step_randk(lay, g[0], e[0], s["seeds"][0], t, s["idx"][0], s["val"][0], s["ws"])
    elif op == "randblock":
        E.ef_step_randblock(lay, g[0], e[0], s["seeds"][0], t, s["idx"][0], s["val"][0])
    elif op == "topk_batch":
        E.ef_step_topk_batch(lay, g, e, s["idx"], s["val"], s["ws"], s["stride"])
    else:
        E.ef_step_randk_batch(lay, g, e, s["seeds"], t, s["idx"], s["val"], s["ws"], s["stride"])
        E.decompress_aggregate_apply(lay, E.EF_MSG_SPARSE, W, s["idx"], s["val"], s["x"], s["m"], MOMENTUM, DECAY, None, s["agg_ws"])
        out.update(x=s["x"], m=s["m"])
    return out


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def work(case):
    offs = _offsets(case)
    d, K, L, W, op = offs[-1], sum(_ks(case, offs)), len(offs) - 1, case["W"], case["op"]
    entry = 4 * K + 4 * L if op in ("randblock", "agg_block") else 8 * K
    if op.startswith("agg"):
        return {"bytes": 4 * d + W * entry, "flops": W * K + d}
    step = (10 if case["dtype"] == "bf16" else 12) * d + entry
    if op == "randk_round":  # and the W messages read, parameters and momentum read and written
        return {"bytes": W * step + 16 * d + W * entry, "flops": W * d + W * K + 6 * d}
    return {"bytes": W * step, "flops": W * d}


def tolerance(case):
    """Every output of the library is defined to the bit: the selections by a total order, the sums by the workers'
    order, each float32 operation rounded on its own."""
    return "exact"


# ---- the same in 64 bits, in plain torch -----------------------------------------------------------------------------
_M = 0xFFFFFFFF


def _mulhilo(a, b):
    """High and low words of a * b (a: a number, b: int64 tensor, both below 2^32)."""
    t = a * (b & 0xFFFF)
    u = a * (b >> 16) + (t >> 16)
    return u >> 16, ((u << 16) | (t & 0xFFFF)) & _M


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 (Salmon et al., SC 2011) on int64 tensors of 32-bit words."""
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, c0)
        h1, l1 = _mulhilo(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & _M, (k1 + 0xBB67AE85) & _M
    return c0, c1, c2, c3


def _random_keys(n, l, step, seed):
    """The random-k keys of a segment's n positions, in pieces of (first position, keys)."""
    for a in range(0, n, 1 << 26):
        m = min(1 << 26, n - a)
        c0 = torch.arange(a // 4, a // 4 + -(-m // 4), device=DEV)
        one = torch.zeros_like(c0)
        x = _philox(c0, one, one + step, one + (0x01000000 | l), seed & _M, seed >> 32)
        yield a, torch.stack(x, 1).reshape(-1)[:m]


def _support(case, offs, ks, acc, seed, step):
    """Indices a worker sends, ascending (block-random-k: in run order), by the definition of its scheme."""
    picked = []
    for l, (o, e, k) in enumerate(zip(offs, offs[1:], ks)):
        n = e - o
        if case["op"].startswith("topk"):  # largest magnitude, then lowest index
            key = (acc[o:e].view(torch.int32).to(torch.int64) & 0x7FFFFFFF) << 32 | (_M - torch.arange(n, device=DEV))
            got = _M - (torch.topk(key, k, sorted=False).values & _M)
        elif case["op"].startswith("randk"):  # smallest key, then lowest index
            most = min(1 << 32, int((k + 8 * math.sqrt(k) + 64) / n * 2.0 ** 32))
            pos, keys = [], []
            for a, u in _random_keys(n, l, step, seed):
                at = (u < most).nonzero().reshape(-1)
                pos.append(at + a)
                keys.append(u[at])
            key = torch.cat(keys) << 31 | torch.cat(pos)
            got = torch.sort(key).values[:k] & 0x7FFFFFFF
        else:
            b = case["block"] if n > case["block"] else 1
            zero = torch.zeros(1, dtype=torch.int64, device=DEV)
            x = _philox(zero, zero, zero + step, zero + (0x02000000 | l), seed & _M, seed >> 32)
            r = int(x[0]) | int(x[1]) << 32
            picked.append((torch.arange(k, device=DEV) + b * (r * -(-n // b) >> 64)) % n + o)
            continue
        picked.append(got.sort().values + o)
    return torch.cat(picked)


def exact(case, seed):
    s = prepare(case, seed)
    op, W = case["op"], case["W"]
    offs = _offsets(case)
    ks, d = _ks(case, offs), offs[-1]
    if op.startswith("agg"):
        if op == "agg_block":
            at = [torch.cat([(torch.arange(k, device=DEV) + st) % (e - o) + o for k, st, o, e in zip(ks, s["idx"][w].cpu().tolist(), offs, offs[1:])]) for w in range(W)]
        else:
            at = [s["idx"][w].to(torch.int64) for w in range(W)]
        q = torch.zeros(d, dtype=torch.float64, device=DEV)
        for w in range(W):
            q[at[w]] += s["val"][w].double()  # a message holds a position once
        return {"out": q / W}
    es, vals, q = [], [], torch.zeros(d, dtype=torch.float64, device=DEV) if op == "randk_round" else None
    for w in range(W):
        g, e = s["g"][0][w], s["e"][w]
        at = _support(case, offs, ks, g.float() + e, s["seeds"][w], 0)
        e64 = g.double() + e.double()
        vals.append(e64[at])
        e64[at] = 0.0
        es.append(e64)
        if q is not None:
            q[at] += vals[-1]
    out = {"e": es, "idx": None, "val": torch.stack(vals)}
    if q is not None:
        m = MOMENTUM * s["m"].double() + (q / W + DECAY * s["x"].double())
        out.update(x=s["x"].double() - m, m=m)
    return out
