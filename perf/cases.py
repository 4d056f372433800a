"""The calls this package is timed on: MoE blocks and stacks as programs run them.

A case is a dict of plain values.  "block" cases run one FarSkip MoE block on
one expert-parallel rank (``MoEBlock.begin`` / ``finish``), "pair" cases the
block with the next layer's linear between its two phases, "replicated" cases
a stack of the replicated-activation inference variant.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, s)    what a program holds before the call: weights, a block
                        or stack with its buffers, token activations
    run(state)          one pass, and its outputs
    work(case)          bytes and flops the pass cannot do without
    tolerance(case)     how far two correct implementations may differ
    exact(case, s)      the same outputs from plain torch in 64 bits
"""

import math
from types import SimpleNamespace

import torch

import paper_2511_11505_amd as fs
from paper_2511_11505_amd.replicated import ReplicatedStack

DEV = "cuda:0"
WEIGHT_STD = 0.02     # all weights ~ N(0, 0.02^2), tokens ~ N(0, 1)
Y_REMOTE_STD = 1.8    # rows returned by the other ranks' experts

# Layer shapes: one DeepSeek-V2-Lite-shaped, Llama-4-Scout-shaped and
# DeepSeek-V3-shaped MoE layer (the last as one rank of EP = 8), and one
# DeepSeek-V2-shaped layer on replicated activations (EP = TP = 8).
DSV2LITE = dict(kind="block", hidden=2048, n_experts=64, top_k=6, ffn=1408, score="softmax",
                norm_topk=False, n_shared=2, ffn_shared=1408, dtype="bf16")
SCOUT = dict(kind="block", hidden=5120, n_experts=16, top_k=1, ffn=8192, score="sigmoid",
             norm_topk=False, n_shared=1, ffn_shared=8192, bias="uniform", dtype="bf16")
DSV3 = dict(kind="block", hidden=7168, n_experts=256, top_k=8, ffn=2048, score="sigmoid",
            norm_topk=True, n_shared=1, ffn_shared=2048, n_groups=8, topk_groups=4, ep_size=8,
            dtype="bf16", comm=True)
DSV2_AR = dict(kind="replicated", layers=1, hidden=5120, n_experts=160, top_k=6, ffn=1536,
               score="softmax", norm_topk=False, n_shared=2, ffn_shared=1536, n_groups=8,
               topk_groups=3, routed_scale=16.0, ep_size=8, dtype="bf16", comm=True)
TINY = dict(kind="pair", hidden=256, n_experts=8, top_k=2, ffn=512, score="softmax",
            norm_topk=True, dtype="f32", comm=True)

DEFAULTS = dict(n_groups=1, topk_groups=1, n_shared=0, ffn_shared=0, routed_scale=1.0, ep_size=1,
                ep_rank=0, bias="none", fp8="none", fragment_order=False, comm=False, layers=1)


def listed():
    return [
        # single-stream generation on one GPU: one token per step, weights
        # laid out for streaming; launches and latency count
        dict(DSV2LITE, name="dsv2lite_one_token", n_tokens=1, fragment_order=True),
        # the fp32 block pair of the smallest workload: every launch is short
        dict(TINY, name="tiny_pair_f32", n_tokens=128),
        # a serving step of one EP rank of eight: 64 tokens per rank, skewed
        # expert popularity, bf16 and FP8 routed experts
        dict(DSV3, name="dsv3_decode", n_tokens=64, bias="zipf", fragment_order=True),
        dict(DSV3, name="dsv3_decode_fp8", n_tokens=64, bias="zipf", fragment_order=True,
             fp8="routed"),
        # a mixed batch (prefill chunks and decode tokens together) on one
        # GPU, row-major weights, a ragged token count
        dict(DSV2LITE, name="dsv2lite_mixed_batch", n_tokens=333),
        # widths that the largest tiles do not divide, odd top-k and tokens
        dict(kind="block", name="odd_widths", hidden=1408, n_experts=24, top_k=3, ffn=960,
             score="sigmoid", norm_topk=True, n_shared=1, ffn_shared=704, bias="uniform",
             dtype="bf16", n_tokens=777),
        # the fp32 block at a model's width (numerics checks, fp32 serving)
        dict(DSV2LITE, name="dsv2lite_f32", n_tokens=512, dtype="f32"),
        # prefill on one GPU
        dict(DSV2LITE, name="dsv2lite_prefill", n_tokens=4096),
        # prefill of the replicated-activation variant, one layer of the stack
        # (a second layer's router would turn roundings into other experts)
        dict(DSV2_AR, name="dsv2_replicated_prefill", n_tokens=4096),
        # prefill of one EP rank of eight, bf16 and FP8 experts
        dict(DSV3, name="dsv3_prefill", n_tokens=4096),
        dict(DSV3, name="dsv3_prefill_fp8", n_tokens=4096, fp8="all"),
        # the largest: the headline prefill
        dict(SCOUT, name="scout_prefill", n_tokens=8192, comm=True),
    ]


def draw(rng):
    def tokens(lo, hi):
        n = round(math.exp(rng.uniform(math.log(lo), math.log(hi))))
        return min(hi, max(lo, n + rng.choice((0, 0, 1, -1, 3))))

    kind = rng.choice(("dsv2lite", "dsv2lite", "dsv3", "dsv3", "scout", "widths", "widths", "f32",
                       "tiny", "replicated"))
    if kind == "dsv2lite":
        c = dict(DSV2LITE, n_tokens=tokens(1, 8192))
    elif kind == "dsv3":
        c = dict(DSV3, n_tokens=tokens(1, 4096), bias=rng.choice(("none", "zipf")))
    elif kind == "scout":
        c = dict(SCOUT, n_tokens=tokens(16, 8000), comm=rng.random() < 0.5)
    elif kind == "widths":
        E = rng.choice((8, 16, 24, 40, 60, 64, 96, 128))
        c = dict(kind="block", hidden=128 * rng.randint(4, 40), n_experts=E,
                 top_k=rng.randint(1, 8), ffn=64 * rng.randint(6, 40),
                 score=rng.choice(("softmax", "sigmoid")), norm_topk=rng.random() < 0.5,
                 n_shared=rng.randint(0, 2), ffn_shared=64 * rng.randint(4, 24), dtype="bf16",
                 n_tokens=tokens(4, 3000))
    elif kind == "f32":
        c = dict(DSV2LITE, n_tokens=tokens(2, 1500), dtype="f32")
    elif kind == "tiny":
        c = dict(TINY, n_tokens=tokens(16, 2000))
    else:
        c = dict(DSV2_AR, n_tokens=tokens(32, 4000))
    if c["kind"] == "block" and c["dtype"] == "bf16" and kind != "widths":
        c["fragment_order"] = c["n_tokens"] <= 512 and rng.random() < 0.6
        c["fp8"] = rng.choice(("none", "none", "routed", "all"))
    return c


# ------------------------------------------------------------------ inputs
def _cfg(case):
    c = SimpleNamespace(**{**DEFAULTS, **case})
    c.n_local = c.n_experts // c.ep_size
    c.ep_mode = "allreduce" if c.kind == "replicated" else "a2a"
    return c


def _normal(shape, std, dtype, seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1009 + tag) & 0x7FFFFFFFFFFF)
    t = torch.empty(shape, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device=DEV)
    t.normal_(0.0, std, generator=g)
    return t


def _bias(c, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1009 + 900) & 0x7FFFFFFFFFFF)
    if c.bias == "uniform":
        return torch.rand(c.n_experts, generator=g, device=DEV) * 0.2 - 0.1
    if c.bias == "zipf":
        rank = torch.randperm(c.n_experts, generator=g, device=DEV).double() + 1.0
        return (-0.05 * 1.2 * torch.log(rank)).float()
    return None


def _weights(c, seed, layer=0):
    """One layer's weights; the shared experts merged into one SwiGLU."""
    d, E, F, El, SF, t = c.hidden, c.n_experts, c.ffn, c.n_local, c.n_shared * c.ffn_shared, 100 * layer
    n = lambda shape, tag: _normal(shape, WEIGHT_STD, c.dtype, seed, t + tag)
    w = SimpleNamespace(router=n((E, d), 1), bias=_bias(c, seed + layer), gate_up=n((El, 2 * F, d), 2),
                        down=n((El, d, F), 3), sh_gate_up=None, sh_down=None, nxt=None, a=None, b=None)
    if c.kind == "replicated":
        W = SF // c.ep_size          # this rank's tensor-parallel share
        w.a, w.b = n((d // c.ep_size, d), 6), n((d, d // c.ep_size), 7)
    else:
        W = SF
    if SF:
        w.sh_gate_up, w.sh_down = n((2 * W, d), 4), n((d, W), 5)
    if c.kind == "pair":
        w.nxt = n((d, d), 8)
    return w


def _tokens(c, seed):
    sources = 1 if c.kind == "replicated" else c.ep_size
    return _normal((sources, c.n_tokens, c.hidden), 1.0, c.dtype, seed, 10)


def _y_remote(c, seed):
    return _normal((c.n_tokens * c.top_k, c.hidden), Y_REMOTE_STD, c.dtype, seed, 11)


def prepare(case, seed):
    c = _cfg(case)
    x_all = _tokens(c, seed)
    comm = torch.cuda.Stream(device=DEV) if c.comm else None
    if c.kind == "replicated":
        layers = []
        for k in range(c.layers):
            w = _weights(c, seed, k)
            layers.append(dict(w_router=w.router, bias=w.bias, w_gate_up=w.gate_up, w_down=w.down,
                               sh_gate_up=w.sh_gate_up, sh_down=w.sh_down, w_a=w.a, w_b=w.b))
        return dict(c=c, x=x_all[0], stack=ReplicatedStack(c, layers, device=DEV), comm=comm)
    w = _weights(c, seed)
    block = fs.MoEBlock(c, w.router, w.bias, w.gate_up, w.down, w.sh_gate_up, w.sh_down, device=DEV,
                        with_comm=c.comm, fp8=None if c.fp8 == "none" else c.fp8,
                        fragment_order=c.fragment_order)
    if c.ep_size > 1:
        # what the other ranks send; rows of y that no local expert writes
        # stay as they are
        block.t["y"].zero_()
        block.set_max_recv_rows(fs.prepare_remote_sources(block, x_all, w.router, w.bias,
                                                          _y_remote(c, seed)))
    x = x_all[c.ep_rank].clone()
    st = dict(c=c, x=x, block=block, comm=comm, w=w, partial=torch.empty_like(x))
    if c.kind == "pair":
        st["nxt"], st["out"] = torch.empty_like(x), torch.empty_like(x)
    return st


def run(state):
    c, x, comm = state["c"], state["x"], state["comm"]
    if c.kind == "replicated":
        stack = state["stack"]
        out = stack.farskip(x, comm=comm)
        return dict(out=out)
    block, partial = state["block"], state["partial"]
    block.begin(x, partial, comm=comm)
    out = partial
    if c.kind == "pair":
        # the far-skipped next layer reads the partial input between phases
        out, nxt = state["out"], state["nxt"]
        fs.fs_dense_linear(block.desc.dtype, c.n_tokens, c.hidden, c.hidden, partial,
                           state["w"].nxt, nxt)
        fs.fs_farskip_residual(block.desc, out, partial, nxt)
    block.finish(x, out, comm=comm)
    res = dict(out=out, topk_ids=block.t["topk_ids"], topk_w=block.t["topk_w"],
               counts=block.t["src_counts"])
    if c.ep_size > 1:
        res["y"] = block.t["y"]
    return res


def work(case):
    c = _cfg(case)
    N, d, E, k, F, R, El = c.n_tokens, c.hidden, c.n_experts, c.top_k, c.ffn, c.ep_size, c.n_local
    SF = c.n_shared * c.ffn_shared
    es = 4 if c.dtype == "f32" else 2
    we = 1 if c.fp8 != "none" else es
    ws = 1 if c.fp8 == "all" else es
    if c.kind == "replicated":
        rows, SF, seen = N * k / R, SF / R, N
    else:
        rows, seen = N * k, N * R     # a balanced rank receives as much as it sends
    active = El * (1.0 - (1.0 - k / E) ** seen)
    flops = 2.0 * N * d * E + 6.0 * rows * d * F + 6.0 * N * d * SF
    bytes_ = active * 3 * d * F * we + 3 * d * SF * ws + E * d * es + 2 * N * d * es
    if c.kind == "pair":
        flops += 2.0 * N * d * d
        bytes_ += d * d * es
    elif c.kind == "replicated":
        flops = c.layers * (flops + 4.0 * N * d * d / R)
        bytes_ = c.layers * (bytes_ - 2 * N * d * es + 2 * d * d / R * es) + 2 * N * d * es
    elif R > 1:
        # rows received from the other ranks and returned to them
        bytes_ += rows * (R - 1) / R * d * (we + es)
    return dict(bytes=float(bytes_), flops=float(flops))


def tolerance(case):
    # about four times what was measured against exact(): fp32 rel 7e-7 and
    # max 6e-6; FP8 rel 9e-3 and max 0.42 (one code of the re-quantised
    # activation more or less); bf16 rel 3.1e-3 and max 0.034
    c = _cfg(case)
    if c.dtype == "f32":
        return {"rel": 3e-6, "max": 3e-5, "differ": 1e-3}
    if c.fp8 != "none":
        return {"rel": 3e-2, "max": 0.95, "differ": 1e-3}
    return {"rel": 1.2e-2, "max": 0.14, "differ": 1e-3}


# ------------------------------------------------------------------ 64 bits
def _logits_f32(x, w):
    """fp32 logits in the router's documented order: products added one at a
    time within slices of 256, the slice sums in ascending order."""
    N, d = x.shape
    E, S = w.shape[0], (d + 255) // 256
    pad = S * 256 - d
    xs = torch.nn.functional.pad(x.float(), (0, pad)).view(N, S, 256)
    ws = torch.nn.functional.pad(w.float(), (0, pad)).view(E, S, 256).permute(2, 0, 1).contiguous()
    out = torch.empty((N, E), dtype=torch.float32, device=x.device)
    step = max(1, (1 << 27) // (E * S))
    for t in range(0, N, step):
        xc = xs[t:t + step].permute(2, 0, 1).contiguous()
        acc = torch.zeros((xc.shape[1], E, S), dtype=torch.float32, device=x.device)
        for i in range(256):
            acc += xc[i][:, None, :] * ws[i][None]
        tot = torch.zeros((xc.shape[1], E), dtype=torch.float32, device=x.device)
        for s in range(S):
            tot = tot + acc[:, :, s]
        out[t:t + step] = tot
    return out


def _route(c, x, w_router, bias):
    """Selected experts (by the fp32 keys) and their 64-bit gate weights."""
    z32 = _logits_f32(x, w_router)
    z = x.double() @ w_router.double().T
    if c.score == "softmax":
        key, p = z32, torch.softmax(z, dim=1)
    else:
        key, p = torch.sigmoid(z32), torch.sigmoid(z)
        if bias is not None:
            key = key + bias
    if c.n_groups > 1:
        N = key.shape[0]
        kg = key.view(N, c.n_groups, -1)
        gs = kg.topk(min(2, kg.shape[2]), dim=2).values.sum(2)
        keep = torch.sort(gs, dim=1, descending=True, stable=True).indices[:, :c.topk_groups]
        mask = torch.ones_like(gs, dtype=torch.bool).scatter_(1, keep, False)
        key = kg.masked_fill(mask[:, :, None], -math.inf).view(N, -1)
    ids = torch.sort(key, dim=1, descending=True, stable=True).indices[:, :c.top_k]
    w = p.gather(1, ids)
    if c.norm_topk:
        w = w / w.sum(1, keepdim=True)
    return ids, w * c.routed_scale


def _fp8(t):
    """Row-wise E4M3 quantisation of t and back, in 64 bits."""
    t = t.float()
    amax = t.abs().amax(-1, keepdim=True)
    scale = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    inv = torch.where(amax > 0, 448.0 / amax, torch.zeros_like(amax))
    code = (t * inv).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return code.to(torch.float64) * scale.double()


def _ffn(x, gate_up, down, fp8):
    F = gate_up.shape[0] // 2
    if fp8:
        gu = _fp8(x) @ _fp8(gate_up).T
        h = torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]
        return _fp8(h.to(torch.bfloat16)) @ _fp8(down).T
    gu = x.double() @ gate_up.double().T
    h = torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]
    return h @ down.double().T


def _rows_of(ids):
    """Send row of every slot: ordered by expert, then token."""
    order = torch.argsort(ids.reshape(-1), stable=True)
    s2r = torch.empty_like(order)
    s2r[order] = torch.arange(order.numel(), device=order.device)
    return s2r


def exact(case, seed):
    c = _cfg(case)
    x_all = _tokens(c, seed)
    if c.kind == "replicated":
        return _exact_replicated(c, seed, x_all[0].double())
    w = _weights(c, seed)
    N, d, k, R, r, El = c.n_tokens, c.hidden, c.top_k, c.ep_size, c.ep_rank, c.n_local
    cap = N * k
    y = torch.zeros((R * cap, d), dtype=torch.float64, device=DEV)
    if R > 1:
        y[r * cap:(r + 1) * cap] = _y_remote(c, seed).double()
    routes = [_route(c, x_all[s], w.router, w.bias) for s in range(R)]
    s2r = [_rows_of(ids) for ids, _ in routes]
    for e in range(El):
        xs, at = [], []
        for s in range(R):
            slots = (routes[s][0].reshape(-1) == r * El + e).nonzero()[:, 0]
            xs.append(x_all[s][slots // k])
            at.append(s * cap + s2r[s][slots])
        xs, at = torch.cat(xs), torch.cat(at)
        if at.numel():
            y[at] = _ffn(xs, w.gate_up[e], w.down[e], c.fp8 != "none")
    ids, gate = routes[r]
    x = x_all[r].double()
    out = x.clone()
    if c.n_shared:
        out += _ffn(x_all[r], w.sh_gate_up, w.sh_down, c.fp8 == "all")
    if c.kind == "pair":
        out = out + out @ w.nxt.double().T
    rows = s2r[r].view(N, k) + r * cap
    for j in range(k):
        out += gate[:, j:j + 1] * y[rows[:, j]]
    counts = torch.stack([torch.bincount(i.reshape(-1), minlength=c.n_experts) for i, _ in routes])
    res = dict(out=out, topk_ids=ids, topk_w=gate, counts=counts)
    if R > 1:
        res["y"] = y
    return res


def _exact_replicated(c, seed, x):
    """p and o are the partial and the full residual; attention reads p, the
    experts read o, and the routed sum joins the residual one layer later."""
    p = o = x
    lo = c.ep_rank * c.n_local
    routed = None
    for k in range(c.layers):
        w = _weights(c, seed, k)
        msg = (p @ w.a.double().T) @ w.b.double().T
        if routed is not None:
            o = p + routed
        if c.n_shared:
            msg = msg + _ffn(o, w.sh_gate_up, w.sh_down, False)
        # the router reads the residual as it is held, in 16 bits
        oh = o.to(torch.float32 if c.dtype == "f32" else torch.bfloat16)
        ids, gate = _route(c, oh, w.router, w.bias)
        routed = torch.zeros_like(o)
        for e in range(c.n_local):
            t, j = (ids == lo + e).nonzero(as_tuple=True)
            if t.numel():
                routed.index_add_(0, t, gate[t, j][:, None] * _ffn(o[t], w.gate_up[e], w.down[e], False))
        p = o + msg
    return dict(out=p + routed)
