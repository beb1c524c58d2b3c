"""The work that this framework is measured on: decode attention, the products of a decoder block,
and whole decode steps, each through the calls that a serving program makes.

A case is a dict of plain values.  Its ``kind``:

* ``attention``  ``layers`` calls of one ``DecodeStepPlan`` each (the sweep of a paged cache in
                 position shards, then the combine), every layer with a cache and a plan of its own;
* ``one_launch`` the same attention through ``attn_decode_noalloc`` (sweep and merge in one launch,
                 nothing allocated), the layers captured in one HIP graph, as a serving loop keeps
                 them;
* ``protocol``   the attention of a decode step with its current token: ``attn_decode_split``, then
                 ``attn_combine_current_append``, the layers captured in one HIP graph;
* ``mlp``        the feed-forward of ``layers`` blocks (``linear`` with the RMS prologue and the gated
                 output, then ``linear`` with the residual), captured in one HIP graph;
* ``step``       a whole decode step of a ``QFirstStack`` (products, sweep, merge, append), captured
                 by ``QFirstStack.capture`` and replayed.

Where a pass appends a position, it first sets the context lengths back (one small copy), so every
pass is the same step: a decode loop that rejects its last token does just that.
"""

import math

import torch

import paper_2608_15473_amd as qf
from paper_2608_15473_amd.stage import LayerCache, QFirstStack

D, P = 128, 16          # head dimension and page size, the library's own
SCALE = 1.0 / math.sqrt(D)
EPS = 1e-6

# (query heads, KV heads, hidden, feed-forward width) of the configurations that this repository
# names: Qwen3-0.6B and Qwen3-4B, and the head counts of Qwen3-32B
SMALL = dict(hq=16, hkv=8, hidden=1024, inter=3072)
MEDIUM = dict(hq=32, hkv=8, hidden=2560, inter=9728)


def _attention(name, kind="attention", batch=1, hq=16, hkv=8, ctx=4608, ragged=False, shards=8,
               layers=1, perm=True, sharp=1.0):
    """``ctx``: every request's cached positions (``ragged``: the longest one's, the others drawn
    log-uniformly below it); ``shards``: of the longest request; ``perm``: pages at random places of
    the pool (else in order); ``sharp``: factor on the queries (larger: a more peaked softmax)."""
    c = dict(kind=kind, batch=batch, hq=hq, hkv=hkv, ctx=ctx, ragged=ragged, shards=shards,
             layers=layers, perm=perm, sharp=sharp)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call in use: one request of 4,608 positions (where Qwen3-0.6B's cache bytes
        # equal its feed-forward's), pages in order, all 28 layers: latency and launches count.
        _attention("attn_b1_n4608", ctx=4608, shards=8, layers=28, perm=False),
        # One GPU's share of a 2^20-position request that 8 GPUs sweep together.
        _attention("attn_b1_n131072", ctx=131072, shards=2, layers=4, sharp=4.0),
        # One request of 2^20 positions on one GPU: the longest context.
        _attention("attn_b1_n1m", ctx=1 << 20, shards=16, sharp=4.0),
        # A full serving batch of medium contexts (Qwen3-0.6B heads), the largest uniform case.
        _attention("attn_b32_n32768", batch=32, ctx=32768, shards=64),
        # The same at Qwen3-4B's heads (four query heads per KV head), an odd context.
        _attention("attn_b16_n36480_g4", batch=16, hq=32, ctx=36480, shards=32),
        # A mixed batch: 64 requests of 512 to 131,072 positions.
        _attention("attn_b64_ragged_g4", batch=64, hq=32, ctx=131072, ragged=True, shards=32),
        # Qwen3-32B's heads: eight query heads per KV head.
        _attention("attn_b16_n32768_g8", batch=16, hq=64, ctx=32768, shards=32),
        # Short ragged chats at Qwen3-4B's heads in one launch per layer, for callers that cannot
        # allocate.
        _attention("one_launch_b4_ragged_g4", kind="one_launch", batch=4, hq=32, ctx=5987,
                   ragged=True, shards=12, layers=12, sharp=2.0),
        # The attention part of a decode step, current token folded in and appended: 12 chats.
        _attention("protocol_b12_ragged", kind="protocol", batch=12, ctx=7003, ragged=True,
                   shards=16, layers=8),
        # The feed-forward of eight requests at Qwen3-4B: weights streamed for a few rows.
        dict(name="mlp_b8_4b", kind="mlp", rows=8, hidden=2560, inter=9728, layers=4),
        # A whole decode step of Qwen3-0.6B, one request: the lowest latency a token can have.
        dict(name="step_b1_06b", kind="step", batch=1, ctx=4608, shards=24, layers=28, **SMALL),
        # The same for eight requests.
        dict(name="step_b8_06b", kind="step", batch=8, ctx=4608, shards=16, layers=28, **SMALL),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attention", "attention", "attention", "one_launch", "protocol", "mlp", "step"])
    if kind == "mlp":
        hidden, inter = rng.choice([(1024, 3072), (2560, 9728), (8 * _log(rng, 64, 640), 8 * _log(rng, 192, 1920))])
        return dict(kind=kind, rows=rng.randint(1, 8), hidden=hidden, inter=inter,
                    layers=rng.randint(2, 6))
    if kind == "step":
        batch, big = _log(rng, 1, 12), rng.random() < 0.3
        ctx = _log(rng, 300, 36480 if big and batch < 3 else 9000)
        return dict(kind=kind, batch=batch, ctx=ctx, shards=max(1, min(128, _log(rng, 8, 32), ctx // 32)),
                    layers=rng.randint(3, 12), **(MEDIUM if big else SMALL))
    g = rng.choice([1, 2, 2, 4, 4, 8])
    hkv = rng.choice([8, 8, 8, 4, 2])
    if kind == "attention":
        batch = _log(rng, 1, 64)
        ctx = _log(rng, 300, min(1 << 20, (1 << 20) // batch))
    else:
        batch = _log(rng, 1, 24)
        ctx = _log(rng, 200, 16000)
    ragged = batch > 1 and rng.random() < 0.5
    shards = max(1, min(64, _log(rng, 1, 64), ctx // 64))
    size = batch * ctx * hkv * D * 4 // (2 if ragged else 1)
    layers = max(1, min(16, (1 << 29) // size))
    return _attention(None, kind=kind, batch=batch, hq=g * hkv, hkv=hkv, ctx=ctx, ragged=ragged,
                      shards=shards, layers=layers, perm=rng.random() < 0.8,
                      sharp=rng.choice([1.0, 2.0, 4.0]))


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed % (1 << 31))


def _lengths(case, seed):
    """Cached positions of each request (host list)."""
    B, n = case["batch"], case["ctx"]
    if not case.get("ragged"):
        return [n] * B
    g = torch.Generator().manual_seed(seed % (1 << 31))
    lo = max(1, n // 256)
    r = torch.rand(B, generator=g, dtype=torch.float64)
    lens = [int(round(math.exp(math.log(lo) + float(x) * (math.log(n) - math.log(lo))))) for x in r]
    lens[int(torch.randint(B, (1,), generator=g))] = n
    return lens


def _caches(case, seed, spare=0):
    """Queries, pools, tables and lengths of every layer, stacked: [layers, ...]."""
    B, L, hq, hkv = case["batch"], case["layers"], case["hq"], case["hkv"]
    lens = _lengths(case, seed)
    g = _gen(seed)
    pages = torch.tensor([-(-(n + spare) // P) for n in lens])
    max_pages, total = int(pages.max()), int(pages.sum())
    perm = case.get("perm", True)
    # where a pass returns its pools, they have a size of their own whatever the lengths
    num = total if perm and not spare else B * max_pages
    q = torch.randn(L, B, hq, D, generator=g, device="cuda", dtype=torch.bfloat16)
    q *= case.get("sharp", 1.0)
    k = torch.randn(L, num, hkv, P, D, generator=g, device="cuda", dtype=torch.bfloat16)
    v = torch.randn(L, num, hkv, P, D, generator=g, device="cuda", dtype=torch.bfloat16)
    if perm:
        table = torch.full((L, B, max_pages), -1, dtype=torch.int32, device="cuda")
        used = (torch.arange(max_pages)[None] < pages[:, None]).cuda()
        for l in range(L):
            table[l][used] = torch.randperm(num, generator=g, device="cuda")[:total].to(torch.int32)
    else:
        table = torch.arange(num, dtype=torch.int32, device="cuda").view(1, B, max_pages).repeat(L, 1, 1)
    ctx = torch.tensor(lens, dtype=torch.int32, device="cuda").repeat(L, 1)
    # shards in proportion to the length, the longest request taking case["shards"]
    per = -(-max(lens) // case["shards"])
    shards = torch.tensor([min(case["shards"], max(1, -(-n // per))) for n in lens],
                          dtype=torch.int32, device="cuda")
    s = dict(q=q, k=k, v=v, table=table, ctx=ctx, shards=shards, lens=lens)
    if spare:
        s["k_cur"] = torch.randn(L, B, hkv, D, generator=g, device="cuda", dtype=torch.bfloat16)
        s["v_cur"] = torch.randn(L, B, hkv, D, generator=g, device="cuda", dtype=torch.bfloat16)
    return s


def _matrix(g, *shape):
    w = torch.randn(*shape, generator=g, device="cuda", dtype=torch.bfloat16)
    return w.mul_(1.0 / math.sqrt(shape[-1]))


def _gain(g, *shape):
    return (torch.rand(*shape, generator=g, device="cuda") + 0.5).to(torch.bfloat16)


def _mlp(case, seed):
    g, L, H, I = _gen(seed), case["layers"], case["hidden"], case["inter"]
    return dict(x=torch.randn(L, case["rows"], H, generator=g, device="cuda", dtype=torch.bfloat16),
                w_gu=_matrix(g, L, 2 * I, H), w_down=_matrix(g, L, H, I), gain=_gain(g, L, H))


def _blocks(case, seed):
    """The weights of every block and the step's input."""
    g, H, I = _gen(seed + 1), case["hidden"], case["inter"]
    layers = []
    for _ in range(case["layers"]):
        w = dict(w_q=_matrix(g, case["hq"] * D, H), w_k=_matrix(g, case["hkv"] * D, H),
                 w_v=_matrix(g, case["hkv"] * D, H), w_o=_matrix(g, H, case["hq"] * D),
                 w_gate=_matrix(g, I, H), w_up=_matrix(g, I, H), w_down=_matrix(g, H, I))
        w["g1"], w["g2"] = _gain(g, H), _gain(g, H)
        layers.append(w)
    u = torch.randn(case["batch"], H, generator=g, device="cuda", dtype=torch.bfloat16)
    return layers, u


def _captured(call):
    """``call`` captured in a HIP graph, after one eager call (first-use set-up is not capturable)."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    return graph


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        s = _mlp(case, seed)
        L, M = case["layers"], case["rows"]
        s["act"] = torch.empty(L, M, case["inter"], device="cuda", dtype=torch.bfloat16)
        s["y"] = torch.empty(L, M, case["hidden"], device="cuda", dtype=torch.bfloat16)

        def call():
            for l in range(L):
                qf.linear(s["x"][l], s["w_gu"][l], "rms_norm", s["gain"][l], EPS, out=s["act"][l],
                          glu_out=True)
                qf.linear(s["act"][l], s["w_down"][l], residual=s["x"][l], out=s["y"][l])

        return dict(s, kind=kind, graph=_captured(call))

    if kind == "step":
        s = _caches(case, seed, spare=1)
        layers, u = _blocks(case, seed)
        caches = [LayerCache(s["k"][l], s["v"][l], s["table"][l], s["ctx"][l], s["shards"])
                  for l in range(case["layers"])]
        stack = QFirstStack(layers, caches, case["hq"], case["hkv"], max_shards=case["shards"],
                            scale=SCALE, eps=EPS)
        start = s["ctx"].clone()
        stack.step(u)                               # first-use set-up, outside the capture
        s["ctx"].copy_(start)
        torch.cuda.synchronize()
        graph, y = stack.capture(u)
        return dict(s, kind=kind, start=start, stack=stack, u=u, graph=graph, y=y)

    s = _caches(case, seed, spare=1 if kind == "protocol" else 0)
    L, B, hq, S = case["layers"], case["batch"], case["hq"], case["shards"]
    out = torch.empty(L, B, hq, D, device="cuda", dtype=torch.bfloat16)
    lse = torch.empty(L, B, hq, device="cuda", dtype=torch.float32)
    s.update(kind=kind, out=out, lse=lse)
    of = [(s["q"][l], s["k"][l], s["v"][l], s["table"][l], s["ctx"][l], s["shards"]) for l in range(L)]
    if kind == "attention":
        s["plans"] = [qf.DecodeStepPlan(*of[l], max_shards=S, scale=SCALE, out=out[l], lse=lse[l],
                                        fold_chunks=False) for l in range(L)]
    elif kind == "one_launch":
        def call():
            for l in range(L):
                qf.attn_decode_noalloc(*of[l], max_shards=S, scale=SCALE, out=out[l], lse=lse[l])
        s["graph"] = _captured(call)
    else:
        desc = qf.make_desc(s["q"][0], s["k"][0], s["table"][0], S, SCALE)
        ws = torch.empty(max(16, qf.workspace_size(desc)), dtype=torch.uint8, device="cuda")
        part_out = torch.empty(B, S, hq, D, device="cuda", dtype=torch.float32)
        part_lse = torch.empty(B, S, hq, device="cuda", dtype=torch.float32)
        s["start"] = s["ctx"].clone()

        def call():
            for l in range(L):
                qf.attn_decode_split(*of[l], max_shards=S, scale=SCALE, part_out=part_out,
                                     part_lse=part_lse, workspace=ws)
                qf.attn_combine_current_append(
                    part_out, part_lse, s["q"][l], s["k_cur"][l], s["v_cur"][l], s["k"][l], s["v"][l],
                    s["table"][l], s["ctx"][l], scale=SCALE, out=out[l], lse=lse[l])
        s["graph"] = _captured(call)
        s["ctx"].copy_(s["start"])
        s["keep"] = (ws, part_out, part_lse)
    return s


def run(s):
    kind = s["kind"]
    if kind == "attention":
        for plan in s["plans"]:
            plan()
        return s["out"], s["lse"]
    if kind == "one_launch":
        s["graph"].replay()
        return s["out"], s["lse"]
    if kind == "mlp":
        s["graph"].replay()
        return s["act"], s["y"]
    s["ctx"].copy_(s["start"])
    s["graph"].replay()
    if kind == "protocol":
        return s["out"], s["lse"], s["k"], s["v"], s["ctx"]
    return s["y"], s["k"], s["v"], s["ctx"]


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without, and what it should give
# ---------------------------------------------------------------------------------------------
def work(case):
    kind, L = case["kind"], case["layers"]
    if kind == "mlp":
        M, H, I = case["rows"], case["hidden"], case["inter"]
        return {"bytes": L * 2 * (3 * H * I + 2 * M * H + 2 * M * I + H),
                "flops": L * 2 * M * 3 * H * I}
    hq, hkv, B = case["hq"], case["hkv"], case["batch"]
    # a ragged batch's lengths are the seed's: their mean is that of the log-uniform range
    n = case["ctx"]
    if case.get("ragged"):
        lo = max(1, n // 256)
        n = (n + (B - 1) * (n - lo) / math.log(n / lo)) / B
    nbytes = B * n * hkv * D * 4 + B * hq * (D * 4 + 4)
    flops = B * n * hq * D * 4
    if kind == "step":
        H, I = case["hidden"], case["inter"]
        weights = H * D * (2 * hq + 2 * hkv) + 3 * H * I
        nbytes += 2 * weights + 4 * H + B * hkv * D * 4
        flops += 2 * B * weights
    return {"bytes": L * nbytes, "flops": L * flops}


def tolerance(case):
    if case["kind"] == "step":
        # seven tensors a block are rounded to bf16, and each rounding travels through the blocks
        # after it: 1.5e-2 measured over 28 blocks
        return {"rel": 3e-2}
    # one rounding to bf16 (2^-9 of an element at most): 1.7e-3 measured
    return {"rel": 7e-3}


def _attend(q, k, v, table, n, extra=None):
    """fp64 attention of one request: q [hq, D] over positions 0..n-1 of the pools, plus ``extra``
    (k, v) [hkv, D]; one KV head at a time.  Returns out [hq, D], lse [hq]."""
    hq, hkv = q.shape[0], k.shape[1]
    G = hq // hkv
    rows = table[: -(-n // P)].long()
    outs, lses = [], []
    for g in range(hkv):
        K = k[rows, g].reshape(-1, D)[:n].double()
        V = v[rows, g].reshape(-1, D)[:n].double()
        if extra is not None:
            K = torch.cat([K, extra[0][g : g + 1].double()])
            V = torch.cat([V, extra[1][g : g + 1].double()])
        s = torch.mm(K, q[g * G : (g + 1) * G].double().t().contiguous()) * SCALE      # [n, G]
        lse = torch.logsumexp(s, 0)
        w = torch.exp(s - lse).t().contiguous()
        outs.append(torch.mm(w, V))
        lses.append(lse)
    return torch.cat(outs), torch.cat(lses)


def _norm(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _bf16(x):
    return x.to(torch.bfloat16).double()


def exact(case, seed):
    kind, L = case["kind"], case["layers"]
    if kind == "mlp":
        s = _mlp(case, seed)
        acts, ys = [], []
        for l in range(L):
            x = s["x"][l].double()
            gu = torch.mm(_norm(x, s["gain"][l]), s["w_gu"][l].double().t().contiguous())
            gate, up = gu[:, 0::2], gu[:, 1::2]
            act = gate / (1 + torch.exp(-gate)) * up
            acts.append(act)
            # the activation is stored in bf16 between the two products
            ys.append(torch.mm(_bf16(act), s["w_down"][l].double().t().contiguous()) + x)
        return torch.stack(acts), torch.stack(ys)
    if kind == "step":
        s = _caches(case, seed, spare=1)
        layers, u = _blocks(case, seed)
        B, hq, hkv = case["batch"], case["hq"], case["hkv"]
        x = u.double()
        for l, w in enumerate(layers):
            m = {k: t.double().t().contiguous() for k, t in w.items() if k.startswith("w_")}
            n1 = _norm(x, w["g1"])
            q = _bf16(torch.mm(n1, m["w_q"]))                 # tensors between calls are bf16
            h = _norm(x, w["g2"])
            gate = torch.mm(h, m["w_gate"])
            act = _bf16(gate / (1 + torch.exp(-gate)) * torch.mm(h, m["w_up"]))
            z = _bf16(x + torch.mm(act, m["w_down"]))
            n1 = _norm(z, w["g1"])
            kc = torch.mm(n1, m["w_k"]).to(torch.bfloat16).view(B, hkv, D)
            vc = torch.mm(n1, m["w_v"]).to(torch.bfloat16).view(B, hkv, D)
            attn = torch.stack([_attend(q[b].view(hq, D), s["k"][l], s["v"][l], s["table"][l, b],
                                        s["lens"][b], (kc[b], vc[b]))[0] for b in range(B)])
            x = _bf16(z + torch.mm(_bf16(attn).view(B, -1), m["w_o"]))
            _append(s, l, kc, vc)
        return x, None, None, None
    s = _caches(case, seed, spare=1 if kind == "protocol" else 0)
    outs, lses = [], []
    for l in range(L):
        for b in range(case["batch"]):
            extra = (s["k_cur"][l, b], s["v_cur"][l, b]) if kind == "protocol" else None
            o, e = _attend(s["q"][l, b], s["k"][l], s["v"][l], s["table"][l, b], s["lens"][b], extra)
            outs.append(o)
            lses.append(e)
    shape = (L, case["batch"], case["hq"])
    out, lse = torch.stack(outs).view(*shape, D), torch.stack(lses).view(shape)
    return (out, lse, None, None, None) if kind == "protocol" else (out, lse)


def _append(s, l, k, v):
    for b, n in enumerate(s["lens"]):
        page = int(s["table"][l, b, n // P])
        s["k"][l, page, :, n % P] = k[b]
        s["v"][l, page, :, n % P] = v[b]
