"""The work whose speed is measured: one dict per case, made into inputs by prepare() and run once by run().

The cases are what a program around this framework has it do in one validation round of retrieval-augmented
speculative decoding, from the smallest call to the largest: attention of the verification positions over contiguous
and paged caches, the drafter's own decode step (recorded once as a graph and replayed, as a decode loop does), the
output head, the accept pass at small, large and ragged-vocabulary batches and in its greedy limit, and one whole round
of a batch.  Sizes are those of the workloads in paper_2502_20330_amd/workloads.py and of the tests, or generic.

Sequence lengths and draft counts of a ragged batch are a fixed spread over the case's range, so that work() is a
function of the case alone; all values come from the seed.
"""
from __future__ import annotations

import math

import torch

from paper_2502_20330_amd import binding


def listed():
    return [
        # the smallest call: 4 query heads on one kv head of 64, a 2K-token context; latency and launches
        dict(name="attn_2k_4h", op="attn", batch=1, hq=4, hkv=1, d=64, ctx_lo=2048, ctx=2048, gamma_lo=4, gamma=4,
             page=0, layout="token", lse=False),
        # one verification layer of an 8B-shaped target at 32K tokens, with the log-sum-exp that a caller who shards
        # the context needs
        dict(name="attn_32k", op="attn", batch=1, hq=32, hkv=8, d=128, ctx_lo=32768, ctx=32768, gamma_lo=8, gamma=8,
             page=0, layout="head", lse=True),
        # the same at 128K tokens: the headline configuration's layer
        dict(name="attn_128k", op="attn", batch=1, hq=32, hkv=8, d=128, ctx_lo=131072, ctx=131072, gamma_lo=8, gamma=8,
             page=0, layout="head", lse=False),
        # a served batch: eight sequences of 16K..128K tokens, 4..8 drafts each, 16-token pages in random order
        dict(name="attn_paged_ragged_b8", op="attn", batch=8, hq=32, hkv=8, d=128, ctx_lo=16385, ctx=131071, gamma_lo=4,
             gamma=8, page=16, layout="head", lse=False),
        # a 70B-shaped layer: 72 packed query rows per kv head
        dict(name="attn_128k_72rows", op="attn", batch=1, hq=64, hkv=8, d=128, ctx_lo=131072, ctx=131072, gamma_lo=8,
             gamma=8, page=0, layout="head", lse=False),
        # the drafter's decode step on the retrieved 8K context: 16 layers, output head for one row, one draw; a graph
        dict(name="drafter_step_8k", op="drafter", batch=1, hq=32, hkv=8, d=128, ctx=8192, layers=16, hidden=2048,
             vocab=128256, layout="head", temperature=1.0),
        # accept pass of one sequence: the latency of every round
        dict(name="accept_b1", op="accept", batch=1, gamma_lo=8, gamma=8, vocab=128256, eta=1.0, temperature=1.0, tail=0.1),
        # accept pass of a large served batch
        dict(name="accept_b64", op="accept", batch=64, gamma_lo=4, gamma=8, vocab=128256, eta=1.0, temperature=1.0,
             tail=0.1),
        # a vocabulary that is not a multiple of four (rows of logits are then not 16-byte aligned), low temperature
        dict(name="accept_odd_vocab_b8", op="accept", batch=8, gamma_lo=10, gamma=10, vocab=50257, eta=5.0,
             temperature=0.7, tail=0.1),
        # greedy decoding of a batch
        dict(name="accept_greedy_b16", op="accept", batch=16, gamma_lo=4, gamma=8, vocab=128256, eta=0.5, temperature=0.0,
             tail=0.1),
        # output head of one sequence's nine verification rows, with the statistics for the accept pass
        dict(name="lm_head_9rows", op="head", rows=9, hidden=4096, vocab=128256, temperature=1.0),
        # one round of a served batch: two layers of append + attention on paged caches, the head for all 72 rows, the
        # accept pass on its statistics, the commit of the accepted lengths
        dict(name="round_b8", op="round", batch=8, hq=32, hkv=8, d=128, ctx_lo=2049, ctx=12289, gamma_lo=4, gamma=8,
             page=16, layout="head", layers=2, hidden=4096, vocab=128256, eta=1.0, temperature=1.0, tail=0.1),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _shape(rng):
    hq, hkv, d = rng.choice([(4, 1, 64), (32, 8, 128), (32, 8, 128), (64, 8, 128), (28, 4, 128), (16, 8, 64)])
    return hq, hkv, d


def draw(rng):
    op = rng.choice(["attn", "attn", "attn", "attn", "accept", "accept", "accept", "head", "head", "drafter", "round"])
    if op == "attn":
        hq, hkv, d = _shape(rng)
        gamma = rng.randint(0, min(10, 96 // (hq // hkv) - 1))
        ctx = _log_int(rng, 2048, 131072)
        per_token = 4 * hkv * d
        batch = min(_log_int(rng, 1, 16), max(1, int(2.2e9 // (per_token * ctx))))
        ragged = batch > 1 and rng.random() < 0.7
        page = rng.choice([0, 0, 16, 64])
        return dict(op=op, batch=batch, hq=hq, hkv=hkv, d=d, ctx_lo=max(1024, ctx // rng.randint(2, 8)) if ragged else ctx,
                    ctx=ctx, gamma_lo=gamma // 2 if ragged else gamma, gamma=gamma, page=page,
                    layout=rng.choice(["head", "head", "token"]), lse=rng.random() < 0.3)
    if op == "accept":
        gamma = rng.randint(1, 10)
        vocab = _log_int(rng, 8192, 152064)
        if rng.random() < 0.5:
            vocab = vocab // 64 * 64
        batch = min(_log_int(rng, 1, 64), max(1, int(5.5e8 // ((2 * gamma + 1) * vocab * 4))))
        return dict(op=op, batch=batch, gamma_lo=rng.randint(max(1, gamma // 2), gamma), gamma=gamma, vocab=vocab,
                    eta=rng.choice([0.0, 0.25, 0.5, 1.0, 5.0]), temperature=rng.choice([0.0, 0.1, 0.7, 1.0]),
                    tail=rng.choice([0.0, 0.1]))
    if op == "head":
        hidden = 128 * _log_int(rng, 8, 64)
        return dict(op=op, rows=_log_int(rng, 1, 96), hidden=hidden, temperature=rng.choice([0.7, 1.0]),
                    vocab=min(_log_int(rng, 8192, 152064), int(1.4e9 // (2 * hidden))))
    if op == "drafter":
        hq, hkv, d = _shape(rng)
        return dict(op=op, batch=_log_int(rng, 1, 4), hq=hq, hkv=hkv, d=d, ctx=_log_int(rng, 2048, 8192),
                    layers=rng.randint(4, 16), hidden=128 * rng.randint(8, 24), vocab=_log_int(rng, 32000, 128256),
                    layout=rng.choice(["head", "token"]), temperature=rng.choice([0.1, 1.0]))
    gamma = rng.randint(3, 8)
    return dict(op=op, batch=rng.randint(1, 96 // (gamma + 1) if gamma > 7 else 8), hq=32, hkv=8, d=128, ctx_lo=1025,
                ctx=_log_int(rng, 2048, 12288), gamma_lo=gamma // 2, gamma=gamma, page=rng.choice([16, 64]), layout="head",
                layers=rng.randint(1, 2), hidden=128 * rng.randint(16, 32), vocab=_log_int(rng, 32000, 128256) // 8 * 8,
                eta=rng.choice([0.25, 1.0]), temperature=rng.choice([0.7, 1.0]), tail=0.1)


# ---------------------------------------------------------------- sizes that follow from a case
def _spread(lo, hi, n):
    """n whole numbers spread over [lo, hi], not sorted; the first one is hi (caches are sized for it)."""
    return [hi if i == 0 else lo + int((hi - lo) * ((i * 0.6180339887498949) % 1.0)) for i in range(n)]


def _lens(case):
    if "ctx_lo" not in case:
        return [case["ctx"]] * case["batch"]
    return _spread(min(case["ctx_lo"], case["ctx"]), case["ctx"], case["batch"])


def _gammas(case):
    return _spread(case["gamma_lo"], case["gamma"], case["batch"])[::-1]


def work(case):
    op = case["op"]
    nbytes = flops = 0
    if op in ("attn", "round", "drafter"):
        gam = [0] * case["batch"] if op == "drafter" else _gammas(case)
        for length, g in zip(_lens(case), gam):
            rows = (g + 1) * case["hq"]
            nbytes += 4 * length * case["hkv"] * case["d"] + 4 * rows * case["d"]
            flops += 4 * rows * length * case["d"]
        nbytes, flops = nbytes * case.get("layers", 1), flops * case.get("layers", 1)
    if op == "round":
        nbytes += case["layers"] * 8 * sum(g + 1 for g in gam) * case["hkv"] * case["d"]     # rows appended: read, written
    if op in ("head", "round", "drafter"):
        rows = case["rows"] if op == "head" else case["batch"] * (case.get("gamma", 0) + 1)
        nbytes += 2 * case["hidden"] * (case["vocab"] + rows) + 4 * rows * case["vocab"]
        flops += 2 * rows * case["hidden"] * case["vocab"]
    if op in ("accept", "round", "drafter"):
        gam = [0] * case["batch"] if op == "drafter" else _gammas(case)
        for g in gam:
            nbytes += 4 * (2 * g + 1) * case["vocab"]
            flops += 10 * (2 * g + 1) * case["vocab"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the path shows against 64 bits (errors of every output: exact())."""
    if case["op"] == "accept":
        # ratios: 2.4e-7 from 32-bit sums over a slice; whole values: a test within 1e-5 of its uniform, or a draw on
        # the edge between two tokens, may fall either way
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.005}
    if case["op"] == "head":
        # 4e-7 on the logits, 9e-7 on the statistics: 32-bit sums over the hidden size
        return {"rel": 4e-6, "max": 4e-5}
    # 2.2e-3: attention results are rounded to bf16 once, and the probabilities before the second product
    return {"rel": 1e-2, "max": 0.06, "differ": 0.01}


# ---------------------------------------------------------------- inputs
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, shape, dtype, std=1.0):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def _int32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def _kv_inputs(case, g, layers):
    """Queries, caches (scores of standard deviation 2, so that attention is neither uniform nor one key), lengths."""
    B, d, hkv, lens = case["batch"], case["d"], case["hkv"], _lens(case)
    page = case.get("page", 0)
    s = dict(lens=_int32(lens), max_ctx=max(lens), ctx_sum=sum(lens), page_table=None)
    if page:
        need = [-(-n // page) for n in lens]
        n_pages = sum(need) + 3                                  # a few pages that nobody owns
        perm = torch.randperm(n_pages, device="cuda", generator=g).to(torch.int32)
        table = torch.full((B, max(need)), -1, dtype=torch.int32, device="cuda")
        at = 0
        for b, n in enumerate(need):
            table[b, :n] = perm[at:at + n]
            at += n
        s["page_table"] = table
        shape = (n_pages, page, hkv, d)
    else:
        shape = (B, max(lens), hkv, d)
    if case["layout"] == "head":                                 # memory order: heads outside tokens
        shape = (shape[0], shape[2], shape[1], shape[3])
    view = (lambda t: t.permute(0, 2, 1, 3)) if case["layout"] == "head" else (lambda t: t)
    rows = case.get("gamma", 0) + 1
    s["q"] = [_randn(g, (B, rows, case["hq"], d), torch.bfloat16) for _ in range(layers)]
    s["k"] = [view(_randn(g, shape, torch.bfloat16, 2.0)) for _ in range(layers)]
    s["v"] = [view(_randn(g, shape, torch.bfloat16)) for _ in range(layers)]
    return s


def _draft_inputs(case, g, target):
    """Drafter's logits = target's + noise, drafted tokens drawn from them, uniforms (target: [B, gamma + 1, V])."""
    B, rows, V = target.shape
    draft = torch.empty((B, rows - 1, V), dtype=torch.float32, device="cuda")
    tokens = torch.empty((B, rows - 1), dtype=torch.int32, device="cuda")
    for b in range(B):
        draft[b] = target[b, :rows - 1] + _randn(g, (rows - 1, V), torch.float32)
        t = case["temperature"]
        noise = torch.empty((rows - 1, V), dtype=torch.float32, device="cuda").exponential_(generator=g).log_().neg_()
        tokens[b] = (draft[b] / t + noise if t > 0 else draft[b]).argmax(-1).to(torch.int32)
    return dict(draft=draft, tokens=tokens, uniforms=torch.rand((B, rows), device="cuda", generator=g))


def _head_inputs(case, g, rows):
    hidden, V = case["hidden"], case["vocab"]
    return dict(h=_randn(g, (rows, hidden), torch.bfloat16),
                w=_randn(g, (V, hidden), torch.bfloat16, 4.0 / math.sqrt(hidden)))


def _inputs(case, seed):
    g = _generator(seed)
    op = case["op"]
    s = dict(case=case)
    if op == "attn":
        s.update(_kv_inputs(case, g, 1), gammas=_int32(_gammas(case)))
    elif op == "accept":
        target = _randn(g, (case["batch"], case["gamma"] + 1, case["vocab"]), torch.float32, 4.0)
        s.update(_draft_inputs(case, g, target), target=target, gammas=_int32(_gammas(case)))
    elif op == "head":
        s.update(_head_inputs(case, g, case["rows"]))
    elif op == "drafter":
        s.update(_kv_inputs(case, g, case["layers"]), **_head_inputs(case, g, case["batch"]))
        s["uniforms"] = torch.rand((case["batch"], 1), device="cuda", generator=g)
        s["no_draft"] = torch.empty((case["batch"], 0, case["vocab"]), dtype=torch.float32, device="cuda")
        s["no_tokens"] = torch.empty((case["batch"], 0), dtype=torch.int32, device="cuda")
    else:
        B, rows = case["batch"], case["gamma"] + 1
        s.update(_kv_inputs(case, g, case["layers"]), **_head_inputs(case, g, B * rows))
        for name, std in (("k_new", 2.0), ("v_new", 1.0)):
            s[name] = [_randn(g, (B, rows, case["hkv"], case["d"]), torch.bfloat16, std) for _ in range(case["layers"])]
        target = (s["h"].float() @ s["w"].float().t()).view(B, rows, case["vocab"])      # only to draw drafts from
        s.update(_draft_inputs(case, g, target), gammas=_int32(_gammas(case)))
    return s


_shared = []


def _handle():
    """The one library handle a program keeps per GPU."""
    if not _shared:
        _shared.append(binding.Rapid(0))
    return _shared[0]


def prepare(case, seed):
    s = _inputs(case, seed)
    op = case["op"]
    if op in ("attn", "drafter", "round"):
        s["out"] = [torch.empty_like(q) for q in s["q"]]
    if op == "attn" and case["lse"]:
        s["lse"] = torch.empty((case["batch"], case["hq"], case["gamma"] + 1), dtype=torch.float32, device="cuda")
    if op == "round":
        s["ctx"] = s["lens"].clone()
    if op == "drafter":
        # a handle of its own: the recorded graph keeps using its workspaces
        s["rapid"], s["graph"] = binding.Rapid(0), torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _drafter_step(s)                                     # the workspaces exist before the recording
        torch.cuda.current_stream().wait_stream(side)
        with torch.cuda.graph(s["graph"]):
            s["result"] = _drafter_step(s)
    else:
        s["rapid"] = _handle()
    return s


# ---------------------------------------------------------------- one pass
def _drafter_step(s):
    r, case = s["rapid"], s["case"]
    for q, k, v, out in zip(s["q"], s["k"], s["v"], s["out"]):
        r.rapid_verify_attn(q, k, v, s["lens"], max_ctx=s["max_ctx"], out=out)
    logits, stats = r.rapid_lm_head(s["h"], s["w"], temperature=case["temperature"])
    _, tokens, _ = r.rapid_accept(logits.view(case["batch"], 1, -1), s["no_draft"], s["no_tokens"], 0.0, s["uniforms"],
                                  temperature=case["temperature"], want_ratio=False, target_stats=stats)
    return {"out": s["out"], "logits": logits, "stats": stats, "tokens": tokens}


def run(s):
    case, r = s["case"], s["rapid"]
    op = case["op"]
    if op == "attn":
        out = r.rapid_verify_attn(s["q"][0], s["k"][0], s["v"][0], s["lens"], gammas=s["gammas"],
                                  page_table=s["page_table"], max_ctx=s["max_ctx"], out=s["out"][0],
                                  lse_out=s.get("lse"), ctx_sum_hint=s["ctx_sum"])
        return {"out": out, "lse": s.get("lse")}
    if op == "accept":
        n, tokens, ratio = r.rapid_accept(s["target"], s["draft"], s["tokens"], case["eta"], s["uniforms"],
                                          gammas=s["gammas"], temperature=case["temperature"], tail_alpha=case["tail"])
        return {"n": n, "tokens": tokens, "ratio": ratio}
    if op == "head":
        logits, stats = r.rapid_lm_head(s["h"], s["w"], temperature=case["temperature"])
        return {"logits": logits, "stats": stats}
    if op == "drafter":
        s["graph"].replay()
        return s["result"]
    s["ctx"].copy_(s["lens"])                                    # the lengths with this round's positions counted
    for i in range(case["layers"]):
        r.rapid_kv_append(s["k"][i], s["v"][i], s["k_new"][i], s["v_new"][i], s["ctx"], gammas=s["gammas"],
                          page_table=s["page_table"], max_ctx=s["max_ctx"])
        r.rapid_verify_attn(s["q"][i], s["k"][i], s["v"][i], s["ctx"], gammas=s["gammas"], page_table=s["page_table"],
                            max_ctx=s["max_ctx"], out=s["out"][i], ctx_sum_hint=s["ctx_sum"])
    logits, stats = r.rapid_lm_head(s["h"], s["w"], temperature=case["temperature"])
    n, tokens, ratio = r.rapid_accept(logits.view(case["batch"], case["gamma"] + 1, -1), s["draft"], s["tokens"],
                                      case["eta"], s["uniforms"], gammas=s["gammas"], temperature=case["temperature"],
                                      tail_alpha=case["tail"], target_stats=stats)
    released, count = r.rapid_kv_commit_pages(s["ctx"], n, s["page_table"], page_size=case["page"],
                                              q_max=case["gamma"] + 1, max_ctx=s["max_ctx"], gammas=s["gammas"],
                                              n_pages=s["k"][0].shape[0])
    return {"out": s["out"], "k": s["k"], "v": s["v"], "logits": logits, "stats": stats, "n": n, "tokens": tokens,
            "ratio": ratio, "ctx": s["ctx"], "released": released, "count": count}


# ---------------------------------------------------------------- the same in 64 bits
def _exact_attn(s, layer, gammas):
    case = s["case"]
    q = s["q"][layer]
    B, rows, hq, d = q.shape
    group = hq // case["hkv"]
    out = torch.zeros((B, rows, hq, d), dtype=torch.float64, device="cuda")
    lse = torch.zeros((B, hq, rows), dtype=torch.float64, device="cuda")
    for b, (length, gamma) in enumerate(zip(_lens(case), gammas)):
        n = gamma + 1
        if s["page_table"] is None:
            k, v = s["k"][layer][b, :length], s["v"][layer][b, :length]
        else:
            ids = s["page_table"][b, :-(-length // case["page"])].long()
            k, v = (t[layer][ids].reshape(-1, case["hkv"], d)[:length] for t in (s["k"], s["v"]))
        hidden = torch.arange(length, device="cuda")[None, :] > (length - n + torch.arange(n, device="cuda"))[:, None]
        for kv in range(case["hkv"]):
            kt = k[:, kv].double().t().contiguous()
            vd = v[:, kv].double().contiguous()
            for h in range(kv * group, (kv + 1) * group):
                score = (q[b, :n, h].double() @ kt) * d ** -0.5
                score.masked_fill_(hidden, -math.inf)
                lse[b, h, :n] = torch.logsumexp(score, -1)
                out[b, :n, h] = torch.softmax(score, -1) @ vd
    return out, lse


def _exact_head(s):
    case = s["case"]
    h, w = s["h"].double(), s["w"]
    logits = torch.cat([h @ w[i:i + 16384].double().t().contiguous() for i in range(0, w.shape[0], 16384)], 1)
    # statistics: one chunk per workgroup, a multiple of 16 entries and at most 512, in whole rounds over the chip
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    blocks = -(-w.shape[0] // 16)
    rounds = -(-blocks // (32 * cus))
    chunk = 16 * min(32, max(1, -(-blocks // (rounds * cus))))
    n = -(-w.shape[0] // chunk)
    z = torch.nn.functional.pad(logits, (0, n * chunk - w.shape[0]), value=-math.inf).view(h.shape[0], n, chunk)
    top = z.amax(-1)
    stats = torch.stack([top, torch.exp((z - top[..., None]) / case["temperature"]).sum(-1)], -1)
    return logits, stats


def _exact_accept(target, draft, tokens, uniforms, gammas, eta, temperature, tail):
    B, rows, V = target.shape
    n_out = torch.zeros(B, dtype=torch.int32)
    tok_out = torch.full((B, rows), -1, dtype=torch.int32)
    ratio = torch.zeros((B, rows - 1), dtype=torch.float64)
    u = uniforms.double().cpu()
    for b in range(B):
        g, n, weight = gammas[b], gammas[b], None
        for k in range(g):
            zt, zd, x = target[b, k].double(), draft[b, k].double(), int(tokens[b, k])
            if temperature == 0:
                a, c = float(zt[x] - zt.max()), float(zd[x] - zd.max())
                rho = math.inf if a > c else 1.0 if a == c else 0.0
            else:
                p, q = torch.softmax(zt / temperature, -1), torch.softmax(zd / temperature, -1)
                mixed = torch.softmax(zt / temperature + eta * (q - p), -1)
                mixed = torch.where(mixed < tail * mixed.max(), p, mixed)
                rho = float(mixed[x] / q[x])
            ratio[b, k] = rho
            if n == g and weight is None and float(u[b, k]) > min(1.0, rho):
                n = k
                weight = False if temperature == 0 else torch.maximum(p - mixed, p - q).clamp_min(0.0)
                if weight is not False and not float(weight.sum()) > 0:
                    weight = p
        tok_out[b, :n] = tokens[b, :n].cpu()
        if temperature == 0:
            tok_out[b, n] = int(target[b, n].argmax())
        else:
            if weight is None:
                weight = torch.softmax(target[b, n].double() / temperature, -1)
            run_sum = torch.cumsum(weight, -1)
            tok_out[b, n] = min(V - 1, int((run_sum <= float(u[b, rows - 1]) * float(run_sum[-1])).sum()))
        n_out[b] = n
    return n_out, tok_out, ratio


def exact(case, seed):
    s = _inputs(case, seed)
    op = case["op"]
    if op == "attn":
        out, lse = _exact_attn(s, 0, _gammas(case))
        return {"out": out, "lse": lse if case["lse"] else None}
    if op == "accept":
        n, tokens, ratio = _exact_accept(s["target"], s["draft"], s["tokens"], s["uniforms"], _gammas(case), case["eta"],
                                         case["temperature"], case["tail"])
        return {"n": n, "tokens": tokens, "ratio": ratio}
    if op == "head":
        logits, stats = _exact_head(s)
        return {"logits": logits, "stats": stats}
    if op == "drafter":
        logits, stats = _exact_head(s)
        _, tokens, _ = _exact_accept(logits[:, None], None, s["no_tokens"], s["uniforms"], [0] * case["batch"], 0.0,
                                     case["temperature"], 0.1)
        return {"out": [_exact_attn(s, i, [0] * case["batch"])[0] for i in range(case["layers"])], "logits": logits,
                "stats": stats, "tokens": tokens}
    gammas, lens = _gammas(case), _lens(case)
    for i in range(case["layers"]):                              # the appended rows
        for b, (length, g) in enumerate(zip(lens, gammas)):
            at = torch.arange(length - g - 1, length, device="cuda")
            pages = s["page_table"][b][at // case["page"]].long()
            s["k"][i][pages, at % case["page"]] = s["k_new"][i][b, :g + 1]
            s["v"][i][pages, at % case["page"]] = s["v_new"][i][b, :g + 1]
    logits, stats = _exact_head(s)
    n, tokens, ratio = _exact_accept(logits.view(case["batch"], case["gamma"] + 1, -1), s["draft"], s["tokens"],
                                     s["uniforms"], gammas, case["eta"], case["temperature"], case["tail"])
    return {"out": [_exact_attn(s, i, gammas)[0] for i in range(case["layers"])], "k": s["k"], "v": s["v"],
            "logits": logits, "stats": stats, "n": n, "tokens": tokens, "ratio": ratio, "ctx": None, "released": None,
            "count": None}
